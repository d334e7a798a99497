"""Restart points: decoding a stream's pieces side by side gives what decoding it from its start gives, with records
that are true, with records that are not, and with words that are damaged; and the records are what the oracle's
decoder holds at their places."""
import numpy as np
import pytest
import torch

from paper_2604_15356_amd.workloads import make_workload
from tests.gpu_util import codec_for, u8, u16, u32

pytestmark = pytest.mark.gpu

GOOD = 0x600D


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2604_15356_amd import plc
    plc.lib()
    return torch.device("cuda:0")


CASES = {
    # name: (path, overrides, layout, records per stream)
    "k8": ("mean", dict(L=2, H=2, n=300, k=8, d=128), "lhnkd", 4),
    "k1_heads_inner": ("mean", dict(L=1, H=3, n=515, k=1, d=40, sigma=0.6), "lnkhd", 3),
    # rows whose chunks a batch does not take whole numbers of, a stream that ends inside a batch, many escapes
    "k5_d24": ("mean", dict(S=2, L=2, H=3, n=461, k=5, d=24, sigma=1.5), "lhnkd", 5),
    # pieces by the thousand: the four-workgroup form of the one-kernel decode, and the three-block ring
    "k4_dense": ("mean", dict(L=8, H=16, n=200, k=4, d=128, sigma=0.5), "lhnkd", 12),
    "k6_dense": ("mean", dict(L=8, H=16, n=200, k=6, d=128, sigma=0.5), "lhnkd", 12),
    # two calls: more candidates than the one-kernel decode takes
    "k20": ("mean", dict(L=2, H=2, n=257, k=20, d=64, sigma=0.8), "lhnkd", 6),
    # more than 1024 pieces: the decoder with two units per wavefront, which counts the tiles' escapes where pieces are
    # whole tiles, and where they are not leaves that to a pass of its own
    "k20_tiles": ("mean", dict(L=8, H=16, n=256, k=20, d=64, sigma=0.8), "lhnkd", 16),
    "k20_no_tiles": ("mean", dict(L=8, H=16, n=257, k=20, d=64, sigma=0.8), "lhnkd", 16),
    # so long pieces that two calls are made
    "k2_two_calls": ("mean", dict(L=16, H=32, n=320, k=2, d=128, sigma=0.5), "lhnkd", 16),
    "cond_k5_two_calls": ("cond", dict(L=8, H=16, n=1024, k=5, d=128, sigma=0.4), "lhnkd", 32),
    "cond_k4": ("cond", dict(L=2, H=2, n=300, k=4, d=128, sigma=0.4), "lhnkd", 4),
    "cond_k8": ("cond", dict(L=2, H=2, n=300, k=8, d=80, sigma=0.4), "lnkhd", 7),
    "adapt": ("adapt", dict(L=2, H=2, n=400, k=8, d=64), "lhnkd", 5),
    "adapt_many": ("adapt", dict(L=12, H=50, n=70, k=3, d=64), "lhnkd", 2),
    # the other forms of the encoders of few units, which all write records: see ENCODERS
    "k20_many": ("mean", dict(L=12, H=50, n=90, k=20, d=64, sigma=0.5), "lhnkd", 2),
    "k20_short": ("mean", dict(L=3, H=7, n=75, k=20, d=64, sigma=0.5), "lhnkd", 2),
    "adapt_two": ("adapt", dict(L=10, H=30, n=165, k=3, d=64), "lhnkd", 3),
    "adapt_three": ("adapt", dict(L=12, H=50, n=169, k=3, d=64), "lhnkd", 3),
    "adapt_short": ("adapt", dict(L=3, H=7, n=75, k=3, d=64), "lhnkd", 2),
}
ENCODERS = {
    "k8": "pipe_kernel<false, 32, true>", "k20_many": "pipe_kernel<false, 16, true>", "adapt": "pipe_kernel<true, 32, true>",
    "adapt_two": "pipe_kernel<true, 32, false>", "adapt_three": "pipe_kernel<true, 16, false>",
    "k20_short": "short_kernel<false, true>", "adapt_short": "short_kernel<true, true>", "adapt_many": "short_kernel<true, false>",
}
THR = (3.0, 3.9)


def _setup(dev, case):
    path, overrides, layout, points = CASES[case]
    w = make_workload("tiny", device=dev, layout=layout, overrides=dict(overrides, seed=7), random_rows=True)
    codec = codec_for(w, esc_frac=1.0)
    from paper_2604_15356_amd import plc
    codec.restart = torch.zeros((codec.n_streams, points, plc.RESTART_WORDS), dtype=torch.int32, device=dev)
    codec._restart_scratch = torch.zeros((codec.n_streams, points, 2), dtype=torch.int32, device=dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(3)
    chosen = torch.randint(-1, w.k, (w.S, w.n), generator=gen, device=dev, dtype=torch.int32)
    from paper_2604_15356_amd.plc import surprisal_thresholds
    thr = surprisal_thresholds(*THR)
    vectors = (w.cand_k, w.cand_v, w.probs, w.act_k, w.act_v)

    def encode():
        if path == "mean":
            codec.encode(*vectors)
        elif path == "cond":
            codec.encode_cond(*vectors, chosen=chosen)
        else:
            codec.encode_adapt(*vectors, chosen, thr, 0.32)
        codec.check_status("encode")

    def decode(with_points):
        """(symbols, K, V, status) of a decode, from buffers that hold something else."""
        keep = codec.restart
        if not with_points:
            codec.restart = None
        codec.dec_symbols.fill_(77)
        codec._restart_scratch.fill_(-1)
        out = [torch.full_like(w.act_k, 3.0), torch.full_like(w.act_v, 3.0)]
        args = (w.cand_k, w.cand_v, w.probs, *out)
        try:
            if path == "mean":
                codec.decode(*args)
            elif path == "cond":
                codec.decode_cond(*args)
            else:
                codec.decode_adapt(*args, thr, 0.32)
        finally:
            codec.restart = keep
        status = int(codec.status.item())
        codec.status.zero_()
        return codec.dec_symbols.clone(), *[o.view(torch.int16) for o in out], status

    return codec, encode, decode


def _same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a[:3], b[:3])) and a[3] == b[3]


def _geometry(codec):
    """Groups of 32 symbols of a stream, and where in them its records stand (from record 1 on)."""
    G = (codec.N + 31) // 32
    head = G % 16 or 16
    rounds = ((G - head) // 16 + 1 + 3) // 4
    per = -(-rounds // codec.restart.shape[1])
    return G, [G - head - (4 * per * r - 1) * 16 for r in range(1, -(-rounds // per))]


def _step(codec, case):
    """Records per piece: the one-kernel decode takes a round of workgroups' worth of pieces."""
    from paper_2604_15356_amd import plc
    path, overrides, _, points = CASES[case]
    one = plc.plc_decode_one_kernel(codec.n_streams, codec.N, 0, overrides["k"], path != "mean", path == "adapt", points)
    assert one == (path != "adapt" and overrides["k"] <= 8 and "two_calls" not in case)
    if not one:
        return 1
    most = (1024 if overrides["k"] <= 4 else 512) // codec.n_streams
    return -(-(len(_geometry(codec)[1]) + 1) // most)


def _pieces_good(codec, case):
    """Streams all of whose pieces were found to fit together, from the decoder's scratch."""
    pieces = -(-(len(_geometry(codec)[1]) + 1) // _step(codec, case))
    assert pieces >= 2
    s = codec._restart_scratch.reshape(-1)
    assert bool((s[codec.n_streams * pieces * 2:] == -1).all())
    return (s[:codec.n_streams * pieces * 2].reshape(codec.n_streams, -1) == GOOD).all(dim=1)


@pytest.mark.parametrize("case", list(CASES))
def test_pieces_equal_the_whole_stream(dev, case):
    codec, encode, decode = _setup(dev, case)
    encode()
    plain = {x: getattr(codec, x).clone() for x in ("states", "words", "n_words")}
    whole = decode(False)
    assert whole[3] == 0 and torch.equal(whole[0], codec.symbols)
    assert _same(decode(True), whole)
    assert bool(_pieces_good(codec, case).all())
    # the encoder writes the same bitstream without records
    keep, codec.restart = codec.restart, None
    encode()
    codec.restart = keep
    used = torch.arange(codec.word_cap, device=dev)[None] < codec.n_words[:, None].long()
    assert torch.equal(codec.states, plain["states"]) and torch.equal(codec.n_words, plain["n_words"])
    assert torch.equal(codec.words.reshape(used.shape)[used], plain["words"].reshape(used.shape)[used])


@pytest.mark.parametrize("case", list(ENCODERS))
def test_records_of_every_encoder_fit_together(dev, case):
    """A record that is not true costs only the time of a second decode, so no other test can tell: every form of the
    encoders of few units writes records by which the pieces fit together."""
    from paper_2604_15356_amd import plc
    codec, encode, decode = _setup(dev, case)
    around = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in around:
        e.record()
    plc.plc_trace_kernel_events(plc.TRACE_RANS_ENCODE, *(e.cuda_event for e in around))
    try:
        encode()
    finally:
        plc.plc_trace_kernel_events(plc.TRACE_RANS_ENCODE)
    name = plc.plc_trace_kernel_name(plc.TRACE_RANS_ENCODE)
    assert ENCODERS[case] in name, name
    decode(True)
    assert bool(_pieces_good(codec, case).all())


@pytest.mark.parametrize("case", list(CASES))
def test_the_kernel_that_decodes_is_the_one_announced(dev, case):
    """One kernel that reconstructs, in pieces or not, or the first of two calls."""
    from paper_2604_15356_amd import plc
    codec, encode, decode = _setup(dev, case)
    path, overrides, _, points = CASES[case]
    encode()
    around = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in around:
        e.record()
    for restart in (True, False):
        plc.plc_trace_kernel_events(plc.TRACE_RANS_DECODE, *(e.cuda_event for e in around))
        try:
            decode(restart)
        finally:
            plc.plc_trace_kernel_events(plc.TRACE_RANS_DECODE)
        one = plc.plc_decode_one_kernel(codec.n_streams, codec.N, 0, overrides["k"], path != "mean", path == "adapt",
                                        points if restart else 0)
        name = plc.plc_trace_kernel_name(plc.TRACE_RANS_DECODE)
        reconstructs = any(name.startswith(f"rans_decode_{x}_kernel<{overrides['k']}, ") for x in ("chain", "depths"))
        assert bool(one) == reconstructs, name


@pytest.mark.parametrize("case", list(CASES))
def test_records_that_are_not_true_change_nothing(dev, case):
    codec, encode, decode = _setup(dev, case)
    encode()
    whole = decode(False)
    true = codec.restart.clone()
    last = codec.n_streams - 1

    def wrong(record, word, change):
        codec.restart.copy_(true)
        codec.restart[last, record, word] = change(codec.restart[last, record, word])

    step = _step(codec, case)
    for record in (step, len(_geometry(codec)[1]) // step * step):
        for word, change in ((0, lambda v: v ^ 1), (31, lambda v: v ^ (1 << 17)), (32, lambda v: v + 1),
                             (32, lambda v: v - 300), (32, lambda v: v * 0 - 1), (33, lambda v: v + 1)):
            if word == 33 and ("two_calls" in case or CASES[case][0] != "mean" or CASES[case][1]["k"] > 8):
                continue  # (two calls: the escapes are counted again, the record's are not looked at)
            wrong(record, word, change)
            assert _same(decode(True), whole), (record, word)
            good = _pieces_good(codec, case)
            assert not bool(good[last]) and bool(good[:last].all())
    for points in (torch.zeros_like(true), torch.full_like(true, -1), true.roll(1, 0), true.roll(1, 1)):
        codec.restart.copy_(points)
        assert _same(decode(True), whole)


@pytest.mark.parametrize("case", ["k8", "k20", "cond_k8", "adapt"])
def test_a_codec_looks_at_records_that_were_written(dev, case):
    """A codec that takes words from elsewhere decodes without records until it is given theirs."""
    codec, encode, decode = _setup(dev, case)
    reader, _, read = _setup(dev, case)
    encode()
    whole = decode(False)
    for x in ("esc_vals", "esc_off", "freq", "states", "words", "n_words", "idx_states", "idx_words", "idx_n_words"):
        getattr(reader, x).copy_(getattr(codec, x))
    if case == "adapt":
        reader._adapt_buffers()
        reader.freq_d.copy_(codec.freq_d)
    reader.restart.copy_(codec.restart)
    untouched = lambda: bool((reader._restart_scratch == -1).all())
    assert _same(read(True), whole) and untouched() and reader.coded().restart is None
    reader.set_restart(codec.coded().restart)
    assert _same(read(True), whole) and bool(_pieces_good(reader, case).all())
    reader.set_restart(None)
    assert _same(read(True), whole) and untouched()
    with pytest.raises(ValueError):
        reader.set_restart(codec.restart[:, 1:])


@pytest.mark.parametrize("case", list(CASES))
def test_records_of_other_words_are_told_by_the_first(dev, case):
    """Record 0 has what the stream starts from: where its word count or first state are others, no piece is decoded."""
    codec, encode, decode = _setup(dev, case)
    encode()
    whole, true = decode(False), codec.restart.clone()
    for word in (0, 32):
        codec.restart.copy_(true)
        codec.restart[0, 0, word] ^= 1
        assert _same(decode(True), whole), word
        good = _pieces_good(codec, case)
        assert not bool(good[0]) and bool(good[1:].all())
        state = codec._restart_scratch.reshape(-1)[:2 * (-(-(len(_geometry(codec)[1]) + 1) // _step(codec, case)))]
        assert not bool((state[::2] == GOOD).any())


@pytest.mark.parametrize("case", list(CASES))
def test_damaged_words_are_reported(dev, case):
    """What the decoder reports of damage does not depend on the records, nor do the streams that have none."""
    codec, encode, decode = _setup(dev, case)
    encode()
    at = codec.n_words.long() // 2
    codec.words.reshape(codec.n_streams, -1)[0, at[0]] ^= 0x155
    whole, pieces = decode(False), decode(True)
    assert whole[3] == pieces[3] == 3
    for a, b in zip(whole[:3], pieces[:3]):   # symbols, K and V, the damaged stream's too
        assert torch.equal(a, b)
    good = _pieces_good(codec, case)
    assert not bool(good[0]) and bool(good[1:].all())


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("what", ["table", "list"])
def test_streams_that_are_refused(dev, case, what):
    """A stream whose table is none, or whose words lie outside the list: reported, and K and V with and without records
    the same, for it as for the others."""
    codec, encode, decode = _setup(dev, case)
    encode()
    if what == "table":
        (codec.freq_d[:, 2] if CASES[case][0] == "adapt" else codec.freq)[0, 127] += 1
    else:
        codec.n_words[0] = 1 << 30
    whole, pieces = decode(False), decode(True)
    assert whole[3] == 3 and _same(pieces, whole)
    good = _pieces_good(codec, case)
    assert not bool(good[0]) and bool(good[1:].all())


def test_records_are_the_oracles_states(oracle, dev):
    """Every record against a decoder in numpy that walks the stream from its start."""
    codec, encode, _ = _setup(dev, "k5_d24")
    encode()
    G, at = _geometry(codec)
    assert len(at) >= 2 and min(at) > 0
    for stream in (0, codec.n_streams - 1):
        rec = u32(codec.restart[stream])
        places = {g: r + 1 for r, g in enumerate(at)}
        sym = u8(codec.symbols[stream])
        freq = u16(codec.freq[stream]).astype(np.int64)
        cum = np.concatenate([[0], np.cumsum(freq)])
        n_words = int(codec.n_words[stream])
        words = u16(codec.words.reshape(codec.n_streams, -1)[stream]).astype(np.int64)
        x, ptr = u32(codec.states[stream]).astype(np.int64), n_words
        seen = 0
        assert np.array_equal(rec[0, :32], x) and rec[0, 32] == n_words and rec[0, 33] == (sym == 255).sum()
        for g in range(G):
            if g in places:
                r = rec[places.pop(g)]
                assert np.array_equal(r[:32], x) and r[32] == ptr and r[33] == (sym == 255).sum() - seen
            s = sym[32 * g:32 * g + 32].astype(np.int64)
            lanes = len(s)
            seen += int((s == 255).sum())
            slot = x[:lanes] & 4095
            x[:lanes] = freq[s] * (x[:lanes] >> 12) + slot - cum[s]
            for l in np.flatnonzero(x[:lanes] < 65536):
                ptr -= 1
                x[l] = (x[l] << 16) | words[ptr]
        assert not places and ptr == 0 and (x == 65536).all()
