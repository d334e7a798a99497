"""The decoder with two units per wavefront: units of every length a chunk may have, odd numbers of them, a last one that
is shorter, tables of one symbol, a table per bit depth; and the tiles' escapes as it counts them."""
import numpy as np
import pytest
import torch

from paper_2604_15356_amd.workloads import make_workload
from tests.gpu_util import codec_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2604_15356_amd import plc
    plc.lib()
    return torch.device("cuda:0")


def _bytes(kind, shape, rng):
    if kind == "one":
        return np.full(shape, 200, dtype=np.uint8)
    if kind == "two":   # a frequency of 4095 and one of 1 in most units
        return np.where(rng.random(shape) < 0.0002, 3, 255).astype(np.uint8)
    if kind == "flat":
        return rng.integers(0, 256, shape, dtype=np.uint8)
    return np.clip(np.round(rng.normal(127, 9, shape)), 0, 255).astype(np.uint8)


@pytest.mark.parametrize("kind", ["flat", "peaked", "one", "two"])
@pytest.mark.parametrize("N,chunk", [(33, 32), (96, 32), (5000, 256), (5000, 512), (7 * 512, 512), (17 * 1024 + 1, 1024),
                                     (9 * 2048 + 1000, 2048), (40960, 4096), (70001, 8192), (3 * 16384, 16384)])
def test_chunks_come_back(dev, kind, N, chunk):
    from paper_2604_15356_amd import plc
    streams, rng = 3, np.random.default_rng(N + chunk)
    data = _bytes(kind, (streams, N), rng)
    symbols = torch.from_numpy(data).to(dev)
    units = streams * plc.plc_units_per_stream(N, chunk)
    i32 = dict(dtype=torch.int32, device=dev)
    i16 = dict(dtype=torch.int16, device=dev)
    status, counts = torch.zeros(1, **i32), torch.empty((streams, 256), **i32)
    freq, cum = torch.empty((streams, 256), **i16), torch.empty((streams, 257), **i16)
    states, n_words = torch.empty((units, 32), **i32), torch.empty(units, **i32)
    cap = chunk + 5      # lists at every place inside a line
    words = torch.empty(units * cap, **i16)
    word_off = torch.arange(units, dtype=torch.int64, device=dev) * cap
    plc.plc_histogram(symbols, streams, N, counts)
    plc.plc_build_freq(counts, streams, freq, cum, status)
    plc.plc_rans_encode(symbols, streams, N, chunk, freq, states, words, word_off, cap, n_words, status)
    out = torch.full_like(symbols, 99)
    plc.plc_rans_decode(freq, states, words, word_off, n_words, streams, N, chunk, out, status)
    assert int(status.item()) == 0 and torch.equal(out, symbols)
    # a word of the middle unit of stream 1 changed: reported, and every other unit as before
    per = units // streams
    bad = per + per // 2
    if int(n_words[bad]) > 2:
        words[int(word_off[bad]) + int(n_words[bad]) - 1] ^= 0x0311
        out.fill_(99)
        plc.plc_rans_decode(freq, states, words, word_off, n_words, streams, N, chunk, out, status)
        assert int(status.item()) == plc.PLC_ERR_CORRUPT
        same = (out == symbols).cpu().numpy().copy()
        at = bad - per
        same[1, at * chunk:(at + 1) * chunk] = True
        assert same.all()


@pytest.mark.parametrize("many", [False, True])   # up to 2560 units have a wavefront each
@pytest.mark.parametrize("n_tables,positions,chunk", [(4, 301, 1024), (4, 64, 96), (3, 100, 4096), (1, 77, 512), (2, 40, 32)])
def test_chunks_come_back_with_a_table_per_depth(dev, n_tables, positions, chunk, many):
    from paper_2604_15356_amd import plc
    spp, sps, rng = 96, 2, np.random.default_rng(positions)
    N = spp * positions
    streams = sps * (-(-2561 // (sps * plc.plc_units_per_stream(N, chunk))) if many else 2)
    bits = rng.integers(1, n_tables + 1, (streams // sps, positions)).astype(np.uint8)
    depth = np.repeat(np.repeat(bits, sps, 0), spp, 1)
    data = np.clip(np.round(rng.normal(127, 2.0 ** depth)), 0, 255).astype(np.uint8)
    data[depth == 2] = 127                      # that depth's table is one of a single symbol
    symbols, bits = torch.from_numpy(data).to(dev), torch.from_numpy(bits).to(dev)
    units = streams * plc.plc_units_per_stream(N, chunk)
    i32 = dict(dtype=torch.int32, device=dev)
    i16 = dict(dtype=torch.int16, device=dev)
    status, counts = torch.zeros(1, **i32), torch.empty((streams, n_tables, 256), **i32)
    freq = torch.empty((streams, n_tables, 256), **i16)
    states, n_words = torch.empty((units, 32), **i32), torch.empty(units, **i32)
    words = torch.empty(units * chunk, **i16)
    word_off = torch.arange(units, dtype=torch.int64, device=dev) * chunk
    plc.plc_histogram_bucketed(symbols, streams, N, spp, sps, bits, n_tables, counts, status)
    plc.plc_build_freq_bucketed(counts, streams, n_tables, freq, status)
    plc.plc_rans_encode_bucketed(symbols, streams, N, chunk, spp, sps, bits, n_tables, freq, states, words, word_off,
                                 chunk, n_words, status)
    out = torch.full_like(symbols, 99)
    plc.plc_rans_decode_bucketed(freq, states, words, word_off, n_words, streams, N, chunk, spp, sps, bits, n_tables,
                                 out, status)
    assert int(status.item()) == 0 and torch.equal(out, symbols)


@pytest.mark.parametrize("path,chunk,n,d,sigma", [("mean", 2048, 300, 128, 1.0), ("mean", 4096, 100, 72, 2.0),
                                                  ("mean", 1024, 300, 128, 1.0), ("mean", 8192, 33, 40, 3.0),
                                                  ("mean", 2048, 8, 128, 3.0), ("adapt", 2048, 300, 128, 1.0),
                                                  # a unit per wavefront, which leaves the counts to a pass
                                                  ("adapt", 131072, 1100, 128, 1.0)])
def test_escapes_counted_by_the_decoder(dev, path, chunk, n, d, sigma):
    """The one call counts each tile's escapes as it decodes (where units are whole tiles), the two calls in a pass."""
    from paper_2604_15356_amd import plc
    w = make_workload("tiny", device=dev, overrides=dict(L=2, H=3, n=n, k=3, d=d, sigma=sigma, seed=5), random_rows=True)
    codec = codec_for(w, esc_frac=1.0, chunk_syms=chunk)
    vectors, adapt = (w.cand_k, w.cand_v, w.probs, w.act_k, w.act_v), path == "adapt"
    thr = plc.surprisal_thresholds(3.0, 3.9)
    if adapt:
        codec.encode_adapt(*vectors, torch.zeros((w.S, w.n), dtype=torch.int32, device=dev), thr, 0.32)
    else:
        codec.encode(*vectors)
    assert int(codec.esc_cnt.sum()) > 0
    outs = []
    for fused in (True, False):
        codec.ws.fill_(0xa5)
        out = [torch.full_like(w.act_k, 3.0), torch.full_like(w.act_v, 3.0)]
        args = (w.cand_k, w.cand_v, w.probs, *out)
        codec.decode_adapt(*args, thr, 0.32, fused=fused) if adapt else codec.decode(*args, fused=fused)
        codec.check_status("decode")
        assert torch.equal(codec.dec_symbols, codec.symbols)
        outs.append([o.view(torch.int16) for o in out])
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])


@pytest.mark.parametrize("path", ["mean", "adapt"])
@pytest.mark.parametrize("what", ["list", "last_list", "table"])
def test_units_that_are_refused_leave_the_others_their_escapes(dev, path, what):
    """A unit whose word list lies outside the words, or whose table is none, is not decoded.  The places of the escapes
    behind it follow from what the symbol buffer holds there, in one call as in two, and not from old workspace."""
    from paper_2604_15356_amd import plc
    w = make_workload("tiny", device=dev, overrides=dict(L=2, H=3, n=300, k=3, d=128, sigma=1.0, seed=5), random_rows=True)
    codec = codec_for(w, esc_frac=1.0, chunk_syms=2048)
    vectors, thr = (w.cand_k, w.cand_v, w.probs, w.act_k, w.act_v), plc.surprisal_thresholds(3.0, 3.9)
    if path == "mean":
        codec.encode(*vectors)
    else:
        codec.encode_adapt(*vectors, torch.zeros((w.S, w.n), dtype=torch.int32, device=dev), thr, 0.32)
    codec.check_status("encode")
    stream, ups = 2, codec.units_per_stream
    if what == "table":
        (codec.freq if path == "mean" else codec.freq_d[:, 2])[stream, 127] += 1
    else:
        codec.n_words[stream * ups + (ups - 1 if what == "last_list" else 4)] = 1 << 30
    held = torch.randint(0, 256, codec.symbols.shape, dtype=torch.uint8, device=dev)
    held[:, ::3] = 255
    outs = []
    for fused in (True, False):
        codec.ws.fill_(0xa5)
        codec.dec_symbols.copy_(held)
        out = [torch.full_like(w.act_k, 3.0), torch.full_like(w.act_v, 3.0)]
        args = (w.cand_k, w.cand_v, w.probs, *out)
        if path == "mean":
            codec.decode(*args, fused=fused)
        else:
            codec.decode_adapt(*args, thr, 0.32, fused=fused)
        assert int(codec.status.item()) == plc.PLC_ERR_CORRUPT
        codec.status.zero_()
        outs.append([codec.dec_symbols.clone()] + [o.view(torch.int16) for o in out])
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    assert torch.equal(outs[0][0][:stream], codec.symbols[:stream])
