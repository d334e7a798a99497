"""The two encoders of few whole-stream units, four wavefronts to a short unit and seven to a long one: which takes which,
and both against the oracle where batches, rounds and rows begin and end."""
import numpy as np
import pytest
import torch

from tests.gpu_util import u16, u32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2604_15356_amd import plc
    plc.lib()
    return torch.device("cuda:0")


class Streams:
    """Streams of one session, a table each or one for each of `tables` bit depths, and their encoding by the oracle;
    rows start at every alignment that N gives them, word lists at odd addresses."""

    def __init__(self, oracle, dev, n_streams, N, tables, seed):
        self.dev, self.n, self.N, self.tables, self.spp = dev, n_streams, N, tables, 32
        rng = np.random.default_rng(seed)
        width = 30.0
        if tables > 1:
            self.bits = rng.integers(1, tables + 1, size=(1, N // self.spp)).astype(np.uint8)
            width = 1.0 * 3.0 ** np.repeat(self.bits, self.spp, axis=1)
            self.bits_t = torch.from_numpy(self.bits).to(dev)
        sym = rng.standard_normal((n_streams, N), dtype=np.float32) * np.float32(width) + 127
        self.sym = np.clip(np.rint(sym), 0, 254).astype(np.uint8)
        if tables > 1:
            freq = oracle.build_freq_sparse(oracle.histogram_bucketed(self.sym, self.spp, n_streams, self.bits,
                                                                      n_tables=tables))
            self.enc = oracle.rans_encode_bucketed(self.sym, freq, self.spp, n_streams, self.bits, word_cap_per_unit=N)
        else:
            freq, _ = oracle.build_freq(oracle.histogram(self.sym))
            self.enc = oracle.rans_encode(self.sym, freq, word_cap_per_unit=N)
        self.sym_t, self.freq_t = torch.from_numpy(self.sym).to(dev), torch.from_numpy(freq.view(np.int16)).to(dev)

    def encode(self, cap):
        """Encodes with room for cap words a stream; (status, kernel), after comparing everything with the oracle."""
        from paper_2604_15356_amd import plc
        n, lead, pitch, guard = self.n, 5, cap + 13, 0x5a5a
        empty = lambda shape, dt: torch.empty(shape, dtype=dt, device=self.dev)
        words = torch.full((lead + n * pitch,), guard, dtype=torch.int16, device=self.dev)
        off = lead + torch.arange(n, dtype=torch.int64, device=self.dev) * pitch
        states, n_words = empty((n, 32), torch.int32), empty(n, torch.int32)
        status = torch.zeros(1, dtype=torch.int32, device=self.dev)
        around = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for e in around:
            e.record()
        print(f"  {n} streams of {self.N} symbols, {self.tables} tables, room for {cap} words", flush=True)
        plc.plc_trace_kernel_events(plc.TRACE_RANS_ENCODE, *(e.cuda_event for e in around))
        try:
            if self.tables > 1:
                plc.plc_rans_encode_bucketed(self.sym_t, n, self.N, 0, self.spp, n, self.bits_t, self.tables, self.freq_t,
                                             states, words, off, cap, n_words, status)
            else:
                plc.plc_rans_encode(self.sym_t, n, self.N, 0, self.freq_t, states, words, off, cap, n_words, status)
        finally:
            plc.plc_trace_kernel_events(plc.TRACE_RANS_ENCODE)
        code = int(status.item())
        enc_words = self.enc["n_words"].astype(np.int64)
        assert np.array_equal(u32(n_words), self.enc["n_words"])
        assert np.array_equal(u32(states), self.enc["states"])
        expect = np.full(lead + n * pitch, guard, dtype=np.uint16)
        lists = expect[lead:].reshape(n, pitch)
        used = np.arange(cap)[None] < enc_words[:, None]
        lists[:, :cap] = np.where(used, self.enc["words"].reshape(n, self.N)[:, :cap], guard)
        assert np.array_equal(u16(words), expect)
        return code, plc.plc_trace_kernel_name(plc.TRACE_RANS_ENCODE)


@pytest.mark.parametrize("n_streams,tables,N,kernel", [
    (2, 1, 10_208, "short_kernel<false, true>"), (2, 1, 10_240, "pipe_kernel<false, 32, true>"),
    (512, 1, 10_239, "short_kernel<false, true>"), (512, 1, 10_251, "pipe_kernel<false, 32, true>"),
    (516, 1, 10_239, "short_kernel<false, true>"), (516, 1, 10_251, "pipe_kernel<false, 16, true>"),
    (1024, 1, 10_208, "short_kernel<false, true>"), (1024, 1, 10_240, "pipe_kernel<false, 16, true>"),
    (256, 4, 12_256, "short_kernel<true, true>"), (256, 4, 12_288, "pipe_kernel<true, 32, true>"),
    (257, 4, 20_448, "short_kernel<true, true>"), (257, 4, 20_480, "pipe_kernel<true, 32, false>"),
    (600, 4, 20_448, "short_kernel<true, false>"), (600, 4, 20_480, "pipe_kernel<true, 16, false>"),
    (1025, 1, 10_208, "pair_kernel<1, true, 4, false>"), (1025, 4, 20_448, "rans_encode_kernel<"),
])
def test_short_units_and_long_ones(oracle, dev, n_streams, tables, N, kernel):
    """Streams below a length take the kernel with four wavefronts, whose start costs less, at any number of units that
    either kernel serves; both sides of each length, also where rows are misaligned and the top group is ragged."""
    s = Streams(oracle, dev, n_streams, N, tables, N + n_streams)
    code, name = s.encode(N)
    assert code == 0 and kernel in name, name


@pytest.mark.parametrize("n_streams,tables,N,kernel", [
    (1028, 1, 32_736, "pair_kernel<1, true, 4, false>"), (1028, 1, 32_768, "pipe_kernel<false, 16, true>"),
    (1792, 1, 32_779, "pipe_kernel<false, 16, true>"), (1028, 4, 49_120, "rans_encode_kernel<"),
    (1028, 4, 49_152, "pipe_kernel<true, 16, false>"), (1537, 4, 49_152, "rans_encode_kernel<"),
    (1793, 4, 49_152, "pipe_kernel<true, 16, false>"), (2304, 4, 49_184, "pipe_kernel<true, 16, false>"),
])
def test_long_units_beyond_a_round(oracle, dev, n_streams, tables, N, kernel):
    """More units than the seven-wavefront kernel takes at any length: where its further rounds win, and where not."""
    test_short_units_and_long_ones(oracle, dev, n_streams, tables, N, kernel)


@pytest.mark.parametrize("n_streams,tables,base,more", [
    (17, 1, 320, [0, 1, 15, 16, 17, 31, 32, 33, 48, 49, 64, 80, 81, 113, 145]), (516, 1, 320, [0, 1, 15, 16, 33]),
    (17, 4, 384, [0, 1, 15, 16, 17, 31, 32, 33, 48, 49, 64, 80, 81, 113, 145]), (260, 4, 640, [0, 1, 16, 17, 33]),
    (516, 4, 640, [0, 1, 15, 16, 33]),
])
def test_long_units_at_the_edges_of_their_batches(oracle, dev, n_streams, tables, base, more):
    """Seven wavefronts, batches of 32 steps and of 16: heads of up to two times 16 groups, a last batch of half its
    steps, and every number of batches left over from whole turns of the rings."""
    for g in more:
        s = Streams(oracle, dev, n_streams, 32 * (base + g), tables, g + tables)
        code, name = s.encode(s.N)
        assert code == 0 and "rans_encode_pipe_kernel" in name, name


@pytest.mark.parametrize("n_streams,tables,N", [
    (3, 1, 10_251), (600, 1, 10_251), (3, 4, 12_320), (300, 4, 20_480), (600, 4, 20_512),  # each form of the long units' kernel
    (600, 1, 5_728), (300, 4, 5_728), (600, 4, 5_728),                                     # and of the short units'
])
def test_word_lists_that_are_too_short_for_few_units(oracle, dev, n_streams, tables, N):
    """Room for fewer words than a stream has: the first words are in place, what lies between the lists is not touched,
    states and counts are the whole stream's, and the shortage is reported."""
    from paper_2604_15356_amd import plc
    s = Streams(oracle, dev, n_streams, N, tables, N + tables)
    least = int(s.enc["n_words"].min())
    for cap in (0, 1, 7, 8, 9, 500, 512, least // 2 // 8 * 8, least // 2 // 8 * 8 + 5, least - 1):
        code, _ = s.encode(cap)
        assert code == plc.PLC_ERR_CAPACITY
