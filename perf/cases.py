"""Workloads that stand for what a user of this package has it do: caches of KV vectors, coded and decoded through
paper_2604_15356_amd.codec.

A case names the path ("mean": the weighted-mean predictor; "cond": token-conditional coding; "adapt": the
surprisal-adaptive quantiser on top of it; "linear": the linear-embedding predictor), the direction ("encode",
"decode", or "both" one after the other, which is what a cache that is evicted and restored goes through), the shape
(S sessions, L layers, H KV heads, n positions, k candidates, d components) and the options in use: rANS units of
`chunk` symbols instead of whole streams, candidates stored heads innermost, positions whose token is none of the
candidates.  listed() are fixed points, most of them this repository's own configurations; draw() gives others of
the same ranges.
"""
import math

import torch

from paper_2604_15356_amd import plc
from paper_2604_15356_amd.codec import KVDeltaCodec

VOCAB = 50_000
ADAPT_B0, ADAPT_HBAR, ADAPT_RANGE = 3.0, math.log2(15.0), 0.32

_BASE = dict(path="mean", what="both", S=1, chunk=0, heads_inner=False, misses=False, sigma=0.05, delta=0.02)


def _case(**kw):
    return {**_BASE, **kw}


def listed():
    return [
        # the smallest: one short cache of a small model, where latency and the number of launches count
        _case(name="tiny", L=2, H=4, n=512, k=4, d=64),
        # sizes nobody tuned for: three sessions, odd counts, rows that are no power of two, heads innermost
        _case(name="ragged", S=3, L=7, H=5, n=777, k=5, d=80, heads_inner=True),
        # an ordinary cache of one session at 4096 positions, each direction by itself
        _case(name="llama8b_encode", what="encode", L=32, H=8, n=4096, k=8, d=128),
        _case(name="llama8b_decode", what="decode", L=32, H=8, n=4096, k=8, d=128),
        # the same cache in independent rANS units of 4096 symbols: random access, and the coder in parallel
        _case(name="llama8b_chunked", L=32, H=8, n=4096, k=8, d=128, chunk=4096),
        # a long context: few streams, each of eight million symbols
        _case(name="long", L=32, H=8, n=32768, k=4, d=128, sigma=0.03),
        # a large model: thousands of streams
        _case(name="70b", L=80, H=64, n=2048, k=4, d=128, sigma=0.08, delta=0.03),
        # a serving batch: a quarter of the 64-session sweep, which with its buffers fills the card
        _case(name="sessions16", S=16, L=32, H=8, n=2048, k=8, d=128, sigma=0.1),
        # many candidates, some tokens outside them
        _case(name="misses_k20", L=32, H=8, n=4096, k=20, d=128, misses=True),
        # coding given the tokens
        _case(name="conditional", path="cond", L=32, H=8, n=4096, k=8, d=128),
        # and with a bit depth per position
        _case(name="adaptive", path="adapt", L=32, H=8, n=4096, k=8, d=128),
        # prediction as two dense contractions over the vocabulary and the embedding
        _case(name="linear", path="linear", L=32, H=8, n=4096, k=1, d=128, V=50016, m=4096),
    ]


_MOST_WORK = 8.6e10   # bytes of one pass: that of "sessions16"
_MOST_STATE = 5.0e10  # bytes of inputs and buffers: about that of "sessions16"
_MOST_FLOPS = 7.8e12  # of one pass: that of "linear"


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        path = rng.choice(["mean", "mean", "mean", "cond", "adapt", "linear"])
        case = _case(path=path, what=rng.choice(["encode", "decode", "both"]), S=_log_int(rng, 1, 16),
                     L=_log_int(rng, 1, 80), H=_log_int(rng, 1, 64), n=_log_int(rng, 32, 32768),
                     k=rng.choice([1, 2, 3, 4, 4, 5, 6, 8, 8, 10, 12, 16, 20, 32]),
                     d=rng.choice([64, 64, 128, 128, 128, 256, 80, 96, 112, 192, 40, 72]),
                     sigma=rng.uniform(0.01, 0.2), delta=rng.choice([0.02, 0.03]))
        if path == "linear":
            # whole tiles of 128 positions and 128 components, any vocabulary that is a multiple of 32
            case.update(S=rng.choice([1, 1, 2]), H=2 * max(1, case["H"] // 8), d=rng.choice([64, 128]), k=1,
                        n=128 * _log_int(rng, 1, 32), V=32 * _log_int(rng, 32, 2048), m=128 * _log_int(rng, 1, 32))
        else:
            case["chunk"] = rng.choice([0, 0, 0, 1024, 4096, 8192])
            case["heads_inner"] = rng.random() < 0.25
            case["misses"] = case["k"] > 1 and rng.random() < 0.25
            if path == "adapt" and case["d"] % 16:
                case["d"] += 8  # a position holds a multiple of 32 symbols
        w = work(case)
        if w["bytes"] <= _MOST_WORK and w["flops"] <= _MOST_FLOPS and 2e5 <= _components(case) \
                and _state_bytes(case) <= _MOST_STATE:
            return case


def _components(c):
    return 2 * c["S"] * c["L"] * c["H"] * c["n"] * c["d"]


def _state_bytes(c):
    # candidates, actual and reconstructed vectors, two sets of symbols, words, escapes
    per = 2 * c["k"] + 2 + 2 + 2 + 2 + 0.3
    if c["path"] == "linear":
        per += 2
    return per * _components(c)


def _coded_bytes(c):
    """Bytes of coded words per component, about: what the paths' entropies come to on these inputs."""
    return {"mean": 0.92, "cond": 0.43, "adapt": 0.17, "linear": 0.92}[c["path"]]


def work(case):
    """One pass reads its candidates (or the one named candidate per position) and the actual vectors and writes
    symbols and words; back, it reads candidates and words and writes symbols and vectors."""
    c = case
    E, both = _components(c), 2 if c["what"] == "both" else 1
    if c["path"] == "linear":
        rows, m, V, N = c["S"] * c["n"], c["m"], c["V"], 2 * c["H"] * c["d"]
        flops = 2.0 * rows * V * m + 2.0 * rows * N * m * c["L"]
        operands = 2.0 * (rows * V + m * V + 2 * rows * m + c["L"] * N * m)
        return {"bytes": both * (operands + E * (2 + 2 + 1 + _coded_bytes(c))), "flops": both * flops}
    cand = 2 * c["k"] if c["path"] == "mean" else 2
    return {"bytes": both * E * (cand + 2 + 1 + _coded_bytes(c)), "flops": both * E * (2.0 * (c["k"] if c["path"] == "mean" else 1) + 4)}


def tolerance(case):
    """Symbols, tables, states and words are whole numbers that decode only if they are exactly these, and the
    prediction's fp32 operations are prescribed one by one.  The contractions of the linear predictor may add in
    any order: an fp16 expected embedding or a residual that lies at a rounding tie then takes its neighbour, a
    symbol's being one step (0.02 or 0.03 against values of root mean square 1.4) away.  With the vocabulary and the
    embedding permuted, "linear" shows 3.3e-4, 0.014 and 5.3e-4 of the symbols; the bounds are four times that."""
    if case["path"] != "linear":
        return "exact"
    return {"rel": 1.3e-3, "max": 0.06, "differ": 2e-3}


def exact(case, seed):
    """The linear predictor's outputs from sums in 64 bits (the expected embedding passes from one contraction to
    the next in fp16: that is the path's definition).  None elsewhere: the outputs are exact already."""
    c = dict(case)
    if c["path"] != "linear":
        return None
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    st = _prepare_linear(c, gen, dev)
    S, L, H, n, d, m = (c[x] for x in ("S", "L", "H", "n", "d", "m"))
    embed = st["embed_t"].double().t()
    ebar = torch.cat([st["probs_full"][r0:r0 + 512].double() @ embed for r0 in range(0, S * n, 512)])
    out = {} if c["what"] == "decode" else {"ebar": ebar, "symbols": None}
    if c["what"] == "encode":
        return out
    delta = float(torch.tensor(c["delta"], dtype=torch.float32))
    mid = ebar.to(torch.float16).double().reshape(S, n, m)
    back = [torch.empty((S, L, H, n, d), dtype=torch.float64, device=dev) for _ in range(2)]
    for s in range(S):
        for l in range(L):
            lin = (mid[s] @ st["A"][l].reshape(2 * H * d, m).double().t()).reshape(n, H, 2, d).permute(1, 2, 0, 3)
            for i, x in enumerate(("k", "v")):
                pred = lin[:, i] + st["bias_" + x][s, l].double()
                act = st["act_" + x][s, l].double()
                q = torch.round((act - pred) / delta)
                back[i][s, l] = torch.where(q.abs() <= 127, pred + q * delta, act)
    out.update(out_k=back[0], out_v=back[1], decoded=None)
    return out


# ---------------------------------------------------------------------------------------------------------------

def _zipf_exponents(S, gen, dev):
    # Zipf exponents at which a vocabulary of 50,000 has perplexities of about 40 down to 5
    return torch.rand(S, generator=gen, device=dev) * (1.75 - 1.3) + 1.3


def _draw_probs(c, gen, dev):
    """Raw top-k probabilities fp32 [S, n, k], descending on average and different at every position, and the index
    of every position's token among them (-1: none)."""
    S, n, k = c["S"], c["n"], c["k"]
    s = _zipf_exponents(S, gen, dev)
    ranks = torch.arange(1, VOCAB + 1, device=dev, dtype=torch.float32)
    full = ranks[None, :] ** -s[:, None]
    head = (full[:, :k] / full.sum(-1, keepdim=True))[:, None, :]
    p = torch.empty((S, n, k), device=dev).exponential_(generator=gen).add_(0.05) * head
    p = (p * (head.sum(-1, keepdim=True) / p.sum(-1, keepdim=True))).contiguous()
    chosen = torch.multinomial(p.reshape(S * n, k), 1, generator=gen).reshape(S, n)
    if c["misses"]:
        miss = torch.rand((S, n), generator=gen, device=dev) < 1.0 - p.sum(-1)
        chosen = torch.where(miss, torch.full_like(chosen, -1), chosen)
    return p, chosen.to(torch.int32)


def _empty_cand(c, dev):
    S, L, H, n, k, d = (c[x] for x in "SLHnkd")
    if c["heads_inner"]:
        return torch.empty((S, L, n, k, H, d), dtype=torch.float16, device=dev).permute(0, 1, 4, 2, 3, 5)
    return torch.empty((S, L, H, n, k, d), dtype=torch.float16, device=dev)


def _draw_vectors(c, chosen, gen, dev):
    """Candidates ~ N(0, 1); the actual vector is the token's candidate plus noise (a fresh draw for a miss)."""
    S, L, H, n, k, d = (c[x] for x in "SLHnkd")
    out = []
    for _ in range(2):
        cand = _empty_cand(c, dev)
        act = torch.empty((S, L, H, n, d), dtype=torch.float16, device=dev)
        for s in range(S):
            pick = chosen[s].long().clamp(min=0)
            at = torch.arange(n, device=dev)
            for l in range(L):
                view = cand[s, l]  # [H, n, k, d]
                view.permute(1, 2, 0, 3).normal_(generator=gen) if c["heads_inner"] else view.normal_(generator=gen)
                true = view[:, at, pick].float()
                if c["misses"]:
                    true = torch.where((chosen[s] < 0)[None, :, None], torch.randn((H, n, d), generator=gen, device=dev), true)
                act[s, l].copy_(true.add_(torch.randn((H, n, d), generator=gen, device=dev), alpha=c["sigma"]))
        out += [cand, act]
    return out


def _codec(c, dev, **kw):
    codec = KVDeltaCodec(c["S"], c["L"], c["H"], c["n"], c["k"], c["d"], c["delta"], chunk_syms=c["chunk"], device=dev, **kw)
    # what an encode leaves unwritten (behind the last word of a unit and the last escape) is always the same
    codec.words.zero_()
    codec.esc_vals.zero_()
    codec.idx_words.zero_()
    return codec


def _prepare_linear(c, gen, dev):
    S, L, H, n, d, m, V = (c[x] for x in ("S", "L", "H", "n", "d", "m", "V"))
    rows = S * n
    # every position ranks the vocabulary its own way: the Zipf row, rotated
    zipf = torch.arange(1, V + 1, device=dev, dtype=torch.float32) ** -1.5
    zipf = zipf / zipf.sum()
    # (drawn through a distribution function summed on the host: torch.multinomial sums on the device, in an order
    # that changes from call to call, and a token at the edge of two would change with it)
    cdf = zipf.double().cpu().cumsum(0).to(dev)
    draws = torch.rand(rows, generator=gen, device=dev, dtype=torch.float64) * cdf[-1]
    token = torch.searchsorted(cdf, draws, right=True).clamp_(max=V - 1)
    shift = torch.randint(0, V, (rows,), generator=gen, device=dev)
    twice = torch.cat([zipf, zipf]).to(torch.float16)
    probs_full = torch.empty((rows, V), dtype=torch.float16, device=dev)
    at = torch.arange(V, device=dev)
    for r0 in range(0, rows, 512):
        probs_full[r0:r0 + 512] = twice[at[None, :] + shift[r0:r0 + 512, None]]
    token = (token - shift) % V
    st = {"probs_full": probs_full}
    st["embed_t"] = torch.empty((m, V), dtype=torch.float16, device=dev).normal_(generator=gen)
    st["A"] = torch.empty((L, H, 2, d, m), dtype=torch.float16, device=dev).normal_(generator=gen).mul_(m ** -0.5)
    for x in ("k", "v"):
        st["bias_" + x] = torch.empty((S, L, H, n, d), dtype=torch.float16, device=dev).normal_(generator=gen)
        st["act_" + x] = torch.empty((S, L, H, n, d), dtype=torch.float16, device=dev)
    e_true = st["embed_t"][:, token].t().contiguous().reshape(S, n, m)
    for s in range(S):
        for l in range(L):
            lin = (e_true[s] @ st["A"][l].reshape(2 * H * d, m).t()).reshape(n, H, 2, d).permute(1, 2, 0, 3).float()
            for i, x in enumerate(("k", "v")):
                z = torch.randn((H, n, d), generator=gen, device=dev)
                st["act_" + x][s, l].copy_(lin[:, i] + st["bias_" + x][s, l] + c["sigma"] * z)
    return st


def prepare(case, seed):
    """Inputs, made on the GPU from the seed, and the codec with its buffers; to decode, a cache that this codec
    has encoded."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    c = dict(case)
    st = {"case": c}
    if c["path"] == "linear":
        st.update(_prepare_linear(c, gen, dev))
        st["codec"] = _codec(c, dev)
    else:
        st["probs"], st["chosen"] = _draw_probs(c, gen, dev)
        st["cand_k"], st["act_k"], st["cand_v"], st["act_v"] = _draw_vectors(c, st["chosen"], gen, dev)
        st["codec"] = _codec(c, dev, cand_stride=st["cand_k"].stride()[:5], act_stride=st["act_k"].stride()[:4])
    if c["path"] == "adapt":
        st["thr"] = plc.surprisal_thresholds(ADAPT_B0, ADAPT_HBAR)
    if c["what"] != "encode":
        st["out_k"], st["out_v"] = torch.zeros_like(st["act_k"]), torch.zeros_like(st["act_v"])
    if c["what"] == "decode":
        _encode(st)
        st["codec"].check_status("encode")
    return st


def _encode(st):
    codec, path = st["codec"], st["case"]["path"]
    if path == "linear":
        return codec.encode_linear(st["probs_full"], st["embed_t"], st["A"], st["bias_k"], st["bias_v"], st["act_k"], st["act_v"])
    vectors = (st["cand_k"], st["cand_v"], st["probs"], st["act_k"], st["act_v"])
    if path == "mean":
        return codec.encode(*vectors)
    if path == "cond":
        return codec.encode_cond(*vectors, chosen=st["chosen"])
    return codec.encode_adapt(*vectors, st["chosen"], st["thr"], ADAPT_RANGE)


def _decode(st):
    codec, path = st["codec"], st["case"]["path"]
    if path == "linear":
        codec.decode_linear(st["probs_full"], st["embed_t"], st["A"], st["bias_k"], st["bias_v"], st["out_k"], st["out_v"])
        return
    vectors = (st["cand_k"], st["cand_v"], st["probs"], st["out_k"], st["out_v"])
    if path == "mean":
        codec.decode(*vectors)
    elif path == "cond":
        codec.decode_cond(*vectors)
    else:
        codec.decode_adapt(*vectors, st["thr"], ADAPT_RANGE)


def run(state):
    st, codec = state, state["codec"]
    path, what = st["case"]["path"], st["case"]["what"]
    out = {}
    if what != "decode":
        coded = _encode(st)
        if path == "linear":
            # (a symbol that a tie moves shifts every word behind it: words, states and tables are compared through
            # what they decode to)
            out = {"ebar": codec.ebar, "symbols": coded.symbols}
        else:
            names = ["symbols", "esc_vals", "esc_cnt", "esc_off", "states", "words", "n_words"]
            if path == "adapt":
                names += ["counts_d", "freq_d", "bits"]
            else:
                names += ["counts", "freq", "cum"]
            if path != "mean":
                names += ["idx_states", "idx_words", "idx_n_words"]
            out = {x: getattr(coded, x) for x in names}
    if what != "encode":
        _decode(st)
        out.update(out_k=st["out_k"], out_v=st["out_v"], decoded=codec.dec_symbols)
        if path in ("cond", "adapt"):
            out["tokens"] = codec.dec_chosen
    return out
