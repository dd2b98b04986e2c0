"""The work whose speed this repository is judged by: calls of the public entry points of paper_2107_06419_amd, from the
smallest launch to the longest sequence.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) device tensors (and the workspace a caller keeps) for one case
    run(state)          one call, as a program that uses the library makes it; returns the output tensor
    work(case)          bytes and flops the call cannot do without
    tolerance(case)     how far two correct implementations of the same precision may be apart

The unfused GEMM -> softmax -> GEMM entry point is not here: it exists as the comparison baseline of the fused dataflow.
"""
import numpy as np
import torch

import paper_2107_06419_amd as fa
from paper_2107_06419_amd import binding, synth


def _case(name, entry, B, H, Nq, Nk, d, mask=0, dtype="bf16", lens=False, keep=1.0, qk_mult=1.0, v_dist="normal"):
    case = {"entry": entry, "B": B, "H": H, "Nq": Nq, "Nk": Nk, "d": d, "mask": mask, "dtype": dtype, "lens": lens,
            "keep": keep, "qk_mult": qk_mult, "v_dist": v_dist}
    return {"name": name, **case} if name else case


def listed():
    return [
        # one request to a BERT-base-sized encoder, 512 tokens: a launch that is mostly latency, in both precisions
        _case("bert_512_bf16", "self", 1, 12, 512, 512, 64),
        _case("bert_512_f32", "self", 1, 12, 512, 512, 64, dtype="f32"),
        # the same encoder over a batch of 64 requests: many short sequences
        _case("batch_512", "self", 64, 12, 512, 512, 64),
        # one long document (the benchmark's headline workload)
        _case("long_16k", "self", 1, 16, 16384, 16384, 64),
        # the longest sequence of the benchmark's set
        _case("extreme_64k", "self", 1, 8, 65536, 65536, 64),
        # causal prefill with wide heads and a peaky softmax (the benchmark's causal workload)
        _case("wide_causal_8k", "self", 2, 8, 8192, 8192, 128, mask=1, qk_mult=2.0, v_dist="uniform"),
        # causal prefill of an odd length with the widest heads
        _case("ragged_causal_d256", "self", 2, 8, 3001, 3001, 256, mask=1),
        # a decoder's cross attention over a padded batch: odd lengths, a key count for every batch entry
        _case("cross_padded", "cross", 16, 12, 250, 1011, 64, lens=True),
        # one new position over a very long cache
        _case("decode_64k", "splitkv", 1, 16, 1, 65536, 64, mask=1),
        # one new position for each request of a batch, caches of different lengths, wide heads
        _case("decode_batch", "splitkv", 16, 16, 1, 4001, 128, lens=True),
        # half of the 256 x 64 blocks pruned at random
        _case("sparse_16k", "blocksparse", 1, 16, 16384, 16384, 64, keep=0.5),
        # training-precision causal attention of a few thousand positions
        _case("causal_2k_f32", "self", 2, 8, 2049, 2049, 128, mask=1, dtype="f32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


MAX_FLOPS = {"bf16": 4e12, "f32": 2e11}  # of a drawn case; the largest listed ones need 8.8e12 and 2e10
MAX_BYTES = 1 << 30


def draw(rng):
    while True:
        entry = rng.choice(("self", "self", "self", "cross", "splitkv", "splitkv", "blocksparse", "f32"))
        d = rng.choice((64, 64, 128, 128, 32, 96, 256))
        H = rng.choice((1, 2, 4, 8, 12, 16, 16, 25, 32))
        if entry == "self":
            N = _log_int(rng, 64, 49152)
            case = _case("", entry, _log_int(rng, 1, 64), H, N, N, d, mask=rng.randrange(2), qk_mult=rng.choice((1.0, 1.0, 2.0)))
        elif entry == "f32":
            N = _log_int(rng, 32, 6000)
            case = _case("", "self", _log_int(rng, 1, 32), H, N, N, rng.choice((64, 128)), mask=rng.randrange(2), dtype="f32")
        elif entry == "cross":
            Nk = _log_int(rng, 64, 16384)
            Nq = min(Nk, _log_int(rng, 16, 4096))
            case = _case("", entry, _log_int(rng, 1, 32), H, Nq, Nk, d, mask=rng.randrange(2), lens=rng.random() < 0.5)
        elif entry == "splitkv":
            Nk = _log_int(rng, 512, 131072)
            Nq = min(Nk, rng.choice((1, 1, 1, _log_int(rng, 2, 64), _log_int(rng, 64, 300))))
            case = _case("", entry, _log_int(rng, 1, 64), H, Nq, Nk, d, mask=rng.randrange(2), lens=rng.random() < 0.5)
        else:
            N = _log_int(rng, 1024, 32768)
            case = _case("", entry, _log_int(rng, 1, 4), H, N, N, d, keep=round(rng.uniform(0.1, 0.9), 2))
        w = work(case)
        if w["flops"] <= MAX_FLOPS[case["dtype"]] and w["bytes"] <= MAX_BYTES:
            return case


def _key_counts(case):
    """Key counts of the batch entries in ascending order: evenly spread from half the keys to all of them."""
    B, Nk = case["B"], case["Nk"]
    if not case["lens"]:
        return np.full(B, Nk, dtype=np.int64)
    return np.linspace((Nk + 1) // 2, Nk, B).astype(np.int64) if B > 1 else np.array([(3 * Nk + 3) // 4], dtype=np.int64)


def prepare(case, seed):
    B, H, Nq, Nk, d = (case[k] for k in ("B", "H", "Nq", "Nk", "d"))
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(n, mult):
        return torch.randn(B, H, n, d, generator=gen, device="cuda").mul_(mult).to(dtype)

    q, k = normal(Nq, case["qk_mult"]), normal(Nk, case["qk_mult"])
    if case["v_dist"] == "uniform":
        v = torch.rand(B, H, Nk, d, generator=gen, device="cuda").mul_(2.0).sub_(1.0).to(dtype)
    else:
        v = normal(Nk, 1.0)
    state = {"entry": case["entry"], "dtype": case["dtype"], "q": q, "k": k, "v": v, "o": torch.empty_like(q),
             "scale": float(np.float32(d ** -0.5)), "mask": case["mask"], "lens": None}
    if case["lens"]:
        order = np.random.RandomState(int(seed) & 0x7fffffff).permutation(B)
        state["lens"] = torch.from_numpy(_key_counts(case)[order].astype(np.int32)).cuda()
    if case["entry"] == "splitkv":  # a serving loop keeps its workspace
        nbytes = fa.flat_attn_fwd_splitkv_workspace_bytes(B, H, Nq, Nk, d, 0)
        state["workspace"] = torch.empty((nbytes + 3) // 4, dtype=torch.float32, device="cuda")
    if case["entry"] == "blocksparse":
        rows, keys = binding.FLAT_SPARSE_BLOCK_ROWS, binding.FLAT_SPARSE_BLOCK_KEYS
        offs, ids = synth.random_block_pattern(B * H * -(-Nq // rows), -(-Nk // keys), case["keep"], int(seed) & 0x7fffffff)
        state["offsets"] = torch.from_numpy(offs.astype(np.int32)).cuda()
        state["ids"] = torch.from_numpy(ids.astype(np.int32)).cuda()
    return state


def run(state):
    q, k, v, o, scale, mask = (state[n] for n in ("q", "k", "v", "o", "scale", "mask"))
    entry = state["entry"]
    if entry == "self":
        (fa.flat_attn_fwd_f32 if state["dtype"] == "f32" else fa.flat_attn_fwd)(q, k, v, o, scale, mask)
    elif entry == "cross":
        fa.flat_attn_fwd_cross(q, k, v, o, scale, mask, state["lens"])
    elif entry == "splitkv":
        fa.flat_attn_fwd_splitkv(q, k, v, o, scale, mask, state["lens"], 0, state["workspace"])
    else:
        fa.flat_attn_fwd_blocksparse(q, k, v, o, scale, state["offsets"], state["ids"])
    return o


def work(case):
    """Q and the keys and values that count read once, O written once; two products over the visible (query, key) pairs."""
    B, H, Nq, Nk, d = (case[k] for k in ("B", "H", "Nq", "Nk", "d"))
    counts = _key_counts(case)
    if case["mask"]:  # query i sees keys 0 .. i + Nk - Nq of those that count
        pairs = sum(int(np.minimum(n, np.arange(Nq, dtype=np.int64) + (Nk - Nq) + 1).sum()) for n in counts)
    else:
        pairs = Nq * int(counts.sum())
    elem = 4 if case["dtype"] == "f32" else 2
    return {"bytes": float(elem * H * d * (2 * B * Nq + 2 * int(counts.sum()))), "flops": 4.0 * H * d * pairs * case["keep"]}


def tolerance(case):
    # Measured against softmax(Q K^T scale) V in 64 bits over the listed cases and a dozen drawn ones: bf16 2.8e-3 (2-norm) and
    # 1.1e-2 (largest element), from rounding P and O; f32 3.6e-7 and 3.5e-6.  About four times that is allowed.
    if case["dtype"] == "f32":
        return {"rel": 1.5e-6, "max": 1.5e-5}
    return {"rel": 1e-2, "max": 4.5e-2}
