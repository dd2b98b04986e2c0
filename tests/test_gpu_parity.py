"""GPU parity: every entry point of the C ABI against the CPU oracle, element by element, on seeded
inputs.  Sizes span several query/key tiles and ragged tails; the full-size workloads are compared on
sampled rows (each oracle row is independent) and through properties that need no oracle."""
import numpy as np
import pytest

import oracle
from paper_2107_06419_amd import synth
from helpers import check_close, errors, oracle_rows, sample_rows, to_device, to_host_f64

pytestmark = pytest.mark.gpu


def run_entry(entry: str, w: synth.Workload, q, k, v):
    import torch
    import paper_2107_06419_amd as fa
    dq, dk, dv = (to_device(x, w.dtype) for x in (q, k, v))
    out = torch.full_like(dq, float("nan"))
    if entry == "fused":
        (fa.flat_attn_fwd if w.dtype == "bf16" else fa.flat_attn_fwd_f32)(dq, dk, dv, out, w.scale, w.mask)
    elif entry == "unfused":
        nbytes = fa.flat_attn_unfused_workspace_bytes(w.B, w.H, w.N, w.d)
        ws = torch.empty(nbytes // 4, dtype=torch.float32, device="cuda")
        fa.flat_attn_unfused(dq, dk, dv, out, w.scale, w.mask, ws)
    else:
        raise ValueError(entry)
    torch.cuda.synchronize()
    return out


SMALL_SHAPES = [  # (B, H, N)
    (1, 1, 1), (1, 2, 17), (2, 1, 64), (1, 3, 100), (1, 2, 256), (2, 2, 257), (1, 2, 640), (1, 1, 1000), (1, 2, 1536),
]


@pytest.mark.parametrize("B,H,N", SMALL_SHAPES)
@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("mask", [0, 1])
def test_fused_bf16_matches_oracle(B, H, N, d, mask):
    w = synth.custom(f"small_{B}_{H}_{N}_{d}_{mask}", B, H, N, d, "bf16", mask, seed=1000 + N + d + mask)
    q, k, v = synth.make_qkv(w)
    print(f"case fused bf16 {w}", flush=True)
    ref = oracle_rows(w, q, k, v)
    check_close(to_host_f64(run_entry("fused", w, q, k, v)), ref, "bf16", w.name)
    # launches this small take the 128-row shape where the head size has one: the 256-row shape (index 0) that large
    # launches run goes through the same ragged cases explicitly
    import torch
    import paper_2107_06419_amd as fa
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    out = torch.full_like(dq, float("nan"))
    fa.flat_attn_fwd_tile(dq, dk, dv, out, w.scale, w.mask, 0)
    torch.cuda.synchronize()
    check_close(to_host_f64(out), ref, "bf16", w.name + " shape 0")


@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("mask", [0, 1])
def test_fused_cross_many_heads_on_the_256_row_shape(d, mask):
    """Cross-length problems with key counts, ragged in both lengths, with enough heads that flat_attn_fwd_cross takes
    the 256-row shape large launches run (fewer rows take a key-group form or the 128-row shape); d = 32 with the causal mask has no such
    range below 8192 positions and runs its 128-row shape here."""
    import torch
    import paper_2107_06419_amd as fa
    B, H, Nq, Nk = 6, 100, 500, 900
    expect = 1 if (d == 32 and mask == 1) else 0
    assert fa.flat_attn_tile_shape_default(B, H, Nq, d, mask) == expect
    rng = np.random.default_rng(77 + d + mask)
    lens = [int(x) for x in rng.integers(Nq if mask else 1, Nk + 1, size=B)]
    lens[0], lens[1] = Nk, (Nq if mask else 1)

    def rounded(shape, tid):
        x = synth.tensor_f32(shape, 6100 + d + mask, tid, "normal", 1.0)
        return synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(x)).reshape(shape)

    q, k, v = rounded((B, H, Nq, d), 0), rounded((B, H, Nk, d), 1), rounded((B, H, Nk, d), 2)
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    out = torch.full_like(dq, float("nan"))
    scale = float(np.float32(d ** -0.5))
    print(f"case cross many heads d={d} mask={mask} lens={lens}", flush=True)
    fa.flat_attn_fwd_cross(dq, dk, dv, out, scale, mask, torch.tensor(lens, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    ref = oracle.attention_cross(q, k, v, scale, mask, kv_lens=np.array(lens))
    check_close(to_host_f64(out), ref, "bf16", f"cross many heads d={d} mask={mask}")


@pytest.mark.parametrize("B,H,N", SMALL_SHAPES)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("mask", [0, 1])
def test_fused_f32_matches_oracle(B, H, N, d, mask):
    w = synth.custom(f"small_{B}_{H}_{N}_{d}_{mask}", B, H, N, d, "f32", mask, seed=2000 + N + d + mask)
    q, k, v = synth.make_qkv(w)
    print(f"case fused f32 {w}", flush=True)
    got = to_host_f64(run_entry("fused", w, q, k, v))
    check_close(got, oracle_rows(w, q, k, v), "f32", w.name)


@pytest.mark.parametrize("B,H,N", SMALL_SHAPES)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("mask", [0, 1])
def test_unfused_bf16_matches_oracle(B, H, N, d, mask):
    w = synth.custom(f"small_{B}_{H}_{N}_{d}_{mask}", B, H, N, d, "bf16", mask, seed=3000 + N + d + mask)
    q, k, v = synth.make_qkv(w)
    print(f"case unfused bf16 {w}", flush=True)
    got = to_host_f64(run_entry("unfused", w, q, k, v))
    check_close(got, oracle_rows(w, q, k, v), "bf16", w.name)


def test_config0_fp32_full():
    w = synth.WORKLOADS["cfg0_bert_base_f32"]
    q, k, v = synth.make_qkv(w)
    got = to_host_f64(run_entry("fused", w, q, k, v))
    print("cfg0 errors", check_close(got, oracle_rows(w, q, k, v), "f32", w.name), flush=True)


@pytest.mark.parametrize("mask", [0, 1])
@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
def test_peaky_softmax_is_stable(d, mask):
    # Q, K ~ 2 N(0,1): scaled logits have std ~4 (d=128) .. ~2.8, row maxima far above the mean;
    # an implementation without max-subtraction or with a wrong running-max rescale fails here
    w = synth.custom("peaky", 1, 2, 777, d, "bf16", mask, qk_mult=2.0, v_dist="uniform", seed=77 + d)
    q, k, v = synth.make_qkv(w)
    q *= 2.0  # still exactly representable in bf16
    for entry in ("fused", "unfused") if d in (64, 128) else ("fused",):  # the unfused baseline has two head sizes
        got = to_host_f64(run_entry(entry, w, q, k, v))
        check_close(got, oracle_rows(w, q, k, v), "bf16", f"{entry} {w.name}")


def test_scale_zero_gives_uniform_weights():
    w = synth.custom("scale0", 1, 2, 300, 64, "bf16", 1, scale=0.0, seed=5)
    q, k, v = synth.make_qkv(w)
    got = to_host_f64(run_entry("fused", w, q, k, v))
    check_close(got, oracle_rows(w, q, k, v), "bf16", w.name)


FULL = ["cfg1_encoder_4k", "cfg2_long_16k", "cfg3_wide_causal_8k", "cfg4_extreme_64k"]


@pytest.mark.parametrize("name", FULL)
def test_full_size_workload_sampled_rows(name):
    """The launch configuration the benchmark times, compared with the oracle on sampled rows of every head."""
    import torch
    w = synth.WORKLOADS[name]
    print(f"generating {name}", flush=True)
    q, k, v = synth.make_qkv(w)
    out = run_entry("fused", w, q, k, v)
    rows = sample_rows(w.N, 24, seed=w.seed)
    print(f"oracle on {rows.size} rows x {w.B * w.H} heads", flush=True)
    ref = oracle_rows(w, q, k, v, rows=rows)
    got = to_host_f64(out[:, :, torch.from_numpy(rows).cuda(), :])
    print(name, "errors", check_close(got, ref, "bf16", name), flush=True)
    # run-to-run bitwise reproducibility (fixed reduction order, no atomics)
    out2 = run_entry("fused", w, q, k, v)
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16))
    # property that needs no oracle: every output lies in the convex hull of the value rows it may see
    vmax = torch.from_numpy(v).cuda().amax(dim=2, keepdim=True)
    vmin = torch.from_numpy(v).cuda().amin(dim=2, keepdim=True)
    o32 = out.to(torch.float32)
    assert bool((o32 <= vmax + 1e-2).all()) and bool((o32 >= vmin - 1e-2).all())


def test_long_causal_d64_default_and_512_row_shape_match_the_oracle():
    """d = 64, causal, 16 heads x 16384 positions: the one problem class where the 8-wavefront, 512-row tile shape
    measures ahead of index 0.  flat_attn_fwd still runs index 0 (bitwise check); both are compared with the oracle
    on sampled rows at this full size."""
    import torch
    import paper_2107_06419_amd as fa
    w = synth.custom("causal_16k_d64", 1, 16, 16384, 64, "bf16", 1, seed=1664)
    q, k, v = synth.make_qkv(w)
    out = run_entry("fused", w, q, k, v)
    rows = sample_rows(w.N, 24, seed=w.seed, tiles=(32, 64, 256, 512))
    ref = oracle_rows(w, q, k, v, rows=rows)
    drows = torch.from_numpy(rows).cuda()
    check_close(to_host_f64(out[:, :, drows, :]), ref, "bf16", w.name)
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    assert fa.flat_attn_tile_shape_get(64, 3).as_dict()["rows_per_workgroup"] == 512
    for index in (0, 3):
        explicit = torch.full_like(dq, float("nan"))
        fa.flat_attn_fwd_tile(dq, dk, dv, explicit, w.scale, w.mask, index)
        torch.cuda.synchronize()
        if index == 0:
            assert torch.equal(out.view(torch.int16), explicit.view(torch.int16))
        else:
            check_close(to_host_f64(explicit[:, :, drows, :]), ref, "bf16", f"{w.name} shape {index}")


@pytest.mark.parametrize("d,B,H,N,mask,index,wg_rows", [
    (64, 2, 64, 512, 1, 7, 128), (64, 1, 129, 512, 0, 0, 256), (64, 1, 128, 2048, 1, 7, 128), (64, 1, 96, 4096, 1, 0, 256),
    (128, 1, 48, 1024, 1, 2, 128), (128, 1, 40, 1024, 0, 0, 256), (32, 2, 16, 8192, 1, 1, 128), (32, 1, 40, 8192, 0, 0, 256),
    (96, 1, 70, 700, 0, 0, 256), (96, 1, 60, 512, 1, 1, 128),
    # key-group forms: four groups on 32 and on 64 rows, two groups on 64 and on 128 rows
    (64, 1, 12, 512, 0, 12, 32), (96, 1, 12, 640, 1, 2, 32), (32, 1, 12, 512, 0, 2, 32), (32, 1, 12, 1024, 0, 3, 64), (64, 1, 16, 777, 0, 13, 64), (64, 8, 16, 256, 0, 14, 64),
    (128, 1, 12, 1024, 0, 6, 64), (256, 1, 8, 512, 1, 1, 64), (96, 1, 48, 2048, 0, 5, 128), (128, 1, 48, 2048, 0, 7, 128)])
def test_launches_take_the_shape_the_dispatch_names(d, B, H, N, mask, index, wg_rows):
    """flat_attn_fwd's choice of tile shape, from the 256-row shape of large launches to the key-group forms of small ones,
    shown by bitwise equality with that shape run explicitly, and the result compared with the oracle."""
    import torch
    import paper_2107_06419_amd as fa
    w = synth.custom(f"small_{d}_{B}_{H}_{N}_{mask}", B, H, N, d, "bf16", mask, seed=3100 + H + N + mask)
    q, k, v = synth.make_qkv(w)
    out = run_entry("fused", w, q, k, v)
    rows = sample_rows(w.N, 12, seed=w.seed)
    check_close(to_host_f64(out[:, :, torch.from_numpy(rows).cuda(), :]), oracle_rows(w, q, k, v, rows=rows), "bf16", w.name)
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    explicit = torch.full_like(dq, float("nan"))
    fa.flat_attn_fwd_tile(dq, dk, dv, explicit, w.scale, w.mask, index)
    torch.cuda.synchronize()
    assert fa.flat_attn_tile_shape_get(d, index).as_dict()["rows_per_workgroup"] == wg_rows
    assert fa.flat_attn_tile_shape_default(B, H, N, d, mask) == index
    assert torch.equal(out.view(torch.int16), explicit.view(torch.int16))


def test_largest_workload_every_row():
    """The 64K-key workload compared with the oracle on EVERY query row of every head (the sampled test above
    looks at a few dozen rows per head).  The oracle takes the rows in slices and reports after each, so a
    slow host shows progress instead of silence."""
    import sys
    import torch
    w = synth.WORKLOADS["cfg4_extreme_64k"]
    q, k, v = synth.make_qkv(w)
    out = run_entry("fused", w, q, k, v)
    q64, k64, v64 = (x.astype(np.float64) for x in (q, k, v))
    worst_abs, num, den = 0.0, 0.0, 0.0
    step = 4096
    for r0 in range(0, w.N, step):
        rows = np.arange(r0, min(r0 + step, w.N), dtype=np.int64)
        ref = oracle.attention(q64, k64, v64, w.scale, w.mask, rows=rows)
        got = to_host_f64(out[:, :, r0:r0 + rows.size, :])
        check_close(got, ref, "bf16", f"{w.name} rows {r0}..{r0 + rows.size - 1}")  # aggregate of the slice + every row of it
        diff = np.abs(got - ref)
        worst_abs, num, den = max(worst_abs, float(diff.max())), num + float(diff.sum()), den + float(np.abs(ref).sum())
        print(f"{w.name}: rows up to {r0 + rows.size} agree", file=sys.__stderr__, flush=True)
    print(f"{w.name} all rows: max|dO| {worst_abs:.3e}, mean rel {num / den:.3e}", flush=True)
    assert num / den <= 5e-3


@pytest.mark.parametrize("name", ["cfg2_long_16k", "cfg3_wide_causal_8k"])
def test_constant_value_columns_full_size(name):
    """V constant along keys => O equals that constant for any Q, K: checks that the row sum and the
    probabilities fed to the second contraction agree, at full size, with no oracle involved."""
    import torch
    import paper_2107_06419_amd as fa
    w = synth.WORKLOADS[name]
    q, k, _ = synth.make_qkv(w)
    dq, dk = to_device(q, "bf16"), to_device(k, "bf16")
    col = (torch.arange(w.d, device="cuda", dtype=torch.float32) - w.d / 2) / 16.0  # exactly representable in bf16
    dv = col.to(torch.bfloat16).expand(w.B, w.H, w.N, w.d).contiguous()
    out = torch.empty_like(dq)
    fa.flat_attn_fwd(dq, dk, dv, out, w.scale, w.mask)
    torch.cuda.synchronize()
    err = (out.to(torch.float32) - dv.to(torch.float32)).abs().max().item()
    assert err <= 2.0 ** -7 * (w.d / 32.0), err  # one bf16 ulp of the largest |value|


def test_unfused_matches_fused_mid_size():
    """Two structurally different GPU paths on a shape with several tiles per dimension; the oracle on sampled rows."""
    import torch
    for mask, d in ((0, 64), (1, 128)):
        w = synth.custom("mid", 2, 4, 2048 + 96, d, "bf16", mask, seed=31 + d)
        q, k, v = synth.make_qkv(w)
        a = run_entry("fused", w, q, k, v)
        b = run_entry("unfused", w, q, k, v)
        rows = sample_rows(w.N, 16, seed=3)
        ref = oracle_rows(w, q, k, v, rows=rows)
        idx = torch.from_numpy(rows).cuda()
        check_close(to_host_f64(a[:, :, idx, :]), ref, "bf16", "fused mid")
        check_close(to_host_f64(b[:, :, idx, :]), ref, "bf16", "unfused mid")
        print("fused vs unfused", errors(to_host_f64(a), to_host_f64(b)), flush=True)


@pytest.mark.parametrize("N", [1000, 1023, 1028, 4096, 4100, 16384, 16388, 40000])
@pytest.mark.parametrize("mask", [0, 1])
def test_unfused_workspace_holds_the_probabilities(N, mask):
    """On return the workspace is A = softmax_row(L) in fp32 (masked keys exactly 0).  The row lengths
    cover every form of the row-softmax kernel: rows held on chip with 1, 4 and 16 vectors per thread of a
    256-thread workgroup, 16 per thread of a 1024-thread one, and the streaming form (N not a multiple of 4)."""
    import torch
    import paper_2107_06419_amd as fa
    w = synth.custom("probs", 1, 1, N, 64, "bf16", mask, seed=77 + N + mask)
    q, k, v = synth.make_qkv(w)
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    out = torch.empty_like(dq)
    ws = torch.full((N * N,), float("nan"), dtype=torch.float32, device="cuda")
    print(f"case unfused probabilities {w}", flush=True)
    fa.flat_attn_unfused(dq, dk, dv, out, w.scale, w.mask, ws)
    torch.cuda.synchronize()
    rows = sample_rows(N, 6, seed=N)
    got = ws.view(N, N)[torch.from_numpy(rows).cuda()].cpu().numpy().astype(np.float64)
    _, A = oracle.logits_softmax(q[0, 0], k[0, 0], w.scale, w.mask, rows=rows)
    assert np.isfinite(got).all()
    assert np.abs(got - A).max() <= 2e-6, np.abs(got - A).max()      # fp32 exp and an fp32 sum of N terms
    assert np.abs(got.sum(axis=1) - 1.0).max() <= 1e-5
    if mask:
        for r, i in enumerate(rows):
            assert (got[r, i + 1:] == 0.0).all()
    check_close(to_host_f64(out[:, :, torch.from_numpy(rows).cuda(), :]), oracle_rows(w, q, k, v, rows=rows), "bf16", w.name)


@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
def test_every_tile_shape_matches_the_oracle(d):
    """Each tile shape the library is built with is held to the same bar as the default one: a ragged length
    spanning several workgroups and ring trips of the largest shape, with and without the causal mask, and the
    degenerate one-key problem."""
    import torch
    import paper_2107_06419_amd as fa
    count = fa.flat_attn_tile_shape_count(d)
    assert count >= (2 if d in (64, 128) else 1)
    for index in range(count):
        shape = fa.flat_attn_tile_shape_get(d, index).as_dict()
        assert fa.flat_attn_tile_shape_occupancy(d, index) >= 1
        for N, mask in ((1, 0), (77, 1), (1500, 0), (1500, 1)):
            w = synth.custom(f"tile_{d}_{index}_{N}_{mask}", 1, 2, N, d, "bf16", mask, seed=500 + 7 * index + N + mask)
            q, k, v = synth.make_qkv(w)
            dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
            out = torch.full_like(dq, float("nan"))
            print(f"case tile shape {index} {shape} {w}", flush=True)
            fa.flat_attn_fwd_tile(dq, dk, dv, out, w.scale, w.mask, index)
            torch.cuda.synchronize()
            check_close(to_host_f64(out), oracle_rows(w, q, k, v), "bf16", w.name)


CROSS_CASES = [  # (B, H, Nq, Nk, kv_lens)
    (1, 2, 1, 1, None), (2, 2, 1, 777, None), (1, 3, 100, 333, None), (2, 2, 300, 300, None), (1, 2, 640, 1700, None),
    (3, 2, 257, 900, [900, 1, 413]), (2, 1, 1000, 1000, [64, 999]), (2, 2, 70, 2100, [2100, 1031]),
]


@pytest.mark.parametrize("B,H,Nq,Nk,lens", CROSS_CASES)
@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("mask", [0, 1])
def test_fused_cross_matches_oracle(B, H, Nq, Nk, lens, d, mask):
    """Nq queries over Nk keys (one decoding step over a long cache, a segment over segment + memory, ragged
    tails on both sides), with and without per-batch key counts; the padding rows hold huge values that must
    not leak into the result."""
    import torch
    import paper_2107_06419_amd as fa
    seed = 3000 + Nq + 3 * Nk + d + mask
    scale = float(np.float32(d ** -0.5))
    q = synth.tensor_f32((B, H, Nq, d), seed, 0, "normal", 1.0)
    k = synth.tensor_f32((B, H, Nk, d), seed, 1, "normal", 1.0)
    v = synth.tensor_f32((B, H, Nk, d), seed, 2, "normal", 1.0)
    q, k, v = (synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(x)).reshape(x.shape) for x in (q, k, v))
    kv_lens = None
    if lens is not None:
        for b, n in enumerate(lens):
            k[b, :, n:, :] = 3.0e4
            v[b, :, n:, :] = -3.0e4
        kv_lens = torch.tensor(lens, dtype=torch.int32, device="cuda")
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    out = torch.full_like(dq, float("nan"))
    print(f"case cross B={B} H={H} Nq={Nq} Nk={Nk} d={d} mask={mask} lens={lens}", flush=True)
    fa.flat_attn_fwd_cross(dq, dk, dv, out, scale, mask, kv_lens)
    torch.cuda.synchronize()
    ref = oracle.attention_cross(q, k, v, scale, mask, kv_lens=None if lens is None else np.array(lens))
    check_close(to_host_f64(out), ref, "bf16", "cross")


def test_cross_with_equal_lengths_is_bitwise_the_self_attention_entry_point():
    import torch
    import paper_2107_06419_amd as fa
    for d, mask in ((64, 0), (64, 1), (128, 1)):
        w = synth.custom("eq", 2, 3, 1111, d, "bf16", mask, seed=17 + d)
        q, k, v = synth.make_qkv(w)
        dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
        a, b = torch.empty_like(dq), torch.empty_like(dq)
        fa.flat_attn_fwd(dq, dk, dv, a, w.scale, w.mask)
        fa.flat_attn_fwd_cross(dq, dk, dv, b, w.scale, w.mask, None)
        torch.cuda.synchronize()
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


def test_cross_long_cache_full_size_rows():
    """A segment of 2048 queries over 32768 cached positions (d=64, causal): sampled rows against the oracle."""
    import torch
    import paper_2107_06419_amd as fa
    B, H, Nq, Nk, d = 1, 8, 2048, 32768, 64
    scale = 0.125
    q = synth.tensor_f32((B, H, Nq, d), 991, 0, "normal", 1.0)
    k = synth.tensor_f32((B, H, Nk, d), 991, 1, "normal", 1.0)
    v = synth.tensor_f32((B, H, Nk, d), 991, 2, "normal", 1.0)
    q, k, v = (synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(x)).reshape(x.shape) for x in (q, k, v))
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    out = torch.full_like(dq, float("nan"))
    fa.flat_attn_fwd_cross(dq, dk, dv, out, scale, 1, None)
    torch.cuda.synchronize()
    rows = sample_rows(Nq, 24, seed=5)
    ref = oracle.attention_cross(q, k, v, scale, 1, rows=rows)
    check_close(to_host_f64(out[:, :, torch.from_numpy(rows).cuda(), :]), ref, "bf16", "cross long cache")
    assert torch.isfinite(out.float()).all()


def _run_blocksparse(w, q, k, v, offs, ids):
    import torch
    import paper_2107_06419_amd as fa
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    out = torch.full_like(dq, float("nan"))
    d_offs = torch.from_numpy(offs.astype(np.int32)).cuda()
    d_ids = torch.from_numpy((ids if ids.size else np.zeros(1, dtype=np.int64)).astype(np.int32)).cuda()[:ids.size]
    fa.flat_attn_fwd_blocksparse(dq, dk, dv, out, w.scale, d_offs, d_ids)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("B,H,N", [(1, 1, 1), (1, 2, 64), (2, 2, 257), (1, 3, 1000), (2, 2, 2304), (1, 2, 5000)])
@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("keep", [0.5, 0.1])
def test_fused_blocksparse_matches_oracle(B, H, N, d, keep):
    """Random block patterns (256 rows x 64 keys) at 50 % and 10 % density, ragged lengths, several row blocks
    per head and ring trips; the oracle gets the same lists."""
    w = synth.custom(f"sparse_{N}_{d}", B, H, N, d, "bf16", 0, seed=700 + N + d)
    q, k, v = synth.make_qkv(w)
    n_rb, n_kt = -(-N // 256), -(-N // 64)
    offs, ids = synth.random_block_pattern(B * H * n_rb, n_kt, keep, seed=N + d + int(100 * keep))
    print(f"case blocksparse {w} keep={keep} listed={ids.size} of {B * H * n_rb * n_kt}", flush=True)
    out = _run_blocksparse(w, q, k, v, offs, ids)
    ref = oracle.attention_blocksparse(q, k, v, w.scale, offs, ids)
    check_close(to_host_f64(out), ref, "bf16", w.name)


def test_blocksparse_with_every_tile_is_bitwise_the_dense_kernel_and_empty_lists_give_zeros():
    import torch
    import paper_2107_06419_amd as fa
    for d in (32, 64, 96, 128, 256):
        w = synth.custom("sparse_full", 2, 2, 1500, d, "bf16", 0, seed=41 + d)
        q, k, v = synth.make_qkv(w)
        n_rb, n_kt = -(-w.N // 256), -(-w.N // 64)
        n_lists = w.B * w.H * n_rb
        offs = np.arange(n_lists + 1, dtype=np.int64) * n_kt
        ids = np.tile(np.arange(n_kt, dtype=np.int64), n_lists)
        out = _run_blocksparse(w, q, k, v, offs, ids)
        dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
        dense = torch.full_like(dq, float("nan"))
        fa.flat_attn_fwd_tile(dq, dk, dv, dense, w.scale, 0, 0)  # the 256-row shape the block-sparse form is built on
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), dense.view(torch.int16))
        # row block 1 of every head sees nothing, the others only tile 3
        counts = np.ones(n_lists, dtype=np.int64)
        counts[1::n_rb] = 0
        offs = np.concatenate([[0], np.cumsum(counts)])
        ids = np.full(int(counts.sum()), 3, dtype=np.int64)
        out = _run_blocksparse(w, q, k, v, offs, ids)
        assert (out[:, :, 256:512, :].float() == 0).all()
        ref = oracle.attention_blocksparse(q, k, v, w.scale, offs, ids)
        check_close(to_host_f64(out), ref, "bf16", "sparse with empty lists")


def test_blocksparse_lists_out_of_range_are_clamped_not_followed():
    """Garbage lists must not fault: offsets and ids outside their ranges are forced into them on the device."""
    import torch
    w = synth.custom("sparse_bad", 1, 2, 700, 64, "bf16", 0, seed=3)
    q, k, v = synth.make_qkv(w)
    offs = np.array([0, 5, -7, 1 << 30, 2, 9, 9], dtype=np.int64)    # 2 heads x 3 row blocks + 1
    ids = np.array([0, 1 << 20, -5, 3, 10, 2, 2, 7, 11], dtype=np.int64)
    out = _run_blocksparse(w, q, k, v, offs, ids)
    assert out.shape == (1, 2, 700, 64)     # completed; values are unspecified for invalid lists


@pytest.mark.parametrize("mask", [0, 1])
def test_f32_large_problem_sampled_rows(mask):
    """fp32 path on a problem of many whole rounds of workgroups, over which the keys need not be divided; in the small shapes
    above the wavefronts of a workgroup share them."""
    import torch
    w = synth.custom("f32_large", 4, 8, 4096 + 40, 64, "f32", mask, seed=123 + mask)
    q, k, v = synth.make_qkv(w)
    out = run_entry("fused", w, q, k, v)
    rows = sample_rows(w.N, 12, seed=9)
    ref = oracle_rows(w, q, k, v, rows=rows)
    check_close(to_host_f64(out[:, :, torch.from_numpy(rows).cuda(), :]), ref, "f32", w.name)
    assert torch.isfinite(out).all()


def test_fused_entry_points_replay_from_a_hip_graph():
    """The library only enqueues kernels on the caller's stream (no allocation, no host synchronisation, no
    memset), so its calls can be captured.  Each replay is compared bit for bit with the eager result, with
    eager work and synchronisations between the replays."""
    import torch
    import paper_2107_06419_amd as fa
    w = synth.custom("graph", 2, 4, 1300, 64, "bf16", 1, seed=77)
    q, k, v = synth.make_qkv(w)
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    kq = dq[:, :, :300, :].contiguous()
    eager_self, eager_cross = torch.empty_like(dq), torch.empty_like(kq)
    fa.flat_attn_fwd(dq, dk, dv, eager_self, w.scale, 1)
    fa.flat_attn_fwd_cross(kq, dk, dv, eager_cross, w.scale, 1, None)
    torch.cuda.synchronize()
    out_self, out_cross = torch.zeros_like(dq), torch.zeros_like(kq)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            fa.flat_attn_fwd(dq, dk, dv, out_self, w.scale, 1, stream=side)
            fa.flat_attn_fwd_cross(kq, dk, dv, out_cross, w.scale, 1, None, stream=side)
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        out_self.fill_(float("nan"))
        out_cross.fill_(float("nan"))
        scratch = (dq.float() * (rep + 1)).sum()   # unrelated eager work between replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_self.view(torch.int16), eager_self.view(torch.int16)), f"replay {rep}"
        assert torch.equal(out_cross.view(torch.int16), eager_cross.view(torch.int16)), f"replay {rep}"
        assert torch.isfinite(scratch)


def test_many_small_heads_every_entry_point():
    """2000 heads of 33 positions: the grid is all heads, every tile is ragged."""
    w = synth.custom("many_heads", 50, 40, 33, 64, "bf16", 1, seed=8)
    q, k, v = synth.make_qkv(w)
    ref = oracle_rows(w, q, k, v)
    check_close(to_host_f64(run_entry("fused", w, q, k, v)), ref, "bf16", "fused many heads")
    check_close(to_host_f64(run_entry("unfused", w, q, k, v)), ref, "bf16", "unfused many heads")
    wf = synth.custom("many_heads_f32", 50, 40, 33, 64, "f32", 1, seed=8)
    qf, kf, vf = synth.make_qkv(wf)
    check_close(to_host_f64(run_entry("fused", wf, qf, kf, vf)), oracle_rows(wf, qf, kf, vf), "f32", "f32 many heads")


def test_cross_with_more_queries_than_keys():
    import torch
    import paper_2107_06419_amd as fa
    for d in (64, 128):
        q = synth.tensor_f32((2, 2, 700, d), 61, 0, "normal", 1.0)
        k = synth.tensor_f32((2, 2, 100, d), 61, 1, "normal", 1.0)
        v = synth.tensor_f32((2, 2, 100, d), 61, 2, "normal", 1.0)
        q, k, v = (synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(x)).reshape(x.shape) for x in (q, k, v))
        dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
        out = torch.full_like(dq, float("nan"))
        fa.flat_attn_fwd_cross(dq, dk, dv, out, 0.1, 0, None)
        torch.cuda.synchronize()
        check_close(to_host_f64(out), oracle.attention_cross(q, k, v, float(np.float32(0.1)), 0), "bf16", "cross Nq > Nk")
        with pytest.raises(fa.FlatAttnError) as e:
            fa.flat_attn_fwd_cross(dq, dk, dv, out, 0.1, 1, None)   # causal needs Nk >= Nq
        assert e.value.status == -3


def test_randomized_small_problems_all_bf16_entry_points():
    """Seeded random shapes (lengths 1..900, every head size, both masks, random key counts and block patterns)
    through the self-attention, cross-length, block-sparse and unfused entry points, each against the oracle."""
    import random
    import torch
    import paper_2107_06419_amd as fa
    rng = random.Random(20210706)

    def rounded(shape, seed, tid, mult=1.0):
        x = synth.tensor_f32(shape, seed, tid, "normal", mult)
        return synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(x)).reshape(shape)

    for case in range(60):
        B, H, d, mask = rng.randint(1, 3), rng.randint(1, 3), rng.choice([32, 64, 96, 128, 256]), rng.randint(0, 1)
        Nk = rng.choice([1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300, 511, 512, 513, 640, 900])
        Nq = rng.choice([1, 17, 64, 100, 256, 257, Nk]) if rng.random() < 0.5 else Nk
        if mask == 1 and Nq > Nk:
            Nq = Nk
        scale = float(np.float32(rng.choice([0.05, 0.125, 0.3])))
        mult = rng.choice([1.0, 2.0])
        seed = 9000 + case
        q = rounded((B, H, Nq, d), seed, 0, mult)
        k = rounded((B, H, Nk, d), seed, 1, mult)
        v = rounded((B, H, Nk, d), seed, 2)
        lens = [rng.randint(1, Nk) for _ in range(B)] if rng.random() < 0.5 else None
        print(f"case {case}: B={B} H={H} Nq={Nq} Nk={Nk} d={d} mask={mask} scale={scale} mult={mult} lens={lens}", flush=True)
        dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
        out = torch.full_like(dq, float("nan"))
        kv = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
        fa.flat_attn_fwd_cross(dq, dk, dv, out, scale, mask, kv)
        torch.cuda.synchronize()
        ref = oracle.attention_cross(q, k, v, scale, mask, kv_lens=None if lens is None else np.array(lens))
        check_close(to_host_f64(out), ref, "bf16", f"random cross {case}")
        if Nq == Nk and lens is None:
            w = synth.custom("rand", B, H, Nk, d, "bf16", mask, scale=scale, seed=seed)
            out2 = torch.full_like(dq, float("nan"))
            fa.flat_attn_fwd(dq, dk, dv, out2, scale, mask)
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), out2.view(torch.int16))
            out0 = torch.full_like(dq, float("nan"))
            fa.flat_attn_fwd_tile(dq, dk, dv, out0, scale, mask, 0)
            torch.cuda.synchronize()
            check_close(to_host_f64(out0), ref, "bf16", f"random shape 0 {case}")
            if d in (64, 128):
                ws = torch.empty(fa.flat_attn_unfused_workspace_bytes(B, H, Nk, d) // 4, dtype=torch.float32, device="cuda")
                out3 = torch.full_like(dq, float("nan"))
                fa.flat_attn_unfused(dq, dk, dv, out3, scale, mask, ws)
                torch.cuda.synchronize()
                check_close(to_host_f64(out3), ref, "bf16", f"random unfused {case}")
            if mask == 0:
                offs, ids = synth.random_block_pattern(B * H * -(-Nk // 256), -(-Nk // 64), rng.choice([0.3, 0.6, 1.0]), seed=seed)
                got = _run_blocksparse(w, q, k, v, offs, ids)
                check_close(to_host_f64(got), oracle.attention_blocksparse(q, k, v, scale, offs, ids), "bf16", f"random sparse {case}")


def test_status_codes_on_device_buffers():
    import torch
    import paper_2107_06419_amd as fa
    t = torch.zeros(1, 1, 64, 64, dtype=torch.bfloat16, device="cuda")
    o = torch.zeros_like(t)
    with pytest.raises(fa.FlatAttnError) as e:
        fa.flat_attn_fwd(t, t, t, t, 1.0, 0)
    assert e.value.status == -7
    with pytest.raises(fa.FlatAttnError) as e:
        fa.flat_attn_fwd(t, t, t, o, 1.0, 5)
    assert e.value.status == -3
    with pytest.raises(fa.FlatAttnError) as e:
        fa.flat_attn_fwd(t, t, t, o, float("nan"), 0)
    assert e.value.status == -3
    ws = torch.zeros(16, dtype=torch.float32, device="cuda")
    with pytest.raises(fa.FlatAttnError) as e:
        fa.flat_attn_unfused(t, t, t, o, 1.0, 0, ws)
    assert e.value.status == -5
    t80 = torch.zeros(1, 1, 64, 80, dtype=torch.bfloat16, device="cuda")  # a head dimension the library is not built for
    with pytest.raises(fa.FlatAttnError) as e:
        fa.flat_attn_fwd(t80, t80, t80, torch.zeros_like(t80), 1.0, 0)
    assert e.value.status == -3
    t96 = torch.zeros(1, 1, 64, 96, dtype=torch.bfloat16, device="cuda")  # fused: built; unfused baseline: not
    with pytest.raises(fa.FlatAttnError) as e:
        fa.flat_attn_unfused(t96, t96, t96, torch.zeros_like(t96), 1.0, 0, torch.zeros(64 * 64, dtype=torch.float32, device="cuda"))
    assert e.value.status == -3


@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("mask", [0, 1])
def test_reference_max_is_raised_when_logits_grow_along_the_sequence(d, mask):
    """Keys whose logits keep growing with the key index, plus one late key far above everything before
    it: the running reference max must be raised many times (and once by a huge step), with O and the
    row sum rescaled each time."""
    w = synth.custom("grow", 1, 2, 1200, d, "bf16", mask, seed=91 + d)
    q, k, v = synth.make_qkv(w)
    ramp = np.linspace(0.25, 6.0, w.N, dtype=np.float32)[None, None, :, None]
    k = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(k * ramp)).reshape(k.shape)
    q = np.abs(q)                      # keeps q.k correlated with |k|: logits grow along the sequence
    k = np.abs(k)
    k[:, :, 900, :] *= 8.0             # exactly representable; a jump of hundreds of log2 units at key 900
    got = to_host_f64(run_entry("fused", w, q, k, v))
    check_close(got, oracle_rows(w, q, k, v), "bf16", w.name)


def test_host_threads_launching_on_their_own_streams_get_the_single_threaded_results():
    """The library keeps no state between calls apart from once-per-kernel launch attributes, so host threads may
    call it at the same time on different streams.  Each thread runs problems of its own head size (so their first
    launches of a kernel coincide) several times; every result must equal, bit for bit, the one computed alone."""
    import threading
    import torch
    import paper_2107_06419_amd as fa
    jobs = []
    for t, (d, N, mask) in enumerate([(64, 1333, 0), (128, 900, 1), (32, 2050, 1), (96, 777, 0), (256, 640, 1), (64, 4100, 1)]):
        w = synth.custom(f"thread_{t}", 1, 3, N, d, "bf16", mask, seed=8800 + t)
        q, k, v = synth.make_qkv(w)
        jobs.append((w, [to_device(x, "bf16") for x in (q, k, v)]))
    alone = []
    for w, (dq, dk, dv) in jobs:
        out = torch.empty_like(dq)
        fa.flat_attn_fwd(dq, dk, dv, out, w.scale, w.mask)
        alone.append(out)
    torch.cuda.synchronize()
    results = [[] for _ in jobs]
    errors = []

    def worker(i):
        try:
            w, (dq, dk, dv) = jobs[i]
            stream = torch.cuda.Stream()
            stream.wait_stream(torch.cuda.default_stream())
            with torch.cuda.stream(stream):  # the poison fill and the call share the stream
                for _ in range(8):
                    out = torch.full_like(dq, float("nan"))
                    fa.flat_attn_fwd(dq, dk, dv, out, w.scale, w.mask, stream=stream)
                    results[i].append(out)
            stream.synchronize()
        except Exception as e:  # noqa: BLE001  (reported by the main thread)
            errors.append((i, repr(e)))

    threads = [threading.Thread(target=worker, args=(i,)) for i in range(len(jobs))]
    for th in threads:
        th.start()
    for th in threads:
        th.join(timeout=100)
        assert not th.is_alive(), "a launching thread did not finish"
    assert not errors, errors
    torch.cuda.synchronize()
    for i, outs in enumerate(results):
        assert len(outs) == 8
        for out in outs:
            assert torch.equal(out.view(torch.int16), alone[i].view(torch.int16)), f"thread {i}"
