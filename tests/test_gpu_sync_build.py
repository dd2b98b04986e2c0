"""Hazard check of the fused bf16 kernel's LDS ring.  The release kernel keeps streaming loads in flight across
steps, waits for them with hand-counted vmcnt values and publishes a tile with a single barrier.  A second build
of the same source (FLAT_SYNC_EVERY_PHASE) awaits every load in full and fences every phase with barriers.  If
the release build's synchronisation were too weak anywhere, the two would differ; they must agree bit for bit."""
import ctypes
import os

import numpy as np
import pytest

import paper_2107_06419_amd as fa
from paper_2107_06419_amd import synth
from helpers import to_device

pytestmark = pytest.mark.gpu

SYNC_LIB = os.path.join(os.path.dirname(fa.library_path()), "libflat_attn_sync.so")


def _sync_lib():
    if not os.path.exists(SYNC_LIB):
        pytest.fail(f"{SYNC_LIB} not built: run `python -c 'import __graft_entry__ as g; g.build()'`")
    import torch  # noqa: F401  (same HIP runtime as the tensors)
    lib = ctypes.CDLL(SYNC_LIB)
    vp, i, f = ctypes.c_void_p, ctypes.c_int, ctypes.c_float
    lib.flat_attn_fwd.restype = i
    lib.flat_attn_fwd.argtypes = [vp, vp, vp, vp, i, i, i, i, f, i, vp]
    lib.flat_attn_fwd_cross.restype = i
    lib.flat_attn_fwd_cross.argtypes = [vp, vp, vp, vp, i, i, i, i, i, f, i, vp, vp]
    return lib


def _both(w, q, k, v):
    import torch
    lib = _sync_lib()
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    rel = torch.full_like(dq, float("nan"))
    chk = torch.full_like(dq, float("nan"))
    fa.flat_attn_fwd(dq, dk, dv, rel, w.scale, w.mask)
    st = torch.cuda.current_stream().cuda_stream
    rc = lib.flat_attn_fwd(dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), chk.data_ptr(), w.B, w.H, w.N, w.d, w.scale, w.mask, st)
    assert rc == 0
    torch.cuda.synchronize()
    return rel, chk


@pytest.mark.parametrize("name", ["cfg2_long_16k", "cfg3_wide_causal_8k"])
def test_release_and_fully_synchronised_builds_agree_at_full_size(name):
    import torch
    w = synth.WORKLOADS[name]
    q, k, v = synth.make_qkv(w)
    print(f"case sync build {name}", flush=True)
    rel, chk = _both(w, q, k, v)
    assert torch.isfinite(rel.float()).all()
    assert torch.equal(rel.view(torch.int16), chk.view(torch.int16))


@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("mask", [0, 1])
def test_release_and_fully_synchronised_builds_agree_on_ragged_shapes(d, mask):
    import torch
    for B, H, N in ((1, 2, 33), (2, 3, 1777), (1, 1, 4100)):
        w = synth.custom(f"sync_{d}_{mask}_{N}", B, H, N, d, "bf16", mask, seed=4242 + d + mask + N)
        q, k, v = synth.make_qkv(w)
        print(f"case sync build {w}", flush=True)
        rel, chk = _both(w, q, k, v)
        assert torch.isfinite(rel.float()).all()
        assert torch.equal(rel.view(torch.int16), chk.view(torch.int16))


@pytest.mark.parametrize("H,Nq,Nk", [(4, 300, 9000), (300, 500, 3000)])
def test_release_and_fully_synchronised_builds_agree_on_cached_keys(H, Nq, Nk):
    """Few queries over many keys with per-batch key counts: short row blocks, long rings.  With 4 heads the launch takes
    a key-group form, with 300 heads the 256-row shape of large launches."""
    import torch
    lib = _sync_lib()
    B, d = 2, 64
    assert fa.flat_attn_tile_shape_default(B, H, Nq, d, 1) == (12 if H == 4 else 0)
    q = synth.tensor_f32((B, H, Nq, d), 77, 0)
    k = synth.tensor_f32((B, H, Nk, d), 77, 1)
    v = synth.tensor_f32((B, H, Nk, d), 77, 2)
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    lens = torch.tensor([Nk, Nk // 2 + 1], dtype=torch.int32, device="cuda")
    rel, chk = torch.full_like(dq, float("nan")), torch.full_like(dq, float("nan"))
    for mask in (0, 1):
        fa.flat_attn_fwd_cross(dq, dk, dv, rel, 0.125, mask, lens)
        rc = lib.flat_attn_fwd_cross(dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), chk.data_ptr(), B, H, Nq, Nk, d, 0.125, mask,
                                     lens.data_ptr(), torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        torch.cuda.synchronize()
        assert torch.isfinite(rel.float()).all()
        assert torch.equal(rel.view(torch.int16), chk.view(torch.int16))


@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
def test_release_and_fully_synchronised_builds_agree_for_every_tile_shape(d):
    """Every shape of the tile table (other ring depths, wavefront counts and keys per tile than the default) keeps its
    own wait counts and barrier placement, so each is compared with its fully synchronised build."""
    import torch
    lib = _sync_lib()
    vp, i, f = ctypes.c_void_p, ctypes.c_int, ctypes.c_float
    lib.flat_attn_fwd_tile.restype = i
    lib.flat_attn_fwd_tile.argtypes = [vp, vp, vp, vp, i, i, i, i, f, i, i, vp]
    for index in range(fa.flat_attn_tile_shape_count(d)):
        for N, mask in ((1777, 0), (2100, 1)):
            w = synth.custom(f"sync_tile_{d}_{index}_{N}", 1, 3, N, d, "bf16", mask, seed=977 + d + index + N)
            q, k, v = synth.make_qkv(w)
            dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
            rel, chk = torch.full_like(dq, float("nan")), torch.full_like(dq, float("nan"))
            print(f"case sync build tile shape {index} {w}", flush=True)
            fa.flat_attn_fwd_tile(dq, dk, dv, rel, w.scale, w.mask, index)
            rc = lib.flat_attn_fwd_tile(dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), chk.data_ptr(), w.B, w.H, w.N, w.d, w.scale,
                                        w.mask, index, torch.cuda.current_stream().cuda_stream)
            assert rc == 0
            torch.cuda.synchronize()
            assert torch.isfinite(rel.float()).all()
            assert torch.equal(rel.view(torch.int16), chk.view(torch.int16))


# from one round of workgroups to a few; one tile (and less), a ragged tail, and as many tiles as the ring has stages
@pytest.mark.parametrize("H,Nq,Nk", [(257, 256, 64), (257, 17, 33), (300, 300, 129), (128, 700, 192), (200, 900, 1000)])
@pytest.mark.parametrize("d", [96, 128])
def test_workgroups_with_several_blocks(d, H, Nq, Nk):
    """Against the fully synchronised build, bit for bit, and against fp32 attention: launches without a mask of about as many blocks as there
    are compute units."""
    import torch
    lib = _sync_lib()
    gen = torch.Generator(device="cuda").manual_seed(d + H + Nq + Nk)
    q, k, v = (torch.randn(1, H, n, d, generator=gen, device="cuda").to(torch.bfloat16) for n in (Nq, Nk, Nk))
    rel, chk = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    scale = float(np.float32(d ** -0.5))
    print(f"case several blocks d={d} H={H} Nq={Nq} Nk={Nk}", flush=True)
    fa.flat_attn_fwd_cross(q, k, v, rel, scale, 0, None)
    assert lib.flat_attn_fwd_cross(q.data_ptr(), k.data_ptr(), v.data_ptr(), chk.data_ptr(), 1, H, Nq, Nk, d, scale, 0, None,
                                   torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(rel.view(torch.int16), chk.view(torch.int16))
    qf, kf, vf = (x.float() for x in (q, k, v))
    ref = torch.softmax(torch.matmul(qf, kf.transpose(-1, -2).contiguous()) * scale, dim=-1) @ vf
    # bf16 rounding of probabilities and results: 2^-9 of the result each, and of the largest results at most 2e-2 as elsewhere
    assert (rel.float() - ref).abs().max() <= 2e-2 and (rel.float() - ref).abs().sum() <= 5e-3 * ref.abs().sum()


# keys: less than a tile, one, two, and as many as every ring has stages and more; heads: four rounds and an odd number of blocks, and more
@pytest.mark.parametrize("H,N", [(1025, 33), (1031, 64), (1500, 129), (2050, 128), (1027, 250), (1100, 300)])
@pytest.mark.parametrize("d,index", [(96, 0), (96, 1), (128, 0), (128, 1), (128, 2), (128, 3)])
def test_workgroups_that_go_on_to_a_second_block(d, index, H, N):
    """Every shape whose workgroups take two blocks in a launch of four rounds or more: against the fully synchronised build, bit for bit,
    and against fp32 attention."""
    import torch
    lib = _sync_lib()
    vp, i, f = ctypes.c_void_p, ctypes.c_int, ctypes.c_float
    lib.flat_attn_fwd_tile.argtypes = [vp, vp, vp, vp, i, i, i, i, f, i, i, vp]
    rows = fa.flat_attn_tile_shape_get(d, index).as_dict()["rows_per_workgroup"]
    assert H * -(-N // rows) >= 4 * 256 * fa.flat_attn_tile_shape_occupancy(d, index)
    gen = torch.Generator(device="cuda").manual_seed(d + index + H + N)
    q, k, v = (torch.randn(1, H, N, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    rel, chk = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    scale = float(np.float32(d ** -0.5))
    print(f"case second block d={d} index={index} H={H} N={N}", flush=True)
    fa.flat_attn_fwd_tile(q, k, v, rel, scale, 0, index)
    assert lib.flat_attn_fwd_tile(q.data_ptr(), k.data_ptr(), v.data_ptr(), chk.data_ptr(), 1, H, N, d, scale, 0, index,
                                  torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(rel.view(torch.int16), chk.view(torch.int16))
    qf, kf, vf = (x.float() for x in (q, k, v))
    ref = torch.softmax(torch.matmul(qf, kf.transpose(-1, -2).contiguous()) * scale, dim=-1) @ vf
    # bf16 rounding of probabilities and results: 2^-9 of the result each, and of the largest results at most 2e-2 as elsewhere
    assert (rel.float() - ref).abs().max() <= 2e-2 and (rel.float() - ref).abs().sum() <= 5e-3 * ref.abs().sum()
