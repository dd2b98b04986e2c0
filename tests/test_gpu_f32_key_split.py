"""fp32 path at the sizes where its key split can go wrong: one to a few 32-key tiles per wavefront, tails of a tile, wavefronts
without a tile, and enough or too few heads for each number of wavefronts per workgroup (1, 2, 4).  From 129 positions on most of these
problems take the split products; test_gpu_f32_forms.py runs every form by name."""
import numpy as np
import pytest

import oracle
import paper_2107_06419_amd as fa
from paper_2107_06419_amd import synth
from helpers import check_close, to_device, to_host_f64

pytestmark = pytest.mark.gpu

HEADS = {1: 1100, 2: 150, 4: 3}  # enough heads for whole rounds of one-wavefront workgroups ... so few that the keys are split in four


@pytest.mark.parametrize("heads", sorted(HEADS.values()))
@pytest.mark.parametrize("N", [1, 31, 32, 33, 64, 65, 96, 129, 160, 289])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("mask", [0, 1])
def test_f32_key_split_edges(heads, N, d, mask):
    import torch
    q, k, v = (synth.tensor_f32((1, heads, N, d), 900 + N + d + mask, t, "normal", 1.0) for t in range(3))
    if N > 64:  # logits that grow along the keys: the reference maximum is passed by less and by more than its slack of 2^8
        k = k * np.linspace(0.1, 8.0, N, dtype=np.float32)[None, None, :, None]
    dq, dk, dv = (to_device(x, "f32") for x in (q, k, v))
    out = torch.full_like(dq, float("nan"))
    print(f"case f32 key split heads={heads} N={N} d={d} mask={mask}", flush=True)
    fa.flat_attn_fwd_f32(dq, dk, dv, out, float(np.float32(d ** -0.5)), mask)
    torch.cuda.synchronize()
    some = sorted({0, 1, heads // 2, heads - 1} & set(range(heads)))
    ref = oracle.attention(q[:, some], k[:, some], v[:, some], float(np.float32(d ** -0.5)), mask)
    check_close(to_host_f64(out[:, some]), ref, "f32", f"heads={heads} N={N} d={d} mask={mask}")
    assert torch.isfinite(out).all()


@pytest.mark.parametrize("heads", sorted(HEADS.values()))
@pytest.mark.parametrize("N", [1, 33, 128, 289])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("mask", [0, 1])
def test_f32_scale_zero_gives_uniform_weights(heads, N, d, mask):
    """scale = 0 is accepted: every visible key weighs the same, masked keys (the diagonal tile, the tail) nothing."""
    import torch
    q, k, v = (synth.tensor_f32((1, heads, N, d), 1700 + N + d + mask, t, "normal", 1.0) for t in range(3))
    dq, dk, dv = (to_device(x, "f32") for x in (q, k, v))
    out = torch.full_like(dq, float("nan"))
    print(f"case f32 scale 0 heads={heads} N={N} d={d} mask={mask}", flush=True)
    fa.flat_attn_fwd_f32(dq, dk, dv, out, 0.0, mask)
    torch.cuda.synchronize()
    some = sorted({0, heads - 1})
    check_close(to_host_f64(out[:, some]), oracle.attention(q[:, some], k[:, some], v[:, some], 0.0, mask), "f32", f"scale 0 N={N} d={d}")
    assert torch.isfinite(out).all()


@pytest.mark.parametrize("heads", sorted(HEADS.values()))
@pytest.mark.parametrize("N", [1, 31, 65, 127])
@pytest.mark.parametrize("d", [64, 128])
def test_f32_infinity_in_the_last_value_row_reaches_its_column_only(heads, N, d):
    """The last tile is filled up with keys that do not exist: they add nothing, whatever the last value row holds."""
    import torch
    q, k, v = (synth.tensor_f32((1, heads, N, d), 1900 + N + d, t, "normal", 1.0) for t in range(3))
    dq, dk, dv = (to_device(x, "f32") for x in (q, k, v))
    dv[:, :, N - 1, 3] = float("inf")
    out = torch.full_like(dq, float("nan"))
    print(f"case f32 infinite value heads={heads} N={N} d={d}", flush=True)
    fa.flat_attn_fwd_f32(dq, dk, dv, out, float(np.float32(d ** -0.5)), 0)
    torch.cuda.synchronize()
    assert torch.isposinf(out[..., 3]).all()
    some, rest = sorted({0, heads - 1}), [c for c in range(d) if c != 3]
    ref = oracle.attention(q[:, some], k[:, some], v[:, some], float(np.float32(d ** -0.5)), 0)
    check_close(to_host_f64(out[:, some])[..., rest], ref[..., rest], "f32", f"infinite value N={N} d={d}")


@pytest.mark.parametrize("heads", sorted(HEADS.values()))
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("magnitude", [1e36, 1e-37])
def test_f32_large_and_small_values_stay_in_range(heads, d, magnitude):
    """Probabilities never exceed 1 against the reference maximum, also while it lags behind the row maximum: the first tile's
    logits lie 7.5 powers of two below the others', and 160 values of 1e36 still sum to less than the largest float.  Nor do they
    become so small that values near the smallest normal float are lost."""
    import torch
    N = 160
    q, k = np.zeros((1, heads, N, d), np.float32), np.zeros((1, heads, N, d), np.float32)
    q[..., 0] = 1.0
    k[:, :, 32:, 0] = 7.5 * np.log(2.0)
    v = (1.0 + 0.1 * synth.tensor_f32((1, heads, N, d), 77, 2, "normal", 1.0)).astype(np.float32)
    dq, dk, dv = (to_device(x, "f32") for x in (q, k, v * np.float32(magnitude)))
    out = torch.full_like(dq, float("nan"))
    print(f"case f32 range heads={heads} d={d} magnitude={magnitude}", flush=True)
    fa.flat_attn_fwd_f32(dq, dk, dv, out, 1.0, 0)
    torch.cuda.synchronize()
    some = sorted({0, heads - 1})
    check_close(to_host_f64(out[:, some]) / float(np.float32(magnitude)), oracle.attention(q[:, some], k[:, some], v[:, some], 1.0, 0), "f32", "range")
    assert torch.isfinite(out).all()


@pytest.mark.parametrize("heads", sorted(HEADS.values()))
@pytest.mark.parametrize("d", [64, 128])
def test_f32_keys_at_minus_infinity_weigh_nothing(heads, d):
    """A wavefront whose own tiles hold only logits of -inf (here every tile but the first) adds nothing to the others' result."""
    import torch
    N, scale = 128, float(np.float32(d ** -0.5))
    q, k, v = (synth.tensor_f32((1, heads, N, d), 2300 + d, t, "normal", 1.0) for t in range(3))
    q = np.abs(q) + 0.1
    dq, dk, dv = (to_device(x, "f32") for x in (q, k, v))
    dk[:, :, 32:] = float("-inf")
    out = torch.full_like(dq, float("nan"))
    print(f"case f32 keys at -inf heads={heads} d={d}", flush=True)
    fa.flat_attn_fwd_f32(dq, dk, dv, out, scale, 0)
    torch.cuda.synchronize()
    some = sorted({0, heads - 1})
    check_close(to_host_f64(out[:, some]), oracle.attention_cross(q[:, some], k[:, some, :32], v[:, some, :32], scale, 0), "f32", "keys at -inf")
