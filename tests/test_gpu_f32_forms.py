"""Every form of the fp32 entry point, taken by number and not by the size of the problem: tails of a tile and of a row block, and thousands of positions."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2107_06419_amd as fa
from paper_2107_06419_amd import synth
from helpers import check_close, sample_rows, to_device, to_host_f64

pytestmark = pytest.mark.gpu

FORMS = {"split, two key groups": -2, "split, one key group": -1, "one wavefront": 1, "two wavefronts": 2, "four wavefronts": 4}


def run(form, q, k, v, scale, mask):
    lib = fa.load_library()
    p, i = ctypes.c_void_p, ctypes.c_int
    call = ctypes.CFUNCTYPE(i, p, p, p, p, i, i, i, ctypes.c_float, i, i, p)(("flat_internal_fwd_f32_form", lib))
    B, H, N, d = q.shape
    assert d in (64, 128) and all(t.shape == q.shape and t.dtype is torch.float32 and t.is_cuda and t.is_contiguous() for t in (q, k, v))
    out = torch.full_like(q, float("nan"))
    print(f"case f32 form {form} {tuple(q.shape)} mask={mask}", flush=True)
    assert call(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), B * H, N, d, scale, mask, FORMS[form], torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    return out


def inputs(heads, N, d, seed):
    return [synth.tensor_f32((1, heads, N, d), seed, t, "normal", 1.0) for t in range(3)]


def off(got, ref):
    """2-norm of the error over that of the result, of everything and of the worst row."""
    e = got - ref
    return np.linalg.norm(e) / np.linalg.norm(ref), (np.linalg.norm(e, axis=-1) / np.linalg.norm(ref, axis=-1)).max()


# Up to 4096 products and sums of either kind are off by 1.3e-6 in the 2-norm (one wavefront, which adds them all up in turn), the split ones by 0.7e-6, a row by
# twice that: with some room 2e-6, 1.2e-6 and 4e-6.  (A piece left out is 2^-12.)
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("mask", [0, 1])
def test_tails(form, d, mask):
    scale = float(np.float32(d ** -0.5))
    for N in (128, 129, 159, 161, 191, 193, 255, 257, 289, 385, 447):
        q, k, v = inputs(2, N, d, 6000 + N + d + mask)
        got = to_host_f64(run(form, *(to_device(x, "f32") for x in (q, k, v)), scale, mask))
        whole, row = off(got, oracle.attention(q, k, v, scale, mask))
        assert whole <= (2e-6 if FORMS[form] > 0 else 1.2e-6) and row <= 4e-6, f"N={N}: {whole:.2e}, worst row {row:.2e}"
        k *= np.linspace(0.1, 8.0, N, dtype=np.float32)[None, None, :, None]  # the reference maximum is raised on the way
        got = to_host_f64(run(form, *(to_device(x, "f32") for x in (q, k, v)), scale, mask))
        check_close(got, oracle.attention(q, k, v, scale, mask), "f32", f"raised, N={N}")


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("N", [2049, 4096])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("mask", [0, 1])
def test_thousands_of_positions(form, N, d, mask):
    scale = float(np.float32(d ** -0.5))
    q, k, v = inputs(3, N, d, 6600 + N + d + mask)
    out = run(form, *(to_device(x, "f32") for x in (q, k, v)), scale, mask)
    rows = sample_rows(N, 24, seed=N + d)
    whole, row = off(to_host_f64(out[:, :, torch.from_numpy(rows).cuda()]), oracle.attention(q, k, v, scale, mask, rows=rows))
    assert whole <= (2e-6 if FORMS[form] > 0 else 1.2e-6) and row <= 4e-6, f"{whole:.2e}, worst row {row:.2e}"
    assert torch.isfinite(out).all()
