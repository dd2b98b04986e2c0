"""fp32 path where its factors are split into fp16 pieces (128 positions and more): tails of a tile and of a row block with one and two key groups, both masks,
and inputs that the pieces cannot hold, which have to give what fp32 arithmetic gives."""
import numpy as np
import pytest
import torch

import oracle
import paper_2107_06419_amd as fa
from paper_2107_06419_amd import synth
from helpers import check_close, to_device, to_host_f64

pytestmark = pytest.mark.gpu

HEADS = [600, 24]  # enough for one key group; so few that two are taken (d = 64: from about 385 positions on, d = 128: at most lengths)


def run(q, k, v, scale, mask):
    out = torch.full_like(q, float("nan"))
    print(f"case f32 pieces {tuple(q.shape)} mask={mask}", flush=True)
    fa.flat_attn_fwd_f32(q, k, v, out, scale, mask)
    torch.cuda.synchronize()
    return out


def inputs(heads, N, d, seed):
    return [synth.tensor_f32((1, heads, N, d), seed, t, "normal", 1.0) for t in range(3)]


@pytest.mark.parametrize("heads", HEADS)
@pytest.mark.parametrize("N", [128, 129, 159, 161, 191, 193, 255, 257, 385])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("mask", [0, 1])
def test_tails(heads, N, d, mask):
    q, k, v = inputs(heads, N, d, 4000 + N + d + mask)
    k *= np.linspace(0.1, 8.0, N, dtype=np.float32)[None, None, :, None]  # the reference maximum is raised on the way
    scale = float(np.float32(d ** -0.5))
    out = run(*(to_device(x, "f32") for x in (q, k, v)), scale, mask)
    some = [0, 1, heads - 1]
    check_close(to_host_f64(out[:, some]), oracle.attention(q[:, some], k[:, some], v[:, some], scale, mask), "f32", f"heads={heads} N={N} d={d} mask={mask}")
    assert torch.isfinite(out).all()


# 390 products and sums of either kind are off by 3e-7 to 4e-7 in the 2-norm (rounded about 200 times in turn, by 2^-25 each in the mean); four times that.
@pytest.mark.parametrize("heads", HEADS)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("q_by,k_by,v_by", [(1, 1, 1e-3), (1, 1, 1e-12), (1, 1, 1e36), (1e-30, 1e30, 1), (1e5, 1e-5, 1), (2e3, 5e-4, 1), (1e-3, 1e3, 1), (1e-6, 1e6, 1),
                                            (1e-20, 1, 1), (1, 0, 0)])
def test_magnitudes(heads, d, q_by, k_by, v_by):
    N, scale = 390, float(np.float32(d ** -0.5))
    q, k, v = (x * np.float32(by) for x, by in zip(inputs(heads, N, d, 4700 + d), (q_by, k_by, v_by)))
    out = run(*(to_device(x, "f32") for x in (q, k, v)), scale, 0)
    some = [0, heads - 1]
    x = [t[:, some].astype(np.float64) for t in (q, k, v)]
    s = np.matmul(x[0], x[1].swapaxes(-1, -2)) * scale
    p = np.exp(s - s.max(-1, keepdims=True))
    ref = np.matmul(p / p.sum(-1, keepdims=True), x[2])
    got = out[:, some].double().cpu().numpy()
    assert np.linalg.norm((got - ref) / (v_by or 1)) <= 1.5e-6 * np.linalg.norm(ref / (v_by or 1))


@pytest.mark.parametrize("heads", HEADS)
@pytest.mark.parametrize("d", [64, 128])
def test_columns_of_small_and_no_values(heads, d):
    """A column of tiny values beside ordinary ones keeps its relative precision; a column of zeros gives zeros."""
    N, scale = 390, float(np.float32(d ** -0.5))
    q, k, v = inputs(heads, N, d, 4800 + d)
    v[..., 5] = 1.0 + 0.1 * v[..., 5]
    tiny = v.copy()
    tiny[..., 5] *= np.float32(1e-9)
    tiny[..., 7] = 0.0
    out = to_host_f64(run(*(to_device(x, "f32") for x in (q, k, tiny)), scale, 0))
    some = [0, heads - 1]
    ref = oracle.attention(q[:, some], k[:, some], v[:, some], scale, 0)
    got = out[:, some]
    assert np.abs(got[..., 5] / float(np.float32(1e-9)) - ref[..., 5]).max() <= 1e-5
    assert (out[..., 7] == 0).all()
    rest = [c for c in range(d) if c not in (5, 7)]
    check_close(got[..., rest], ref[..., rest], "f32", "beside tiny values")


@pytest.mark.parametrize("heads", HEADS)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("low", [-1e5, -3.4e38, float("-inf")])
def test_low_keys_and_infinite_values(heads, d, low):
    """Keys marked by a low number in a feature column weigh nothing; an infinite value reaches its column only, a NaN in Q its row."""
    N, scale = 390, float(np.float32(d ** -0.5))
    q, k, v = inputs(heads, N, d, 4900 + d)
    q[..., d - 1], k[..., d - 1] = 1.0, 0.0
    k[:, :, 200:, d - 1] = low
    dq, dk, dv = (to_device(x, "f32") for x in (q, k, v))
    dv[:, :, 17, 3] = float("inf")
    dq[:, :, 250, 0] = float("nan")
    out = run(dq, dk, dv, scale, 0)
    assert out[:, :, 250].isnan().all()
    some, rows, rest = [0, heads - 1], [r for r in range(N) if r != 250], [c for c in range(d) if c != 3]
    assert torch.isposinf(out[:, some][:, :, rows][..., 3]).all()
    ref = oracle.attention_cross(q[:, some], k[:, some, :200], v[:, some, :200], scale, 0)
    check_close(to_host_f64(out[:, some][:, :, rows])[..., rest], ref[:, :, rows][..., rest], "f32", f"low keys {low}")


def elementwise_excess(got, q, k, v, scale, mask, bound):
    """How far the worst element is off, in units of `bound` times the sum of |p v| that makes it up (64 bits)."""
    x = [t.astype(np.float64) for t in (q, k, v)]
    s = np.matmul(x[0], x[1].swapaxes(-1, -2)) * scale
    if mask:
        s = np.where(np.tri(s.shape[-2], dtype=bool), s, -np.inf)
    p = np.exp(s - s.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    made_of = np.matmul(p, np.abs(x[2]))
    return float((np.abs(got - np.matmul(p, x[2])) / np.maximum(made_of * bound, 1e-300)).max())


# A row's own exponents, up to 16 here (64 with one heavy key), are off by 2^-25 of that and the sums by a few 2^-24: 3e-6 and 1e-5.
@pytest.mark.parametrize("heads", HEADS)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("small", [1e-7, 1e-12])
@pytest.mark.parametrize("where", ["first keys", "first keys of a column", "heavy key", "heavy key in a column"])
def test_rows_that_see_small_values(heads, d, small, where):
    """What a row gets keeps its relative precision, element by element, also where keys that it does not see, or barely, have far larger values."""
    N, scale, causal = 390, float(np.float32(d ** -0.5)), where.startswith("first")
    q, k, v = inputs(heads, N, d, 5000 + d)
    columns = slice(9, 10) if where.endswith("column") else slice(None)
    if causal:
        v[:, :, :40, columns] *= np.float32(small)
    else:
        q[..., 0], k[..., 0] = 8.0, 0.0
        k[:, :, 200, :], k[:, :, 200, 0] = 0.0, 5.0 / scale
        v[:, :, 200, columns] *= np.float32(small)
    out = to_host_f64(run(*(to_device(x, "f32") for x in (q, k, v)), scale, int(causal)))
    some = [0, heads - 1]
    assert elementwise_excess(out[:, some], q[:, some], k[:, some], v[:, some], scale, causal, 3e-6 if causal else 1e-5) <= 1.0


@pytest.mark.parametrize("heads", HEADS)
@pytest.mark.parametrize("d", [64, 128])
def test_values_that_select_keys(heads, d):
    """V of zeros and one 1 per key: a result is the weight of some keys, from all of it to 1e-13, and keeps its relative precision.  (Exponents up to 64 are off by 2^-19.)"""
    N = 390
    q, k, v = (np.zeros((1, heads, N, d), np.float32) for _ in range(3))
    of = np.arange(N) % d
    v[:, :, np.arange(N), of] = 1.0
    q[..., 0] = 1.0 + 0.1 * np.arange(N, dtype=np.float32) / N
    k[..., 0] = -27.0 * of.astype(np.float32) / d
    out = to_host_f64(run(*(to_device(x, "f32") for x in (q, k, v)), 1.0, 0))
    some = [0, heads - 1]
    assert elementwise_excess(out[:, some], q[:, some], k[:, some], v[:, some], 1.0, 0, 1e-5) <= 1.0


@pytest.mark.parametrize("heads", HEADS)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("q_by", [1e-30, 1e-36])
def test_small_queries_and_a_large_scale(heads, d, q_by):
    """The logits are ordinary ones, however far apart Q and the scale are.  (Bound: as for the magnitudes above.)"""
    N = 390
    q, k, v = inputs(heads, N, d, 5200 + d)
    q *= np.float32(q_by)
    scale = float(np.float32(d ** -0.5 / q_by))
    out = run(*(to_device(x, "f32") for x in (q, k, v)), scale, 0)
    some = [0, heads - 1]
    x = [t[:, some].astype(np.float64) for t in (q, k, v)]
    s = np.matmul(x[0], x[1].swapaxes(-1, -2)) * scale
    p = np.exp(s - s.max(-1, keepdims=True))
    ref = np.matmul(p / p.sum(-1, keepdims=True), x[2])
    assert np.linalg.norm(out[:, some].double().cpu().numpy() - ref) <= 1.5e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("heads", HEADS)
@pytest.mark.parametrize("d", [64, 128])
def test_a_row_of_one_key_is_its_value(heads, d):
    """The causal mask leaves query 0 one key, of weight 1: its result is that key's value, bit for bit."""
    q, k, v = (to_device(x, "f32") for x in inputs(heads, 390, d, 5300 + d))
    out = run(q, k, v, float(np.float32(d ** -0.5)), 1)
    assert torch.equal(out[:, :, 0], v[:, :, 0])


@pytest.mark.parametrize("heads", HEADS)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("weak", [1e-3, 1e-4, 1e-5, 1e-6])
@pytest.mark.parametrize("mask", [0, 1])
def test_a_weak_column(heads, d, weak, mask):
    """A column of V far below the others keeps its relative precision, whether that shows in the first keys or in the results.  (Bound: as for rows above.)"""
    N, scale = 390, float(np.float32(d ** -0.5))
    q, k, v = inputs(heads, N, d, 5400 + d + mask)
    v[..., 11] *= np.float32(weak)
    out = to_host_f64(run(*(to_device(x, "f32") for x in (q, k, v)), scale, mask))
    some = [0, heads - 1]
    assert elementwise_excess(out[:, some], q[:, some], k[:, some], v[:, some], scale, mask, 3e-6) <= 1.0
