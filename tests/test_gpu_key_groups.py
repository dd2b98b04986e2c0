"""The key-group forms of the fused bf16 kernel (launches of few query rows), against the CPU oracle and, bit for bit, against
the fully synchronised build."""
import ctypes
import os

import numpy as np
import pytest

import oracle
import paper_2107_06419_amd as fa
from paper_2107_06419_amd import synth
from helpers import check_close, to_device, to_host_f64

pytestmark = pytest.mark.gpu


def rounded(shape, seed, tid, mult=1.0):
    x = synth.tensor_f32(shape, seed, tid, "normal", mult)
    return synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(x)).reshape(shape)


def run_both(q, k, v, scale, mask, lens):
    """The release library's output, after comparing it with the fully synchronised library's."""
    import torch
    lib = ctypes.CDLL(os.path.join(os.path.dirname(fa.library_path()), "libflat_attn_sync.so"))
    vp, i, f = ctypes.c_void_p, ctypes.c_int, ctypes.c_float
    lib.flat_attn_fwd_cross.argtypes = [vp, vp, vp, vp, i, i, i, i, i, f, i, vp, vp]
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    kv = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    out, chk = torch.full_like(dq, float("nan")), torch.full_like(dq, float("nan"))
    fa.flat_attn_fwd_cross(dq, dk, dv, out, scale, mask, kv)
    rc = lib.flat_attn_fwd_cross(dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), chk.data_ptr(), *q.shape[:3], k.shape[2], q.shape[3],
                                 scale, mask, None if kv is None else kv.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0 and torch.equal(out.view(torch.int16), chk.view(torch.int16))
    return to_host_f64(out)


# (B, H, Nq, Nk, kv_lens): one row and one tile; tails of one key and one row on both sides of a tile and of a group's share;
# then sizes at which the 64-row forms (four groups, two groups) and the 128-row form are chosen; last, one round of
# 128-row workgroups or more, where no form is
CASES = [
    (1, 1, 1, 65, None), (2, 2, 31, 128, [128, 1]), (1, 3, 33, 129, None), (2, 2, 65, 161, [33, 161]), (2, 1, 257, 545, [385, 416]),
    (1, 45, 257, 2500, None), (3, 15, 250, 2049, [2049, 250, 1111]), (2, 45, 257, 1100, [1100, 513]), (2, 16, 513, 513, None),
    (1, 27, 1025, 1025, None), (2, 64, 300, 700, [700, 333]),
]


@pytest.mark.parametrize("B,H,Nq,Nk,lens", CASES)
@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("mask", [0, 1])
def test_few_rows_match_the_oracle_and_the_synchronised_build(B, H, Nq, Nk, lens, d, mask):
    seed = 52000 + Nq + Nk + d + mask
    q, k, v = rounded((B, H, Nq, d), seed, 0), rounded((B, H, Nk, d), seed, 1), rounded((B, H, Nk, d), seed, 2)
    scale = float(np.float32(d ** -0.5))
    print(f"case key groups B={B} H={H} Nq={Nq} Nk={Nk} d={d} mask={mask} lens={lens}", flush=True)
    got = run_both(q, k, v, scale, mask, lens)
    ref = oracle.attention_cross(q, k, v, scale, mask, kv_lens=None if lens is None else np.array(lens))
    check_close(got, ref, "bf16", "key groups")


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("rising", [True, False])
def test_groups_with_very_different_maxima_merge(d, rising):
    """Logits that grow (or fall) along the keys by hundreds of log2 units: the groups end with different reference maxima,
    or with sums that vanish beside another group's."""
    B, H, Nq, Nk = 1, 2, 70, 1500
    q, k = np.abs(rounded((B, H, Nq, d), 9, 0)), np.abs(rounded((B, H, Nk, d), 9, 1))
    ramp = np.linspace(0.1, 6.0, Nk, dtype=np.float32)[:: 1 if rising else -1][None, None, :, None]
    k = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(k * ramp)).reshape(k.shape)
    v = rounded((B, H, Nk, d), 9, 2)
    for mask in (0, 1):
        check_close(run_both(q, k, v, 0.125, mask, None), oracle.attention_cross(q, k, v, 0.125, mask), "bf16", "ramp")


@pytest.mark.parametrize("Nq,Nk", [(100, 100), (64, 161), (32, 160), (1, 33)])
@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
def test_a_group_whose_keys_a_row_does_not_see_weighs_nothing(d, Nq, Nk):
    """Causal, with logits of hundreds of log2 units from a row's first unseen key on: each group takes its reference maximum from the
    first key of its share, which must not count in the merge where the row sees none of the share.  The split form, too."""
    import torch
    q, k, v = np.abs(rounded((1, 2, Nq, d), 77, 0)), rounded((1, 2, Nk, d), 77, 1), rounded((1, 2, Nk, d), 77, 2)
    k[:, :, Nk - Nq + 1:] = np.abs(k[:, :, Nk - Nq + 1:]) * 16.0  # exact in bf16; visible to the last rows only
    scale = float(np.float32(d ** -0.5))
    ref = oracle.attention_cross(q, k, v, scale, 1)
    check_close(run_both(q, k, v, scale, 1, None), ref, "bf16", "unseen shares")
    dq, dk, dv = (to_device(x, "bf16") for x in (q, k, v))
    out = torch.full_like(dq, float("nan"))
    ws = torch.empty(fa.flat_attn_fwd_splitkv_workspace_bytes(1, 2, Nq, Nk, d, 2) // 4 + 1, dtype=torch.float32, device="cuda")
    fa.flat_attn_fwd_splitkv(dq, dk, dv, out, scale, 1, None, 2, ws)
    torch.cuda.synchronize()
    check_close(to_host_f64(out), ref, "bf16", "unseen shares, two splits")


@pytest.mark.parametrize("B,H,Nq,Nk", [(2, 65, 40, 90), (3, 43, 300, 310), (1, 8, 33, 100), (15, 16, 129, 140)])
@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
def test_heads_dealt_over_the_xcds(B, H, Nq, Nk, d):
    """Key counts over fewer than 16 batch entries, with head counts that eight divides and (from 128 heads on) does not."""
    q, k, v = rounded((B, H, Nq, d), 88, 0), rounded((B, H, Nk, d), 88, 1), rounded((B, H, Nk, d), 88, 2)
    lens = np.linspace(1, Nk, B).astype(np.int64) if B > 1 else np.array([Nk - 7])
    scale = float(np.float32(d ** -0.5))
    print(f"case dealt heads B={B} H={H} Nq={Nq} Nk={Nk} d={d}", flush=True)
    check_close(run_both(q, k, v, scale, 0, [int(x) for x in lens]), oracle.attention_cross(q, k, v, scale, 0, kv_lens=lens), "bf16", "dealt heads")


# (B, H, Nq, Nk, d, mask): launches on the edge of a key-group form, which a rule of its own for key counts would take
@pytest.mark.parametrize("B,H,Nq,Nk,d,mask", [(6, 16, 300, 900, 64, 1), (16, 12, 250, 1011, 128, 1), (12, 16, 160, 600, 128, 1), (8, 16, 200, 500, 32, 1),
                                              (8, 12, 250, 700, 96, 0), (8, 12, 250, 700, 96, 1)])
def test_counts_of_all_keys_change_nothing(B, H, Nq, Nk, d, mask):
    """Key counts that name every key divide the keys as no counts do: the same sums in the same order."""
    import torch
    q, k, v = (to_device(rounded((B, H, n, d), 53000 + Nq + d + mask, t), "bf16") for n, t in ((Nq, 0), (Nk, 1), (Nk, 2)))
    counts = torch.full((B,), Nk, dtype=torch.int32, device="cuda")
    with_counts, without = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    print(f"case all keys counted B={B} H={H} Nq={Nq} Nk={Nk} d={d} mask={mask}", flush=True)
    fa.flat_attn_fwd_cross(q, k, v, with_counts, float(np.float32(d ** -0.5)), mask, counts)
    fa.flat_attn_fwd_cross(q, k, v, without, float(np.float32(d ** -0.5)), mask, None)
    torch.cuda.synchronize()
    assert torch.isfinite(without).all() and torch.equal(with_counts.view(torch.int16), without.view(torch.int16))
