"""Keys whose logits lie far below the others' (padding marked in a feature column of K): they weigh nothing and must not touch the weights
of the other keys, wherever they stand.  A wavefront starts from the logit of the first key it takes, so the places are the
first and last keys of the 32-key blocks that open a share, whole blocks and tiles, and all keys but a few."""
import numpy as np
import pytest
import torch

import oracle
import paper_2107_06419_amd as fa
from paper_2107_06419_amd import binding, synth
from helpers import check_close, to_host_f64

pytestmark = pytest.mark.gpu

PLACES = {"0": [0], "31": [31], "32": [32], "64": [64], "96": [96], "0, 32, 64, 96": [0, 32, 64, 96], "a block": range(32),
          "a tile and one": range(65), "every other block": [j for j in range(330) if j % 64 < 32], "all but three": range(327)}
LOW = [-1e5, -1e7, -1e9, -3.3895314e38, float("-inf")]  # before scaling; the fourth is the lowest bf16 number
B, H, N = 1, 1, 330


def inputs(Nq, Nk, d, low, keys, dtype="bf16"):
    """The tensors on the device, and their values for the oracle."""
    q, k, v = (synth.tensor_f32((B, H, n, d), 6400 + d, t, "normal", 1.0) for n, t in ((Nq, 0), (Nk, 1), (Nk, 2)))
    q[..., d - 1], k[..., d - 1] = 1.0, 0.0
    k[:, :, list(keys), d - 1] = low
    dev = [torch.from_numpy(x).to(torch.float32 if dtype == "f32" else torch.bfloat16) for x in (q, k, v)]
    return [x.cuda() for x in dev], [x.float().numpy() for x in dev]


def agree(run, dev, ref, what, dtype="bf16"):
    out = torch.full_like(dev[0], float("nan"))
    run(*dev, out)
    torch.cuda.synchronize()
    check_close(to_host_f64(out), ref, dtype, what)


@pytest.mark.parametrize("low", LOW)
@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
def test_keys_of_low_logits_weigh_nothing(d, low):
    scale = float(np.float32(d ** -0.5))
    blocks, tiles = B * H * -(-N // binding.FLAT_SPARSE_BLOCK_ROWS), -(-N // binding.FLAT_SPARSE_BLOCK_KEYS)
    offs = torch.arange(0, blocks * tiles + 1, tiles, dtype=torch.int32, device="cuda")
    ids = torch.arange(tiles, dtype=torch.int32, device="cuda").repeat(blocks)
    for place, keys in PLACES.items():
        print(f"case low logits d={d} low={low} keys {place}", flush=True)
        what = f"low keys {place}"
        # self-attention: every tile shape, and the block-sparse variant with every tile listed
        dev, host = inputs(N, N, d, low, keys)
        ref = oracle.attention(*host, scale, 0)
        for index in range(fa.flat_attn_tile_shape_count(d)):
            agree(lambda *t: fa.flat_attn_fwd_tile(*t, scale, 0, index), dev, ref, f"{what}, tile shape {index}")
        agree(lambda *t: fa.flat_attn_fwd_blocksparse(*t, scale, offs, ids), dev, ref, f"{what}, block-sparse")
        # few rows over the same keys, on their own and in splits; the mask leaves each row some of the other keys
        for Nq in (1, 40, 70):
            for mask in (0, 1):
                if mask and place == "all but three":
                    continue
                dev, host = inputs(Nq, N, d, low, keys)
                ref = oracle.attention_cross(*host, scale, mask)
                agree(lambda *t: fa.flat_attn_fwd_cross(*t, scale, mask, None), dev, ref, f"{what}, {Nq} rows, mask {mask}")
                for splits in (2, 5):
                    ws = torch.empty(fa.flat_attn_fwd_splitkv_workspace_bytes(B, H, Nq, N, d, splits) // 4 + 1, dtype=torch.float32, device="cuda")
                    agree(lambda *t: fa.flat_attn_fwd_splitkv(*t, scale, mask, None, splits, ws), dev, ref,
                          f"{what}, {Nq} rows, mask {mask}, {splits} splits")


@pytest.mark.parametrize("low", LOW[:3])
@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
def test_keys_of_one_low_logit_weigh_the_same(d, low):
    """All keys at the same logit: a row is the mean of the values, however coarse the numbers are at that logit."""
    scale = float(np.float32(d ** -0.5))
    dev, host = inputs(N, N, d, low, range(N))
    dev[0][..., :-1] = 0.0
    ref = np.broadcast_to(host[2].astype(np.float64).mean(axis=2, keepdims=True), host[2].shape)
    for index in range(fa.flat_attn_tile_shape_count(d)):
        agree(lambda *t: fa.flat_attn_fwd_tile(*t, scale, 0, index), dev, ref, f"one low logit, tile shape {index}")
    if d in (64, 128):
        agree(lambda *t: fa.flat_attn_fwd_f32(*t, scale, 0), [x.float() for x in dev], ref, "one low logit", "f32")


@pytest.mark.parametrize("low", LOW)
@pytest.mark.parametrize("d", [64, 128])
def test_keys_of_low_logits_weigh_nothing_fp32(d, low):
    scale = float(np.float32(d ** -0.5))
    for place, keys in PLACES.items():
        print(f"case low logits fp32 d={d} low={low} keys {place}", flush=True)
        dev, host = inputs(N, N, d, low, keys, "f32")
        agree(lambda *t: fa.flat_attn_fwd_f32(*t, scale, 0), dev, oracle.attention(*host, scale, 0), f"low keys {place}", "f32")
