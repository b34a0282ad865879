"""Sizes of the scratch memory, on the host: a buffer made for the longest call
serves every shorter one, and the part that only holds partial sums is bounded."""
import os

import pytest

from paper_2609_13141_amd import configs, sas

pytestmark = pytest.mark.skipif(not os.path.exists(sas.LIB_PATH), reason="libsas.so not built")

SHAPES = [(32, 32, 128, 64, 8), (32, 32, 128, 64, 16), (28, 4, 128, 64, 32), (8, 2, 64, 16, 4), (4, 1, 64, 128, 2)]


def never_falls(sizes):
    return all(0 < a <= b for a, b in zip(sizes, sizes[1:]))


@pytest.mark.parametrize("H,Hkv,dh,B,K", SHAPES)
def test_attention_backward(H, Hkv, dh, B, K):
    w = configs.L7B_1K.with_(n_heads=H, n_kv_heads=Hkv, head_dim=dh, block_size=B, top_k=K)
    cfg, dense = sas.make_config(w, "gated"), sas.make_config(w, "dense")
    size = lambda c, b, n: sas.workspace_size(c, sas.OP_ATTENTION_BACKWARD, b, n)  # noqa: E731
    assert never_falls([size(cfg, 1, n) for n in range(1, 6000, 13)])
    for n in (100, 700, 911, 4096):
        assert never_falls([size(cfg, b, n) for b in range(1, 20)])
        assert never_falls([size(sas.make_config(w.with_(top_k=k), "gated"), 1, n) for k in range(1, 33)])
    # what the divided row lists add: nothing of note where no list is long enough to be
    # divided, at most 1024 parts of dK and dV of 64 keys anywhere
    assert size(cfg, 1, 256) - size(dense, 1, 256) < 1 << 16
    for b, n in ((1, 2048), (1, 16384), (4, 4096)):
        assert size(cfg, b, n) - size(dense, b, n) < 1024 * 2 * 64 * dh * 4 + (1 << 20)


@pytest.mark.parametrize("d,F,H,Hkv", [(4096, 11008, 32, 32), (3584, 18944, 28, 4), (1536, 8960, 12, 2), (256, 688, 4, 4)])
def test_products(d, F, H, Hkv):
    w = configs.L7B_1K.with_(d_model=d, d_ff=F, n_heads=H, n_kv_heads=Hkv)
    cfg = sas.make_config(w)
    mlp = [sas.workspace_size(cfg, sas.OP_MLP, n, 0) for n in range(1, 20000, 61)]
    assert never_falls(mlp)
    # activations [n, d] and [n, d_ff], and at most 256 MiB of sums
    for n, s in zip(range(1, 20000, 61), mlp):
        assert s <= 2 * n * (d + F) + 512 + (256 << 20)
    # (from 1024 query tiles on, the layer's attention no longer splits its keys)
    assert never_falls([sas.workspace_size(cfg, sas.OP_LAYER, 1, n) for n in range(1, 128 * (1023 // H), 61)])
