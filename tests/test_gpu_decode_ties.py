"""The long caches' Top-K where its digits run out at different places: scores
that part in their first digits, only in their lowest ones, or not at all at
the K-th place (lower blocks win); exact against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_13141_amd import inputs, sas

from helpers import f64, spec_of
from test_gpu_decode_long import _select_cache, _w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels,step", [(1, 1.0), (3, 1.0), (40, 0.5), (4096, 2.0**-23), (17, 2.0**-23)])
@pytest.mark.parametrize("blocks,K,sign", [(257, 1, 1), (600, 32, -1), (3000, 16, 1)])
def test_topk_among_ties(levels, step, blocks, K, sign):
    print(f"\n[case] decode Top-K {levels} levels {step:g} apart, {blocks} blocks, K={K}, sign {sign}", flush=True)
    w = _w("f32", 64, K, index=131)
    r = np.random.default_rng(blocks + levels)
    kb = np.zeros((w.batch, w.n_kv_heads, blocks, 64), np.float32)
    kb[..., 3] = 1 + r.integers(0, levels, kb.shape[:3]) * np.float32(step)
    q = inputs.normal(w, "q_t", (w.batch, w.n_heads, 64), 1.0)
    q[..., 3] = sign * (1 + np.abs(q[..., 3]))
    pos = [blocks * w.block_size - 1, (K + 1) * w.block_size + 3]
    sel = sas.decode_select(sas.make_config(w), sas.to_device(q, "f32"),
                            torch.tensor(pos, dtype=torch.int32, device="cuda"),
                            _select_cache(w, blocks, sas.to_device(kb, "f32")))
    ref, _ = oracle.decode_select(f64(q), np.array(pos), f64(kb), spec_of(w))
    np.testing.assert_array_equal(sel.cpu().numpy(), ref)
