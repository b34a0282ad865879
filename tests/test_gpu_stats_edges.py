"""Selection statistics at the edges of the bf16 pass: ragged lengths, every
sub-block width, grouped queries, value norms that span many magnitudes (the
sums' references change from tile to tile, products of weight and norm leave
the range of float) and logits far apart, and the reference Top-K's list sizes,
words and ties; against the fp64 oracle."""
import numpy as np
import pytest

from oracle.stats import block_mass_topk, majority_vote
from paper_2609_13141_amd import configs, inputs, sas

from helpers import assert_close, f64
from test_gpu_stats import _bits, _clear_rows

pytestmark = pytest.mark.gpu


#                                              n   H Hkv dh   B   K  norms logits
@pytest.mark.parametrize("n,H,Hkv,dh,B,K,norms,logits", [
    (1, 2, 2, 128, 64, 1, 0, 1.0), (64, 2, 1, 64, 16, 2, 0, 1.0), (129, 3, 1, 128, 32, 2, 20, 1.0),
    (300, 2, 2, 64, 64, 2, 30, 4.0), (400, 2, 2, 128, 128, 1, 10, 1.0), (260, 2, 1, 128, 16, 4, 40, 4.0),
    (200, 2, 1, 128, 32, 2, 60, 16.0), (150, 1, 1, 64, 64, 1, 60, 30.0)])
def test_coverage(n, H, Hkv, dh, B, K, norms, logits):
    print(f"\n[case] stats n={n} H={H}/{Hkv} dh={dh} B={B} K={K} norms 2^+-{norms} logits x{logits}", flush=True)
    w = configs.L7B_1K.with_(seq_len=n, n_heads=H, n_kv_heads=Hkv, head_dim=dh, block_size=B, top_k=K,
                             segments=(("txt", n),), index=127)
    q, k, v = inputs.qkv(w)
    q = inputs.as_dtype(q * np.float32(logits), "bf16")
    r = np.random.default_rng(n)
    # one magnitude per key and group: norms are what the statistic weights by
    v = inputs.as_dtype(v * np.exp2(r.uniform(-norms, norms, v.shape[:3] + (1,))).astype(np.float32), "bf16")
    cfg = sas.make_config(w, "gated")
    dq, dk, dv = (sas.to_device(a, "bf16") for a in (q, k, v))
    sel = sas.attention_prefill(cfg, dq, dk, dv)["sel_idx"]
    out = sas.selection_stats(cfg, dq, dk, dv, sel)
    # a logit z (log2 domain, |z| up to some 8 x logits x 1.44) carries fp32 rounding of about
    # 2^-24 |z| from its dot product and again from z + log2 norm; that is the relative error
    # of its weight
    tol = max(2e-5, 2 * 2.0**-24 * (12 * logits + norms))
    Q, Kk, V, S = f64(q[0]), f64(k[0]), f64(v[0]), sel[0].cpu().numpy()
    for h in range(H):
        g = h // (H // Hkv)
        z = Q[:, h] @ Kk[:, g].T / np.sqrt(dh)
        vn = np.linalg.norm(V[:, g], axis=-1)
        cov, cov_v = np.zeros(n), np.zeros(n)
        for t in range(n):
            keep = np.array([j // B == t // B or j // B in S[g, t] for j in range(t + 1)])
            p = np.exp(z[t, :t + 1] - z[t, :t + 1].max())
            cov[t], cov_v[t] = p[keep].sum() / p.sum(), (p * vn[:t + 1])[keep].sum() / (p * vn[:t + 1]).sum()
        assert_close(out["cov"][0, h].cpu().numpy(), cov, "f32", f"cov {h}", tol=tol)
        assert_close(out["cov_v"][0, h].cpu().numpy(), cov_v, "f32", f"cov_v {h}", tol=tol)


@pytest.mark.parametrize("n,B,K", [(700, 16, 8), (700, 16, 9), (1200, 16, 32), (600, 64, 16), (100, 64, 4)])
def test_reference_topk(n, B, K):
    print(f"\n[case] reference Top-K n={n} B={B} K={K}", flush=True)
    w = configs.L7B_1K.with_(seq_len=n, n_heads=2, n_kv_heads=2, head_dim=64, block_size=B, top_k=K,
                             segments=(("txt", n),), index=128)
    q, k, v = inputs.qkv(w)
    cfg = sas.make_config(w, "gated")
    NB = -(-n // B)
    for zero in (False, True):
        dq, dk, dv = (sas.to_device(a, "bf16") for a in (q * 0 if zero else q, k, v))
        sel = sas.attention_prefill(cfg, dq, dk, dv)["sel_idx"]
        ru = sas.alloc_union(cfg, 1, n)
        sas.selection_stats(cfg, dq, dk, dv, sel, ref_union=ru)
        got = _bits(ru, NB)[0]
        if zero:  # every block's mass is the same: the lower blocks win
            want = np.arange(NB)[None] < np.minimum(K, np.arange(n) // B)[:, None]
            np.testing.assert_array_equal(got, np.stack([want, want]))
            continue
        hs, lmass = block_mass_topk(f64(q[0]), f64(k[0]), B, K)
        ok = _clear_rows(lmass, K, 1)
        assert ok.mean() > 0.9
        np.testing.assert_array_equal(got[ok], majority_vote(hs, 1)[ok])
