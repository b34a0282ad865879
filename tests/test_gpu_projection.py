"""The selector's learned projections on the GPU: projected summaries and the
selection from projected gate queries, bit-exact against the fp64 oracle at
row counts around the kernel's 64-row tiles (one tile per workgroup), and with
two to four tiles per workgroup (2048 tiles and more over all sequences and
groups) bit-equal to the same sequences one by one."""
import numpy as np
import pytest
import torch

from oracle.selector import normalized_log_gate, select
from paper_2609_13141_amd import configs, inputs, sas

from helpers import assert_close_with_infs, f64

pytestmark = pytest.mark.gpu

#        dtype   b   n   H Hkv dh   B   K
CASES = [("bf16", 1, 1, 2, 2, 128, 16, 2), ("bf16", 2, 63, 2, 1, 64, 16, 2), ("bf16", 1, 64, 4, 4, 128, 16, 3),
         ("bf16", 1, 65, 7, 1, 128, 16, 3), ("bf16", 2, 1100, 4, 2, 128, 16, 8), ("f32", 1, 129, 2, 2, 64, 16, 3),
         ("f32", 1, 200, 4, 2, 128, 32, 2)]


@pytest.mark.parametrize("dtype,b,n,H,Hkv,dh,B,K", CASES)
def test_projected_selection_is_exact(dtype, b, n, H, Hkv, dh, B, K):
    print(f"\n[case] projection {dtype} b={b} n={n} H={H}/{Hkv} dh={dh} B={B} K={K}", flush=True)
    w = configs.TINY.with_(dtype=dtype, batch=b, seq_len=n, n_heads=H, n_kv_heads=Hkv, head_dim=dh, block_size=B,
                           top_k=K, segments=(("txt", n),), index=90)
    q, k, v = inputs.qkv(w)
    wgq = inputs.normal(w, "w_gq", (Hkv, dh, dh), 0.1)
    wgk = inputs.normal(w, "w_gk", (Hkv, dh, dh), 0.1)
    cfg = sas.make_config(w, "gated")
    dev = [sas.to_device(a, dtype) for a in (q, k, v, wgq, wgk)]
    out = sas.attention_prefill(cfg, *dev, log_gate=True)
    torch.cuda.synchronize()
    NB = -(-n // B)
    for i in range(b):
        ref = select(f64(q[i]), f64(k[i]), B, K, dtype, w_gq=f64(wgq), w_gk=f64(wgk))
        np.testing.assert_array_equal(out["sel_idx"][i].cpu().numpy(), ref["sel"])
        nf = n // B
        got = out["k_summary"][i].float().cpu().numpy()
        np.testing.assert_array_equal(got[:, :nf], ref["kbar_proj"])
        assert not got[:, nf:].any()  # incomplete blocks
        lg = np.full((Hkv, n, NB), -np.inf)
        lg[:, :, :nf] = normalized_log_gate(ref["r"], ref["ct"], H // Hkv, dh)
        # scores are exact: the gate differs by its fp32 rounding and the fp32 sum of the normalizer
        assert_close_with_infs(out["log_gate"][i].cpu().numpy(), lg, dtype, "log_gate", tol=1e-5)


@pytest.mark.parametrize("dtype,b,n,dh,tiles", [("bf16", 4, 1090, 64, 2), ("bf16", 6, 1090, 128, 3),
                                                ("f32", 8, 1090, 64, 4), ("f32", 4, 1037, 128, 2)])
def test_several_tiles_per_workgroup(dtype, b, n, dh, tiles):
    H = 32
    print(f"\n[case] projection tiles {dtype} b={b} n={n} dh={dh}: {tiles} per workgroup", flush=True)
    assert -(-n // 64) * b * H // 1024 == tiles and -(-n // 64) * H // 1024 == 0
    w = configs.TINY.with_(dtype=dtype, batch=b, seq_len=n, n_heads=H, n_kv_heads=H, head_dim=dh, block_size=16,
                           top_k=4, segments=(("txt", n),), index=91)
    dev = [sas.to_device(a, dtype) for a in inputs.qkv(w)]
    wgq = sas.to_device(inputs.normal(w, "w_gq", (H, dh, dh), 0.1), dtype)
    cfg = sas.make_config(w, "gated")
    out = sas.attention_prefill(cfg, *dev, wgq, log_gate=True, tau=True)
    for i in range(b):
        one = sas.attention_prefill(cfg, *(t[i:i + 1].contiguous() for t in dev), wgq, log_gate=True, tau=True)
        for f in ("sel_idx", "log_gate", "tau"):
            assert torch.equal(out[f][i], one[f][0]), (f, i)
