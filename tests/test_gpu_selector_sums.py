"""The selector backward's products at the edges of their tiles: 64-block and
32-row stages, a ragged last block, more blocks than a tile, split sums over t,
a batch summed into the projections' gradients, and which outputs are asked
for; against fp64.  fp32 operands: the error is that of fp32 sums of up to n
terms of mixed sign, 1e-5 of the largest; bf16 operands enter exactly, so the
same bound holds for both."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2609_13141_amd import configs, inputs, sas

from helpers import assert_close, f64

pytestmark = pytest.mark.gpu

#        dtype   b   n    H Hkv  dh  B   K
CASES = [("bf16", 1, 17, 2, 2, 64, 16, 2), ("bf16", 2, 1040, 2, 1, 128, 16, 4), ("bf16", 1, 1100, 3, 1, 64, 16, 8),
         ("bf16", 3, 333, 2, 2, 128, 64, 3), ("f32", 2, 300, 2, 1, 128, 32, 3)]


@pytest.mark.parametrize("proj", [False, True])
@pytest.mark.parametrize("dtype,b,n,H,Hkv,dh,B,K", CASES)
def test_selector_products(dtype, b, n, H, Hkv, dh, B, K, proj):
    print(f"\n[case] selector sums {dtype} b={b} n={n} H={H}/{Hkv} dh={dh} B={B} K={K} proj={proj}", flush=True)
    w = configs.TINY.with_(dtype=dtype, batch=b, seq_len=n, n_heads=H, n_kv_heads=Hkv, head_dim=dh, block_size=B,
                           top_k=K, segments=(("txt", n),), index=126)
    q, k, v = inputs.qkv(w)
    wgq = inputs.normal(w, "w_gq", (Hkv, dh, dh), 0.1) if proj else None
    wgk = inputs.normal(w, "w_gk", (Hkv, dh, dh), 0.1) if proj else None
    to = lambda a: None if a is None else sas.to_device(a, dtype)  # noqa: E731
    dev = [to(a) for a in (q, k, v, wgq, wgk)]
    cfg = sas.make_config(w, "gated")
    f = sas.attention_prefill(cfg, *dev, log_gate=True)
    dlg = torch.randn(b, Hkv, n, K, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda")
    full = sas.selector_backward(cfg, dev[0], dev[1], f["sel_idx"], f["log_gate"], dlg, dev[3], dev[4])
    few = sas.selector_backward(cfg, dev[0], dev[1], f["sel_idx"], f["log_gate"], dlg, dev[3], dev[4], ds=False,
                                dqhat=False, dkbar=False)
    G, NB, nf, c = H // Hkv, -(-n // B), n // B, 1.0 / (H // Hkv * math.sqrt(dh))
    dw = {"dw_gq": np.zeros((Hkv, dh, dh)), "dw_gk": np.zeros((Hkv, dh, dh))}
    for i in range(b):
        st = oracle.select(f64(q[i]), f64(k[i]), B, K, dtype, w_gq=None if not proj else f64(wgq),
                           w_gk=None if not proj else f64(wgk))
        sel, lg = f["sel_idx"][i].cpu().numpy(), f["log_gate"][i].double().cpu().numpy()
        dl = np.zeros((Hkv, n, NB))
        for g in range(Hkv):
            for t in range(n):
                for s in range(K):
                    if sel[g, t, s] >= 0:
                        dl[g, t, sel[g, t, s]] = float(dlg[i, g, t, s])
        ds = dl - np.exp(lg) * dl.sum(-1, keepdims=True)
        ds[np.isneginf(lg)] = 0.0
        assert_close(full["ds"][i].cpu().numpy(), ds, "f32", "ds")
        dq = c * np.einsum("gtm,gmj->gtj", ds[:, :, :nf], st["kbar_proj"])
        dk = np.zeros((Hkv, NB, dh))
        dk[:, :nf] = c * np.einsum("gtm,gtj->gmj", ds[:, :, :nf], st["qhat"])
        assert_close(full["dqhat"][i].cpu().numpy(), dq, "f32", "dqhat")
        assert_close(full["dkbar"][i].cpu().numpy(), dk, "f32", "dkbar")
        if proj:
            q0 = oracle.select(f64(q[i]), f64(k[i]), B, K, dtype)["qhat"]
            dw["dw_gq"] += np.einsum("gtk,gtj->gkj", dq, q0)
            dw["dw_gk"] += np.einsum("gmk,gmj->gkj", dk[:, :nf], st["kbar"])
    if proj:
        for name, want in dw.items():
            assert_close(full[name].cpu().numpy(), want, "f32", name)
            assert torch.equal(full[name], few[name])


@pytest.mark.parametrize("n,B,K,full", [(4096, 64, 16, False), (1100, 16, 8, True)])
def test_projection_gradient_of_keys_with_a_common_part(n, B, K, full):
    """Summaries that share a component many times their spread: the rows of ds
    add to zero, so the common part cancels out of dW_gq, and has to cancel
    before fp32 sums over the rows round it (the bound of this file; about 6e-6
    when it cancels row by row, 3e-5 when only the last sum over blocks does)."""
    print(f"\n[case] selector sums with offset n={n} B={B} K={K} full={full}", flush=True)
    dh = 128
    w = configs.TINY.with_(dtype="bf16", seq_len=n, n_heads=1, n_kv_heads=1, head_dim=dh, block_size=B, top_k=K,
                           segments=(("txt", n),), index=127)
    q, k, v = inputs.qkv(w)
    off = inputs.normal(w, "offset", (dh,), 40.0 / math.sqrt(B), dtype="f32")  # 40 times the summaries' spread
    k = (k + off).astype(np.float32)
    wgq = (np.eye(dh) + inputs.normal(w, "w_gq", (1, dh, dh), 0.02)).astype(np.float32)
    dev = [sas.to_device(a, "bf16") for a in (q, k, v, wgq)]
    cfg = sas.make_config(w, "gated", scope="full" if full else "sparse")
    f = sas.attention_prefill(cfg, *dev, log_gate=True)
    NB, nf = -(-n // B), n // B
    gen = torch.Generator(device="cuda").manual_seed(n)
    dlg = torch.randn(1, 1, n, NB if full else K, generator=gen, device="cuda")
    got = sas.selector_backward(cfg, dev[0], dev[1], f["sel_idx"], f["log_gate"], None if full else dlg, dev[3], None,
                                ds=False, dqhat=False, dkbar=False, dlog_gate_full=dlg if full else None)
    lg = f["log_gate"][0, 0].double().cpu()
    hist = torch.isfinite(lg)
    if full:
        dl = torch.where(hist, dlg[0, 0].double().cpu(), 0.0)
    else:
        sel = f["sel_idx"][0, 0].long().cpu()
        dl = torch.zeros(n, NB + 1, dtype=torch.float64)
        dl.scatter_(1, torch.where(sel >= 0, sel, NB), dlg[0, 0].double().cpu())
        dl = dl[:, :NB]
    ds = torch.where(hist, dl - lg.exp() * dl.sum(1, keepdim=True), 0.0)[:, :nf]
    q0 = torch.from_numpy(q[0, :, 0]).double()
    kb = f["k_summary"][0, 0, :nf].double().cpu()
    want = ((ds @ kb).T @ q0) / math.sqrt(dh)
    assert_close(got["dw_gq"][0].cpu().numpy(), want.numpy(), "f32", "dw_gq")
