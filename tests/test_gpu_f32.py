"""The fp32 kernels at the edges of their tiles (16 rows, 16 or 32 columns, 16
keys, K split over four waves): the MLP's two products and the attention in
every mode, against fp64.  Sums are fp32 chains of at most K / 4 terms joined
by three additions, so errors stay far below the 1e-5 of the dtype."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_13141_amd import configs, inputs, sas

from helpers import assert_close, f64, spec_of

pytestmark = pytest.mark.gpu


#                    T     d   d_ff
@pytest.mark.parametrize("T,d,F", [(1, 8, 8), (15, 40, 24), (17, 264, 72), (33, 256, 688), (600, 72, 2056),
                                   (2048, 256, 688)])
def test_mlp_f32(T, d, F):
    print(f"\n[case] f32 mlp T={T} d={d} F={F}", flush=True)
    w = configs.TINY.with_(d_model=d, d_ff=F, index=91)
    cfg = sas.make_config(w, "dense")
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn(T, d, generator=g, device="cuda")
    W = {"rms2": torch.randn(d, generator=g, device="cuda"),
         "w_gate": torch.randn(F, d, generator=g, device="cuda") * 0.1,
         "w_up": torch.randn(F, d, generator=g, device="cuda") * 0.1,
         "w_down": torch.randn(d, F, generator=g, device="cuda") * 0.1}
    y = sas.mlp_forward(cfg, x, W)
    D = {k: v.double().cpu() for k, v in W.items()}
    xd = x.double().cpu()
    u = xd * torch.rsqrt(xd.square().mean(-1, keepdim=True) + w.rms_eps) * D["rms2"]
    ref = xd + (torch.nn.functional.silu(u @ D["w_gate"].T) * (u @ D["w_up"].T)) @ D["w_down"].T
    assert_close(y.cpu().numpy(), ref.numpy(), "f32", "mlp")


@pytest.mark.parametrize("mode", ["gated", "sparse", "dense"])
@pytest.mark.parametrize("n,H,Hkv,dh,B,K", [(1, 2, 2, 64, 16, 1), (15, 2, 1, 128, 16, 2), (17, 2, 2, 64, 16, 1),
                                            (160, 7, 1, 64, 16, 3), (210, 2, 2, 128, 64, 1), (270, 2, 1, 64, 128, 2)])
def test_attention_f32(n, H, Hkv, dh, B, K, mode):
    print(f"\n[case] f32 attention n={n} H={H}/{Hkv} dh={dh} B={B} K={K} {mode}", flush=True)
    w = configs.TINY.with_(batch=2, seq_len=n, n_heads=H, n_kv_heads=Hkv, head_dim=dh, block_size=B, top_k=K,
                           mode=mode, segments=(("txt", n),), index=92)
    q, k, v = inputs.qkv(w)
    out = sas.attention_prefill(sas.make_config(w, mode), *(sas.to_device(a, "f32") for a in (q, k, v)))
    ref = oracle.attention_prefill(f64(q), f64(k), f64(v), spec_of(w, mode))
    assert_close(out["o"].cpu().numpy(), ref["O_exact"], "f32", "O")
    assert_close(out["lse"].cpu().numpy(), ref["LSE"], "f32", "LSE")


@pytest.mark.parametrize("dh", [64, 128])
def test_attention_f32_keeps_values_outside_the_attended_set_out(dh):
    """A non-finite value reaches exactly the queries that attend its key."""
    n, B = 40, 16
    w = configs.TINY.with_(batch=1, seq_len=n, n_heads=2, n_kv_heads=2, head_dim=dh, block_size=B, top_k=1,
                           mode="sparse", segments=(("txt", n),), index=93)
    q, k, v = inputs.qkv(w)
    cfg = sas.make_config(w, "sparse")
    dq, dk, dv = (sas.to_device(a, "f32") for a in (q, k, v))
    clean = sas.attention_prefill(cfg, dq, dk, dv)
    sel = clean["sel_idx"].cpu().numpy()
    for key in (5, 20):
        bad = dv.clone()
        bad[:, key] = float("inf")
        out = sas.attention_prefill(cfg, dq, dk, bad)["o"].cpu().numpy()
        for h in range(2):
            for t in range(n):
                attends = key <= t and (t // B == key // B or key // B in sel[0, h, t])
                if attends:
                    assert not np.isfinite(out[0, t, h]).any(), (key, h, t)
                else:
                    assert_close(out[0, t, h], clean["o"][0, t, h].cpu().numpy(), "f32", f"key {key} head {h} row {t}")
