"""Products of 1 to 64 rows (the weight-streaming kernel, its 16-row tiles and
column-group choices) and the first row count past them, through the MLP, the
decode step and the prefill into a cache.  bf16 results differ between tilings
by the order of fp32 sums only: the dtype's tolerance is far above that."""
import pytest
import torch

from paper_2609_13141_amd import configs, sas

from helpers import assert_close

pytestmark = pytest.mark.gpu


def weights(w, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = lambda *s: (torch.randn(*s, generator=g, device="cuda") * 0.05).bfloat16()  # noqa: E731
    d, H, Hkv, dh, F = w.d_model, w.n_heads, w.n_kv_heads, w.head_dim, w.d_ff
    return {"rms1": 1 + n(d), "wq": n(H * dh, d), "wk": n(Hkv * dh, d), "wv": n(Hkv * dh, d), "wo": n(d, H * dh),
            "rms2": 1 + n(d), "w_gate": n(F, d), "w_up": n(F, d), "w_down": n(d, F)}


def W_(**kw):
    return configs.L7B_1K.with_(**{**dict(d_model=256, n_heads=4, n_kv_heads=2, head_dim=64, d_ff=640, block_size=16,
                                          top_k=32, rope_base=1000.0, index=94), **kw})


@pytest.mark.parametrize("d,F", [(128, 128), (384, 4096 + 128), (1152, 256)])
@pytest.mark.parametrize("T", [1, 16, 17, 32, 33, 48, 49, 64, 65])
def test_mlp_rows(T, d, F):
    print(f"\n[case] mlp T={T} d={d} F={F}", flush=True)
    w = W_(d_model=d, d_ff=F)
    W = weights(w, T)
    x = torch.randn(T, d, generator=torch.Generator(device="cuda").manual_seed(d), device="cuda").bfloat16()
    y = sas.mlp_forward(sas.make_config(w, "dense"), x, W)
    D = {k: v.double().cpu() for k, v in W.items()}
    xd = x.double().cpu()
    u = xd * torch.rsqrt(xd.square().mean(-1, keepdim=True) + w.rms_eps) * D["rms2"]
    ref = xd + (torch.nn.functional.silu(u @ D["w_gate"].T) * (u @ D["w_up"].T)) @ D["w_down"].T
    assert_close(y.float().cpu().numpy(), ref.numpy(), "bf16", "mlp")


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("b", [17, 40, 64, 65])
def test_decode_rows_match_small_batches(b, packed):
    """A step of b sequences against the same sequences in steps of 8 (every
    block is kept, so that no near-tie separates them)."""
    print(f"\n[case] decode rows b={b} packed={packed}", flush=True)
    w = W_()
    cfg = sas.make_config(w, "sparse")
    W = weights(w, b)
    if packed:
        W = sas.pack_decode_weights(cfg, W)
    g = torch.Generator(device="cuda").manual_seed(b)
    ctx = 80
    whole = sas.alloc_cache(cfg, b, ctx, page_size=16)
    whole.k_pages.copy_(torch.randn(whole.k_pages.shape, generator=g, device="cuda"))
    whole.v_pages.copy_(torch.randn(whole.v_pages.shape, generator=g, device="cuda"))
    whole.k_summary.copy_(torch.randn(whole.k_summary.shape, generator=g, device="cuda"))
    x = torch.randn(b, w.d_model, generator=g, device="cuda").bfloat16()
    pos = (48 + torch.arange(b, device="cuda", dtype=torch.int32) % 32).contiguous()  # some complete a block
    parts = sas.PagedCache(whole.k_pages.clone(), whole.v_pages.clone(), whole.block_table, whole.k_summary.clone(), 16)
    y, sel, tap = sas.decode_step(cfg, x, pos, W, whole, taps=True)
    for i in range(0, b, 8):
        j = min(b, i + 8)
        sub = sas.PagedCache(parts.k_pages, parts.v_pages, parts.block_table[i:j].contiguous(),
                             parts.k_summary[i:j].contiguous(), 16)
        yi, si, ti = sas.decode_step(cfg, x[i:j].contiguous(), pos[i:j].contiguous(), W, sub, taps=True)
        parts.k_summary[i:j] = sub.k_summary
        assert torch.equal(sel[i:j], si)
        assert_close(y[i:j].float().cpu().numpy(), yi.float().cpu().numpy(), "bf16", f"y {i}")
        for f in ("q", "k", "v", "h1"):
            assert_close(tap[f][i:j].float().cpu().numpy(), ti[f].float().cpu().numpy(), "bf16", f"{f} {i}")
    for f in ("k_pages", "v_pages", "k_summary"):
        assert_close(getattr(whole, f).float().cpu().numpy(), getattr(parts, f).float().cpu().numpy(), "bf16", f)


@pytest.mark.parametrize("b,n", [(1, 1), (3, 19), (4, 16)])
def test_short_prefill_is_a_prefix_of_a_longer_one(b, n):
    print(f"\n[case] short prefill b={b} n={n}", flush=True)
    w = W_()
    cfg = sas.make_config(w, "dense")
    W = weights(w, n)
    x = torch.randn(b, 70, w.d_model, generator=torch.Generator(device="cuda").manual_seed(n),
                    device="cuda").bfloat16()
    long = sas.alloc_cache(cfg, b, 96, page_size=16)
    short = sas.alloc_cache(cfg, b, 96, page_size=16)
    yl = sas.layer_forward(cfg, x, W, stats=False, cache=long)["y"]
    ys = sas.layer_forward(cfg, x[:, :n].contiguous(), W, stats=False, cache=short)["y"]
    assert_close(ys.float().cpu().numpy(), yl[:, :n].float().cpu().numpy(), "bf16", "y")
    for f in ("k_pages", "v_pages"):
        for i in range(b):
            for p in range(n):
                page = int(short.block_table[i, p // 16])
                assert_close(getattr(short, f)[page, :, p % 16].float().cpu().numpy(),
                             getattr(long, f)[page, :, p % 16].float().cpu().numpy(), "bf16", f"{f} {i} {p}")
    nf = n // 16
    assert_close(short.k_summary[:, :, :nf].float().cpu().numpy(), long.k_summary[:, :, :nf].float().cpu().numpy(),
                 "bf16", "summaries")
