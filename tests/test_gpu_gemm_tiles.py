"""The tiled products over every tile shape, with K whole and split over
workgroups, for each epilogue (SwiGLU, residual, QKV with rotary pairs and
pages), ragged rows and columns, against fp64.  The split adds up to 8 fp32
partial sums in order: far below the bf16 tolerance."""
import pytest
import torch

from paper_2609_13141_amd import configs, sas

from helpers import assert_close

pytestmark = pytest.mark.gpu


def draw(seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return lambda *s, std=1.0: (torch.randn(*s, generator=g, device="cuda") * std).bfloat16()


# (tokens, d, d_ff): the tiles and splits of gate/up and down that the launch takes there
MLP = [(65, 256, 4096),     # 128x128; 128x128 in 6
       (130, 2048, 256),    # 128x128 in several; 128x128
       (200, 1096, 2056),   # columns that end inside a tile (and K % 64 != 0: the register-staged kernel)
       (700, 2048, 8192),   # 256x256; 256x128 in 5
       (2100, 1024, 8192),  # one round of 256x256 and 256x128 for the other columns; 128x256 in 3
       (1300, 3584, 8192),  # 256x128; 256x256 in 3
       (700, 256, 11000),   # one round of 256x256 and 256x128 for the other columns, ragged; K % 64 != 0
       (520, 3072, 12288),  # 128x256 in 4
       (300, 128, 128)]


@pytest.mark.parametrize("T,d,F", MLP)
def test_mlp_tiles(T, d, F):
    print(f"\n[case] mlp tiles T={T} d={d} F={F}", flush=True)
    n = draw(T)
    w = configs.L7B_1K.with_(d_model=d, d_ff=F)
    W = {"rms2": 1 + n(d, std=0.1), "w_gate": n(F, d, std=d ** -0.5), "w_up": n(F, d, std=d ** -0.5),
         "w_down": n(d, F, std=F ** -0.5)}
    x = n(T, d)
    y = [sas.mlp_forward(sas.make_config(w, "dense"), x, W) for _ in range(2)]
    D = {k: v.double() for k, v in W.items()}
    xd = x.double()
    u = xd * torch.rsqrt(xd.square().mean(-1, keepdim=True) + w.rms_eps) * D["rms2"]
    ref = xd + (torch.nn.functional.silu(u @ D["w_gate"].T) * (u @ D["w_up"].T)) @ D["w_down"].T
    assert_close(y[0].float().cpu().numpy(), ref.cpu().numpy(), "bf16", "mlp")
    assert torch.equal(y[0], y[1])


@pytest.mark.parametrize("b,n,d,H,Hkv,dh", [(1, 100, 2048, 4, 2, 64), (2, 75, 4096, 2, 1, 128), (3, 150, 512, 7, 1, 128),
                                            (1, 600, 3072, 16, 4, 128),
                                            (1, 1400, 256, 64, 16, 128)])  # the last in two launches of columns
def test_qkv_tiles(b, n, d, H, Hkv, dh):
    print(f"\n[case] qkv tiles b={b} n={n} d={d} H={H}/{Hkv} dh={dh}", flush=True)
    r = draw(n)
    w = configs.L7B_1K.with_(d_model=d, d_ff=256, n_heads=H, n_kv_heads=Hkv, head_dim=dh, block_size=16, top_k=2)
    std = d ** -0.5
    W = {"rms1": 1 + r(d, std=0.1), "wq": r(H * dh, d, std=std), "wk": r(Hkv * dh, d, std=std),
         "wv": r(Hkv * dh, d, std=std), "wo": r(d, H * dh, std=std), "rms2": 1 + r(d, std=0.1),
         "w_gate": r(256, d, std=std), "w_up": r(256, d, std=std), "w_down": r(d, 256, std=0.05)}
    x = r(b, n, d)
    cfg = sas.make_config(w, "dense")
    cache = sas.alloc_cache(cfg, b, n, page_size=16)
    out = sas.layer_forward(cfg, x, W, taps=True, cache=cache)
    xd = x.double()
    u = xd * torch.rsqrt(xd.square().mean(-1, keepdim=True) + w.rms_eps) * W["rms1"].double()
    h = dh // 2
    a = torch.arange(n, device="cuda").double()[:, None, None] * \
        (w.rope_base ** (-torch.arange(h, device="cuda", dtype=torch.float64) / h))
    for name, rot in (("q", True), ("k", True), ("v", False)):
        t = (u.view(b * n, d) @ W["w" + name].double().T).view(b, n, -1, dh)
        if rot:
            t = torch.cat((t[..., :h] * a.cos() - t[..., h:] * a.sin(), t[..., h:] * a.cos() + t[..., :h] * a.sin()), -1)
        assert_close(out[name].float().cpu().numpy(), t.cpu().numpy(), "bf16", name)
        if name != "q":
            pages = cache.k_pages if name == "k" else cache.v_pages
            pos = torch.arange(n, device="cuda")
            for i in range(b):  # the pages hold the same bits as the contiguous rows
                got = pages[cache.block_table[i].long()[pos // 16], :, pos % 16]
                assert torch.equal(got, out[name][i])
    o = out["o"].double().view(b, n, -1)
    h1 = xd + (o.view(b * n, -1) @ W["wo"].double().T).view(b, n, d)
    assert_close(out["h1"].float().cpu().numpy(), h1.cpu().numpy(), "bf16", "h1")
