"""Scratch memory for partial sums is optional: with a smaller workspace a call
divides less, down to not at all, and gives the same result but for the order of
fp32 sums; below that it is refused before anything is written."""
import pytest
import torch

from paper_2609_13141_amd import configs, inputs, sas

from helpers import assert_close

pytestmark = pytest.mark.gpu


class Fixed(sas.Workspace):
    """A workspace of a fixed number of bytes, whatever is asked for; a guard follows it."""

    def __init__(self, nbytes):
        super().__init__()
        self.n = nbytes
        self.buf = torch.full((nbytes + 4096,), 0x5A, dtype=torch.uint8, device="cuda")

    def get(self, nbytes):
        return self.buf, self.n

    def intact(self):
        return bool((self.buf[self.n:] == 0x5A).all())


def shrink(full, run, check):
    """Runs with less and less scratch until it is refused; at least two smaller sizes have to work."""
    ran = 0
    for part in (0.999, 0.9, 0.8, 0.7, 0.6, 0.5, 0.4, 0.3, 0.2, 0.1, 0.05, 0.01):
        ws = Fixed(int(full * part) // 16 * 16)
        try:
            out = run(ws)
        except sas.SasError as e:
            assert e.status == sas.SAS_ERR_WORKSPACE
            assert ran >= 2, f"refused at {part} of the workspace"
            return
        torch.cuda.synchronize()
        assert ws.intact()
        check(out)
        ran += 1
    raise AssertionError("never refused")


def test_attention_backward_with_less_scratch():
    w = configs.L7B_1K.with_(seq_len=1500, n_heads=7, n_kv_heads=1, top_k=8, segments=(("txt", 1500),), index=161)
    print("\n[case] attention backward, shrinking workspace", flush=True)
    cfg = sas.make_config(w)
    dev = [sas.to_device(a, "bf16") for a in (*inputs.qkv(w), inputs.normal(w, "d_o", (1, 1500, 7, 128), 1.0))]
    f = sas.attention_prefill(cfg, *dev[:3], log_gate=True)
    run = lambda ws: sas.attention_backward(cfg, *dev[:3], f["o"], dev[3], f["lse"], f["sel_idx"],  # noqa: E731
                                            f["log_gate"], ws=ws)
    full = sas.workspace_size(cfg, sas.OP_ATTENTION_BACKWARD, 1, 1500)
    best = {k: v.float().cpu() for k, v in run(Fixed(full)).items()}

    def check(out):
        assert torch.equal(out["dq"].float().cpu(), best["dq"])
        assert torch.equal(out["dlog_gate"].cpu(), best["dlog_gate"])
        for k in ("dk", "dv"):  # fp32 sums in another order, rounded to bf16: an ulp here and there
            assert_close(out[k].float().cpu().numpy(), best[k].numpy(), "bf16", k, tol=2 ** -8)

    shrink(full, run, check)


@pytest.mark.parametrize("what", ["mlp", "layer"])
def test_split_products_with_less_scratch(what):
    T = 300
    w = configs.L7B_1K.with_(seq_len=T, d_model=512, n_heads=4, n_kv_heads=2, d_ff=8192, segments=(("txt", T),),
                             index=162)
    print(f"\n[case] split products, shrinking workspace: {what}", flush=True)
    cfg = sas.make_config(w, "dense")
    W = sas.weights_to_device(inputs.layer_weights(w), "bf16")
    x = sas.to_device(inputs.embeddings(w), "bf16")
    if what == "mlp":
        run = lambda ws: sas.mlp_forward(cfg, x, W, ws=ws)  # noqa: E731
        full = sas.workspace_size(cfg, sas.OP_MLP, T, 0)
    else:
        run = lambda ws: sas.layer_forward(cfg, x, W, stats=False, ws=ws)["y"]  # noqa: E731
        full = sas.workspace_size(cfg, sas.OP_LAYER, 1, T)
    best = run(Fixed(full)).float().cpu().numpy()
    # sums in another order before each product's rounding to bf16
    shrink(full, run, lambda y: assert_close(y.float().cpu().numpy(), best, "bf16", what, tol=2 ** -7))
