"""The backward of the full scope with grouped queries when blocks are masked:
score noise of -inf, or of the lowest float, gives every row of a wave a block
whose gate is zero.  Such a block's log-gate gradient is 0 and has to be written
(the scratch memory is NaN beforehand), and the selector's gradients follow from
it; against the fp64 oracle, for blocks within and across the 64-key tiles."""
import numpy as np
import pytest
import torch

from oracle.variants import gate_backward_act, select_variant, variant_attention_backward
from paper_2609_13141_amd import configs, inputs, sas

from helpers import assert_close, f64

pytestmark = pytest.mark.gpu

#        n   H Hkv dh   B
CASES = [(200, 4, 1, 64, 16), (330, 7, 1, 128, 64), (450, 4, 2, 64, 128), (450, 7, 1, 128, 128)]


@pytest.mark.parametrize("mask", [-np.inf, np.finfo(np.float32).min], ids=["inf", "lowest"])
@pytest.mark.parametrize("n,H,Hkv,dh,B", CASES)
def test_masked_blocks_get_a_zero_gradient(n, H, Hkv, dh, B, mask):
    print(f"\n[case] masked backward n={n} H={H}/{Hkv} dh={dh} B={B} mask={mask}", flush=True)
    K = 2
    w = configs.L7B_1K.with_(seq_len=n, n_heads=H, n_kv_heads=Hkv, head_dim=dh, block_size=B, top_k=K,
                             segments=(("txt", n),), index=160)
    q, k, v = inputs.qkv(w)
    d_o = inputs.normal(w, "d_o", q.shape, 1.0)
    NB, nf = -(-n // B), n // B
    eps = np.zeros((1, Hkv, n, NB), np.float32)
    masked = np.arange(NB) * B // max(B, 64) % 2 == 1
    eps[..., masked] = mask                   # every second key tile (or block), for every row; block 0 stays
    cfg = sas.make_config(w, "gated", scope="full")
    dev = [sas.to_device(a, "bf16") for a in (q, k, v, d_o)]
    fw = sas.attention_prefill(cfg, *dev[:3], log_gate=True, noise=torch.from_numpy(eps).cuda())
    ws = sas.Workspace()
    ws.buf = torch.full((1 << 24,), float("nan"), device="cuda").view(torch.uint8)
    assert ws.buf.numel() >= sas.workspace_size(cfg, sas.OP_ATTENTION_BACKWARD, 1, n)
    bw = sas.attention_backward(cfg, *dev[:3], fw["o"], dev[3], fw["lse"], fw["sel_idx"], fw["log_gate"],
                                dlog_gate=False, dlog_gate_full=True, ws=ws)
    sb = sas.selector_backward(cfg, dev[0], dev[1], None, fw["log_gate"], None, dlog_gate_full=bw["dlog_gate_full"])
    torch.cuda.synchronize()
    st = select_variant(f64(q[0]), f64(k[0]), B, K, "bf16", act="softmax", noise=f64(eps[0]))
    dQ, dK, dV, dLG = variant_attention_backward(f64(q[0]), f64(k[0]), f64(v[0]), f64(d_o[0]), B, st["sel"],
                                                 st["log_gate"], "inner", "full", False)
    got = bw["dlog_gate_full"][0].cpu().numpy()
    assert np.all(got[:, :, masked] == 0), "gradient of a masked block"
    assert_close(got, dLG, "bf16", "dlog_gate_full")
    assert_close(bw["dq"][0].float().cpu().numpy(), dQ, "bf16", "dQ")
    assert_close(bw["dk"][0].float().cpu().numpy(), dK, "bf16", "dK")
    assert_close(bw["dv"][0].float().cpu().numpy(), dV, "bf16", "dV")
    ds = gate_backward_act(dLG[:, :, :nf], st["s"], st["ct"], "softmax")
    assert_close(sb["ds"][0, :, :, :nf].cpu().numpy(), ds, "bf16", "ds")
    assert torch.isfinite(sb["dqhat"]).all() and torch.isfinite(sb["dkbar"]).all()
