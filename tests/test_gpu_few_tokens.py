"""GPU parity of the few-token stage (one launch between the gate/up and the down product): token, pair,
expert and rank counts at the edges of what it takes, forward and backward against the oracle; tolerance
as everywhere for bf16 storage (2e-2)."""
import numpy as np
import pytest
import torch

from oracle import mixlora_oracle as orc
from paper_2404_15159_amd import binding as B, synth
from paper_2404_15159_amd.runner import MixLoraFFN

import parity_utils as pu
from test_gpu_multi import compare_multi, run_multi

pytestmark = pytest.mark.gpu

BASE = synth.CONFIGS["llama2_7b"]

# T, d, d_ff, N, k, r: one and two tokens (the rank term in the matrix-vector launch) and more; 256 pairs; one,
# two, three, five experts (several waves per expert), 9, 17 and 32 (several experts per wave); ranks below 8, of 8
# and 16; a last column block of 16 columns is not possible here (d_ff is in whole 64-wide tiles but for T <= 2)
SHAPES = [(1, 256, 512, 8, 2, 16), (1, 264, 520, 5, 3, 4), (2, 256, 1032, 8, 4, 16), (2, 8320, 256, 9, 2, 8),
          (3, 192, 448, 8, 2, 16), (31, 256, 512, 1, 1, 16), (33, 256, 512, 3, 2, 12), (40, 256, 576, 17, 1, 16),
          (64, 192, 448, 32, 4, 8), (85, 256, 640, 5, 3, 16), (128, 256, 576, 8, 2, 16), (128, 128, 320, 2, 2, 2),
          (100, 576, 256, 9, 2, 8)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "T%d_d%d_f%d_N%d_k%d_r%d" % s)
def test_few_tokens_match_oracle(shape):
    T, d, f, N, k, r = shape
    cfg = synth.scaled(BASE, name="few", T=T, d=d, d_ff=f, N=N, k=k, r=r, alpha=2.0 * r)
    print(f"case few {shape}", flush=True)
    host = synth.make_inputs(cfg)
    m = MixLoraFFN(cfg, host)
    m.workspace.fill_(0xFF)          # NaN patterns: nothing may be read before it is written
    m.forward()
    m.backward(d_aux=1.0)
    res = m.results()
    W = {n: host[n] for n in synth.WEIGHT_NAMES}
    bw = orc.backward(host["x"], W, cfg.k, cfg.lora_scale, host["dy"], 1.0, cfg.aux_coeff, "top1")
    if T >= 16:
        pu.compare_all(res, bw["forward"], bw, cfg)
    else:   # (with fewer tokens the router gradient is a difference of nearly equal bf16 numbers)
        pu.compare_all(res, bw["forward"], None, cfg)
        for n in pu.GRAD_NAMES[:-1]:
            pu.assert_close(n, res[n], bw[n], 2e-2)
    # a workspace for the forward alone: the same results
    one = MixLoraFFN(cfg, host, with_backward=False)
    one.workspace.fill_(0xFF)
    one.forward()
    for n in ("y", "topk_idx", "topk_w", "counts", "aux_loss"):
        assert np.array_equal(res[n], one.results()[n]), n


def test_one_expert_takes_all_tokens():
    cfg = synth.scaled(BASE, name="few_skew", T=96, d=256, d_ff=512, N=8, k=2, r=16, structure="skew0")
    host = synth.make_inputs(cfg)
    host["W_router"][0, -1] += 30.0          # every token's first choice
    m = MixLoraFFN(cfg, host, with_backward=False)
    m.workspace.fill_(0xFF)
    m.forward()
    assert int(m.counts[0]) == cfg.T
    W = {n: host[n] for n in synth.WEIGHT_NAMES}
    pu.compare_all(m.results(), orc.forward(host["x"], W, cfg.k, cfg.lora_scale, cfg.aux_coeff, "top1"), None, cfg)


@pytest.mark.parametrize("T,M,N,pattern", [(120, 3, 5, "skip_last"), (60, 2, 8, "uneven"), (2, 2, 8, "round_robin")])
def test_few_tokens_of_several_adapters(T, M, N, pattern):
    cfg = synth.scaled(BASE, name="few_multi", T=T, d=256, d_ff=512, N=N, k=2, r=8, alpha=16.0, M=M, seq_len=max(1, T // 10))
    host = synth.make_inputs(cfg)
    if T < 16:
        tm = synth.token_model(cfg, pattern)
        m = MixLoraFFN(cfg, host, token_model=tm)
        m.forward()
        fw = orc.multi_forward(host["x"], tm, synth.split_adapters(cfg, host), cfg.k, cfg.lora_scale, cfg.aux_coeff, "top1")
        pu.assert_close("y", m.results()["y"], fw["y"], 2e-2)
        return
    res, fw, bw, tm = run_multi(cfg, host, pattern)
    compare_multi(res, fw, bw, cfg, tm)


@pytest.mark.parametrize("T", [2, 40])
def test_non_finite_logits_stay_to_themselves(T):
    """As for longer batches: such a token goes to k different experts, every other token's outputs are those
    of a clean batch."""
    cfg = synth.scaled(BASE, name="few_nonfinite", T=T, d=256, d_ff=768, N=8, k=2, r=8, alpha=16.0)
    host = synth.make_inputs(cfg)
    host["W_router"][:, 0] = 0.015625       # one feature that reaches every logit with the same sign
    bad = {0: (0, -np.inf)}
    if T > 2:
        bad = {0: (slice(None), np.nan), T // 3: (0, np.inf), T // 2: (0, -np.inf), T - 1: (3, np.inf)}
    clean, dirty = host["x"].copy(), host["x"].copy()
    for t, (col, v) in bad.items():
        clean[t] = 0.0
        dirty[t, col] = v
    rest = np.setdiff1d(np.arange(T), list(bad))
    out = []
    for x in (clean, dirty):
        m = MixLoraFFN(cfg, dict(host, x=x))
        m.workspace.fill_(0)
        m.forward()
        idx = m.topk_idx.cpu().numpy()
        assert ((idx >= 0) & (idx < cfg.N)).all() and (idx[:, 0] != idx[:, 1]).all()
        assert int(m.counts.sum()) == cfg.k * T
        m.backward(d_aux=0.0)
        out.append(m.results())
    assert np.isnan(out[1]["topk_w"][list(bad)]).all()
    for n in ("topk_idx", "topk_w", "y", "dx"):
        assert np.array_equal(out[0][n][rest], out[1][n][rest]), n


def test_capture_and_replay():
    cfg = synth.scaled(BASE, name="few_graph", T=24, d=256, d_ff=512, N=8, k=2, r=16)
    host = synth.make_inputs(cfg)
    m = MixLoraFFN(cfg, host, with_backward=False)
    m.forward()
    ref = m.results()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        m.forward()
    for _ in range(3):
        m.y.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(m.results()["y"], ref["y"])


@pytest.mark.parametrize("T,f", [(2, 512), (40, 768), (128, 512), (300, 768), (1100, 4648)])
def test_backward_does_not_depend_on_the_size_named_to_the_forward(T, f):
    """The forward may be told of the forward's own workspace size: in the same (larger) buffer it leaves all that a
    backward pass reads, also beside the two stages above that end in the weighted combination."""
    cfg = synth.scaled(BASE, name="few_ws", T=T, d=64, d_ff=f, N=8, k=2, r=16)
    host = synth.make_inputs(cfg)
    out = []
    for size in (B.mixlora_workspace_bytes(MixLoraFFN(cfg, host).dims, True),
                 B.mixlora_workspace_bytes(MixLoraFFN(cfg, host).dims, False)):
        print(f"case T={T} f={f} size={size}", flush=True)
        m = MixLoraFFN(cfg, host)
        m.workspace.fill_(0xFF)
        whole, m.ws_bytes = m.ws_bytes, size
        m.forward()
        m.ws_bytes = whole
        m.backward(d_aux=1.0)
        out.append(m.results())
    for n in ("dx",) + pu.GRAD_NAMES:
        assert np.isfinite(out[1][n]).all() and np.array_equal(out[0][n], out[1][n]), n
