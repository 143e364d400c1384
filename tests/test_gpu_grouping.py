"""GPU parity of routing and grouping in workgroups that count all experts at once: token counts around a
wave's 64, around the limit up to which every workgroup routes for itself, and the largest the launch takes;
eight and sixteen experts and odd numbers of them; one to four slots; several adapters.  Tables are pinned
through the outputs: indices and counts exactly, y, gradients and the auxiliary loss against the oracle."""
import numpy as np
import pytest

from oracle import mixlora_oracle as orc
from paper_2404_15159_amd import synth
from paper_2404_15159_amd.runner import MixLoraFFN

import parity_utils as pu
from test_gpu_multi import compare_multi, run_multi

pytestmark = pytest.mark.gpu

SHAPES = [("llama2_7b", 129, 8, 2), ("llama2_7b", 1024, 8, 2), ("llama2_7b", 1025, 8, 2), ("llama2_7b", 1087, 7, 3),
          ("llama2_7b", 4096, 8, 2), ("llama2_7b", 2048, 16, 4), ("llama2_7b", 300, 13, 2), ("llama2_7b", 8192, 4, 1),
          ("llama2_7b", 200, 17, 2), ("tiny_f32", 63, 5, 4), ("tiny_f32", 1030, 16, 2), ("tiny_f32", 200, 9, 5)]


@pytest.mark.parametrize("base,T,N,k", SHAPES)
def test_grouping_matches_oracle(base, T, N, k):
    cfg = synth.scaled(synth.CONFIGS[base], name="grouping", T=T, d=64, d_ff=136, N=N, k=k, r=8, alpha=16.0)
    print(f"case {base} T={T} N={N} k={k}", flush=True)
    host = synth.make_inputs(cfg)
    host["W_router"] = synth._store(host["W_router"] * 8.0, cfg.dtype)
    m = MixLoraFFN(cfg, host)
    m.workspace.fill_(0xFF)          # NaN patterns: nothing may be read before it is written
    m.forward()
    m.backward(d_aux=1.0)
    W = {n: host[n] for n in synth.WEIGHT_NAMES}
    bw = orc.backward(host["x"], W, cfg.k, cfg.lora_scale, host["dy"], 1.0, cfg.aux_coeff, "top1")
    pu.compare_all(m.results(), bw["forward"], bw, cfg)


@pytest.mark.parametrize("T,M,N", [(500, 2, 4), (1500, 4, 4), (900, 3, 5)])
def test_grouping_of_several_adapters(T, M, N):
    cfg = synth.scaled(synth.CONFIGS["llama2_7b"], name="grouping_multi", T=T, d=64, d_ff=136, N=N, k=2, r=8, alpha=16.0,
                       M=M, seq_len=37)
    host = synth.make_inputs(cfg)
    host["W_router"] = synth._store(host["W_router"] * 8.0, cfg.dtype)
    res, fw, bw, tm = run_multi(cfg, host, "uneven")
    compare_multi(res, fw, bw, cfg, tm)


@pytest.mark.parametrize("T,d,f,N", [(300, 4096, 64, 8), (37, 4096, 136, 13), (2000, 4096, 1024, 16)])
def test_f32_logits_are_summed_in_short_chains(T, d, f, N):
    """Routing weights of fp32 storage against 64 bits.  A logit is the sum of 64 chains of d / 64 = 64 terms of
    RMS 0.02; with rounding errors of RMS 0.58 * 2^-24 per addition on partial sums that grow as a random walk
    it is off by 2e-7 (z itself 1.28), w0 = 1 / (1 + e^(z1 - z0)) by at most a quarter of sqrt(2) times
    that, 1.4e-7 of its size of about 1/2 with the exponential's share; in chains of d / 8 it would be 3.5e-7."""
    cfg = synth.scaled(synth.CONFIGS["tiny_f32"], name="f32_logits", T=T, d=d, d_ff=f, N=N, k=2, r=8, alpha=16.0)
    host = synth.make_inputs(cfg)
    print(f"case T={T} d={d} f={f} N={N}", flush=True)
    m = MixLoraFFN(cfg, host, with_backward=False)
    m.workspace.fill_(0xFF)
    m.forward()
    res = m.results()
    z = host["x"].astype(np.float64) @ host["W_router"].astype(np.float64).T
    zk = np.take_along_axis(z, res["topk_idx"].astype(np.int64), 1)
    w = np.exp(zk - zk.max(1, keepdims=True))
    w /= w.sum(1, keepdims=True)
    assert np.linalg.norm(res["topk_w"] - w) / np.linalg.norm(w) < 2e-7
