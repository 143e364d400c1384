"""GPU parity of routing and grouping in workgroups that count all experts at once: token counts around a
wave's 64, around the limit up to which every workgroup routes for itself, and the largest the launch takes;
eight and sixteen experts and odd numbers of them; one to four slots; several adapters.  Tables are pinned
through the outputs: indices and counts exactly, y, gradients and the auxiliary loss against the oracle."""
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
