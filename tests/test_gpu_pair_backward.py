"""GPU parity of the backward stage on pair-grouped tiles, which makes the gradient sums of B_gate, B_up and
A_down itself: token counts on both sides of its limit, column blocks that end inside a wavefront's columns
or leave a wavefront without any, ranks of one and two 8-entry pieces, runs that cross column blocks, experts
that come back after others, every token at one pair, several adapters.  Against the oracle, bf16 tolerance
(2e-2).  And what a non-finite value of one feature or one token may reach, here and in the pair-grouped forward."""
import numpy as np
import pytest

from oracle import mixlora_oracle as orc
from paper_2404_15159_amd import synth
from paper_2404_15159_amd.runner import MixLoraFFN

import parity_utils as pu
from test_gpu_multi import compare_multi, run_multi

pytestmark = pytest.mark.gpu
BASE = synth.CONFIGS["llama2_7b"]


@pytest.mark.parametrize("T,f,N,r", [(783, 5632, 8, 16), (784, 5632, 8, 16), (1000, 4648, 8, 8), (1100, 4168, 3, 16),
                                     (3400, 1288, 16, 8), (900, 4688, 2, 4), (2048, 2064, 7, 12), (1007, 10304, 8, 16),
                                     (1008, 10304, 8, 16), (671, 6912, 8, 8), (672, 6912, 8, 8), (3399, 1408, 16, 16),
                                     (3400, 1408, 16, 16), (3808, 1280, 4, 16), (3840, 1280, 4, 16)])
def test_pair_backward_matches_oracle(T, f, N, r):
    cfg = synth.scaled(BASE, name="pair_bwd", T=T, d=64, d_ff=f, N=N, k=2, r=r, alpha=2.0 * r)
    print(f"case T={T} f={f} N={N} r={r}", flush=True)
    host = synth.make_inputs(cfg)
    host["W_router"] = synth._store(host["W_router"] * 8.0, cfg.dtype)
    m = MixLoraFFN(cfg, host)
    m.workspace.fill_(0xFF)          # NaN patterns: nothing may be read before it is written
    m.forward()
    m.backward(d_aux=1.0)
    res = m.results()
    W = {n: host[n] for n in synth.WEIGHT_NAMES}
    bw = orc.backward(host["x"], W, cfg.k, cfg.lora_scale, host["dy"], 1.0, cfg.aux_coeff, "top1")
    pu.compare_all(res, bw["forward"], bw, cfg)
    m.backward(d_aux=1.0)            # the same workspace again: sums start afresh, bit for bit
    again = m.results()
    for n in ("dx",) + pu.GRAD_NAMES:
        assert np.array_equal(res[n], again[n]), n


def test_all_tokens_at_one_pair():
    cfg = synth.scaled(BASE, name="pair_bwd_one", T=1200, d=64, d_ff=4608, N=6, k=2, r=16)
    host = synth.make_inputs(cfg)
    host["x"][:, 0] = 1.0
    host["W_router"][1, 0], host["W_router"][4, 0] = 30.0, 20.0
    m = MixLoraFFN(cfg, host)
    m.workspace.fill_(0xFF)
    m.forward()
    m.backward(d_aux=0.0)
    res = m.results()
    W = {n: host[n] for n in synth.WEIGHT_NAMES}
    bw = orc.backward(host["x"], W, cfg.k, cfg.lora_scale, host["dy"], 0.0, cfg.aux_coeff, "top1")
    for n in ("dx", "dA_gate", "dB_gate", "dA_up", "dB_up", "dA_down", "dB_down"):
        pu.assert_close(n, res[n], bw[n], 2e-2)
    for n in ("dB_gate", "dB_up", "dA_down"):   # experts without a token: exact zeros
        assert not res[n][[0, 2, 3, 5]].any(), n


@pytest.mark.parametrize("T,M,N", [(700, 2, 4), (900, 3, 3)])
def test_pair_backward_of_several_adapters(T, M, N):
    cfg = synth.scaled(BASE, name="pair_bwd_multi", T=T, d=64, d_ff=6088, N=N, k=2, r=8, alpha=16.0, M=M, seq_len=61)
    host = synth.make_inputs(cfg)
    host["W_router"] = synth._store(host["W_router"] * 8.0, cfg.dtype)
    res, fw, bw, tm = run_multi(cfg, host, "uneven")
    compare_multi(res, fw, bw, cfg, tm)


# (the second: pair-grouped forward, expert-grouped backward)
@pytest.mark.parametrize("T,f", [(1100, 4648), (300, 776)])
@pytest.mark.parametrize("name", ["W_gate", "W_up", "W_down"])
def test_non_finite_feature_stays_to_itself(T, f, name):
    """One infinite element of a frozen matrix makes one feature (a column of G, U or dy W_down) non-finite for every
    token: the gradients of every other feature are those of a clean pass, bit for bit."""
    cfg = synth.scaled(BASE, name="pair_bwd_inf", T=T, d=64, d_ff=f, N=8, k=2, r=16)
    host = synth.make_inputs(cfg)
    c = f // 2 + 5
    out = []
    for v in (0.0, np.inf):
        W = host[name].copy()
        W[(7, c) if name == "W_down" else (c, 7)] = v
        print(f"case T={T} f={f} {name} {v}", flush=True)
        m = MixLoraFFN(cfg, dict(host, **{name: W}))
        m.workspace.fill_(0xFF)
        m.forward()
        m.backward(d_aux=0.0)
        out.append(m.results())
    rest = np.delete(np.arange(f), c)
    for n in ("dB_gate", "dB_up"):
        assert not np.isfinite(out[1][n][:, c]).all() or (n, name) == ("dB_up", "W_up"), n
        assert np.array_equal(out[0][n][:, rest], out[1][n][:, rest]), n
    assert np.array_equal(out[0]["dA_down"][:, :, rest], out[1]["dA_down"][:, :, rest])


@pytest.mark.parametrize("T,f", [(1100, 4648), (300, 776)])
def test_non_finite_tokens_stay_to_themselves(T, f):
    cfg = synth.scaled(BASE, name="pair_bwd_nan", T=T, d=64, d_ff=f, N=8, k=2, r=16)
    host = synth.make_inputs(cfg)
    bad = {5: np.nan, T // 2: np.inf, T - 1: -np.inf}
    rest = np.setdiff1d(np.arange(T), list(bad))
    clean, dirty = host["x"].copy(), host["x"].copy()
    for t, v in bad.items():
        clean[t] = 0.0
        dirty[t, 3] = v
    out = []
    for x in (clean, dirty):
        print(f"case T={T} f={f} tokens", flush=True)
        m = MixLoraFFN(cfg, dict(host, x=x))
        m.workspace.fill_(0xFF)
        m.forward()
        m.backward(d_aux=0.0)
        out.append(m.results())
    assert not np.isfinite(out[1]["y"][list(bad)]).all()
    for n in ("topk_idx", "topk_w", "y", "dx"):
        assert np.array_equal(out[0][n][rest], out[1][n][rest]), n
