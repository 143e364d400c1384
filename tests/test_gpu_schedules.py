"""GPU parity of the paper's own execution schedules (Section 3.3, Figure 3) against the oracle.

The shared (Figure 3b) and unshared (Figure 3a) schedules compute the same block as the
library's default schedule, with the frozen matrices applied per (token, expert) pair row where
the figure has them per expert.  The oracle is the definition of the block and does not depend
on the schedule, so every schedule is compared with the same oracle results, to the same bar.
"""
import numpy as np
import pytest

from oracle import mixlora_oracle as orc
from paper_2404_15159_amd import binding as B
from paper_2404_15159_amd import synth
from paper_2404_15159_amd.runner import MixLoraFFN

import parity_utils as pu

pytestmark = pytest.mark.gpu

BASE = synth.CONFIGS["llama2_7b"]
SCHEDULES = [("shared", B.SCHEDULE_SHARED), ("vanilla", B.SCHEDULE_VANILLA)]

CASES = [
    ("ragged", dict(T=300, d=256, d_ff=520, N=8, k=2, r=16)),
    ("multi_tile", dict(T=1000, d=512, d_ff=1288, N=16, k=2, r=8, alpha=16.0)),
    ("top3_r32", dict(T=257, d=136, d_ff=264, N=5, k=3, r=32, alpha=64.0)),
    ("top1", dict(T=200, d=128, d_ff=384, N=8, k=1, r=16)),
    ("k_eq_N", dict(T=130, d=128, d_ff=256, N=4, k=4, r=8, alpha=16.0)),
    ("few_tokens", dict(T=17, d=512, d_ff=704, N=8, k=2, r=16)),
    ("one_token", dict(T=1, d=64, d_ff=128, N=8, k=2, r=16)),
]


def _inputs(name, over):
    cfg = synth.scaled(BASE, name="sched_" + name, **over)
    host = synth.make_inputs(cfg)
    for n in ("B_gate", "B_up", "B_down"):      # livelier LoRA paths than the large-shape recipe
        host[n] = synth.round_to_bf16(host[n] * 4.0)
    return cfg, host


@pytest.mark.parametrize("sname,schedule", SCHEDULES, ids=[s[0] for s in SCHEDULES])
@pytest.mark.parametrize("name,over", CASES, ids=[c[0] for c in CASES])
def test_schedule_matches_oracle(name, over, sname, schedule):
    cfg, host = _inputs(name, over)
    print(f"\ncase {cfg.name} schedule={sname}: T={cfg.T} d={cfg.d} f={cfg.d_ff} N={cfg.N} "
          f"k={cfg.k} r={cfg.r}", flush=True)
    m = MixLoraFFN(cfg, host, schedule=schedule)
    m.forward()
    m.backward(d_aux=1.5)
    res = m.results()
    W = {n: host[n] for n in synth.WEIGHT_NAMES}
    bw = orc.backward(host["x"], W, cfg.k, cfg.lora_scale, host["dy"], 1.5, cfg.aux_coeff, "top1")
    pu.compare_all(res, bw["forward"], bw, cfg)


def test_schedules_agree_on_routing_and_need_more_workspace():
    """Same routing decisions bit for bit (the router does not depend on the schedule); outputs
    within the bf16 bar of each other; workspace grows with the per-pair rows."""
    cfg, host = _inputs("agree", dict(T=700, d=256, d_ff=1032, N=8, k=2, r=16))
    out, ws = {}, {}
    for sname, schedule in [("linear", B.SCHEDULE_LINEAR_DOWN)] + SCHEDULES:
        m = MixLoraFFN(cfg, host, schedule=schedule)
        m.forward()
        m.backward()
        out[sname] = m.results()
        ws[sname] = m.ws_bytes
    for sname in ("shared", "vanilla"):
        assert np.array_equal(out[sname]["topk_idx"], out["linear"]["topk_idx"])
        assert np.array_equal(out[sname]["counts"], out["linear"]["counts"])
        assert np.array_equal(out[sname]["topk_w"], out["linear"]["topk_w"])
        assert out[sname]["aux_loss"] == out["linear"]["aux_loss"]
        for n in ("y", "dx") + pu.GRAD_NAMES:
            pu.assert_close(f"{sname}:{n}", out[sname][n], out["linear"][n], 2e-2)
    assert ws["linear"] < ws["shared"] < ws["vanilla"]


# launches whose tiles are all cut along K (the router's among them), a few rows on either side of the
# matrix-vector products' limit, ragged contractions of few and of many rows, no cut
@pytest.mark.parametrize("T,d,f,N", [(150, 1024, 2752, 8), (300, 1032, 2744, 5), (1, 512, 704, 8), (2, 264, 712, 8),
                                     (4, 512, 1408, 8), (4, 264, 2744, 8), (30, 264, 712, 8), (100, 1032, 2744, 3),
                                     (120, 512, 1408, 8), (1500, 512, 1408, 16)])
def test_schedules_sum_the_logits_alike(T, d, f, N):
    cfg, host = _inputs("logits", dict(T=T, d=d, d_ff=f, N=N, k=2, r=16))
    out = []
    for schedule in (B.SCHEDULE_LINEAR_DOWN, B.SCHEDULE_SHARED, B.SCHEDULE_VANILLA):
        m = MixLoraFFN(cfg, host, schedule=schedule, with_backward=False)
        m.forward()
        out.append(m.results())
    for o in out[1:]:
        for n in ("topk_idx", "topk_w", "counts"):
            assert np.array_equal(o[n], out[0][n]), n


def test_schedule_argument_errors():
    cfg, host = _inputs("errors", dict(T=64, d=64, d_ff=128, N=4, k=2, r=8, alpha=16.0))
    m = MixLoraFFN(cfg, host)
    with pytest.raises(B.MixLoraError):      # unknown schedule
        B.mixlora_ffn_forward_schedule(m.dims, 7, m.weights, m.t["x"], m.y, m.topk_idx, m.topk_w,
                                       m.counts, m.aux, m.workspace, m.ws_bytes)
    need = B.mixlora_schedule_workspace_bytes(m.dims, B.SCHEDULE_VANILLA, False)
    with pytest.raises(B.MixLoraError):      # workspace too small for this schedule
        B.mixlora_ffn_forward_schedule(m.dims, B.SCHEDULE_VANILLA, m.weights, m.t["x"], m.y,
                                       m.topk_idx, m.topk_w, m.counts, m.aux, m.workspace,
                                       need - 256)
    assert B.mixlora_schedule_workspace_bytes(m.dims, 7, True) == 0


@pytest.mark.parametrize("sname,schedule", SCHEDULES, ids=[s[0] for s in SCHEDULES])
def test_schedule_full_size_sampled(sname, schedule):
    """LLaMA-2-7B shape, the configuration bench.py --schedule times: outputs of sampled tokens
    against the oracle (per-token outputs are independent), routing of all tokens."""
    cfg = BASE
    host = synth.make_inputs(cfg)
    m = MixLoraFFN(cfg, host, schedule=schedule)
    m.forward()
    m.backward()
    res = m.results()
    W = {n: host[n] for n in synth.WEIGHT_NAMES}
    rng = np.random.default_rng(11)
    sample = np.sort(rng.choice(cfg.T, size=96, replace=False))
    fw = orc.forward(host["x"][sample], W, cfg.k, cfg.lora_scale, cfg.aux_coeff, "top1")
    set_safe, order_safe = pu.routing_masks(fw["logits"], cfg.k)
    gi = res["topk_idx"][sample].astype(np.int64)
    assert (np.sort(gi[set_safe], axis=1) == np.sort(fw["topk_idx"][set_safe], axis=1)).all()
    same = (gi == fw["topk_idx"]).all(axis=1)
    assert same.sum() >= 90
    pu.assert_close("y", res["y"][sample][same], fw["y"][same], 2e-2)
    assert res["counts"].sum() == cfg.k * cfg.T
    # backward at this size: against the default schedule (itself compared with the oracle at
    # this size by the parity tests), same routing, so every tensor must agree to the bf16 bar
    del m
    ref = MixLoraFFN(cfg, host)
    ref.forward()
    ref.backward()
    rr = ref.results()
    assert np.array_equal(res["topk_idx"], rr["topk_idx"])
    for n in ("y", "dx") + pu.GRAD_NAMES:
        pu.assert_close(n, res[n], rr[n], 2e-2)
