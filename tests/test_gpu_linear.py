"""GPU parity of the plain LoRA linear (attention-projection form, Eq. 1) against the oracle."""
import numpy as np
import pytest

from oracle import mixlora_oracle as orc
from paper_2404_15159_amd import synth
from paper_2404_15159_amd.runner import LoraLinear

import parity_utils as pu

pytestmark = pytest.mark.gpu

CASES = [
    # name, T, d_in, d_out, r, dtype, pretransposed
    ("f32_small", 130, 72, 200, 8, "f32", True),
    ("f32_r16_untransposed", 97, 64, 136, 16, "f32", False),
    ("bf16_ragged", 300, 256, 520, 16, "bf16", True),
    ("bf16_r64", 257, 136, 264, 64, "bf16", True),
    ("bf16_r24_untransposed", 513, 192, 320, 24, "bf16", False),
    ("bf16_multi_tile", 1000, 512, 1288, 8, "bf16", True),
    ("bf16_few_rows", 17, 512, 704, 16, "bf16", True),
    ("bf16_one_row", 1, 64, 128, 8, "bf16", True),
    # both sides of the row counts from which the rank-r term rides in the frozen product (5 into fewer
    # than 8192 columns, 129 into any); square (one launch for both gradient sums), column blocks of 16
    # that are not full, cut K ranges
    ("bf16_128_rows", 128, 264, 264, 40, "bf16", True),
    ("bf16_129_rows", 129, 264, 264, 40, "bf16", True),
    ("bf16_square_split", 200, 1024, 1024, 8, "bf16", True),
    ("bf16_r12_square", 331, 1032, 1032, 12, "bf16", False),
    ("bf16_2_rows", 2, 1032, 520, 16, "bf16", True),
    ("bf16_4_rows", 4, 520, 1032, 8, "bf16", True),
    ("bf16_5_rows", 5, 520, 1032, 8, "bf16", True),
    ("bf16_60_rows_wide", 60, 264, 8200, 16, "bf16", True),
    ("bf16_128_rows_wide", 128, 264, 8200, 8, "bf16", True),
    ("bf16_129_rows_wide", 129, 264, 8200, 8, "bf16", True),
    ("bf16_40_rows_8184", 40, 264, 8184, 16, "bf16", True),
]


@pytest.mark.parametrize("name,T,d_in,d_out,r,dtype,pre", CASES, ids=[c[0] for c in CASES])
def test_lora_linear_small(name, T, d_in, d_out, r, dtype, pre):
    s = 2.0
    host = synth.make_linear_inputs(T, d_in, d_out, r, dtype, seed=synth.SEED_BASE + 100 + len(name),
                                    b_std=0.08)
    print(f"\nlinear case {name}: T={T} d_in={d_in} d_out={d_out} r={r} {dtype}", flush=True)
    m = LoraLinear(T, d_in, d_out, r, s, dtype, host, pretransposed=pre)
    m.forward(); m.backward()
    res = m.results()
    y = orc.lora_linear_forward(host["x"], host["W"], host["A"], host["B"], s)
    g = orc.lora_linear_backward(host["x"], host["W"], host["A"], host["B"], s, host["dy"])
    tol = pu.TOL[dtype]
    rep = {"y": pu.assert_close("y", res["y"], y, tol)}
    for n in ("dx", "dA", "dB"):
        rep[n] = pu.assert_close(n, res[n], g[n], tol)
    print({k: tuple(f"{v:.2e}" for v in e) for k, e in rep.items()}, flush=True)
    # the LoRA path is really there: the frozen product alone is off by more than the tolerance
    base = host["x"].astype(np.float64) @ host["W"].astype(np.float64).T
    assert pu.rel_errors(base, y)[0] > 5 * tol


@pytest.mark.parametrize("T,r", [(5, 16), (100, 8), (131, 64), (300, 12)])
def test_rank_term_keeps_24_bits(T, r):
    """W cancels the rank-r term but for an identity, in whole numbers: x A^T reaches 2^22, every product
    and partial sum is below 2^24, so the result is exact unless the term is held in fewer bits.  Forward
    with large A and B of +-1, backward (s (dy B) A) the other way round."""
    rng = np.random.default_rng(T)
    n, cols = 512, 264
    big = lambda shape: rng.integers(-127, 128, size=shape).astype(np.float32)
    x, dy = np.abs(big((T, n))), np.abs(big((T, n)))      # (absolute values: sums of one sign)
    pick = np.zeros((cols, r), np.float32)                # row c picks rank entry c % r, with a sign
    pick[np.arange(cols), np.arange(cols) % r] = np.where(np.arange(cols) // r % 2, 1.0, -1.0)
    bank = np.abs(big((r, n)))
    keep = np.zeros((cols, n), np.float32)
    keep[np.arange(cols), np.arange(cols) * 5 % n] = 1.0
    host = dict(x=x, W=keep - pick @ bank, A=bank, B=pick, dy=big((T, cols)))
    print(f"case forward T={T} r={r}", flush=True)
    m = LoraLinear(T, n, cols, r, 1.0, "bf16", host)
    m.forward()
    assert np.array_equal(m.results()["y"], x @ keep.T)
    host = dict(x=big((T, cols)), W=(keep - pick @ bank).T.copy(), A=pick.T.copy(), B=bank.T.copy(), dy=dy)
    print(f"case backward T={T} r={r}", flush=True)
    m = LoraLinear(T, cols, n, r, 1.0, "bf16", host)
    m.forward(); m.backward()
    assert np.array_equal(m.results()["dx"], dy @ keep.T)


@pytest.mark.parametrize("T", [5, 131, 300])
def test_rank_term_with_infinite_and_huge_weights(T):
    """An infinite element of B (forward) or A (backward) gives the infinities that 64-bit arithmetic
    gives; a projection that only overflows once it is scaled does not."""
    r, s = 16, 3.0
    host = synth.make_linear_inputs(T, 256, 264, r, "bf16", seed=77)
    with np.errstate(invalid="ignore", over="ignore"):
        for n, at in (("B", (3, 1)), ("A", (2, 5))):
            h = dict(host, **{n: host[n].copy()})
            h[n][at] = -np.inf
            m = LoraLinear(T, 256, 264, r, s, "bf16", h)
            m.forward(); m.backward()
            h64 = {k: v.astype(np.float64) for k, v in h.items()}
            ref = dict(y=h64["x"] @ h64["W"].T + s * (h64["x"] @ h64["A"].T) @ h64["B"].T,
                       dx=h64["dy"] @ h64["W"] + s * (h64["dy"] @ h64["B"]) @ h64["A"])
            res = m.results()
            for out in ("y", "dx"):
                assert np.array_equal(np.isnan(res[out]), np.isnan(ref[out])), (n, out)
                assert np.array_equal(np.isinf(res[out]) * np.sign(res[out]),
                                      np.isinf(ref[out]) * np.sign(ref[out])), (n, out)
        h = {n: host[n].copy() for n in host}
        h["x"][:, 5], h["A"][2, 5], h["B"][:, 2] = 1.0, synth.round_to_bf16(np.float32([3e38]))[0], 0.01
        h["B"] = synth.round_to_bf16(h["B"])
        m = LoraLinear(T, 256, 264, r, s, "bf16", h)
        m.forward()
        pu.assert_close("y", m.results()["y"], orc.lora_linear_forward(h["x"], h["W"], h["A"], h["B"], s), 2e-2)


def test_lora_linear_full_size_attention_projection():
    """A q/k/v/o-sized projection of the LLaMA-2-7B shape (4096 -> 4096, rank 16, 4096 tokens),
    as bench.py --workload llama2_7b_attn_proj times it: sampled outputs and the full A/B
    gradients against the oracle."""
    T, d, r, s = 4096, 4096, 16, 2.0
    host = synth.make_linear_inputs(T, d, d, r, "bf16", seed=synth.SEED_BASE + 8)
    m = LoraLinear(T, d, d, r, s, "bf16", host)
    m.forward(); m.backward()
    res = m.results()
    rng = np.random.default_rng(4)
    rows = rng.choice(T, size=64, replace=False)
    y = orc.lora_linear_forward(host["x"][rows], host["W"], host["A"], host["B"], s)
    pu.assert_close("y", res["y"][rows], y, pu.TOL["bf16"])
    g = orc.lora_linear_backward(host["x"], host["W"], host["A"], host["B"], s, host["dy"])
    for n in ("dx", "dA", "dB"):
        pu.assert_close(n, res[n], g[n], pu.TOL["bf16"])


def test_adamw_step_matches_oracle():
    """Three AdamW steps on 100003 parameters: float32 master values and moments against the
    float64 oracle, and the bf16 copy equal to the rounded master values."""
    import torch
    from paper_2404_15159_amd import binding as B
    n = 100003
    rng = np.random.default_rng(21)
    p0 = rng.standard_normal(n).astype(np.float32)
    p = torch.from_numpy(p0.copy()).cuda()
    m = torch.zeros(n, dtype=torch.float32, device="cuda:0")
    v = torch.zeros_like(m)
    low = torch.empty(n, dtype=torch.bfloat16, device="cuda:0")
    rp, rm, rv = p0.astype(np.float64), np.zeros(n), np.zeros(n)
    # the C struct carries the hyper-parameters as float32: the oracle gets the same values
    lr, b1, b2, eps, wd = (float(np.float32(h)) for h in (2e-4, 0.9, 0.999, 1e-8, 0.01))
    for t in range(1, 4):
        g = (rng.standard_normal(n) * 0.3).astype(np.float32)
        gd = torch.from_numpy(g).cuda()
        B.mixlora_adamw_step(B.AdamW(lr, b1, b2, eps, wd, t), n, p, gd, m, v, low, B.BF16)
        rp, rm, rv = orc.adamw_step(rp, g, rm, rv, t, lr, b1, b2, eps, wd)
    torch.cuda.synchronize()
    pu.assert_close("param", p.cpu().numpy(), rp, 1e-6)
    pu.assert_close("m", m.cpu().numpy(), rm, 1e-6)
    pu.assert_close("v", v.cpu().numpy(), rv, 1e-6)
    assert torch.equal(low, p.to(torch.bfloat16))
    # the update really moved the parameters by about lr per step
    assert 1e-4 < np.abs(p.cpu().numpy() - p0).mean() < 1e-3
