"""GPU calibration (ssdi8_calibrate) against the oracle's calibration (oracle/calibrate.py, pinned
by the oracle tests) on the same seeded draw.

  alpha_B, alpha_C, alpha_Xs   bit-exact: the same fp32 values are reduced with max and divided
                               once in fp32 (X_scaled with the fp32 operations of ChunkState)
  alpha_CB                     relative 1e-5 for fp16 B, C (products exact in fp32, fp32 sums
                               of 128 terms, then / 127 rounded to fp32); fp32 inputs are rounded
                               to fp16 first: relative 2e-3 (2 * 2^-11 per product plus slack)
  alpha_S                      relative 1e-5: X_scaled split into two fp16 parts (22 bits) times
                               fp16 B, 2 x 256-term fp32 sums, fp64 passing; fp32 B: 2e-3
  corr                         (a) equal, to 1e-5 of its scale, to eta * mean(y_fp - y_q)
                               recomputed on the host from the FP16 layer and the INT8 layer run
                               through their own entry points with the calibrated steps;
                               (b) against the oracle's mean correction with the same steps:
                               |d corr[h,p]| <= eta * 2 TOL_RELL2 * rms(y[.,.,h,p])
                               since |mean e| <= rms e (Cauchy-Schwarz) and the y errors of the
                               INT8 and the FP16 layer are each bounded by the y tolerance
                               (1e-3 relative L2; the rounding errors are correlated over tokens,
                               so no averaging over B L is assumed); plus 1e-4 of max |corr| for
                               the fp32 rounding of corr itself
"""
import dataclasses

import numpy as np
import pytest

from helpers import TOL_RELL2, dev, say
from oracle import calibrate as ocal
from oracle import exact as oex
from oracle import int8 as oq
from paper_2608_21952_amd import synth

pytestmark = pytest.mark.gpu

ETA = 0.15


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    assert _t.cuda.is_available(), "GPU tests need a GPU"
    return _t


@pytest.fixture(scope="module")
def ssdi8(torch):
    from paper_2608_21952_amd import ssdi8 as _s
    _s.lib()
    return _s


CASES = [
    ("tiny", {}),
    ("mamba2-130m", dict(batch=2, seqlen=1024, nheads=8)),
    ("mamba2-8b-g8", dict(batch=1, seqlen=768, nheads=16, ngroups=4)),
]


def _gpu_calibrate(torch, ssdi8, inp, cfg):
    f = lambda v: dev(np.asarray(v, np.float32), torch)
    out = ssdi8.calibrate(dev(inp["x"], torch), f(inp["dt_raw"]), f(inp["A"]),
                          dev(inp["B"], torch), dev(inp["C"], torch), D=f(inp["D"]),
                          chunk=cfg.chunk, xs_per_head=cfg.xs_per_head, eta=ETA)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


def _oracle_y_rms(inp, cfg):
    """Per-channel (h, p) rms of the fp64 SSD output (the scale of y and of its errors)."""
    H, G = cfg.nheads, cfg.ngroups
    gi = oex.head_group(H, G)
    dt32 = oq.dt_post(inp["dt_raw"], True)
    ss = np.zeros((H, cfg.headdim))
    for b in range(cfg.batch):
        for h in range(H):
            y = oex.ssd_chunked_bh(inp["x"][b, :, h], dt32[b, :, h].astype(np.float64),
                                   float(np.float32(inp["A"][h])),
                                   np.asarray(inp["B"][b, :, gi[h]], np.float32),
                                   np.asarray(inp["C"][b, :, gi[h]], np.float32),
                                   float(np.float32(inp["D"][h])), cfg.chunk)["y"]
            ss[h] += np.square(y).sum(axis=0)
    return np.sqrt(ss / (cfg.batch * cfg.seqlen))


def _rel(g, r):
    g = np.asarray(g, np.float64)
    r = np.asarray(r, np.float64)
    return float(np.abs(g - r).max() / np.abs(r).max())


@pytest.mark.parametrize("name,over", CASES)
def test_calibrated_steps_match_oracle(torch, ssdi8, name, over):
    cfg = dataclasses.replace(synth.CONFIGS[name], name=name + "-cal", **over)
    say(f"calibrate {cfg.name}: B={cfg.batch} L={cfg.seqlen} H={cfg.nheads} G={cfg.ngroups} "
        f"{cfg.dtype} xs_per_head={cfg.xs_per_head}")
    inp = synth.draw(cfg, 2)
    g = _gpu_calibrate(torch, ssdi8, inp, cfg)
    ref = ocal.calibrate(inp["x"], inp["dt_raw"], inp["A"], inp["B"], inp["C"], inp["D"],
                         chunk=cfg.chunk, xs_per_head=cfg.xs_per_head, eta=ETA)
    for k in ("alpha_B", "alpha_C", "alpha_Xs"):
        assert g[k].shape == ref[k].shape, k
        assert np.array_equal(g[k], ref[k]), (k, g[k], ref[k])
    fp16_in = cfg.dtype == "fp16"
    tol_cb = 1e-5 if fp16_in else 2e-3
    tol_s = 1e-5 if fp16_in else 2e-3
    r_cb, r_s = _rel(g["alpha_CB"], ref["alpha_CB"]), _rel(g["alpha_S"], ref["alpha_S"])
    say(f"  alpha_CB rel {r_cb:.2e}  alpha_S rel {r_s:.2e}")
    assert r_cb <= tol_cb
    assert r_s <= tol_s
    # the correction against the oracle's Eq. 10 with the GPU's own steps (so that both INT8
    # layers quantize identically and only floating-point rounding separates them)
    sc = {k: g[k] for k in ("alpha_B", "alpha_C", "alpha_Xs", "alpha_S", "alpha_CB")}
    corr_ref = ocal.mean_correction(inp["x"], inp["dt_raw"], inp["A"], inp["B"], inp["C"],
                                    inp["D"], sc, chunk=cfg.chunk, eta=ETA)
    y_rms = _oracle_y_rms(inp, cfg)
    dcorr = np.abs(g["corr"].astype(np.float64) - corr_ref)
    tol = ETA * 2 * TOL_RELL2 * y_rms + 1e-4 * float(np.abs(corr_ref).max())
    say(f"  corr max|ref| {np.abs(corr_ref).max():.3e}  max|d| {dcorr.max():.3e}  "
        f"max |d|/tol {(dcorr / tol).max():.3f}")
    assert (dcorr <= tol).all(), np.argwhere(dcorr > tol)[:5]


def test_correction_is_the_damped_mean_of_the_layer_difference(torch, ssdi8):
    cfg = dataclasses.replace(synth.CONFIGS["mamba2-130m"], name="cal-host", batch=2,
                              seqlen=1024, nheads=8)
    inp = synth.draw(cfg, 2)
    g = _gpu_calibrate(torch, ssdi8, inp, cfg)
    f = lambda v: dev(np.asarray(v, np.float32), torch)
    x, dt, A, D = dev(inp["x"], torch), f(inp["dt_raw"]), f(inp["A"]), f(inp["D"])
    B, C = dev(inp["B"], torch), dev(inp["C"], torch)
    yfp = ssdi8.ssd_chunk_scan_fp16(x, dt, A, B, C, D=D, y_dtype=torch.float32,
                                    final_state=False)["y"]
    aB, aC = f(g["alpha_B"]), f(g["alpha_C"])
    Bq, _ = ssdi8.quantize_act(B, "group", aB)
    Cq, _ = ssdi8.quantize_act(C, "group", aC)
    run = lambda corr: ssdi8.ssd_chunk_scan(x, dt, A, Bq, Cq, aB, aC, f(g["alpha_Xs"]),
                                            f(g["alpha_S"]), f(g["alpha_CB"]), D=D, corr=corr,
                                            y_dtype=torch.float32, final_state=False)["y"]
    yq = run(None)
    torch.cuda.synchronize()
    d = (yfp.double() - yq.double()).cpu().numpy()
    host = ETA * d.mean(axis=(0, 1))
    err = float(np.abs(g["corr"] - host).max())
    say(f"  corr vs host mean: max|corr| {np.abs(host).max():.3e}  max|d| {err:.3e}")
    assert err <= 1e-5 * float(np.abs(host).max()) + 1e-12
    # applying the correction removes eta of each channel's mean difference (Eq. 10 is additive
    # at the SSD output)
    yc = run(f(g["corr"]))
    torch.cuda.synchronize()
    rest = (yfp.double() - yc.double()).cpu().numpy().mean(axis=(0, 1))
    before = d.mean(axis=(0, 1))
    np.testing.assert_allclose(rest, (1 - ETA) * before,
                               atol=1e-6 * float(np.abs(before).max()) + 1e-7)


@pytest.mark.parametrize("B,L,H,G,dtype,single", [
    (1, 256, 3, 3, "fp16", True),      # one chunk: one row per layer
    (1, 1280, 5, 1, "fp16", True),     # five chunks of few sequences
    (1, 1536, 5, 1, "fp16", False),    # six of them: the separate kernels
    (3, 768, 6, 2, "fp32", False),     # fp32 x, nine rows
    (2, 1280, 60, 4, "fp16", True),    # the walked FP16 states
    (4, 1280, 104, 2, "fp16", True),   # more than eight items per CU: no speculative loads
])
def test_correction_from_channel_sums(torch, ssdi8, B, L, H, G, dtype, single):
    """corr is eta times the mean of the two layers' own fp32 outputs: the kernels sum the same
    fp32 values in fp64, so only the order of those sums (2^-53 of the sum of |y| each) and the
    last rounding to fp32 differ.  alpha_CB is the largest causal entry of fp16 C B^T / 127, summed
    in fp32 here and there: 128 terms, 1e-5 of it."""
    torch.manual_seed(B + L + H)
    dt_ = torch.float16 if dtype == "fp16" else torch.float32
    assert ssdi8.uses_single_pass(ssdi8.dims(B, L, H, G), dt_) == single
    x = (torch.randn(B, L, H, 64, device="cuda") * 3).to(dt_)
    dt = torch.randn(B, L, H, device="cuda") * 0.5 - 2
    A, D = -torch.exp(torch.rand(H, device="cuda") * 6 - 4), torch.rand(H, device="cuda")
    Bt, Ct = (torch.randn(B, L, G, 128, device="cuda").to(dt_) for _ in range(2))
    s = ssdi8.calibrate(x, dt, A, Bt, Ct, D=D, eta=0.5)
    yf = ssdi8.ssd_chunk_scan_fp16(x, dt, A, Bt, Ct, D=D, y_dtype=torch.float32)["y"].double()
    yq = ssdi8.ssd_chunk_scan(x, dt, A, None, None, s["alpha_B"], s["alpha_C"], s["alpha_Xs"],
                              s["alpha_S"], s["alpha_CB"], D=D, B=Bt, C=Ct,
                              y_dtype=torch.float32)["y"].double()
    ref = 0.5 * (yf - yq).mean((0, 1))
    slack = 2.0 ** -24 * ref.abs() + 2.0 ** -48 * (yf.abs() + yq.abs()).mean((0, 1))
    assert bool(((s["corr"].double() - ref).abs() <= slack).all())
    c, b = (t.half().float().view(B, L // 256, 256, G, 128).permute(0, 1, 3, 2, 4).contiguous()
            for t in (Ct, Bt))
    cb = (c @ b.transpose(3, 4).contiguous()).tril().abs().amax((0, 1, 3, 4)) / 127.0
    assert bool(((s["alpha_CB"] - cb).abs() <= 1e-5 * cb).all())


@pytest.mark.parametrize("dtype", ["fp16", "fp32"])
def test_nan_does_not_count_in_the_steps_of_b_and_c(torch, ssdi8, dtype):
    """A token whose B or C is zero but for a NaN leaves the steps of B, C and C B^T as a zero row
    does: the maxima leave NaNs out."""
    torch.manual_seed(8)
    dt_ = torch.float16 if dtype == "fp16" else torch.float32
    B, L, H, G = 1, 512, 4, 2
    x = torch.randn(B, L, H, 64, device="cuda").to(dt_)
    dt, A = torch.randn(B, L, H, device="cuda") - 2, -torch.rand(H, device="cuda")
    Bt, Ct = (torch.randn(B, L, G, 128, device="cuda").to(dt_) for _ in range(2))
    Bt[0, 300, 0], Ct[0, 40, 1] = 0, 0
    names = ("alpha_B", "alpha_C", "alpha_CB")
    zero = ssdi8.calibrate(x, dt, A, Bt, Ct)
    Bt[0, 300, 0, 5], Ct[0, 40, 1, 99] = float("nan"), float("nan")
    nan = ssdi8.calibrate(x, dt, A, Bt, Ct)
    for k in names:
        assert torch.equal(nan[k], zero[k]), (k, nan[k], zero[k])
