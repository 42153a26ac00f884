"""GPU parity of the FP16 baseline (ssdi8_ssd_chunk_scan_fp16) against its oracle
(oracle/fp16.py, itself pinned against the fp64 forms): y within the stated tolerance and the
fp32 final state within 1e-5 relative L2, whole layers and sampled full-size slabs."""
import dataclasses

import numpy as np
import pytest

from helpers import assert_close, dev, rel_errors, say
from oracle import fp16 as ofp
from paper_2608_21952_amd import synth

pytestmark = pytest.mark.gpu

STATE_RELL2 = 1e-5


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


def _run(torch, ssdi8, inp, init=None, y_dtype=None):
    f = lambda v: dev(np.asarray(v, np.float32), torch)
    return ssdi8.ssd_chunk_scan_fp16(dev(inp["x"], torch), f(inp["dt_raw"]), f(inp["A"]),
                                     dev(inp["B"], torch), dev(inp["C"], torch), D=f(inp["D"]),
                                     init_state=None if init is None else f(init),
                                     y_dtype=y_dtype)


def _check_state(gpu, ref, what):
    _, rel = rel_errors(gpu, ref)
    say(f"  {what}: relL2 = {rel:.3e}")
    assert rel <= STATE_RELL2, f"{what}: relative L2 {rel:.3e} > {STATE_RELL2}"


@pytest.mark.parametrize("name,over", [
    ("tiny", {}),
    ("mamba2-130m", dict(batch=2, seqlen=1024, nheads=8)),
    ("mamba2-8b-g8", dict(batch=1, seqlen=768, nheads=16, ngroups=4)),
])
def test_fp16_layer_matches_oracle(torch, ssdi8, name, over):
    cfg = dataclasses.replace(synth.CONFIGS[name], name=name + "-fp16", **over)
    say(f"fp16 layer {cfg.name}: B={cfg.batch} L={cfg.seqlen} H={cfg.nheads} G={cfg.ngroups} "
        f"{cfg.dtype}")
    inp = synth.draw(cfg, 1)
    g = _run(torch, ssdi8, inp)
    ref = ofp.ssd_fp16_forward(inp["x"], inp["dt_raw"], inp["A"], inp["B"], inp["C"], inp["D"],
                               chunk=cfg.chunk)
    assert_close(g["y"].float().cpu().numpy(), ref["y64"], "y")
    _check_state(g["final_state"].cpu().numpy(), ref["final_state"], "final state")


def test_fp16_initial_state_and_fp32_output(torch, ssdi8):
    cfg = dataclasses.replace(synth.CONFIGS["mamba2-130m"], name="fp16-init", batch=2,
                              seqlen=512, nheads=4)
    inp = synth.draw(cfg, 2)
    rng = np.random.default_rng(4)
    init = rng.standard_normal((2, 4, 64, 128)).astype(np.float32)
    g = _run(torch, ssdi8, inp, init=init, y_dtype=torch.float32)
    ref = ofp.ssd_fp16_forward(inp["x"], inp["dt_raw"], inp["A"], inp["B"], inp["C"], inp["D"],
                               chunk=cfg.chunk, init=init)
    assert g["y"].dtype == torch.float32
    assert_close(g["y"].cpu().numpy(), ref["y64"], "y (fp32 out, initial state)")
    _check_state(g["final_state"].cpu().numpy(), ref["final_state"], "final state")


@pytest.mark.parametrize("name", ["mamba2-130m", "mamba2-2.7b"])
def test_fp16_full_size_sampled_slabs(torch, ssdi8, name):
    """Full-size layers, the 2.7B-shaped one with x and y streamed through the caches."""
    cfg = synth.CONFIGS[name]
    say(f"fp16 layer full size {name}")
    inp = synth.draw(cfg, 1)
    g = _run(torch, ssdi8, inp)
    y = g["y"].float().cpu().numpy()
    fin = g["final_state"].cpu().numpy()
    picks = [(0, 0), (cfg.batch - 1, cfg.nheads - 1), (cfg.batch // 2, cfg.nheads // 2)]
    ref = ofp.ssd_fp16_forward(inp["x"], inp["dt_raw"], inp["A"], inp["B"], inp["C"], inp["D"],
                               chunk=cfg.chunk, heads=picks)
    for (b, h) in picks:
        r = ref["slabs"][(b, h)]
        assert_close(y[b, :, h], r["y64"], f"y slab ({b},{h})")
        _check_state(fin[b, h], r["final"], f"final state slab ({b},{h})")


def test_fp16_empty_sequence_returns_initial_state(torch, ssdi8):
    init = torch.randn((2, 4, 64, 128), device="cuda")
    z = lambda *s: torch.zeros(s, dtype=torch.float32, device="cuda")
    h16 = lambda *s: torch.zeros(s, dtype=torch.float16, device="cuda")
    out = ssdi8.ssd_chunk_scan_fp16(h16(2, 0, 4, 64), z(2, 0, 4), z(4), h16(2, 0, 1, 128),
                                    h16(2, 0, 1, 128), init_state=init)
    assert torch.equal(out["final_state"], init)


@pytest.mark.parametrize("batch,seqlen,nheads,ngroups,dtype,y_dtype,a_lo,a_hi", [
    (1, 256, 5, 5, "fp16", "fp16", 0.0, 2.77),       # one chunk, narrow state passing
    (1, 2304, 3, 1, "fp16", "fp32", -4.0, 0.0),      # nine chunks, no block skipped
    (2, 768, 64, 2, "fp32", "fp32", -4.0, 4.0),      # wide state passing, mixed decays
    (2, 512, 65, 5, "fp16", "fp16", 3.0, 6.0),       # every off-diagonal block a zero weight
    (1, 512, 6, 3, "fp32", "fp16", 2.0, 5.0),        # diagonal spans on both sides of 64
])
def test_fp16_scan_edges(torch, ssdi8, batch, seqlen, nheads, ngroups, dtype, y_dtype, a_lo, a_hi):
    """Skipped and kept ChunkScan2 blocks, both output stages, both widths of state passing."""
    cfg = dataclasses.replace(synth.CONFIGS["mamba2-130m"], name="fp16-edges", batch=batch,
                              seqlen=seqlen, nheads=nheads, ngroups=ngroups, dtype=dtype,
                              a_lo=a_lo, a_hi=a_hi, x_outliers=min(31, nheads), dt_sigma=0.7)
    inp = synth.draw(cfg, 1)
    rng = np.random.default_rng(5)
    init = rng.standard_normal((batch, nheads, 64, 128)).astype(np.float32)
    g = _run(torch, ssdi8, inp, init=init, y_dtype={"fp16": torch.float16,
                                                    "fp32": torch.float32}[y_dtype])
    y, fin = g["y"].float().cpu().numpy(), g["final_state"].cpu().numpy()
    picks = sorted({(0, 0), (batch - 1, nheads - 1), (batch - 1, nheads // 2)})
    ref = ofp.ssd_fp16_forward(inp["x"], inp["dt_raw"], inp["A"], inp["B"], inp["C"], inp["D"],
                               chunk=cfg.chunk, heads=picks, init=init)
    for (b, h) in picks:
        assert_close(y[b, :, h], ref["slabs"][(b, h)]["y64"], f"y slab ({b},{h})")
        _check_state(fin[b, h], ref["slabs"][(b, h)]["final"], f"final state slab ({b},{h})")


@pytest.mark.parametrize("batch,seqlen,nheads,ngroups,dtype,init", [
    (2, 256, 48, 1, "fp16", True),      # the fewest sequences walked, one chunk
    (1, 768, 113, 1, "fp32", False),    # odd chunks and heads, one chunk of x ahead
    (4, 1024, 30, 5, "fp16", True),     # even chunks, groups
    (1, 512, 95, 5, "fp16", True),      # one sequence too few: the separate kernels
])
def test_fp16_walk_matches_oracle(torch, ssdi8, batch, seqlen, nheads, ngroups, dtype, init):
    """ChunkState and StatePassing as one walk over each sequence: odd and even chunk counts, both
    x types, an initial state, and a chunk whose dt spans over 21 binades (the exact scan)."""
    cfg = dataclasses.replace(synth.CONFIGS["mamba2-130m"], name="fp16-walk", batch=batch,
                              seqlen=seqlen, nheads=nheads, ngroups=ngroups, dtype=dtype,
                              a_lo=-4.0)
    inp = synth.draw(cfg, 1)
    inp["dt_raw"][0, :256:3, 0] = -18.0   # softplus 1.5e-8 beside 0.1
    rng = np.random.default_rng(6)
    st = rng.standard_normal((batch, nheads, 64, 128)).astype(np.float32) if init else None
    g = _run(torch, ssdi8, inp, init=st)
    y, fin = g["y"].float().cpu().numpy(), g["final_state"].cpu().numpy()
    picks = sorted({(0, 0), (batch - 1, nheads - 1), (batch // 2, nheads // 2)})
    ref = ofp.ssd_fp16_forward(inp["x"], inp["dt_raw"], inp["A"], inp["B"], inp["C"], inp["D"],
                               chunk=cfg.chunk, heads=picks, init=st)
    for (b, h) in picks:
        assert_close(y[b, :, h], ref["slabs"][(b, h)]["y64"], f"y slab ({b},{h})")
        _check_state(fin[b, h], ref["slabs"][(b, h)]["final"], f"final state slab ({b},{h})")


@pytest.mark.parametrize("dtype", ["fp16", "fp32"])
@pytest.mark.parametrize("chunks", [1, 2, 9, 33])
def test_fp16_walk_equals_separate_kernels(torch, ssdi8, chunks, dtype):
    """A sequence's result does not depend on how many others share the call: 2 x 48 sequences
    (walked) and each 48 on their own (the separate kernels) agree bit for bit, very slow heads and
    an inexact scan among them."""
    torch.manual_seed(chunks)
    dt_ = torch.float16 if dtype == "fp16" else torch.float32
    B, L, H = 2, chunks * 256, 48
    x, Bt, Ct = (torch.randn(B, L, *s, device="cuda").to(dt_)
                 for s in ((H, 64), (1, 128), (1, 128)))
    dt = torch.randn(B, L, H, device="cuda") * 0.5 - 2
    dt[1, :256:3, 7] = -18.0
    A = -torch.exp(torch.rand(H, device="cuda") * 7 - 7)
    init = torch.randn(B, H, 64, 128, device="cuda")
    run = lambda s: ssdi8.ssd_chunk_scan_fp16(x[s], dt[s], A, Bt[s], Ct[s], init_state=init[s],
                                              y_dtype=torch.float32)
    both, one = run(slice(0, 2)), [run(slice(b, b + 1)) for b in range(B)]
    for k in ("final_state", "y"):
        assert torch.equal(both[k], torch.cat([o[k] for o in one])), k


@pytest.mark.parametrize("dtype", ["fp16", "fp32"])
@pytest.mark.parametrize("value,token", [(float("inf"), 3), (float("nan"), 70),
                                         (float("-inf"), 255)])
def test_fp16_scan_non_finite_x(torch, ssdi8, dtype, value, token):
    """An infinite or NaN x reaches every later row of its channel, also through blocks whose
    weights decay to zero (zero times infinity is NaN), and no other channel."""
    torch.manual_seed(3)
    dt_ = torch.float16 if dtype == "fp16" else torch.float32
    B, L, H = 1, 512, 2
    x = torch.randn(B, L, H, 64, device="cuda").to(dt_)
    dt = torch.zeros(B, L, H, device="cuda")
    A = torch.tensor([-200.0, -0.1], device="cuda")
    Bt, Ct = (torch.randn(B, L, 1, 128, device="cuda").to(dt_) for _ in range(2))
    x[0, token, :, 5] = value
    y = ssdi8.ssd_chunk_scan_fp16(x, dt, A, Bt, Ct, D=torch.ones(H, device="cuda"))["y"]
    fin = torch.isfinite(y)
    assert not bool(fin[0, token:, :, 5].any())
    fin[..., 5] = True
    assert bool(fin.all())


@pytest.mark.parametrize("dtype", ["fp16", "fp32"])
def test_fp16_scan_decay_that_rises_again(torch, ssdi8, dtype):
    """dt of both signs without the softplus: cs falls by 32 over one block of 32 tokens and rises by
    32 over the next, so weights that are zero at that block's first row are of order one at its
    last.  The tokens in between have B = 0 (their weights would leave the fp16 range).  Against 64
    bits: weights rounded to fp16 (2^-11 relative each), twice that for the fp32 factors of the
    decay, of the sum of |W x|."""
    torch.manual_seed(9)
    dt_ = torch.float16 if dtype == "fp16" else torch.float32
    B, L, H = 1, 256, 3
    x, Bt, Ct = (torch.randn(B, L, *s, device="cuda").half().to(dt_)
                 for s in ((H, 64), (1, 128), (1, 128)))
    Bt[:, 32:96] = 0
    dt = torch.full((B, L, H), 0.02, device="cuda")
    dt[:, :32], dt[:, 32:64], dt[:, 64:96] = 0.05, 1.0, -1.0
    A = torch.tensor([-1.0, -0.9, -1.1], device="cuda")
    y = ssdi8.ssd_chunk_scan_fp16(x, dt, A, Bt, Ct, dt_softplus=False,
                                  y_dtype=torch.float32)["y"].double()
    cs = torch.cumsum((dt * A).double(), 1)[0].T.contiguous()                  # (H, L)
    cb = (Ct[0, :, 0].double() @ Bt[0, :, 0].double().T.contiguous()).tril()
    W = cb * dt[0].T.double()[:, None] * torch.exp((cs[:, :, None] - cs[:, None]).tril())
    xh = x[0].double().permute(1, 0, 2).contiguous()
    ref = (W @ xh).permute(1, 0, 2)
    bound = (W.abs() @ xh.abs()).permute(1, 0, 2) * 2.0 ** -10 + 2.0 ** -20
    assert bool(((y[0] - ref).abs() <= bound).all())
    assert float(ref[88:96].abs().max()) > 0.1    # the rows in question are not small


def test_fp16_scan_nan_in_b(torch, ssdi8):
    """A NaN in B reaches every later row of its chunk, also through weights that decay to zero."""
    torch.manual_seed(4)
    B, L, H = 1, 256, 2
    x, Bt, Ct = (torch.randn(B, L, *s, device="cuda").half() for s in ((H, 64), (1, 128), (1, 128)))
    Bt[0, 3, 0, 77] = float("nan")
    y = ssdi8.ssd_chunk_scan_fp16(x, torch.zeros(B, L, H, device="cuda"),
                                  torch.tensor([-200.0, -0.1], device="cuda"), Bt, Ct)["y"]
    assert bool(torch.isnan(y[0, 3:]).all()) and bool(torch.isfinite(y[0, :3]).all())
