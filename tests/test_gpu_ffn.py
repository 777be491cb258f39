"""The feed-forward glue between two Float8 linears (h = silu(a) * b and its backward) and the
whole feed-forward chain X -> [W1; W3] -> glue -> W2 -> Y, forward and backward."""
import numpy as np
import pytest
import torch

import oracle as o
from paper_2410_06511_amd import f8
from paper_2410_06511_amd import workloads as wl
from helpers import bits, u8, f32, assert_gemm_close, codes_t

pytestmark = pytest.mark.gpu


def _from_bits(b):
    return torch.from_numpy(np.ascontiguousarray(b).view(np.int16)).view(torch.bfloat16)


def assert_bf16_close(got_bits, ref_bits, what=""):
    """fp32 arithmetic against the fp64 definition: equal up to one bf16 unit in the last place
    (a rounding boundary can fall between the two), and never off in sign or by a binade."""
    got = o.bf16_to_f32(got_bits).astype(np.float64)
    ref = o.bf16_to_f32(ref_bits).astype(np.float64)
    assert np.isfinite(got).all(), what
    ulp = np.maximum(np.abs(ref), 2.0 ** -126) * 2.0 ** -7          # >= one bf16 ulp at |ref|
    bad = np.abs(got - ref) > ulp
    assert not bad.any(), (what, int(bad.sum()), np.argwhere(bad)[:3])
    # the overwhelming majority is bit-identical
    assert (got_bits == ref_bits).mean() > 0.98, what


@pytest.mark.parametrize("M,H", [(16, 16), (272, 336), (512, 1792)])
def test_silu_mul_forward_and_backward(M, H):
    g = torch.Generator("cpu")
    g.manual_seed(M + H)
    ab = wl.randn_bf16((M, 2 * H), 2.0, 0, generator=g)
    ab[0, :8] = torch.tensor([0.0, -0.0, 30.0, -30.0, 100.0, -100.0, 1e-3, -1e-3]).bfloat16()
    dh = wl.randn_bf16((M, H), 1e-3, 0, generator=g)
    ws = f8.new_workspace(M, 2 * H)
    h = torch.empty((M, H), dtype=torch.bfloat16, device="cuda")
    dab = torch.empty((M, 2 * H), dtype=torch.bfloat16, device="cuda")
    a_h, a_d = torch.full((1,), -1.0, device="cuda"), torch.full((1,), -1.0, device="cuda")
    f8.silu_mul(ab.cuda(), h, a_h, ws)
    f8.silu_mul_bwd(ab.cuda(), dh.cuda(), dab, a_d, ws)
    torch.cuda.synchronize()
    rh, ra_h = o.silu_mul(bits(ab))
    rd, ra_d = o.silu_mul_bwd(bits(ab), bits(dh))
    assert_bf16_close(bits(h), rh, "h")
    assert_bf16_close(bits(dab), rd, "dab")
    # the amax is exactly that of the values written, and within an ulp of the oracle's
    assert a_h.item() == o.amax(bits(h))[0] and a_d.item() == o.amax(bits(dab))[0]
    assert abs(a_h.item() - ra_h[0]) <= 2.0 ** -7 * ra_h[0] and abs(a_d.item() - ra_d[0]) <= 2.0 ** -7 * ra_d[0]
    # without an amax output no workspace is needed and the values are the same
    h2 = torch.empty_like(h)
    f8.silu_mul(ab.cuda(), h2)
    torch.cuda.synchronize()
    assert torch.equal(h.view(torch.int16), h2.view(torch.int16))


@pytest.mark.parametrize("M,H", [(16, 128), (16, 272), (512, 1024), (528, 1024), (1040, 4112), (2048, 4080), (2048, 4096),
                                 (2064, 4112)])
def test_silu_mul_at_the_edges_of_a_block(M, H):
    """Up to 256 blocks take one chunk of 16 bytes a thread: one whole block, two and a remainder, all of them.  Above that
    two in turn: some threads only one, a remainder, all of them.  From 2^20 chunks on, past the caches, 1024 blocks take two
    chunks a thread side by side: two whole rounds, a third with a remainder.  In place too: a chunk is read and written by
    one thread."""
    g = torch.Generator("cpu")
    g.manual_seed(M + H)
    ab, dh = wl.randn_bf16((M, 2 * H), 2.0, 0, generator=g), wl.randn_bf16((M, H), 1e-3, 0, generator=g)
    ws = f8.new_workspace(M, 2 * H)
    h, dab = torch.empty((M, H), dtype=torch.bfloat16, device="cuda"), ab.cuda()
    a_h, a_d = torch.full((1,), -1.0, device="cuda"), torch.full((1,), -1.0, device="cuda")
    f8.silu_mul(ab.cuda(), h, a_h, ws)
    f8.silu_mul_bwd(dab, dh.cuda(), dab, a_d, ws)
    torch.cuda.synchronize()
    assert_bf16_close(bits(h), o.silu_mul(bits(ab))[0], "h")
    assert_bf16_close(bits(dab), o.silu_mul_bwd(bits(ab), bits(dh))[0], "dab")
    assert a_h.item() == o.amax(bits(h))[0] and a_d.item() == o.amax(bits(dab))[0]


def test_glue_argument_errors():
    t = torch.zeros((16, 32), dtype=torch.bfloat16, device="cuda")
    h = torch.zeros((16, 16), dtype=torch.bfloat16, device="cuda")
    a = torch.zeros(1, device="cuda")
    with pytest.raises(f8.F8Error) as e:       # amax requested without a workspace
        f8.silu_mul(t, h, a, None)
    assert e.value.code == 5
    with pytest.raises(f8.F8Error) as e:
        f8._check(f8.lib().f8_silu_mul(t.data_ptr(), 16, 24, h.data_ptr(), None, None, 0, None))
    assert e.value.code == 2


class FFN:
    """Device buffers and the call sequence of one feed-forward block."""

    def __init__(self, M, D, H, gfmt=f8.E4M3):
        bf = dict(dtype=torch.bfloat16, device="cuda")
        self.M, self.D, self.H = M, D, H
        self.d13, self.d2 = f8.linear_desc(M, D, 2 * H, False, gfmt), f8.linear_desc(M, H, D, False, gfmt)
        self.s13, self.s2 = f8.Saved(M, D, 2 * H), f8.Saved(M, H, D)
        self.ws = f8.new_workspace(max(M, D, 2 * H), max(M, D, 2 * H))
        self.AB, self.Hh, self.Y = torch.empty((M, 2 * H), **bf), torch.empty((M, H), **bf), torch.empty((M, D), **bf)
        self.dH, self.dAB, self.dX = torch.empty((M, H), **bf), torch.empty((M, 2 * H), **bf), torch.empty((M, D), **bf)
        self.dW13, self.dW2 = torch.empty((2 * H, D), **bf), torch.empty((D, H), **bf)
        self.a_h, self.a_dab = torch.empty(1, device="cuda"), torch.empty(1, device="cuda")

    def forward(self, X, W13, W2, chained=True):
        if chained:
            f8.linear_fwd_chained(self.d13, X, None, W13, self.AB, None, self.s13, self.ws)
            f8.silu_mul(self.AB, self.Hh, self.a_h, self.ws)
            f8.linear_fwd_chained(self.d2, self.Hh, self.a_h, W2, self.Y, None, self.s2, self.ws)
        else:
            f8.linear_fwd(self.d13, X, W13, self.AB, self.s13, self.ws)
            f8.silu_mul(self.AB, self.Hh)
            f8.linear_fwd(self.d2, self.Hh, W2, self.Y, self.s2, self.ws)

    def backward(self, dY, chained=True):
        if chained:
            f8.linear_bwd_chained(self.d2, dY, None, self.s2, self.dH, None, self.dW2, self.ws)
            f8.silu_mul_bwd(self.AB, self.dH, self.dAB, self.a_dab, self.ws)
            f8.linear_bwd_chained(self.d13, self.dAB, self.a_dab, self.s13, self.dX, None, self.dW13, self.ws)
        else:
            f8.linear_bwd(self.d2, dY, self.s2, self.dH, self.dW2, self.ws)
            f8.silu_mul_bwd(self.AB, self.dH, self.dAB)
            f8.linear_bwd(self.d13, self.dAB, self.s13, self.dX, self.dW13, self.ws)


def _ffn_inputs(M, D, H, seed):
    g = torch.Generator("cpu")
    g.manual_seed(seed)
    return (wl.randn_bf16((M, D), 1.0, 0, generator=g), wl.randn_bf16((2 * H, D), 0.02, 0, generator=g),
            wl.randn_bf16((D, H), 0.02, 0, generator=g), wl.randn_bf16((M, D), 1e-3, 0, generator=g))


@pytest.mark.parametrize("M,D,H", [(272, 336, 208), (1024, 1024, 1792)])
def test_ffn_chained_equals_unchained(M, D, H):
    X, W13, W2, dY = (t.cuda() for t in _ffn_inputs(M, D, H, 5))
    outs = []
    for chained in (True, False):
        f = FFN(M, D, H)
        f.forward(X, W13, W2, chained)
        f.backward(dY, chained)
        torch.cuda.synchronize()
        outs.append((f.Y, f.dX, f.dW13, f.dW2, f.Hh, f.dAB, f.s2.x.q, codes_t(f.s13.dy), f.s2.x.scale, f.s13.dy.scale))
    for a, b in zip(*outs):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


def test_ffn_stage_by_stage_against_oracle():
    """Every stage of the chain is fed the ORACLE's output of the stage before and compared with
    the oracle's output of this stage: codes and scales bit-exact, GEMMs and glue within their
    tolerances."""
    M, D, H = 512, 768, 1024
    X, W13, W2, dY = _ffn_inputs(M, D, H, 6)
    # oracle chain
    rAB, xq, w13q = o.linear_fwd(bits(X), bits(W13))
    rH, ra_h = o.silu_mul(rAB)
    rY, hq, w2q = o.linear_fwd(rH, bits(W2))
    rdH, rdW2, dyq = o.linear_bwd(bits(dY), hq, w2q)
    rdAB, ra_dab = o.silu_mul_bwd(rAB, rdH)
    rdX, rdW13, dabq = o.linear_bwd(rdAB, xq, w13q)

    f = FFN(M, D, H)
    # stage 1: stacked linear
    f8.linear_fwd_chained(f.d13, X.cuda(), None, W13.cuda(), f.AB, None, f.s13, f.ws)
    torch.cuda.synchronize()
    assert np.array_equal(u8(f.s13.x.q), xq.q) and np.array_equal(u8(f.s13.w.q), w13q.q)
    assert_gemm_close(bits(f.AB), rAB, "AB")
    # stage 2: glue on the oracle's AB
    f.AB.copy_(_from_bits(rAB))
    f8.silu_mul(f.AB, f.Hh, f.a_h, f.ws)
    torch.cuda.synchronize()
    assert_bf16_close(bits(f.Hh), rH, "h")
    # stage 3: second linear on the oracle's h and its amax
    f.Hh.copy_(_from_bits(rH))
    f.a_h.copy_(torch.from_numpy(ra_h))
    f8.linear_fwd_chained(f.d2, f.Hh, f.a_h, W2.cuda(), f.Y, None, f.s2, f.ws)
    torch.cuda.synchronize()
    assert np.array_equal(u8(f.s2.x.q), hq.q) and f32(f.s2.x.scale)[0] == hq.scale[0] and f32(f.s2.x.amax)[0] == hq.amax[0]
    assert_gemm_close(bits(f.Y), rY, "Y")
    # stage 4: backward of the second linear
    f8.linear_bwd_chained(f.d2, dY.cuda(), None, f.s2, f.dH, None, f.dW2, f.ws)
    torch.cuda.synchronize()
    assert np.array_equal(u8(f.s2.dy.q), dyq.q)
    assert_gemm_close(bits(f.dH), rdH, "dH"), assert_gemm_close(bits(f.dW2), rdW2, "dW2")
    # stage 5: glue backward on the oracle's dH
    f.dH.copy_(_from_bits(rdH))
    f8.silu_mul_bwd(f.AB, f.dH, f.dAB, f.a_dab, f.ws)
    torch.cuda.synchronize()
    assert_bf16_close(bits(f.dAB), rdAB, "dAB")
    # stage 6: backward of the stacked linear on the oracle's dAB and its amax
    f.dAB.copy_(_from_bits(rdAB))
    f.a_dab.copy_(torch.from_numpy(ra_dab))
    f8.linear_bwd_chained(f.d13, f.dAB, f.a_dab, f.s13, f.dX, None, f.dW13, f.ws)
    torch.cuda.synchronize()
    assert np.array_equal(u8(f.s13.dy.q), dabq.q) and f32(f.s13.dy.scale)[0] == dabq.scale[0]
    assert_gemm_close(bits(f.dX), rdX, "dX"), assert_gemm_close(bits(f.dW13), rdW13, "dW13")


def test_ffn_end_to_end_close_to_oracle():
    """The whole chain on the GPU against the whole chain in the oracle: quantisation noise of
    one stage moves the next stage's inputs, so the bar is the fp8 noise level, not the GEMM
    tolerance: relative error of Y and dX below 3 %."""
    M, D, H = 512, 768, 1024
    X, W13, W2, dY = _ffn_inputs(M, D, H, 7)
    rAB, xq, w13q = o.linear_fwd(bits(X), bits(W13))
    rH, _ = o.silu_mul(rAB)
    rY, hq, w2q = o.linear_fwd(rH, bits(W2))
    rdH, rdW2, _ = o.linear_bwd(bits(dY), hq, w2q)
    rdAB, _ = o.silu_mul_bwd(rAB, rdH)
    rdX, rdW13, _ = o.linear_bwd(rdAB, xq, w13q)
    f = FFN(M, D, H)
    f.forward(X.cuda(), W13.cuda(), W2.cuda())
    f.backward(dY.cuda())
    torch.cuda.synchronize()
    for name, got, ref in (("Y", f.Y, rY), ("dX", f.dX, rdX), ("dW13", f.dW13, rdW13), ("dW2", f.dW2, rdW2)):
        gv, rv = o.bf16_to_f32(bits(got)).astype(np.float64), o.bf16_to_f32(ref).astype(np.float64)
        assert np.abs(gv - rv).max() <= 3e-2 * np.abs(rv).max(), name


@pytest.mark.parametrize("M,D", [(16, 16), (272, 336), (512, 4096), (64, 16384)])
def test_rmsnorm_forward(M, D):
    g_ = torch.Generator("cpu")
    g_.manual_seed(M + D)
    x = wl.randn_bf16((M, D), 3.0, 0, generator=g_)
    x[1] = 0.0                                    # an all-zero row: rstd = 1 / sqrt(eps), y = 0
    gw = (1.0 + 0.1 * torch.randn(D, generator=g_)).to(torch.bfloat16)
    eps = 1e-5
    ws = f8.new_workspace(M, D)
    y = torch.empty((M, D), dtype=torch.bfloat16, device="cuda")
    rstd = torch.empty(M, device="cuda")
    amax = torch.full((1,), -1.0, device="cuda")
    f8.rmsnorm(x.cuda(), gw.cuda(), eps, y, rstd, amax, ws)
    torch.cuda.synchronize()
    ry, rr, ra = o.rmsnorm(bits(x), bits(gw), eps)
    assert_bf16_close(bits(y), ry, "y")
    assert np.allclose(f32(rstd), rr, rtol=2e-6)
    assert amax.item() == o.amax(bits(y))[0] and abs(amax.item() - ra[0]) <= 2.0 ** -7 * ra[0]
    y2 = torch.empty_like(y)
    f8.rmsnorm(x.cuda(), gw.cuda(), eps, y2)      # no rstd, no amax, no workspace
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), y2.view(torch.int16))


@pytest.mark.parametrize("M,D", [(4096, 4096), (4112, 4080), (2064, 8192)])
def test_rmsnorm_of_large_tensors(M, D):
    """Tensors of 16 M elements and more go past the caches: the bits of the call on pieces of the rows, which do not."""
    x = torch.randn((M, D), device="cuda").to(torch.bfloat16)
    gw = (1.0 + 0.1 * torch.randn(D, device="cuda")).to(torch.bfloat16)
    ws, a, b = f8.new_workspace(M, D), torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
    y, y2, r, r2 = torch.empty_like(x), torch.empty_like(x), torch.empty(M, device="cuda"), torch.empty(M, device="cuda")
    f8.rmsnorm(x, gw, 1e-5, y, r, a, ws)
    top = 0.0
    for i in range(0, M, 1024):
        f8.rmsnorm(x[i:i + 1024], gw, 1e-5, y2[i:i + 1024], r2[i:i + 1024], b, ws)
        top = max(top, b.item())
    assert torch.equal(y.view(torch.int16), y2.view(torch.int16)) and torch.equal(r, r2) and a.item() == top


def test_norm_then_feed_forward_chain():
    """rmsnorm -> w1|w3 -> silu(a) * b -> w2 with every amax handed over: identical to the same
    sequence with each linear taking its own amax."""
    M, D, H = 512, 768, 1024
    X, W13, W2, _ = (t.cuda() for t in _ffn_inputs(M, D, H, 8))
    gw = torch.ones(D, dtype=torch.bfloat16, device="cuda")
    outs = []
    for chained in (True, False):
        f = FFN(M, D, H)
        xn = torch.empty((M, D), dtype=torch.bfloat16, device="cuda")
        a_xn = torch.empty(1, device="cuda")
        f8.rmsnorm(X, gw, 1e-5, xn, None, a_xn if chained else None, f.ws)
        if chained:
            f8.linear_fwd_chained(f.d13, xn, a_xn, W13, f.AB, None, f.s13, f.ws)
            f8.silu_mul(f.AB, f.Hh, f.a_h, f.ws)
            f8.linear_fwd_chained(f.d2, f.Hh, f.a_h, W2, f.Y, None, f.s2, f.ws)
        else:
            f.forward(xn, W13, W2, chained=False)
        torch.cuda.synchronize()
        outs.append((f.Y, f.s13.x.q, f.s13.x.scale, codes_t(f.s2.x)))
    for a, b in zip(*outs):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("M,D,H", [(272, 336, 208), (512, 768, 1024)])
def test_glue_fused_into_the_delayed_cast(M, D, H):
    """silu(a) * b formed inside the cast of the next linear's input (delayed scaling): over
    several steps, codes, scales, amax, history, next scale and Y are bit-identical to writing h
    with f8_silu_mul and quantising it in the linear."""
    g = torch.Generator("cpu")
    g.manual_seed(M)
    W2 = wl.randn_bf16((D, H), 0.02, 0, generator=g).cuda()
    desc = f8.linear_desc(M, H, D)
    ws = f8.new_workspace(max(M, D, H), max(M, D, 2 * H))
    results = []
    steps = [wl.randn_bf16((M, 2 * H), 1.0 + 0.7 * i, 0, generator=g).cuda() for i in range(4)]
    for fused in (False, True):
        st = f8.ScalingState(f8.DELAYED, 2)
        st.scale_x.fill_(300.0), st.scale_w.fill_(5000.0)
        saved = f8.Saved(M, H, D)
        Y = torch.empty((M, D), dtype=torch.bfloat16, device="cuda")
        h = torch.empty((M, H), dtype=torch.bfloat16, device="cuda")
        snaps = []
        for AB in steps:
            if fused:
                f8.silu_mul_quantise_delayed(AB, f8.E4M3, st.hist_x, st.scale_x, saved.x, ws)
                f8.linear_fwd_xq(desc, st, W2, Y, saved, ws)
            else:
                f8.silu_mul(AB, h)
                f8.linear_fwd_scaled(desc, st, h, W2, Y, saved, ws)
            torch.cuda.synchronize()
            snaps.append([t.clone() for t in (Y, saved.x.q, codes_t(saved.x), saved.x.amax, saved.x.scale, saved.x.inv_scale,
                                              saved.w.q, st.hist_x, st.scale_x, st.hist_w, st.scale_w)])
        results.append(snaps)
    for a_step, b_step in zip(*results):
        for a, b in zip(a_step, b_step):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    # and against the oracle on the last step: where the GPU's h equals the oracle's h bit for bit
    # (almost everywhere), the codes are the oracle's codes for the scale that was used
    rh, _ = o.silu_mul(bits(steps[-1]))
    used_scale = f32(results[1][-1][4])
    ref_codes = o.cast(rh, used_scale, o.TENSORWISE, o.E4M3)
    got_codes = u8(results[1][-1][1])
    f8.silu_mul(steps[-1], h)
    torch.cuda.synchronize()
    same_h = bits(h) == rh
    assert same_h.mean() > 0.98 and np.array_equal(got_codes[same_h], ref_codes[same_h])


@pytest.mark.parametrize("M,D,H", [(272, 336, 208), (512, 768, 1024)])
def test_glue_backward_fused_into_the_delayed_cast(M, D, H):
    """The backward of silu(a) * b formed inside the cast of dAB, the output gradient of the stacked
    w1|w3 linear (delayed scaling): over several steps the codes in both orientations, scales,
    amax, history, next scale, dX and dW are bit-identical to writing dAB with f8_silu_mul_bwd and
    quantising it in the linear's backward."""
    g = torch.Generator("cpu")
    g.manual_seed(M + 1)
    W13 = wl.randn_bf16((2 * H, D), 0.02, 0, generator=g).cuda()
    X = wl.randn_bf16((M, D), 1.0, 0, generator=g).cuda()
    desc = f8.linear_desc(M, D, 2 * H)
    ws = f8.new_workspace(max(M, D, 2 * H), max(M, D, 2 * H))
    steps = [(wl.randn_bf16((M, 2 * H), 1.0 + 0.5 * i, 0, generator=g).cuda(),
              wl.randn_bf16((M, H), 1e-3 * (1 + i), 0, generator=g).cuda()) for i in range(4)]
    results = []
    for fused in (False, True):
        st = f8.ScalingState(f8.DELAYED, 2)
        st.scale_x.fill_(100.0), st.scale_w.fill_(5000.0), st.scale_dy.fill_(2.0e4)
        saved = f8.Saved(M, D, 2 * H)
        AB0 = torch.empty((M, 2 * H), dtype=torch.bfloat16, device="cuda")
        f8.linear_fwd_scaled(desc, st, X, W13, AB0, saved, ws)       # fills saved.x, saved.w
        dAB = torch.empty((M, 2 * H), dtype=torch.bfloat16, device="cuda")
        dX = torch.empty((M, D), dtype=torch.bfloat16, device="cuda")
        dW = torch.empty((2 * H, D), dtype=torch.bfloat16, device="cuda")
        snaps = []
        for AB, dh in steps:
            if fused:
                f8.silu_mul_bwd_quantise_delayed(AB, dh, f8.E4M3, st.hist_dy, st.scale_dy, saved.dy, ws)
                f8.linear_bwd_dyq(desc, saved, dX, dW)
            else:
                f8.silu_mul_bwd(AB, dh, dAB)
                f8.linear_bwd_scaled(desc, st, dAB, saved, dX, dW, ws)
            torch.cuda.synchronize()
            snaps.append([t.clone() for t in (dX, dW, saved.dy.q, codes_t(saved.dy), saved.dy.amax, saved.dy.scale,
                                              saved.dy.inv_scale, st.hist_dy, st.scale_dy)])
        results.append(snaps)
    for a_step, b_step in zip(*results):
        for a, b in zip(a_step, b_step):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    # against the oracle on the last step, where the GPU's dAB equals the oracle's bit for bit
    AB, dh = steps[-1]
    rd, _ = o.silu_mul_bwd(bits(AB), bits(dh))
    used_scale = f32(results[1][-1][5])
    ref_codes = o.cast(rd, used_scale, o.TENSORWISE, o.E4M3)
    got = u8(results[1][-1][2])
    f8.silu_mul_bwd(AB, dh, dAB)
    torch.cuda.synchronize()
    same = bits(dAB) == rd
    assert same.mean() > 0.97 and np.array_equal(got[same], ref_codes[same])


def test_fused_glue_backward_argument_checks():
    M, D, H = 64, 64, 64
    ws = f8.new_workspace(256, 256)
    ab = torch.zeros((M, 2 * H), dtype=torch.bfloat16, device="cuda")
    dh = torch.zeros((M, H), dtype=torch.bfloat16, device="cuda")
    st = f8.ScalingState(f8.DELAYED, 2)
    saved = f8.Saved(M, D, 2 * H)
    with pytest.raises(f8.F8Error):
        f8.silu_mul_bwd_quantise_delayed(ab, dh, 7, st.hist_dy, st.scale_dy, saved.dy, ws)
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    with pytest.raises(f8.F8Error):
        f8.silu_mul_bwd_quantise_delayed(ab, dh, f8.E4M3, st.hist_dy, st.scale_dy, saved.dy, small)
    rw = f8.linear_desc(M, D, 2 * H, rowwise=True)
    dX = torch.empty((M, D), dtype=torch.bfloat16, device="cuda")
    dW = torch.empty((2 * H, D), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(f8.F8Error):
        f8.linear_bwd_dyq(rw, saved, dX, dW)


# Less than a block; the last size with a chunk a thread (256 blocks) and the next; and from 8 M elements on two chunks side by
# side: one round of all blocks, and 12320 chunks more, 24 pairs of a block and 32 chunks.
@pytest.mark.parametrize("fmt", [f8.E4M3, f8.E5M2])
@pytest.mark.parametrize("M,H", [(16, 16), (512, 1024), (528, 1024), (1008, 2800), (2048, 4096), (2064, 4112)])
def test_streamed_glue_casts_equal_the_glue_and_a_cast(M, H, fmt, transposed=False):
    g = torch.Generator("cuda")
    g.manual_seed(M + H)
    R = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std).to(torch.bfloat16)
    ab, dh = R(1.5, M, 2 * H), R(1e-2, M, H)
    ws, hist = f8.new_workspace(M, 2 * H), torch.zeros(3, device="cuda")
    h, dab, amax = torch.empty_like(dh), torch.empty_like(ab), torch.empty(1, device="cuda")
    for plain, fused, t, s0 in ((lambda: f8.silu_mul(ab, h, amax, ws), lambda q, sc: f8.silu_mul_quantise_delayed(ab, fmt, hist, sc, q, ws), h, 30.0),
                                (lambda: f8.silu_mul_bwd(ab, dh, dab, amax, ws),
                                 lambda q, sc: f8.silu_mul_bwd_quantise_delayed(ab, dh, fmt, hist, sc, q, ws), dab, 5000.0)):
        plain()
        used, sc, q = torch.full((1,), s0, device="cuda"), torch.full((1,), s0, device="cuda"), f8.QTensor(M, t.shape[1], False, transposed=transposed)
        codes = torch.empty_like(q.q)
        f8.cast(t, used, f8.TENSORWISE, fmt, codes)
        fused(q, sc)
        torch.cuda.synchronize()
        assert torch.equal(codes, q.q) and torch.equal(amax, q.amax) and q.scale.item() == s0 and hist[0].item() == amax.item()
        assert not transposed or torch.equal(codes.t(), q.q_t)


# With a transposed copy in 128x128 tiles: part of one, and ragged rows and columns of several.
@pytest.mark.parametrize("fmt", [f8.E4M3, f8.E5M2])
@pytest.mark.parametrize("M,H", [(16, 16), (144, 272), (1008, 2800)])
def test_tiled_glue_casts_equal_the_glue_and_a_cast(M, H, fmt):
    test_streamed_glue_casts_equal_the_glue_and_a_cast(M, H, fmt, transposed=True)
