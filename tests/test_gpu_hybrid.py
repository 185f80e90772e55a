"""GPU parity of the HYBRID recipe's gradient path (Sec. 4.3: E4M3 activations and weights, E5M2
gradients): E5M2 quantize-cast bit-exact against the CPU oracle, dgrad / wgrad with E5M2 dY within
the FP8 GEMM tolerance, through the C ABI."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_23225_amd as tw
from paper_2511_23225_amd import synth
from gpu_util import DEV, to_dev_bf16, to_dev, bf16_bits, scalar_f32, workspace, check_gemm

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


def is_nan_code(q):
    return ((q & 0x7C) == 0x7C) & ((q & 0x03) != 0)


def gpu_quantize_e5m2(x_dev, amax_dev, transpose=True):
    r, c = x_dev.shape
    q = torch.empty((r, c), dtype=torch.uint8, device=DEV)
    qT = torch.empty((c, r), dtype=torch.uint8, device=DEV) if transpose else None
    s, si = scalar_f32(), scalar_f32()
    tw.tweo_quantize_e5m2(x_dev, amax_dev, q, qT, s, si)
    return q, qT, s, si


def test_quantize_e5m2_all_bf16_patterns_times_scales():
    # every bf16 bit pattern, for scales that exercise flush, subnormal, normal, saturate
    allx = np.arange(65536, dtype=np.uint32).astype(np.uint16).reshape(256, 256)
    amaxes = [57344.0, 1.0, 9873.0, 3.0e4, 0.013, 1e-30, 3.0e38, 57344.0 * 8, 5000.0, 0.0, np.inf, np.nan]
    xd = to_dev_bf16(allx)
    for amax in amaxes:
        say("quantize e5m2 all patterns, amax=%r" % amax)
        q, qT, s, si = gpu_quantize_e5m2(xd, scalar_f32(amax))
        scale, scale_inv = oracle.scale_from_amax_e5m2(np.float32(amax))
        assert s.cpu().numpy()[0] == scale and si.cpu().numpy()[0] == scale_inv
        want, wantT = oracle.quantize_e5m2(allx, scale)
        got, gotT = q.cpu().numpy(), qT.cpu().numpy()
        nan = is_nan_code(want)
        assert np.array_equal(is_nan_code(got), nan)  # NaN -> a NaN code (which one is unpinned)
        assert np.array_equal(got[~nan], want[~nan])
        assert np.array_equal(gotT, got.T)
        assert not (((got & 0x7F) == 0x7C) & ~nan).any()  # a cast never produces an infinity


@pytest.mark.parametrize("shape", [(8, 8), (24, 40), (100, 72), (256, 512), (1000, 1024), (16, 65536)])
def test_quantize_e5m2_shapes(shape):
    r, c = shape
    say("quantize e5m2 shape %dx%d" % shape)
    rng = np.random.default_rng(r * 131 + c)
    x = synth.f32_to_bf16_bits((rng.standard_normal((r, c)) * np.exp(rng.uniform(-8, 3, (r, c)))).astype(np.float32))
    amax = oracle.amax_bf16(x)
    q, qT, _, _ = gpu_quantize_e5m2(to_dev_bf16(x), scalar_f32(amax))
    scale, _ = oracle.scale_from_amax_e5m2(amax)
    want, wantT = oracle.quantize_e5m2(x, scale)
    assert np.array_equal(q.cpu().numpy(), want) and np.array_equal(qT.cpu().numpy(), wantT)
    assert (want & 0x7F).max() == 0x7B  # the element that attains amax saturates the range


def oracle_e4m3(x):
    s, si = oracle.scale_from_amax(oracle.amax_bf16(x))
    q, qT = oracle.quantize_e4m3(x, s)
    return q, qT, si


def oracle_e5m2(x):
    s, si = oracle.scale_from_amax_e5m2(oracle.amax_bf16(x))
    q, qT = oracle.quantize_e5m2(x, s)
    return q, qT, si


# tiny (64x64 tiles), ragged, mid-sized (register-staged 128 / 256 tiles), whole-tile shapes for
# the deferred-epilogue kernel (dgrad: rows M, contraction N; wgrad: rows N, contraction M) with
# one and with several tiles per workgroup, and a long contraction that takes the 192-row tiles
HYBRID_CASES = [
    (0, 0, 64, 64, 48, 0),
    (1, 0, 208, 264, 144, 0),
    (0, 0, 256, 512, 512, 0),
    (3, 0, 1024, 1024, 1024, 0),
    (3, 1, 4352, 2048, 4096, 0),
    (3, 2, 2304, 512, 4608, 15),
    (1, 1, 2048, 768, 2304, 16),
    (3, 0, 16400, 264, 528, 0),  # few tiles, long contraction: the K split with an E5M2 operand
    (1, 1, 16384, 768, 768, 0),  # the same on whole 256x256 tiles: the deferred-epilogue kernel's K split
]


@pytest.mark.parametrize("case", HYBRID_CASES)
def test_bwd_hybrid(case):
    cfg, gi, M, K, N, tile = case
    say("bwd hybrid cfg=%d M=%d K=%d N=%d tile=%d" % (cfg, M, K, N, tile))
    x, w, dy = synth.fp8_linear_inputs(cfg, gi, M=M, K=K, N=N)
    xq, xqT, sxi = oracle_e4m3(x)
    wq, wqT, swi = oracle_e4m3(w)
    dyq, dyqT, sdyi = oracle_e5m2(dy)
    dx_ref, dx_abs = oracle.fp8_linear_dgrad(dyq, wq, sdyi, swi, dy_e5m2=True)
    dw_ref, dw_abs = oracle.fp8_linear_wgrad(dyq, xq, sdyi, sxi, dy_e5m2=True)
    dx = torch.full((M, K), float('nan'), dtype=torch.bfloat16, device=DEV)
    dw = torch.full((N, K), float('nan'), dtype=torch.bfloat16, device=DEV)
    tw.tweo_set_gemm_tile(tile)
    try:
        tw.tweo_fp8_linear_bwd_hybrid(to_dev(dyq), to_dev(dyqT), scalar_f32(sdyi), to_dev(wqT),
                                      scalar_f32(swi), to_dev(xqT), scalar_f32(sxi), M, N, K, dx, dw,
                                      workspace(tw.TWEO_OP_FP8_LINEAR_BWD, M, N, K))
        torch.cuda.synchronize()
    finally:
        tw.tweo_set_gemm_tile(0)
    check_gemm(bf16_bits(dx), dx_ref, dx_abs, N, "dgrad")
    check_gemm(bf16_bits(dw), dw_ref, dw_abs, M, "wgrad")


def test_hybrid_whole_backward_from_bf16():
    cfg, gi, M, K, N = 0, 0, 256, 512, 512
    say("hybrid bf16 path M=%d K=%d N=%d" % (M, K, N))
    x, w, dy = synth.fp8_linear_inputs(cfg, gi)
    u8 = lambda *s: torch.empty(s, dtype=torch.uint8, device=DEV)
    xq, xqT, wq, wqT, dyq, dyqT = u8(M, K), u8(K, M), u8(N, K), u8(K, N), u8(M, N), u8(N, M)
    sc = torch.zeros(16, dtype=torch.float32, device=DEV)
    saved = tw.make_saved(xq, xqT, wq, wqT, sc)
    y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    dx = torch.full((M, K), float('nan'), dtype=torch.bfloat16, device=DEV)
    dw = torch.full((N, K), float('nan'), dtype=torch.bfloat16, device=DEV)
    ws = workspace(tw.TWEO_OP_FP8_LINEAR_FWD_BF16, M, N, K)
    tw.tweo_fp8_linear_fwd_bf16(to_dev_bf16(x), to_dev_bf16(w), y, saved, workspace=ws)
    tw.tweo_fp8_linear_bwd_bf16_hybrid(to_dev_bf16(dy), saved, K, dyq, dyqT, dx, dw, ws)
    torch.cuda.synchronize()
    oxq, _, sxi = oracle_e4m3(x)
    owq, _, swi = oracle_e4m3(w)
    odyq, odyqT, sdyi = oracle_e5m2(dy)
    assert np.array_equal(dyq.cpu().numpy(), odyq) and np.array_equal(dyqT.cpu().numpy(), odyqT)
    assert sc.cpu().numpy()[8] == sdyi
    dx_ref, dx_abs = oracle.fp8_linear_dgrad(odyq, owq, sdyi, swi, dy_e5m2=True)
    dw_ref, dw_abs = oracle.fp8_linear_wgrad(odyq, oxq, sdyi, sxi, dy_e5m2=True)
    check_gemm(bf16_bits(dx), dx_ref, dx_abs, N, "dgrad")
    check_gemm(bf16_bits(dw), dw_ref, dw_abs, M, "wgrad")


@pytest.mark.parametrize("shape", [(256, 512), (200, 136), (1024, 768)])
def test_delayed_scaling_sequence_e5m2(shape):
    # the gradient tensors under the paper's own recipe (Sec. 4.3: HYBRID formats, delayed scaling
    # with an amax history of 16): 20 steps with a spike and an all-zero step, bytes and the
    # scales in the state bit-exact against the oracle
    rows, cols = shape
    say("delayed scaling, E5M2", shape)
    ref = oracle.DelayedScaling(e5m2=True)
    state = torch.full((tw.DELAYED_STATE_WORDS,), -7.0, dtype=torch.float32, device=DEV)
    tw.tweo_delayed_state_init(state)
    q = torch.empty((rows, cols), dtype=torch.uint8, device=DEV)
    qT = torch.empty((cols, rows), dtype=torch.uint8, device=DEV)
    rng = np.random.default_rng(rows + 3 * cols)
    for step in range(20):
        v = (rng.standard_normal((rows, cols)) * (1.0 + 0.1 * step)).astype(np.float32)
        if step == 3:
            v[rng.integers(rows), rng.integers(cols)] = -4321.0
        if step == 7:
            v[:] = 0.0
        x = synth.f32_to_bf16_bits(v)
        oq, oqT, used, used_inv = ref.cast(x)
        q.fill_(0x55)
        qT.fill_(0x55)
        tw.tweo_quantize_e5m2_delayed(to_dev_bf16(x), state, q, qT, bootstrap=(step == 0))
        torch.cuda.synchronize()
        st = state.cpu().numpy()
        assert np.array_equal(q.cpu().numpy(), oq), step
        assert np.array_equal(qT.cpu().numpy(), oqT), step
        assert st[tw.DELAYED_USED_SCALE].view(np.uint32) == np.float32(used).view(np.uint32), step
        assert st[tw.DELAYED_USED_SCALE_INV].view(np.uint32) == np.float32(used_inv).view(np.uint32), step
        assert st[tw.DELAYED_NEXT_SCALE].view(np.uint32) == np.float32(ref.next_scale).view(np.uint32), step


@pytest.mark.parametrize("pen", [(3.0, 1e-6, 4), (2.0, 0.0, 3)])
@pytest.mark.parametrize("e5m2", [False, True])
def test_backward_with_fused_penalty_gradient_injection(e5m2, pen):
    # the injection as a prologue of the gradient's amax and cast: every downstream bit equals what
    # the stand-alone injection kernel followed by the plain backward call gives, and the codes
    # equal the oracle's (injection -> bf16 -> amax -> cast)
    cfg, gi, M, K, N = 0, 0, 256, 512, 512
    say("fused injection e5m2=%s pen=%s" % (e5m2, pen))
    x, w, dy = synth.fp8_linear_inputs(cfg, gi)
    u8 = lambda *s: torch.empty(s, dtype=torch.uint8, device=DEV)
    bf = lambda *s: torch.full(s, float("nan"), dtype=torch.bfloat16, device=DEV)
    g = 0.37 / (M * N)
    results = []
    for fused in (True, False):
        xq, xqT, wq, wqT, dyq, dyqT = u8(M, K), u8(K, M), u8(N, K), u8(K, N), u8(M, N), u8(N, M)
        sc = torch.zeros(16, dtype=torch.float32, device=DEV)
        saved = tw.make_saved(xq, xqT, wq, wqT, sc)
        y, dx, dw = bf(M, N), bf(M, K), bf(N, K)
        ws = torch.empty(max(tw.tweo_workspace_bytes(op, M, N, K) for op in
                             (tw.TWEO_OP_FP8_LINEAR_FWD_BF16, tw.TWEO_OP_FP8_LINEAR_BWD_BF16)),
                         dtype=torch.uint8, device=DEV)
        tw.tweo_fp8_linear_fwd_bf16(to_dev_bf16(x), to_dev_bf16(w), y, saved, workspace=ws)
        dyd = to_dev_bf16(dy)
        if fused:
            tw.tweo_fp8_linear_bwd_bf16_inject(dyd, y, pen, g, saved, K, dyq, dyqT, dx, dw, ws, dy_e5m2=e5m2)
        else:
            dy2 = torch.empty_like(dyd)
            tw.tweo_penalty_grad_inject(dyd, y, pen, g, dy2)
            (tw.tweo_fp8_linear_bwd_bf16_hybrid if e5m2 else tw.tweo_fp8_linear_bwd_bf16)(
                dy2, saved, K, dyq, dyqT, dx, dw, ws)
        torch.cuda.synchronize()
        results.append([t.clone() for t in (dyq, dyqT, sc, dx.view(torch.int16), dw.view(torch.int16))])
        y_bits = bf16_bits(y)
    for a, b in zip(*results):
        assert torch.equal(a, b)
    # against the oracle (fp64 injection): the GPU forms the gradient in fp32, so a value that sits at a
    # bf16 rounding boundary may come out one ulp apart (tests of the stand-alone kernel); hence the
    # amax within one bf16 ulp, and, when it is the same, the same codes on all but the odd element
    dy2_ref, _ = oracle.penalty_grad_inject(dy, y_bits, pen[0], pen[1], pen[2], g)
    amax = oracle.amax_bf16(dy2_ref)
    dyq, dyqT, sc = results[0][0], results[0][1], results[0][2].cpu().numpy()
    got_amax_bits = int(sc[6:7].view(np.uint32)[0])
    assert abs(got_amax_bits - int(np.float32(amax).view(np.uint32))) <= 1 << 16
    if sc[6] == amax:
        if e5m2:
            s_ref, si_ref = oracle.scale_from_amax_e5m2(amax)
            q_ref, qT_ref = oracle.quantize_e5m2(dy2_ref, s_ref)
        else:
            s_ref, si_ref = oracle.scale_from_amax(amax)
            q_ref, qT_ref = oracle.quantize_e4m3(dy2_ref, s_ref)
        assert sc[7] == s_ref and sc[8] == si_ref
        assert np.mean(dyq.cpu().numpy() == q_ref) > 0.99 and np.mean(dyqT.cpu().numpy() == qT_ref) > 0.99
        assert np.array_equal(dyqT.cpu().numpy(), dyq.cpu().numpy().T)


# E5M2 gradients on every kernel that the same product of E4M3 codes can run on: whole 128-byte stages
# (11, 13, 14), whole 64-byte stages (6, 8), K split of ragged tiles (no override), ragged rows and columns
@pytest.mark.parametrize("tile,shape", [(11, (384, 640, 520)), (13, (384, 640, 520)), (14, (640, 384, 264)), (6, (448, 576, 520)),
                                        (8, (448, 576, 520)), (0, (16448, 200 // 8 * 8, 264)), (0, (2048, 336, 136)),
                                        (0, (96, 1872, 1120))])
def test_e5m2_gradients_on_the_tiled_kernels(tile, shape):
    M, N, K = shape
    N = (N + 15) // 16 * 16
    say("e5m2 tile=%d M=%d N=%d K=%d" % (tile, M, N, K))
    x, w, dy = synth.fp8_linear_inputs(1, 0, M=M, K=K, N=N)
    sx, sxi = oracle.scale_from_amax(oracle.amax_bf16(x))
    sw, swi = oracle.scale_from_amax(oracle.amax_bf16(w))
    sd, sdi = oracle.scale_from_amax_e5m2(oracle.amax_bf16(dy))
    xq, xqT = oracle.quantize_e4m3(x, sx)
    wq, wqT = oracle.quantize_e4m3(w, sw)
    dyq, dyqT = oracle.quantize_e5m2(dy, sd)
    ws = workspace(tw.TWEO_OP_FP8_LINEAR_BWD, M, N, K)
    dx = torch.full((M, K), float("nan"), dtype=torch.bfloat16, device=DEV)
    dw = torch.full((N, K), float("nan"), dtype=torch.bfloat16, device=DEV)
    d = [to_dev(np.ascontiguousarray(t)) for t in (dyq, dyqT, wqT, xqT)]
    tw.tweo_set_gemm_tile(tile)
    try:
        for out in (dict(dx_bf16=dx), dict(dw_bf16=dw)):  # one product at a time
            tw.tweo_fp8_linear_bwd_hybrid(d[0], d[1], scalar_f32(sdi), d[2], scalar_f32(swi), d[3], scalar_f32(sxi), M, N, K,
                                          workspace=ws, **out)
        torch.cuda.synchronize()
    finally:
        tw.tweo_set_gemm_tile(0)
    ref, refabs = oracle.fp8_linear_dgrad(dyq, wq, sdi, swi, dy_e5m2=True)
    check_gemm(bf16_bits(dx), ref, refabs, N, "dgrad")
    ref, refabs = oracle.fp8_linear_wgrad(dyq, xq, sdi, sxi, dy_e5m2=True)
    check_gemm(bf16_bits(dw), ref, refabs, M, "wgrad")
