"""The ring GEMM (128-byte stages in a deep ring, one tile per workgroup): every tile shape against the oracle where
it can go wrong - edges of tiles, fewer stages than the ring, one more, contractions that end inside a stage -
in every operand format and with everything its way out can do; runs of a K split; both gradients in one launch."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_23225_amd as tw
from paper_2511_23225_amd import synth
from gpu_util import DEV, PEN, to_dev, bf16_bits, scalar_f32, workspace, check_gemm, check_penalty
from test_gpu_fp8_linear import run_fwd, oracle_quantized, check_bwd_pair
from test_gpu_w8a8_rows import run_scaled

pytestmark = pytest.mark.gpu

# 64x64, 64x64 and 64x128 in two groups of waves, 64x128, 128x128, 96x128; stages in the ring: 4, 8, 3, 6, 4, 5
RING = [4, 18, 19, 20, 21, 22]


def say(*a):
    print(*a, flush=True)


@pytest.fixture
def tile(request):
    tw.tweo_set_gemm_tile(request.param)
    yield request.param
    tw.tweo_set_gemm_tile(0)


# one chunk, one stage, inside the second, as many stages as each ring has and one more, many; rows and columns
# on the edges of tiles and just past them
@pytest.mark.parametrize("tile", RING, indirect=True)
@pytest.mark.parametrize("shape", [(64, 64, 16), (1, 8, 128), (96, 128, 144), (128, 128, 384), (129, 136, 512), (97, 264, 528),
                                   (200, 520, 640), (192, 192, 784), (65, 72, 1024), (256, 128, 1152), (130, 200, 2064)])
def test_forward(shape, tile):
    M, N, K = shape
    say("ring fwd M=%d N=%d K=%d tile=%d" % (M, N, K, tile))
    x, w, _ = synth.fp8_linear_inputs(1, 0, M=M, K=K, N=N)
    xq, _, sxi = oracle_quantized(x)
    wq, _, swi = oracle_quantized(w)
    for res, pen in ((None, None), (None, PEN), (synth.residual_input(1, 0, M, N), PEN), (None, (2.0, 0.5, 3))):
        ref, refabs, refbf = oracle.fp8_linear_fwd(xq, wq, sxi, swi, residual=res)
        got, S = run_fwd(xq, wq, sxi, swi, M, N, K, residual=res, pen=pen)
        check_gemm(got, ref, refabs, K, "fwd")
        if pen:
            check_penalty(S, got, refbf, oracle.penalty_sum(refbf, *pen), pen, strict=False)


@pytest.mark.parametrize("tile", RING, indirect=True)
@pytest.mark.parametrize("K", [48, 144, 1040, 1056])
def test_a_nan_stays_in_its_column(K, tile):
    # in the chunk that stands in for those past a contraction's end
    M, N = 70, 136
    say("ring NaN K=%d tile=%d" % (K, tile))
    x, w, _ = synth.fp8_linear_inputs(1, 0, M=M, K=K, N=N)
    xq, _, sxi = oracle_quantized(x)
    wq = oracle_quantized(w)[0].copy()
    wq[5, 0] = 0x7F
    got, _ = run_fwd(xq, wq, sxi, np.float32(1.0), M, N, K, pen=None)
    val = (got.astype(np.uint32) << 16).view(np.float32)
    assert np.isnan(val[:, 5]).all() and not np.isnan(np.delete(val, 5, axis=1)).any()


@pytest.mark.parametrize("tile", RING, indirect=True)
@pytest.mark.parametrize("shape", [(65, 72, 1040), (129, 264, 528), (96, 128, 1152), (40, 136, 80)])
def test_int8(shape, tile):
    M, N, K = shape
    say("ring INT8 M=%d N=%d K=%d tile=%d" % (M, N, K, tile))
    rng = np.random.default_rng(M + K)
    xq, wq = (rng.integers(-127, 128, (n, K), dtype=np.int8) for n in (M, N))
    y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    tw.tweo_w8a8_linear(to_dev(xq), to_dev(wq), 0.001, y)
    torch.cuda.synchronize()
    assert np.array_equal(bf16_bits(y), oracle.w8a8_linear(xq, wq, 0.001))
    sx, sw = (rng.uniform(1e-3, 1e-2, n).astype(np.float32) for n in (M, N))
    assert np.array_equal(run_scaled(xq, wq, sx, sw, tile), oracle.w8a8_linear_scaled(xq, wq, sx, sw))
    tw.tweo_set_gemm_tile(tile)
    out = torch.zeros((M, N), dtype=torch.int8, device=DEV)
    tw.tweo_w8a8_linear_scaled_i8out(to_dev(xq), to_dev(wq), to_dev(sx), to_dev(sw), 0.7, out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), oracle.w8a8_linear_scaled_i8out(xq, wq, sx, sw, np.float32(0.7)))


# every XCD starts at its own stage; fewer stages than XCDs, no whole number of eighths, and tiles alone or two on a CU
@pytest.mark.parametrize("shape", [(100, 6200, 1152), (128, 12288, 384), (192, 12288, 512), (70, 4104, 1664), (512, 4096, 2176)])
def test_int8_as_dispatched(shape):
    M, N, K = shape
    say("ring INT8 as dispatched M=%d N=%d K=%d" % (M, N, K))
    rng = np.random.default_rng(M + K)
    xq, wq = (rng.integers(-127, 128, (n, K), dtype=np.int8) for n in (M, N))
    y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    tw.tweo_w8a8_linear(to_dev(xq), to_dev(wq), 0.001, y)
    torch.cuda.synchronize()
    assert np.array_equal(bf16_bits(y), oracle.w8a8_linear(xq, wq, 0.001))


@pytest.mark.parametrize("tile", RING, indirect=True)
@pytest.mark.parametrize("shape", [(208, 272, 144), (1040, 128, 264)])
def test_e5m2_gradients(shape, tile):
    M, N, K = shape
    say("ring E5M2 M=%d N=%d K=%d tile=%d" % (M, N, K, tile))
    check_bwd_pair(shape, True)


# default dispatch: runs of small tiles under a long contraction (a stage count they do not divide, ragged
# rows, a tile and a bit), and both products in one launch on each shape that takes pairs
@pytest.mark.parametrize("hybrid", [False, True])
@pytest.mark.parametrize("shape", [(8576, 256, 256), (20480, 256, 256), (16400, 272, 264), (12288, 512, 512),
                                   (256, 512, 512), (1024, 512, 1024), (2048, 1024, 1024), (4096, 704, 512), (672, 768, 3072),
                                   (1552, 1040, 2064), (4096, 3072, 768)])
def test_backward(shape, hybrid):
    check_bwd_pair(shape, hybrid)


# contractions over more than 4096 rows: both products in one launch, the weight gradient in two to seven runs (a stage count
# that they do not divide, ragged rows and not, tiles past every edge); without a workspace whole
@pytest.mark.parametrize("hybrid", [False, True])
@pytest.mark.parametrize("shape", [(4112, 272, 272), (8240, 880, 336), (14208, 688, 384), (12208, 2736, 400), (5248, 672, 1552)])
def test_backward_over_many_rows(shape, hybrid):
    check_bwd_pair(shape, hybrid)


# scratch for fewer runs than were asked for, down to none: the bytes past it stay as they are
@pytest.mark.parametrize("runs", [6.5, 3.0, 1.9, 0.0])
def test_backward_over_many_rows_in_less_scratch(runs):
    M, N, K = 8240, 880, 336
    say("ring backward over many rows, scratch of %.1f runs" % runs)
    x, w, dy = synth.fp8_linear_inputs(1, 0, M=M, K=K, N=N)
    (xq, xqT, sxi), (wq, wqT, swi), (dyq, dyqT, sdi) = (oracle_quantized(t) for t in (x, w, dy))
    whole = torch.full((tw.tweo_workspace_bytes(tw.TWEO_OP_FP8_LINEAR_BWD, M, N, K) + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    size = 256 + int(runs * N * K * 4)
    dx = torch.full((M, K), float("nan"), dtype=torch.bfloat16, device=DEV)
    dw = torch.full((N, K), float("nan"), dtype=torch.bfloat16, device=DEV)
    args = [to_dev(np.ascontiguousarray(t)) for t in (dyq, dyqT, wqT, xqT)]
    tw.tweo_fp8_linear_bwd(args[0], args[1], scalar_f32(sdi), args[2], scalar_f32(swi), args[3], scalar_f32(sxi), M, N, K, dx, dw,
                           whole[:size])
    torch.cuda.synchronize()
    assert bool((whole[size:] == 0xA5).all())
    check_gemm(bf16_bits(dx), *oracle.fp8_linear_dgrad(dyq, wq, sdi, swi), N, "dgrad")
    check_gemm(bf16_bits(dw), *oracle.fp8_linear_wgrad(dyq, xq, sdi, sxi), M, "wgrad")


def penalised_layer(seed, M, N, K, delayed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    u8 = lambda *s: torch.zeros(s, dtype=torch.uint8, device=DEV)
    t = dict(x=torch.randn((M, K), generator=g, device=DEV).bfloat16(), w=(torch.randn((N, K), generator=g, device=DEV) * 0.1).bfloat16(),
             y=torch.empty((M, N), dtype=torch.bfloat16, device=DEV), sc=torch.full((16,), 7.0, dtype=torch.float32, device=DEV),
             codes=[u8(M, K), u8(K, M), u8(N, K), u8(K, N)], ws=workspace(tw.TWEO_OP_FP8_LINEAR_FWD_BF16, M, N, K))
    t["saved"] = tw.make_saved(*t["codes"], t["sc"])
    if delayed:
        t["states"] = [torch.zeros(tw.DELAYED_STATE_WORDS, dtype=torch.float32, device=DEV) for _ in range(2)]
        for st in t["states"]:
            tw.tweo_delayed_state_init(st)
    return t


def forward(t, S, **more):
    if "states" in t:
        tw.tweo_fp8_linear_fwd_bf16_delayed(t["x"], t["w"], t["y"], t["saved"], *t["states"], pen=PEN, penalty_sum=S, workspace=t["ws"], **more)
    else:
        tw.tweo_fp8_linear_fwd_bf16(t["x"], t["w"], t["y"], t["saved"], pen=PEN, penalty_sum=S, workspace=t["ws"], **more)


# the penalty finished by the last workgroup of the GEMM (up to one workgroup per CU, behind a cast that clears its sum)
# against the finishing kernel on the same codes: the same bits, call after call, over a poisoned sum
@pytest.mark.parametrize("shape", [(16, 16, 64), (256, 512, 512), (1024, 1024, 256), (1040, 1024, 256), (2048, 1024, 1024),
                                   (816, 608, 2064), (2048, 2048, 256)])
def test_penalty_finished_by_the_last_workgroup(shape):
    M, N, K = shape
    say("ring penalty finish M=%d N=%d K=%d" % shape)
    g = torch.Generator(device=DEV)
    g.manual_seed(M + N)
    u8 = lambda *s: torch.zeros(s, dtype=torch.uint8, device=DEV)
    sc = torch.zeros(16, dtype=torch.float32, device=DEV)
    xq, xqT, wq, wqT = u8(M, K), u8(K, M), u8(N, K), u8(K, N)
    saved = tw.make_saved(xq, xqT, wq, wqT, sc)
    ws = workspace(tw.TWEO_OP_FP8_LINEAR_FWD_BF16, M, N, K)
    y, y2 = (torch.empty((M, N), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    S, S2 = (torch.full((1,), float("nan"), dtype=torch.float64, device=DEV) for _ in range(2))
    w = (torch.randn((N, K), generator=g, device=DEV) * 0.1).bfloat16()
    for pen in (PEN, PEN, (2.0, 0.5, 3)):
        x = torch.randn((M, K), generator=g, device=DEV).bfloat16()
        tw.tweo_fp8_linear_fwd_bf16(x, w, y, saved, pen=pen, penalty_sum=S, workspace=ws)
        tw.tweo_fp8_linear_fwd(xq, sc[2:3], wq, sc[5:6], y2, pen=pen, penalty_sum=S2, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(y, y2) and S.item() > 0.0
        assert torch.equal(S.view(torch.int64), S2.view(torch.int64))
        S.fill_(float("nan"))


# ... on every tile shape (two groups of waves, one of which has left by then, 96 and 128 rows), edges and whole tiles, with
# a residual; what the counter and the sum held before does not matter
@pytest.mark.parametrize("tile", RING, indirect=True)
@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("shape", [(16, 16, 64), (208, 272, 528), (384, 512, 1152)])
def test_penalty_finished_on_every_shape(shape, residual, tile):
    M, N, K = shape
    say("ring penalty finish M=%d N=%d K=%d residual=%s tile=%d" % (shape + (residual, tile)))
    t = penalised_layer(M + N, M, N, K, False)
    g = torch.Generator(device=DEV)
    g.manual_seed(K)
    r = torch.randn((M, N), generator=g, device=DEV).bfloat16() if residual else None
    y2 = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    S, S2 = (torch.zeros(1, dtype=torch.float64, device=DEV) for _ in range(2))
    for poison in (0x5555555555555555, -1, 0):
        S.view(torch.int64).fill_(poison)
        t["sc"][15:].view(torch.int32).fill_(poison >> 32)
        forward(t, S, residual_bf16=r)
        tw.tweo_fp8_linear_fwd(t["codes"][0], t["sc"][2:3], t["codes"][2], t["sc"][5:6], y2, residual_bf16=r, pen=PEN, penalty_sum=S2,
                               workspace=t["ws"])
        torch.cuda.synchronize()
        assert torch.equal(t["y"], y2) and S.item() > 0.0
        assert torch.equal(S.view(torch.int64), S2.view(torch.int64)) and t["sc"][15:].view(torch.int32).item() == 0
        t["x"].mul_(1.25)


# an argument that is refused only behind the cast: nothing has written the sum by then
@pytest.mark.parametrize("delayed", [False, True])
def test_a_refused_call_leaves_the_sum(delayed):
    M, N, K = 256, 512, 512
    t = penalised_layer(1, M, N, K, delayed)
    S = torch.full((1,), 0x5555555512345678, dtype=torch.int64, device=DEV).view(torch.float64)
    if delayed:
        forward(t, torch.zeros(1, dtype=torch.float64, device=DEV), bootstrap=True)
    t["y"] = torch.empty(M * N + 8, dtype=torch.bfloat16, device=DEV)[1:1 + M * N].view(M, N)
    with pytest.raises(tw.TweoError) as e:
        forward(t, S)
    torch.cuda.synchronize()
    assert e.value.status == tw.TWEO_ERR_INVALID_ARG
    assert S.view(torch.int64).item() == 0x5555555512345678


# calls on two streams with one sum that nobody reads: their histories and scalars are those of calls with sums of
# their own, and the words that the last workgroups counted in are 0 again
@pytest.mark.parametrize("shape", [(256, 512, 512), (1024, 1024, 256)])
def test_calls_in_flight_may_share_a_sum(shape):
    M, N, K = shape
    alone, shared = ([penalised_layer(3 + i, M, N, K, True) for i in range(2)] for _ in range(2))
    S = torch.zeros(3, dtype=torch.float64, device=DEV)
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for step in range(40):
        for i in range(2):
            forward(alone[i], S[i:i + 1], bootstrap=step == 0)
            with torch.cuda.stream(streams[i]):
                forward(shared[i], S[2:3], bootstrap=step == 0)
                shared[i]["x"].mul_(1.0 + 0.25 * (step % 3 - 1))
            alone[i]["x"].mul_(1.0 + 0.25 * (step % 3 - 1))
    torch.cuda.synchronize()
    for a, b in zip(alone, shared):
        assert torch.equal(a["y"], b["y"]) and torch.equal(a["sc"], b["sc"]) and a["sc"][15].item() == 0.0
        for k in range(2):
            assert torch.equal(a["states"][k].view(torch.int32), b["states"][k].view(torch.int32))
        assert int(b["states"][0].view(torch.int32)[19]) == 40 % 16


# INT8 into more columns than the ring kernel has tiles resident for: the stream, 64-byte stages and the streaming kernel, as
# estimated, on both sides of a round of 128x128 tiles
@pytest.mark.parametrize("shape", [(33, 66048, 4096), (65, 66048, 512), (64, 65536, 1024), (48, 131080, 1024), (17, 32000, 2048), (128, 66056, 1088)])
def test_int8_into_wide_outputs(shape):
    M, N, K = shape
    say("ring INT8 wide M=%d N=%d K=%d" % (M, N, K))
    g = torch.Generator(device=DEV)
    g.manual_seed(N + K)
    xq, wq = (torch.randint(-127, 128, (n, K), generator=g, device=DEV, dtype=torch.int8) for n in (M, N))
    y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    tw.tweo_w8a8_linear(xq, wq, 0.001, y)
    rows = torch.cat([torch.arange(64), torch.randint(0, N, (512,)), torch.arange(N - 64, N)]).to(DEV)
    torch.cuda.synchronize()
    want = oracle.w8a8_linear(xq.cpu().numpy(), wq[rows].cpu().numpy(), 0.001)
    assert np.array_equal(bf16_bits(y[:, rows].contiguous()), want) and not bool(y.isnan().any())
