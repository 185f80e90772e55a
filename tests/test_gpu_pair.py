"""Both gradient products of a layer in one launch of the deferred-epilogue GEMM."""
import pytest
import torch

import paper_2511_23225_amd as tw
from gpu_util import DEV, scalar_f32

pytestmark = pytest.mark.gpu


# both products in one launch of the deferred-epilogue kernel: the weight gradient whole and in runs, tiles for some of the
# workgroups only, contractions of four to 44 stages under the input gradient's tiles, E5M2; against the products
# one by one in float64, and against the scratch of fewer runs
@pytest.mark.parametrize("hybrid", [False, True])
@pytest.mark.parametrize("shape,scratch", [((1024, 1024, 5632), None), ((8192, 3072, 768), None), ((8192, 768, 3072), None),
                                           ((13312, 512, 2304), None), ((16384, 1024, 1024), 2.0), ((16384, 1024, 1024), 0.0),
                                           ((3328, 5632, 1280), None), ((31488, 3584, 256), 5.5),
                                           # rows that end inside a stage of the weight gradient and inside a tile
                                           ((1872, 3072, 1792), None), ((3696, 3584, 1280), None), ((8208, 768, 3072), None),
                                           ((7200, 1536, 768), None), ((16400, 1024, 1024), 2.0), ((7088, 3072, 4608), None)])
def test_backward_of_whole_tiles_in_one_launch(shape, scratch, hybrid):
    M, N, K = shape
    print("deferred pair M=%d N=%d K=%d scratch %s hybrid %s" % (*shape, scratch, hybrid), flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(M + N + K)
    f8, dyt = torch.float8_e4m3fn, torch.float8_e5m2 if hybrid else torch.float8_e4m3fn
    rnd = lambda r, c, t: (torch.randn((r, c), generator=g, device=DEV) * 4).to(t)
    dyq, wq, xq = rnd(M, N, dyt), rnd(N, K, f8), rnd(M, K, f8)
    u8 = lambda t: t.contiguous().view(torch.uint8)
    tr = lambda t: u8(t.view(torch.uint8).t())
    one = scalar_f32(1.0)
    size = tw.tweo_workspace_bytes(tw.TWEO_OP_FP8_LINEAR_BWD, M, N, K) if scratch is None else 256 + int(scratch * N * K * 4)
    whole = torch.full((size + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    dx = torch.full((M, K), float("nan"), dtype=torch.bfloat16, device=DEV)
    dw = torch.full((N, K), float("nan"), dtype=torch.bfloat16, device=DEV)
    bwd = tw.tweo_fp8_linear_bwd_hybrid if hybrid else tw.tweo_fp8_linear_bwd
    for _ in range(2):  # a second call over the first one's runs
        bwd(u8(dyq), tr(dyq), one, tr(wq), one, tr(xq), one, M, N, K, dx, dw, whole[:size])
    torch.cuda.synchronize()
    assert bool((whole[size:] == 0xA5).all())
    for got, a, b in ((dx, dyq, wq), (dw, dyq.view(torch.uint8).t().view(dyt), xq)):
        a, b = a.double(), b.double()
        ref, refabs = a @ b, a.abs() @ b.abs()
        diff = (got.double() - ref).abs()
        # bf16 rounding, and what one FP8 MFMA loses (check_gemm)
        assert bool((diff <= 2.0 ** -8 * ref.abs() + (2.0 ** -10 + a.shape[1] * 2.0 ** -24) * refabs).all())
        assert float(diff.norm() / ref.norm()) < 3e-3


# The kernel that such a layer runs on, as tweo_gemm_plan names it, and on that kernel: two tiles and more for some workgroups, write-outs
# over three, five, seven and fifteen stages on either tile height, the scratch of fewer runs and of none
@pytest.mark.parametrize("hybrid", [False, True])
@pytest.mark.parametrize("shape,scratch,plan", [
    ((13312, 3072, 2048), None, (15, 1)), ((16384, 1024, 3072), None, (15, 3)), ((16384, 1024, 3072), 2.0, (15, 2)),
    ((10240, 1792, 3072), None, (15, 2)), ((10240, 1792, 3072), 0.0, (15, 1)),
    ((1872, 3072, 2304), None, (16, 1)), ((16400, 1280, 1280), None, (16, 5)), ((12304, 1024, 3072), 2.0, (16, 2)),
    ((6160, 1792, 4096), 0.0, (16, 1)), ((16400, 2048, 1536), 2.0, (16, 2)), ((12304, 2048, 2048), None, (16, 2))])
def test_backward_on_the_deferred_kernel(shape, scratch, plan, hybrid):
    assert backward_plan(shape, scratch) == plan
    test_backward_of_whole_tiles_in_one_launch(shape, scratch, hybrid)


# what the layers above the last test run on: eight of the shapes the ring kernel's launch, or the products one after the other
@pytest.mark.parametrize("shape,scratch,plan", [
    ((8192, 3072, 768), None, (15, 3)), ((8192, 768, 3072), None, (15, 3)), ((13312, 512, 2304), None, (15, 5)),
    ((8208, 768, 3072), None, (16, 3)), ((7088, 3072, 4608), None, (16, 1)),
    ((1024, 1024, 5632), None, (21, 1)), ((16384, 1024, 1024), 2.0, (21, 2)), ((3328, 5632, 1280), None, (21, 1)),
    ((31488, 3584, 256), 5.5, (21, 5)), ((3696, 3584, 1280), None, (21, 1)), ((7200, 1536, 768), None, (21, 3)),
    ((16384, 1024, 1024), 0.0, None), ((16400, 1024, 1024), 2.0, None)])
def test_plan_of_a_backward(shape, scratch, plan):
    assert backward_plan(shape, scratch) == plan


def backward_plan(shape, scratch):
    """(kernel, runs) of both products in one launch with that scratch, None of one after the other."""
    M, N, K = shape
    size = tw.tweo_workspace_bytes(tw.TWEO_OP_FP8_LINEAR_BWD, M, N, K) if scratch is None else 256 + int(scratch * N * K * 4)
    kernel, runs, shared = tw.tweo_gemm_plan(tw.TWEO_OP_FP8_LINEAR_BWD, M, N, K, workspace_bytes=size)
    return (kernel, runs) if shared else None


# events armed for both products of a backward call whose products share a launch of the deferred-epilogue kernel: two pairs, as the
# products apart record, the second for the addition of runs or empty; the next GEMM finds none of them
@pytest.mark.parametrize("shape,plan", [((13312, 3072, 2048), (15, 1, True)), ((1872, 3072, 2304), (16, 1, True)), ((8208, 768, 3072), (16, 3, True))])
def test_profile_events_of_a_shared_launch(shape, plan):
    M, N, K = shape
    print("profile events M=%d N=%d K=%d" % shape, flush=True)
    u8 = lambda *s: torch.full(s, 0x30, dtype=torch.uint8, device=DEV)
    dyq, dyqT, wqT, xqT = u8(M, N), u8(N, M), u8(K, N), u8(K, M)
    dx, dw = (torch.empty(s, dtype=torch.bfloat16, device=DEV) for s in ((M, K), (N, K)))
    ws = torch.empty(tw.tweo_workspace_bytes(tw.TWEO_OP_FP8_LINEAR_BWD, M, N, K), dtype=torch.uint8, device=DEV)
    assert tw.tweo_gemm_plan(tw.TWEO_OP_FP8_LINEAR_BWD, M, N, K, workspace_bytes=ws.numel()) == plan
    one = scalar_f32(1.0)
    call = lambda: tw.tweo_fp8_linear_bwd(dyq, dyqT, one, wqT, one, xqT, one, M, N, K, dx, dw, ws)
    call()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(8)]
    for e in ev:
        e.record()  # creates the handle, in front of the call
    tw.tweo_profile_gemm_launches([e.cuda_event for e in ev[:6]])
    call()
    tw.tweo_profile_gemm_launches([])
    ev[7].record()
    torch.cuda.synchronize()
    assert [ev[6].elapsed_time(e) > 0.0 for e in ev[:6]] == [True] * 4 + [False] * 2
    assert 0.0 < ev[0].elapsed_time(ev[1]) < ev[6].elapsed_time(ev[7])
    assert ev[1].elapsed_time(ev[2]) >= 0.0 and ev[2].elapsed_time(ev[3]) >= 0.0 and ev[3].elapsed_time(ev[7]) >= 0.0


# the weight gradient alone, in runs over a contraction that ends 16, 48 and 112 into a stage, and at one; a NaN of either
# operand stays in its row or column, also where a lane past the end loads its row's first chunk
@pytest.mark.parametrize("hybrid", [False, True])
@pytest.mark.parametrize("shape", [(16400, 512, 768), (15408, 768, 1536), (16496, 256, 512), (16512, 256, 512)])
def test_weight_gradient_of_ragged_rows(shape, hybrid):
    M, N, K = shape
    print("weight gradient M=%d N=%d K=%d hybrid %s" % (*shape, hybrid), flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(M + N + K)
    dyt = torch.float8_e5m2 if hybrid else torch.float8_e4m3fn
    dyT = (torch.randn((N, M), generator=g, device=DEV) * 4).to(dyt)
    xT = (torch.randn((K, M), generator=g, device=DEV) * 4).to(torch.float8_e4m3fn)
    one = scalar_f32(1.0)
    ws = torch.full((tw.tweo_workspace_bytes(tw.TWEO_OP_FP8_LINEAR_BWD, M, N, K),), 0xA5, dtype=torch.uint8, device=DEV)
    bwd = tw.tweo_fp8_linear_bwd_hybrid if hybrid else tw.tweo_fp8_linear_bwd

    def run():
        dw = torch.full((N, K), float("nan"), dtype=torch.bfloat16, device=DEV)
        bwd(None, dyT.view(torch.uint8), one, None, None, xT.view(torch.uint8), one, M, N, K, None, dw, ws)
        torch.cuda.synchronize()
        return dw.double()

    got, a, b = run(), dyT.double(), xT.double()
    ref, refabs = a @ b.t(), a.abs() @ b.abs().t()
    assert bool(((got - ref).abs() <= 2.0 ** -8 * ref.abs() + (2.0 ** -10 + M * 2.0 ** -24) * refabs).all())
    dyT.view(torch.uint8)[3, 5] = xT.view(torch.uint8)[7, 11] = 0x7F
    xT.view(torch.uint8)[9, M - 1] = 0x7F
    nan = run().isnan()
    want = torch.zeros_like(nan)
    want[3, :] = want[:, 7] = want[:, 9] = True
    assert torch.equal(nan, want)


# contractions that end 16, 80 and 112 into a stage, in runs of the deferred-epilogue kernel; the first four shapes of the test above run
# on the ring kernel, in runs and whole
@pytest.mark.parametrize("hybrid", [False, True])
@pytest.mark.parametrize("shape,plan", [
    ((16400, 1280, 1280), (15, 8)), ((16752, 1280, 1280), (15, 8)), ((19408, 768, 1536), (15, 9)), ((30064, 256, 2304), (15, 14))])
def test_weight_gradient_in_ragged_runs(shape, plan, hybrid):
    assert weight_gradient_plan(shape) == plan
    test_weight_gradient_of_ragged_rows(shape, hybrid)


@pytest.mark.parametrize("shape,plan", [((16400, 512, 768), (19, 5)), ((15408, 768, 1536), (20, 1)), ((16496, 256, 512), (4, 8)),
                                        ((16512, 256, 512), (4, 7))])
def test_plan_of_a_weight_gradient(shape, plan):
    assert weight_gradient_plan(shape) == plan


def weight_gradient_plan(shape):
    """(kernel, runs) of the weight gradient alone, with the backward's workspace."""
    M, N, K = shape
    # (the scratch lies behind 256 bytes there, in the forward call, which takes the product here, behind the penalty's)
    scratch = tw.tweo_workspace_bytes(tw.TWEO_OP_FP8_LINEAR_FWD, N, K, 16) + tw.tweo_workspace_bytes(tw.TWEO_OP_FP8_LINEAR_BWD, M, N, K) - 256
    return tw.tweo_gemm_plan(tw.TWEO_OP_FP8_LINEAR_FWD, N, K, M, workspace_bytes=scratch)[:2]
