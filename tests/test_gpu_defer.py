"""The deferred-epilogue GEMM: the residual under contractions of as few stages as it takes, two tile heights in one
launch, edges on every side."""
import pytest
import torch

import paper_2511_23225_amd as tw
from gpu_util import DEV, PEN, scalar_f32, workspace
from test_gpu_fp8_linear import test_fwd_residual_on_the_deferred_kernels as check_residual

pytestmark = pytest.mark.gpu


# five stages of write-out, five of the residual and the last one (11 in all), one more; one tile and a second one
@pytest.mark.parametrize("case", [(15, 256, 1408, 256, PEN), (15, 512, 1408, 512, None), (15, 8448, 1408, 2048, PEN),
                                  (15, 8448, 1536, 2048, None)])
def test_residual_under_short_contractions(case):
    check_residual(case)


# 192-row tiles alone and behind 256-row ones under 11 and 15 stages; 18 stages and more: the residual over eight of them
@pytest.mark.parametrize("case", [(23, 200, 1408, 512, PEN), (23, 4112, 1408, 6144, PEN), (23, 4112, 1920, 6144, None),
                                  (15, 8448, 2304, 2048, None), (16, 4160, 2304, 3072, PEN), (16, 200, 2432, 512, None), (23, 4112, 2304, 6144, PEN)])
def test_residual_on_either_tile_height(case):
    check_residual(case)


def kernel_of(kind, tile, shape):
    """The kernel that products(kind, *shape)(tile) runs on (INT8 calls go by the same rule and are not asked for)."""
    pen = kind in ("penalty", "residual")
    tw.tweo_set_gemm_tile(tile)
    try:
        return tw.tweo_gemm_plan(tw.TWEO_OP_FP8_LINEAR_FWD, *shape, p=4 if pen else 0, residual=kind == "residual",
                                 workspace_bytes=tw.tweo_workspace_bytes(tw.TWEO_OP_FP8_LINEAR_FWD, *shape))[0]
    finally:
        tw.tweo_set_gemm_tile(0)


def products(kind, M, N, K):
    """What computes the product into y (and the penalty's sum into S) on the kernel that is set."""
    g = torch.Generator(device=DEV)
    g.manual_seed(M + N + K)
    u8 = lambda t: t.contiguous().view(torch.uint8)
    rnd = lambda r, c, t: u8((torch.randn((r, c), generator=g, device=DEV) * 4).to(t))
    one = scalar_f32(0.01)
    a = rnd(M, K, torch.int8 if kind == "int8" else torch.float8_e5m2 if kind == "e5m2" else torch.float8_e4m3fn)
    b = rnd(N, K, torch.int8 if kind == "int8" else torch.float8_e4m3fn)
    res = torch.randn((M, N), generator=g, device=DEV).bfloat16() if kind == "residual" else None
    ws = workspace(tw.TWEO_OP_FP8_LINEAR_FWD, M, N, K)

    def run(tile):
        y = torch.full((M + 1, N), float("nan"), dtype=torch.bfloat16, device=DEV)
        S = torch.zeros(2, dtype=torch.float64, device=DEV)
        tw.tweo_set_gemm_tile(tile)
        try:
            if kind == "int8":
                tw.tweo_w8a8_linear(a.view(torch.int8), b.view(torch.int8), 0.01, y[:M])
            elif kind == "e5m2":  # an input gradient of a layer [K, N] -> dx [M, N]
                tw.tweo_fp8_linear_bwd_hybrid(a, None, one, b, one, None, None, M, K, N, y[:M], None, ws)
            else:
                tw.tweo_fp8_linear_fwd(a, one, b, one, y[:M], residual_bf16=res, pen=PEN if kind != "plain" else None,
                                       penalty_sum=S if kind != "plain" else None, workspace=ws)
            torch.cuda.synchronize()
        finally:
            tw.tweo_set_gemm_tile(0)
        assert bool(y[M].isnan().all())  # nothing behind the last row
        return y[:M], float(S[0].cpu())

    return run


# contractions over five, seven and fifteen stages of write-out; 192-row tiles alone (the first two), one and two rounds of either
# height, workgroups without a tile of one of them; rows that end inside a tile, and inside the first quad of one; against the 8-wave
# kernel, with a residual (one rounding less) the 192-row tiles: the same bits
@pytest.mark.parametrize("shape,kinds", [((200, 512, 768), "plain penalty"), ((4104, 512, 1152), "penalty int8"),
                                         ((4112, 6144, 768), "plain penalty int8 e5m2"), ((4097, 6144, 1152), "penalty e5m2"),
                                         ((8193, 4864, 2048), "plain penalty residual int8 e5m2"), ((512, 256, 2048), "penalty residual"),
                                         ((20000, 2048, 2176), "penalty residual"), ((50432, 768, 2304), "residual int8")])
def test_two_tile_heights_in_one_launch(shape, kinds):
    M, N, K = shape
    for kind in kinds.split():
        if kind == "e5m2" and M % 16 != 0:
            continue
        print("two tile heights M=%d N=%d K=%d %s" % (M, N, K, kind), flush=True)
        run = products(kind, M, N, K)
        y, S = run(23)
        ref, Sref = run(16 if kind == "residual" else 11)
        assert torch.equal(y.view(torch.int16), ref.view(torch.int16)), kind
        # (fp32 sums of each wave's own tiles: some thousand terms a lane)
        assert abs(S - Sref) <= 2e-6 * Sref, kind
        again, S2 = run(23)
        assert torch.equal(y.view(torch.int16), again.view(torch.int16)) and S == S2


# in the place of the 128x128 streaming tiles, which the shape alone decides: three to six rounds of those, rows that end inside a tile,
# one height and two; full rounds, which stay (the last)
@pytest.mark.parametrize("shape,kinds", [((8704, 2304, 768), "plain penalty int8 e5m2"), ((10737, 2048, 896), "penalty int8"),
                                         ((6224, 6144, 1664), "plain penalty residual e5m2"), ((7388, 5120, 1408), "residual"),
                                         ((8192, 3072, 768), "plain penalty")])
def test_two_tile_heights_by_the_shape(shape, kinds):
    M, N, K = shape
    for kind in kinds.split():
        print("by the shape M=%d N=%d K=%d %s" % (M, N, K, kind), flush=True)
        run = products(kind, M, N, K)
        (y, S), (ref, Sref) = run(0), run(23 if kind == "residual" else 11)
        assert torch.equal(y.view(torch.int16), ref.view(torch.int16)), kind
        assert abs(S - Sref) <= 2e-6 * Sref, kind


# columns, rows and contractions that end inside a tile, inside a stage, at one; eight stages and more under write-outs of five,
# seven and fifteen; one tile, several for some workgroups; against the register-staged kernel, which takes any of them: the same bits
@pytest.mark.parametrize("shape,kinds", [((193, 136, 912), "plain penalty int8"), ((10, 264, 1008), "penalty int8"), ((208, 512, 1040), "penalty e5m2"),
                                         ((8193, 1608, 912), "plain penalty int8"), ((8208, 1616, 1200), "penalty e5m2 int8"),
                                         ((8193, 1544, 2416), "penalty int8"), ((8208, 1552, 2320), "plain e5m2"),
                                         ((50000, 264, 2304), "penalty")])
def test_edges_on_every_side(shape, kinds):
    M, N, K = shape
    for kind in kinds.split():
        print("edges on every side M=%d N=%d K=%d %s" % (M, N, K, kind), flush=True)
        run = products(kind, M, N, K)
        y, S = run(24)
        ref, Sref = run(3)
        assert torch.equal(y.view(torch.int16), ref.view(torch.int16)), kind
        assert abs(S - Sref) <= 2e-6 * Sref, kind
        again, S2 = run(24)
        assert torch.equal(y.view(torch.int16), again.view(torch.int16)) and S == S2


# a NaN of the weight stays in its column and one of the activation in its row, also where a row's first chunk is loaded again
def test_nan_under_edges_on_every_side():
    M, N, K = 8193, 1608, 912
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    a, b = ((torch.randn(s, generator=g, device=DEV) * 4).to(torch.float8_e4m3fn).view(torch.uint8) for s in ((M, K), (N, K)))
    a[3, 5] = a[8192, K - 1] = b[7, 11] = b[1607, K - 1] = 0x7F
    y = torch.zeros((M, N), dtype=torch.bfloat16, device=DEV)
    tw.tweo_set_gemm_tile(24)
    try:
        tw.tweo_fp8_linear_fwd(a, scalar_f32(1.0), b, scalar_f32(1.0), y)
        torch.cuda.synchronize()
    finally:
        tw.tweo_set_gemm_tile(0)
    want = torch.zeros((M, N), dtype=torch.bool, device=DEV)
    want[3] = want[8192] = want[:, 7] = want[:, 1607] = True
    assert torch.equal(y.isnan(), want)


# as dispatched: ragged rows under a short contraction, whole rows with a badly filled last round of 256
@pytest.mark.parametrize("shape", [(7400, 3584, 1664), (50432, 768, 3072)])
def test_two_tile_heights_as_dispatched(shape):
    run = products("penalty", *shape)
    (y, S), (ref, Sref) = run(0), run(23)
    assert torch.equal(y.view(torch.int16), ref.view(torch.int16)) and S == Sref


# Which kernel the products above run on.  As first written 512x2048 -> 256 leaves no rows for a second height and compares
# the 192-row kernel with itself, 10x1008 -> 264 the register-staged one: neighbours that do not stand beside them.
@pytest.mark.parametrize("tile,shape,kinds", [(23, (520, 256, 2048), "penalty residual"), (24, (10, 504, 1008), "penalty int8")])
def test_small_products_on_the_kernel_they_are_for(tile, shape, kinds):
    for kind in kinds.split():
        assert kind == "int8" or kernel_of(kind, tile, shape) == tile
    (test_two_tile_heights_in_one_launch if tile == 23 else test_edges_on_every_side)(shape, kinds)


@pytest.mark.parametrize("tile,ran,kinds,shapes", [
    (23, 23, "plain penalty", ((200, 512, 768), (4104, 512, 1152), (4112, 6144, 768), (4097, 6144, 1152))),
    (23, 23, "plain penalty residual", ((8193, 4864, 2048), (20000, 2048, 2176), (50432, 768, 2304))),
    (11, 11, "plain penalty", ((200, 512, 768), (4104, 512, 1152), (4112, 6144, 768), (8193, 4864, 2048))),
    (16, 16, "residual", ((8193, 4864, 2048), (20000, 2048, 2176), (50432, 768, 2304))),
    (24, 24, "plain penalty", ((193, 136, 912), (208, 512, 1040), (8193, 1608, 912), (8208, 1616, 1200), (8193, 1544, 2416),
                               (8208, 1552, 2320), (50000, 264, 2304))),
    (3, 3, "plain penalty", ((193, 136, 912), (8193, 1608, 912), (50000, 264, 2304))),
    # by the shape (a residual under 11 to 15 stages has no other kernel of one rounding: its values are checked above)
    (0, 23, "plain penalty", ((8704, 2304, 768), (10737, 2048, 896), (6224, 6144, 1664))),
    (0, 23, "residual", ((6224, 6144, 1664), (7388, 5120, 1408))), (0, 13, "plain penalty", ((8192, 3072, 768),)),
    (0, 23, "penalty", ((7400, 3584, 1664), (50432, 768, 3072)))])
def test_products_run_on_the_kernel_they_are_for(tile, ran, kinds, shapes):
    for shape in shapes:
        for kind in kinds.split():
            assert kernel_of(kind, tile, shape) == ran, (shape, kind)
