"""The fragment-B GEMM's tile plans (dn::frag_plan, a host function of the library): plans only
name kernels that run, and the shapes of the GPU operator tests reach every kernel."""

import pytest

from tests.plans import CONV, COVER, FP8, LINEAR, VT, plan, plan_fp32


def test_vt_output_never_plans_a_kernel_that_does_not_run():
    """Projections with a V^T output run unsplit and not on the four-wave 128 x 160 tile:
    the plan may not price that tile for them, at any size of the sublayers."""
    for heads, K in ((20, 1280), (10, 640), (8, 320), (5, 320), (20, 2048), (10, 768), (8, 768)):
        for n in (1, 2, 4, 8):
            for tokens in [77, *range(64, 1100, 31), *range(1100, 4200, 293)]:
                g = plan(n * tokens, 3 * 64 * heads, K, VT)
                assert (g.x5, g.split, g.frag) == (0, 1, 1), (n * tokens, heads, K)
    # the same sizes without V^T do use it
    assert any(plan(2 * t, 960, 320, LINEAR).x5 for t in range(64, 4200, 31))


def test_gpu_shapes_reach_every_kernel():
    """The shapes of the GPU operator tests take the tile and split each is there for, and
    together every tile, split and unsplit, that some shape of a wide range is given."""
    for (kind, M, N, K, geglu, out_f32), want in COVER.items():
        g = plan(M, N, K, kind, geglu=geglu, out_f32=out_f32)
        assert (g.bm, g.bn, g.x5, g.split) == want, (kind, M, N, K)
        assert M % g.bm and N % g.bn, "ragged tiles"
    have = {(k[0], v[0], v[1], v[2], v[3] > 1, k[4]) for k, v in COVER.items()}
    for kind in (LINEAR, VT, CONV, FP8):
        for geglu in ((False, True) if kind in (LINEAR, FP8) else (False,)):
            for M in (33, 154, 512, 1000, 2048, 2100, 4096, 8192, 12000, 16384, 32768, 262144):
                for N in (64, 128, 320, 512, 640, 1280, 1920, 2560, 3840, 10240):
                    for K in (128, 320, 640, 1280, 2560, 2880, 5120, 5760, 11520, 23040):
                        if K % 64 or (kind == FP8 and K % 128):
                            continue
                        for out_f32 in (False, True):
                            g = plan(M, N, K, kind, geglu=geglu, out_f32=out_f32)
                            assert (kind, g.bm, g.bn, g.x5, g.split > 1, geglu) in have, (M, N, K)


@pytest.mark.parametrize("M,N,K,want,us,other", [
    (2048, 1280, 11520, (128, 160, 1, 4), 82.9, "128 x 256 in three parts 98.8 (upsampled input)"),
    (2048, 1280, 17280, (128, 256, 0, 6), 104.2, "three parts 108.6"),
    (2048, 1280, 23040, (128, 256, 0, 6), 133.2, "three parts 142.3"),
    (8192, 640, 8640, (128, 160, 1, 1), 105.1, "two parts 112.3"),
])
def test_convolution_plans_are_the_measured_best(M, N, K, want, us, other):
    """SD-XL convolutions whose plans lie close together in the cost model and far apart on the
    device (us measured for the wanted plan and for its nearest rival)."""
    g = plan(M, N, K, CONV)
    assert (g.bm, g.bn, g.x5, g.split) == want, f"{us} us wanted, {other}"


@pytest.mark.parametrize("M,N,K,want,us,other", [
    (16384, 320, 1280, (128, 128, 1), 20.5, "128 x 256 24.0"),
    (1152, 320, 1280, (128, 128, 3), 11.1, "unsplit 11.9"),
    (2048, 320, 1280, (128, 128, 1), 12.0, "two parts 13.0"),
])
def test_fp8_plans_are_the_measured_best(M, N, K, want, us, other):
    """Feed-forward outputs of 320 channels with an fp32 residual (as above)."""
    g = plan(M, N, K, FP8, out_f32=True)
    assert (g.bm, g.bn, g.split) == want, f"{us} us wanted, {other}"


@pytest.mark.parametrize("M,N,K,kind,waves,us,other", [
    (512, 512, 576, "linear", True, 10.8, 18.6), (512, 512, 64, "linear", False, 5.7, 6.2),
    (1024, 512, 2560, "linear", True, 50.0, 65.3), (1024, 512, 64, "linear", False, 6.6, 11.2),
    (8192, 64, 1280, "linear", False, 36.6, 39.6), (1024, 960, 1280, "linear", False, 36.1, 57.0),
    (16256, 64, 5120, "linear", False, 133.3, 299.6), (64, 16320, 576, "linear", False, 20.8, 41.9),
    (512, 1024, 64, "geglu", True, 8.2, 11.5), (512, 1280, 64, "geglu", False, 11.6, 14.7),
    (512, 1280, 320, "geglu", True, 18.7, 29.0), (8192, 64, 576, "conv", True, 17.4, 21.6),
    (4096, 192, 1152, "conv", True, 34.0, 38.2), (4096, 192, 288, "conv", False, 12.9, 15.3),
    (2048, 448, 2880, "conv", False, 87.8, 102.2)])
def test_fp32_launches_split_k_over_waves_only_where_faster(M, N, K, kind, waves, us, other):
    """Both forms measured (us of the wanted one, then of the other) on each side of every line
    of the rule."""
    g = plan_fp32(M, N, K, geglu=kind == "geglu", conv=kind == "conv")
    assert (g.bm == 32) == waves, f"{us} us wanted, {other}"
