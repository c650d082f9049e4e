"""How a render call is cut into launches and tiles, without a GPU: every ray is
rendered by one tile, every launch fits the 32-bit grid of the dispatch packet,
and its split tail fits the scratch."""
import random

import pytest

from paper_2103_03231_amd import binding as b

PREC = {"fp32": b.FP32, "bf16": b.BF16, "fp8": b.FP8}
# every tile a precision has a kernel for, and that kernel's threads
TILES = {"fp32": {64: 512, 32: 512}, "bf16": {256: 512, 64: 512, 32: 512}, "fp8": {128: 256, 64: 512, 32: 512}}
SCRATCH = 5 * 256 * 256   # floats of the split tail's scratch at 256 compute units


def plan(precision, P, H, W, N, n_cu=256, **cfg):
    c = b.Config(precision=PREC[precision], n_max=16, **cfg)
    out = []
    while True:
        p = b.donerf_debug_plan(c, P, H, W, N, launch=len(out), n_cu=n_cu)
        if not p:
            return out
        out.append(p)


def check(precision, launches, P, H, W, n_cu=256):
    assert sum(p["poses"] for p in launches) == P
    for p in launches:
        assert 1 <= p["poses"] <= 32
        assert TILES[precision][p["tile_rays"]] == p["threads"], p
        tiles = -(-p["poses"] * H * W // p["tile_rays"])
        assert p["n_full"] + p["n_split"] == tiles, p
        groups = p["n_full"] + p["n_split"] * p["split"]
        assert groups * p["threads"] < 2 ** 32, p
        if p["split"] > 1:
            assert 5 * p["n_split"] * p["split"] * p["tile_rays"] <= SCRATCH * n_cu // 256, p


# fp32 tiles of 64 rays are rendered by 512 threads: 32 views of 2^24 rays are
# 2^32 work-items, one more than a launch can have
@pytest.mark.parametrize("P,H,W", [(32, 4096, 4096), (127, 4096, 4096), (32, 1, (1 << 24) - 1), (35, 4095, 4097),
                                   (1, 4096, 4096), (33, 4000, 4000)])
@pytest.mark.parametrize("precision", PREC)
def test_launches_fit_the_grid_at_the_size_limits(precision, P, H, W):
    for N in (1, 4, 16):
        check(precision, plan(precision, P, H, W, N), P, H, W)


@pytest.mark.parametrize("precision", PREC)
def test_plans_cover_every_ray_within_the_scratch(precision):
    rng = random.Random(7)
    for _ in range(400):
        P = rng.choice([1, 1, 2, 5, 32, 33])
        H, W = (int(2 ** rng.uniform(0, 10.5)) for _ in range(2))
        N, n_cu = rng.randrange(1, 17), rng.choice([256, 256, 304, 64, 1])
        kw = {"n_bins": rng.choice([64, 128, 192, 256]), "select": rng.choice([b.SELECT_TOPN, b.SELECT_CDF]),
              "depth_input": rng.choice([b.DEPTH_ENCODED, b.DEPTH_POSITIONS])}
        check(precision, plan(precision, P, H, W, N, n_cu, **kw), P, H, W, n_cu)


def test_plan_refuses_what_render_refuses():
    c = b.Config(n_max=4)
    for args in ((0, 4, 4, 4), (1, 4, 4, 5), (1, 4, 4, 0), (1, 4097, 4096, 4), (128, 4096, 4096, 4)):
        with pytest.raises(b.DonerfError) as e:
            b.donerf_debug_plan(c, *args)
        assert e.value.status == b.E_INVALID_ARG
    with pytest.raises(b.DonerfError) as e:
        b.donerf_debug_plan(b.Config(n_bins=100), 1, 4, 4, 4)
    assert e.value.status == b.E_UNSUPPORTED


# Microseconds of one call of an fp8 network on an MI355X, by (rays per tile,
# workgroups per tile of the last round): every tile and several splits timed.
MEASURED_FP8 = [
    ("cdf", "positions", 256, 4422, 7, {(32, 1): 48.2, (64, 1): 61.8, (64, 3): 41.3, (128, 1): 119.3, (128, 3): 73.8,
                                        (128, 7): 54.2}),
    ("cdf", "encoded", 192, 7310, 16, {(32, 1): 92.6, (64, 1): 119.8, (64, 2): 76.1, (128, 1): 229.3, (128, 2): 135.8,
                                       (128, 4): 92.3, (128, 8): 90.9}),
    ("cdf", "encoded", 192, 12100, 9, {(32, 1): 114.1, (32, 2): 98.5, (64, 1): 77.5, (128, 1): 142.4, (128, 2): 99.7,
                                       (128, 5): 86.4}),
    ("cdf", "positions", 64, 5550, 5, {(32, 1): 37.8, (64, 1): 47.1, (64, 2): 37.8, (128, 1): 85.1, (128, 2): 63.1,
                                       (128, 5): 41.6}),
    ("cdf", "positions", 64, 39800, 8, {(32, 1): 257.4, (64, 1): 209.3, (64, 2): 187.8, (128, 1): 172.4}),
    ("topn", "positions", 64, 5852, 16, {(32, 1): 90.0, (64, 1): 119.0, (64, 2): 71.0, (128, 1): 216.6, (128, 2): 122.7,
                                         (128, 5): 76.9, (128, 11): 77.6}),
    ("topn", "encoded", 128, 24964, 4, {(32, 1): 116.4, (32, 4): 104.3, (64, 1): 78.6, (128, 1): 69.7, (128, 2): 64.8}),
    ("topn", "encoded", 192, 25440, 4, {(32, 1): 120.1, (32, 4): 107.2, (64, 1): 81.7, (128, 1): 75.3, (128, 2): 71.5}),
    ("topn", "encoded", 64, 5929, 4, {(32, 1): 30.5, (64, 1): 38.2, (64, 2): 28.9, (128, 1): 67.7, (128, 2): 45.9,
                                      (128, 4): 35.1}),
]


@pytest.mark.parametrize("select,din,B,rays,N,us", MEASURED_FP8)
def test_fp8_plan_is_near_the_fastest_measured(select, din, B, rays, N, us):
    (p,) = plan("fp8", 1, 1, rays, N, n_bins=B, select=b.SELECT_CDF if select == "cdf" else b.SELECT_TOPN,
                depth_input=b.DEPTH_POSITIONS if din == "positions" else b.DEPTH_ENCODED)
    assert us[p["tile_rays"], p["split"]] <= 1.05 * min(us.values()), p
