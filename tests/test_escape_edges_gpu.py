"""Escape-time counts where the blocked loop, its escape test and its cycle
test could go wrong: caps around the block length, |c| near 2 (the plain
loop's border, the tip of the real axis and c = -2, whose orbit is a cycle),
components of c near the smallest it scales, zero, denormal, huge and NaN
coordinates. Counts are whole numbers and equal the oracle's."""
import numpy as np
import pytest
import torch

import paper_1805_02755_amd as ce
from oracle import oracle as O

pytestmark = pytest.mark.gpu

# (x0, y0, dx, dy)
REGIONS = {
    "set": (-2.0, -1.5, 3.0 / 128, 3.0 / 96),
    "tip": (-2.0, -2e-5, 1e-6, 1e-6),
    "tip_outside": (-2.00001, 0.0, 2.4e-7, 1e-6),
    "circle": (1.3, 1.3, 0.002, 0.002),
    "border_of_plain": (-1.99999, -0.02, 1e-7, 5e-4),
    "seahorse": (-0.75, 0.1, 2e-4, 2e-4),
    "near_zero": (-2e-6, -2e-6, 4e-8, 4e-8),
    "zero_row": (-2.0, 0.0, 3.0 / 128, 0.0),
    "zero_column": (0.0, -1.5, 0.0, 3.0 / 96),
    "least_imaginary": (-1.9, -4e-18, 0.01, 1e-19),
    "denormal_imaginary": (-1.9, 0.0, 0.01, 1e-40),
    "tiny_real": (0.0, 0.3, 1e-38, 0.01),
    "huge": (-1e30, -1e38, 1e28, 3e36),
    "nan": (float("nan"), -1.0, 0.01, 0.02),
}


@pytest.mark.parametrize("max_iter", [1, 2, 7, 8, 9, 16, 17, 100, 1003])
@pytest.mark.parametrize("region", sorted(REGIONS))
def test_counts_equal_the_oracles(region, max_iter):
    w, h = 131, 96
    x0, y0, dx, dy = (float(np.float32(v)) for v in REGIONS[region])
    out = torch.full((h, w), -1, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    ce.ce_bare_run(ce.CE_KERNEL_ESCAPE, ce.ce_escape_params(w, h, x0, y0, dx, dy, max_iter), [], out)
    ref = O.escape(w, h, x0, y0, dx, dy, max_iter)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref)


# Around the discs that no orbit leaves: the fixed point's border at c = 1/4, at
# -3/4 (where the cycle of two takes over) and in between, the cycle's at -5/4
# and above, and the seahorse and elephant valleys, where orbits escape late.
DISCS = {
    "root": (0.2499, -3e-4, 4e-6, 6e-6),
    "root_wide": (0.15, -0.12, 0.002, 0.0025),
    "neck": (-0.7512, -0.0031, 2e-5, 6e-5),
    "neck_wide": (-0.85, -0.12, 0.0015, 0.0025),
    "two_left": (-1.2512, -0.002, 2e-5, 4e-5),
    "two_top": (-1.02, 0.23, 3e-4, 4e-4),
    "cusp_side": (0.27, 0.48, 2e-4, 2e-4),
    "elephant": (0.255, 0.0, 2e-5, 2e-5),
    "real_axis": (-2.0, 0.0, 0.018, 0.0),
}


@pytest.mark.parametrize("max_iter", [64, 20011])
@pytest.mark.parametrize("region", sorted(DISCS))
def test_orbits_near_the_discs(region, max_iter):
    w, h = 128, 96
    x0, y0, dx, dy = (float(np.float32(v)) for v in DISCS[region])
    out = torch.full((h, w), -1, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    ce.ce_bare_run(ce.CE_KERNEL_ESCAPE, ce.ce_escape_params(w, h, x0, y0, dx, dy, max_iter), [], out)
    ref = O.escape(w, h, x0, y0, dx, dy, max_iter)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref)


@pytest.mark.parametrize("w,h", [(1, 1), (1, 700), (15, 3), (16, 4), (17, 5), (131, 96), (513, 33), (1025, 301),
                                 (4100, 67)])
def test_every_pixel_once_however_the_blocks_are_dealt(w, h):
    """The direct sweep (GPU alone; also with one workgroup and with more than
    it has blocks), tiles dealt by tickets and in packages, and the plain
    launch write every pixel of a ragged grid."""
    x0, y0, dx, dy = (float(np.float32(v)) for v in (-2.0, -1.5, 3.0 / w, 3.0 / h))
    prm = ce.ce_escape_params(w, h, x0, y0, dx, dy, 300)
    ref = O.escape(w, h, x0, y0, dx, dy, 300)
    out = torch.full((h, w), -1, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    ce.ce_bare_run(ce.CE_KERNEL_ESCAPE, prm, [], out)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref)
    with ce.Engine() as eng:
        eng.use(ce.CE_DEV_GPU, 0, 0)
        for workgroups in (0, 1, 7, 5000):
            for sched in (dict(kind=ce.CE_SCHED_STATIC), dict(kind=ce.CE_SCHED_DYNAMIC, package_granules=7),
                          dict(kind=ce.CE_SCHED_HGUIDED, power=[1], k=2, min_granules=[1])):
                out.fill_(-1)
                torch.cuda.synchronize()
                eng.gpu_workgroups(workgroups)
                eng.work_items([w, h])
                eng.scheduler(**sched)
                eng.program_kernel(ce.CE_KERNEL_ESCAPE, prm)
                eng.program_out(0, dev=out, nbytes=w * h * 4)
                eng.run()
                assert np.array_equal(out.cpu().numpy().view(np.uint32), ref), (workgroups, sched)


@pytest.mark.parametrize("workgroups,max_iter", [(3, 256), (64, 600), (64, 5000), (200, 2000), (0, 300)])
@pytest.mark.parametrize("host", [False, True])
def test_deep_caps_in_packages(host, workgroups, max_iter):
    """Waves that take the blocks of their workgroup's tiles on their own, over
    many packages, with and without the host; repeated runs of one engine."""
    w, h = 700, 501
    x0, y0, dx, dy = (float(np.float32(v)) for v in (-2.0, -1.5, 3.0 / w, 3.0 / h))
    prm = ce.ce_escape_params(w, h, x0, y0, dx, dy, max_iter)
    ref = O.escape(w, h, x0, y0, dx, dy, max_iter)
    out = torch.empty((h, w), dtype=torch.int32, device="cuda:0")
    with ce.Engine() as eng:
        eng.use(ce.CE_DEV_GPU | (ce.CE_DEV_HOST if host else 0), 0, 4 if host else 0)
        eng.gpu_workgroups(workgroups)
        eng.work_items([w, h])
        power = [4096, 64] if host else [1]
        for sched in (dict(kind=ce.CE_SCHED_HGUIDED, k=2, power=power, min_granules=[1] * len(power)),
                      dict(kind=ce.CE_SCHED_DYNAMIC, package_granules=5),
                      dict(kind=ce.CE_SCHED_DYNAMIC, package_granules=64)):
            eng.scheduler(**sched)
            eng.program_kernel(ce.CE_KERNEL_ESCAPE, prm)
            eng.program_out(0, dev=out, nbytes=w * h * 4)
            for run in range(3):
                out.fill_(-1)
                torch.cuda.synchronize()
                eng.run()
                assert np.array_equal(out.cpu().numpy().view(np.uint32), ref), (sched, run)


@pytest.mark.parametrize("w", [1, 15, 17, 31, 33, 63, 65, 511, 513, 1500])
@pytest.mark.parametrize("rows", [1, 2, 3, 5])
def test_packages_of_few_rows(rows, w):
    """Packages of one and two rows are cut into blocks of their own shape: the
    image in packages of so many rows, and as one package of so few, with a cap
    where waves take blocks on their own and one where they do not."""
    with ce.Engine() as eng:
        for h, cap in ((rows, 100), (301, 100), (301, 5000)):
            prm = ce.ce_escape_params(w, h, -2.0, -1.5, float(np.float32(3.0 / w)), float(np.float32(3.0 / h)), cap)
            out = torch.full((h, w), -1, dtype=torch.int32, device="cuda:0")
            eng.use(ce.CE_DEV_GPU, 0, 0)
            eng.gpu_workgroups(50 if cap == 5000 else 0)
            eng.work_items([w, h])
            eng.program_kernel(ce.CE_KERNEL_ESCAPE, prm)
            eng.program_out(0, dev=out, nbytes=out.numel() * 4)
            ref = O.escape(w, h, -2.0, -1.5, prm.dx, prm.dy, cap)
            for sched in (dict(kind=ce.CE_SCHED_DYNAMIC, package_granules=rows), dict(kind=ce.CE_SCHED_STATIC)):
                out.fill_(-1)
                torch.cuda.synchronize()
                eng.scheduler(**sched)
                eng.run()
                assert np.array_equal(out.cpu().numpy().view(np.uint32), ref), (h, cap, sched)
            out.fill_(-1)
            torch.cuda.synchronize()
            ce.ce_bare_run(ce.CE_KERNEL_ESCAPE, prm, [], out)
            assert np.array_equal(out.cpu().numpy().view(np.uint32), ref), (h, cap)


@pytest.mark.parametrize("cap", [64, 300, 600])
@pytest.mark.parametrize("w,h", [(3, 65536), (3, 65537), (515, 40000), (700, 300)])
def test_many_tiles_and_many_bands(w, h, cap):
    """Around 65,536 tiles, and in 31, 32 and 64 bands, where tiles go from the
    round-robin to tickets, with caps on either side of the one from which waves
    take blocks on their own."""
    prm = ce.ce_escape_params(w, h, -2.0, -1.5, float(np.float32(3.0 / w)), float(np.float32(3.0 / h)), cap)
    ref = O.escape(w, h, -2.0, -1.5, prm.dx, prm.dy, cap)
    out = torch.empty((h, w), dtype=torch.int32, device="cuda:0")
    with ce.Engine() as eng:
        eng.use(ce.CE_DEV_GPU, 0, 0)
        eng.work_items([w, h])
        eng.program_kernel(ce.CE_KERNEL_ESCAPE, prm)
        eng.program_out(0, dev=out, nbytes=out.numel() * 4)
        for sched in (dict(kind=ce.CE_SCHED_HGUIDED, k=2, power=[1]), dict(kind=ce.CE_SCHED_DYNAMIC, n_packages=50),
                      dict(kind=ce.CE_SCHED_STATIC, n_packages=31), dict(kind=ce.CE_SCHED_STATIC, n_packages=32),
                      dict(kind=ce.CE_SCHED_STATIC, n_packages=64)):
            eng.scheduler(**sched)
            for _ in range(2):
                out.fill_(-1)
                torch.cuda.synchronize()
                eng.run()
                assert np.array_equal(out.cpu().numpy().view(np.uint32), ref), sched


@pytest.mark.parametrize("w,h", [(512, 4095), (512, 4096), (515, 2049), (1920, 1080)])
def test_grid_of_packages_around_two_rounds(w, h):
    """In packages, escape-time takes whole rounds of tiles below two rounds of
    resident workgroups (eight per compute unit) and all of them from there on."""
    prm = ce.ce_escape_params(w, h, -2.0, -1.5, float(np.float32(3.0 / w)), float(np.float32(3.0 / h)), 300)
    ref = O.escape(w, h, -2.0, -1.5, prm.dx, prm.dy, 300)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    resident, tiles = 8 * cus, h * -(-w // 512)
    out = torch.empty((h, w), dtype=torch.int32, device="cuda:0")
    with ce.Engine() as eng:
        for devs in (ce.CE_DEV_GPU, ce.CE_DEV_GPU | ce.CE_DEV_HOST):
            eng.use(devs, 0, 0 if devs == ce.CE_DEV_GPU else 4)
            eng.work_items([w, h])
            eng.program_kernel(ce.CE_KERNEL_ESCAPE, prm)
            eng.program_out(0, dev=out, nbytes=out.numel() * 4)
            for sched in (dict(kind=ce.CE_SCHED_HGUIDED, k=2, power=[9, 1][:1 if devs == ce.CE_DEV_GPU else 2]),
                          dict(kind=ce.CE_SCHED_DYNAMIC, package_granules=16)):
                eng.scheduler(**sched)
                out.fill_(-1)
                torch.cuda.synchronize()
                eng.run()
                assert np.array_equal(out.cpu().numpy().view(np.uint32), ref), sched
                g = eng.stats().gpu_workgroups
                if tiles >= 2 * resident:
                    assert g == resident, (g, tiles)
                else:
                    assert -(-tiles // g) * -(-g // cus) == -(-tiles // cus), (g, tiles)
