"""N-body sizes where the order of the sums could go wrong: around a chunk (8,
24, 48 bodies) and a round of chunks over a workgroup's waves, a phase of the
terms fed to an adding wave (48, 56), a group of 16 or 64 bodies, a granule, and
the borders between the forms (fed groups, wide groups, groups, whole granules);
in the direct, persistent, plain and serving kernels. The
strict form equals the oracle bit for bit; the hardware 1/sqrt lies within
1e-5 of the sum of the terms' lengths."""
import numpy as np
import pytest
import torch

import paper_1805_02755_amd as ce
from paper_1805_02755_amd import synth
from oracle import oracle as O

from gpu_util import DEV

pytestmark = pytest.mark.gpu
EPS2 = 1e-6
SIZES = [1, 2, 7, 8, 9, 23, 24, 25, 47, 48, 49, 55, 56, 57, 63, 64, 65, 95, 96, 97, 111, 112, 113,
         167, 168, 169, 191, 192, 193, 255, 256, 257, 383, 384, 385, 767, 768, 769, 1000]
BORDERS = [8192, 8193, 8207, 8208, 8209, 16384, 16385, 32767, 32768, 98304, 98305, 114688, 114689, 131072, 131073]


@pytest.fixture(scope="module")
def eng():
    e = ce.Engine()
    yield e
    e.close()


def forms(eng, pos, strict, which):
    """(name, output) of the acceleration in each form of the kernel."""
    n = pos.shape[0]
    p_d = torch.from_numpy(pos).to(DEV)
    prm = ce.ce_nbody_params(n, EPS2, strict)
    out = torch.full((n, 4), float("nan"), device=DEV)
    torch.cuda.synchronize()
    if "plain" in which:
        ce.ce_bare_run(ce.CE_KERNEL_NBODY_ACC, prm, [p_d], out)
        yield "plain", out.cpu().numpy()
    for name, sched in (("direct", dict(kind=ce.CE_SCHED_STATIC)),
                        ("persistent", dict(kind=ce.CE_SCHED_DYNAMIC, package_granules=1))):
        if name not in which:
            continue
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        eng.use(ce.CE_DEV_GPU, 0, 0)
        eng.work_items([n], [256])
        eng.scheduler(**sched)
        eng.program_kernel(ce.CE_KERNEL_NBODY_ACC, prm)
        eng.program_in(0, dev=p_d, nbytes=n * 16)
        eng.program_out(0, dev=out, nbytes=n * 16)
        eng.run()
        yield name, out.cpu().numpy()
    if "serve" in which:
        with ce.Server(64 << 20, keep_outputs=True, session_timeout_s=30.0) as srv:
            t = srv.submit(ce.CE_KERNEL_NBODY_ACC, prm, p_d)
            srv.wait(t, 60.0)
            res = np.empty((n, 4), np.float32)
            srv.copy_output(t, res)
            srv.drain(60.0)
        yield "serve", res


def same(a, b):
    return np.array_equal(np.ascontiguousarray(a).view(np.uint32), np.ascontiguousarray(b).view(np.uint32))


@pytest.mark.parametrize("n", SIZES)
def test_small_sizes_every_body(eng, n):
    pos = synth.nbody_bodies(n, seed=1000 + n)
    ref = O.nbody_acc(pos, EPS2, True)
    for name, out in forms(eng, pos, 1, ("plain", "direct", "persistent")):
        assert same(out, ref), (name, n)
    if n > 1:
        ref64 = O.nbody_acc_f64(pos, EPS2)
        for name, out in forms(eng, pos, 0, ("plain", "direct", "persistent")):
            d = pos[None, :, :3].astype(np.float64) - pos[:, None, :3]
            r2 = (d * d).sum(-1) + np.float64(np.float32(EPS2))
            bound = 1e-5 * (pos[None, :, 3] * np.sqrt((d * d).sum(-1)) * r2 ** -1.5).sum(1)
            assert np.all(np.linalg.norm(out[:, :3] - ref64[:, :3], axis=1) <= bound), (name, n)


def test_serving_sizes(eng):
    for n in (1, 9, 65, 385, 1000):
        pos = synth.nbody_bodies(n, seed=2000 + n)
        ref = O.nbody_acc(pos, EPS2, True)
        for name, out in forms(eng, pos, 1, ("serve",)):
            assert same(out, ref), (name, n)


@pytest.mark.parametrize("n", BORDERS)
def test_borders_between_forms_sampled(eng, n):
    pos = synth.nbody_bodies(n, seed=n)
    which = ("plain", "direct", "persistent") + (("serve",) if n in (32767, 32768) else ())
    at = sorted({0, 63, 64, n // 2, n - 65, n - 2, n - 1})
    ref = {i: O.nbody_acc_body(pos, EPS2, i, True) for i in at}
    for name, out in forms(eng, pos, 1, which):
        assert not np.isnan(out).any(), (name, n)
        for i in at:
            assert same(out[i], ref[i]), (name, n, i)


SHARES = [dict(props=[0.125]), dict(props=[0.5]), dict(props=[0.6]), dict(props=[0.75]),
          dict(props=[0.125], n_packages=8)]


def bound_f64(pos, i):
    """64-bit acceleration of body i and 1e-5 of the sum of its terms' lengths."""
    d = pos[:, :3].astype(np.float64) - pos[i, :3]
    r2 = (d * d).sum(-1) + np.float64(np.float32(EPS2))
    return O.nbody_acc_f64(pos, EPS2, i, i + 1)[0, :3], 1e-5 * (pos[:, 3] * np.sqrt((d * d).sum(-1)) * r2 ** -1.5).sum()


@pytest.mark.parametrize("kind", ["acc", "step"])
@pytest.mark.parametrize("strict", [1, 0])
@pytest.mark.parametrize("n", [98304, 98305, 114688, 114689, 120000, 131072, 131073])
def test_static_share_of_the_gpu_around_whole_granules(eng, n, strict, kind):
    """The GPU's share in one package of a space beside the host: the form of the
    tiles follows from the bodies, the kernel from the share's tiles too. Every
    body is written, sampled ones over the share are right."""
    pos, vel = synth.nbody_bodies(n, seed=n), synth.nbody_velocities(n, seed=n)
    p_d, v_d = torch.from_numpy(pos).to(DEV), torch.from_numpy(vel).to(DEV)
    dt = 0.002
    outs = [torch.empty((n, 4), device=DEV) for _ in range(1 if kind == "acc" else 2)]
    eng.use(ce.CE_DEV_GPU | ce.CE_DEV_HOST, 0, 0)
    eng.work_items([n], [256])
    if kind == "acc":
        eng.program_kernel(ce.CE_KERNEL_NBODY_ACC, ce.ce_nbody_params(n, EPS2, strict))
    else:
        eng.program_kernel(ce.CE_KERNEL_NBODY_STEP, ce.ce_nbody_step_params(n, EPS2, dt, strict))
        eng.program_in(1, host=vel, dev=v_d, nbytes=n * 16)
    eng.program_in(0, host=pos, dev=p_d, nbytes=n * 16)
    for s, o in enumerate(outs):
        eng.program_out(s, dev=o, nbytes=n * 16)
    at = sorted(set(range(0, n, n // 24)) | {n - 1})
    if strict:
        ref = {i: ([O.nbody_acc_body(pos, EPS2, i, True)] if kind == "acc" else
                   O.nbody_step_body(pos, vel, EPS2, dt, i, True)) for i in at}
    else:
        ref = {i: bound_f64(pos, i) for i in at}
    for share in SHARES:
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        eng.scheduler(kind=ce.CE_SCHED_STATIC, order=ce.CE_ORDER_GPU_FIRST, **share)
        eng.run()
        got = [o.cpu().numpy() for o in outs]
        for g in got:
            assert not np.isnan(g).any(), (share, int(np.isnan(g).any(1).sum()))
        for i in at:
            if strict:
                assert all(same(g[i], r) for g, r in zip(got, ref[i])), (share, i)
                continue
            a, bound = ref[i]
            if kind == "acc":
                assert np.linalg.norm(got[0][i, :3] - a) <= bound, (share, i)
                continue
            x, v = pos[i, :3].astype(np.float64), vel[i, :3].astype(np.float64)
            h = dt * dt / 2
            # four roundings at most of sums and products no larger than these
            slack = 2.0 ** -22 * (np.abs(x) + np.abs(v * dt) + np.abs(a * h) + bound * h)
            assert np.all(np.abs(got[0][i, :3] - (x + v * dt + a * h)) <= bound * h + slack), (share, i)
            slack = 2.0 ** -22 * (np.abs(v) + np.abs(a * dt) + bound * dt)
            assert np.all(np.abs(got[1][i, :3] - (v + a * dt)) <= bound * dt + slack), (share, i)


def gpu_runs(eng, kid, prm, ins, n, n_out):
    """The payload's outputs in the plain launch, on the GPU alone and in packages."""
    outs = [torch.empty((n, 4), device=DEV) for _ in range(n_out)]
    for name, sched in (("plain", None), ("direct", dict(kind=ce.CE_SCHED_STATIC)),
                        ("persistent", dict(kind=ce.CE_SCHED_DYNAMIC, package_granules=1))):
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        if sched is None:
            ce.ce_bare_run_outs(kid, prm, ins, outs)
        else:
            eng.use(ce.CE_DEV_GPU, 0, 0)
            eng.work_items([n], [256])
            eng.scheduler(**sched)
            eng.program_kernel(kid, prm)
            for s, t in enumerate(ins):
                eng.program_in(s, dev=t, nbytes=n * 16)
            for s, o in enumerate(outs):
                eng.program_out(s, dev=o, nbytes=n * 16)
            eng.run()
        yield name, [o.cpu().numpy() for o in outs]


@pytest.mark.parametrize("n", BORDERS)
def test_borders_of_the_hardware_rsqrt_and_the_step(eng, n):
    """What the borders above leave out: the hardware 1/sqrt, whose whole granules
    begin elsewhere, and the step's own stores in either."""
    pos, vel = synth.nbody_bodies(n, seed=n + 1), synth.nbody_velocities(n, seed=n + 1)
    p_d, v_d = torch.from_numpy(pos).to(DEV), torch.from_numpy(vel).to(DEV)
    dt = 0.002
    at = sorted({0, 63, 64, n // 2, n - 65, n - 2, n - 1})
    bounds = {i: bound_f64(pos, i) for i in at}
    for name, (a,) in gpu_runs(eng, ce.CE_KERNEL_NBODY_ACC, ce.ce_nbody_params(n, EPS2, 0), [p_d], n, 1):
        assert not np.isnan(a).any(), name
        assert all(np.linalg.norm(a[i, :3] - bounds[i][0]) <= bounds[i][1] for i in at), name
    steps = {i: O.nbody_step_body(pos, vel, EPS2, dt, i, True) for i in at}
    for name, (x, v) in gpu_runs(eng, ce.CE_KERNEL_NBODY_STEP, ce.ce_nbody_step_params(n, EPS2, dt, 1), [p_d, v_d], n, 2):
        assert not np.isnan(x).any() and not np.isnan(v).any(), name
        assert all(same(x[i], steps[i][0]) and same(v[i], steps[i][1]) for i in at), name
    for name, (x, v) in gpu_runs(eng, ce.CE_KERNEL_NBODY_STEP, ce.ce_nbody_step_params(n, EPS2, dt, 0), [p_d, v_d], n, 2):
        assert not np.isnan(x).any() and not np.isnan(v).any(), name
        for i in at:
            a, bound = bounds[i]
            v64 = vel[i, :3].astype(np.float64)
            slack = 2.0 ** -22 * (np.abs(v64) + np.abs(a * dt) + bound * dt)
            assert np.all(np.abs(v[i, :3] - (v64 + a * dt)) <= bound * dt + slack), (name, i)
