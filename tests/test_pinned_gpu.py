"""Host-resident runs over pinned host buffers (section 7.3 counts the
transfers in T): the GPU streams a pinned input over PCIe and writes its
rows of a pinned output in place, while the host workers use the same
buffers; every output bit-exact against the oracle, for every scheduler and
device set, including payloads whose inputs are copied to HBM first
(n-body re-reads its positions) and the full 8192 x 8192 blur."""
import numpy as np
import pytest

import paper_1805_02755_amd as ce
from paper_1805_02755_amd import synth
from oracle import oracle as O

from gpu_util import BOTH, check_trace, diff_report, escape_params, run_payload

pytestmark = pytest.mark.gpu

DEVS = {"gpu": ce.CE_DEV_GPU, "both": BOTH}
SCHEDS = ["static", "static_rev", "dynamic", "hguided"]


@pytest.fixture(scope="module")
def eng():
    e = ce.Engine()
    yield e
    e.close()


@pytest.mark.parametrize("devs", list(DEVS))
@pytest.mark.parametrize("sched", SCHEDS)
def test_escape_pinned(eng, devs, sched):
    p = synth.escape_region(1000, 300, -2.0, 0.6, -1.2, 1.2, 256)
    ref = O.escape(p.w, p.h, *[float(v) for v in p.as_f32()], p.max_iter)
    out, st, tr = run_payload(eng, ce.CE_KERNEL_ESCAPE, escape_params(p), [p.w, p.h], None, [], (p.h, p.w),
                              np.uint32, DEVS[devs], sched, mode="pinned")
    assert np.array_equal(out, ref), diff_report(out, ref, tr)
    check_trace(tr, p.h, st.n_devices)


@pytest.mark.parametrize("devs", list(DEVS))
@pytest.mark.parametrize("sched", SCHEDS)
@pytest.mark.parametrize("w,h", [(1001, 37), (4096, 300), (3, 2000)])
def test_blur_pinned(eng, devs, sched, w, h):
    img = synth.blur_image(w, h, seed=w * 3 + h)
    wt = ce.ce_gauss5_weights(1.0)
    ref = O.blur5(img, O.gauss5_weights(1.0))
    out, st, tr = run_payload(eng, ce.CE_KERNEL_BLUR5, ce.ce_blur5_params(w, h), [w, h], None, [img, wt], (h, w),
                              np.float32, DEVS[devs], sched, mode="pinned")
    assert np.array_equal(out.view(np.uint32), ref.view(np.uint32)), diff_report(out, ref, tr)
    check_trace(tr, h, st.n_devices)


@pytest.mark.parametrize("devs", list(DEVS))
def test_nbody_pinned(eng, devs):
    n = 5000
    pos = synth.nbody_bodies(n, seed=17)
    ref = O.nbody_acc(pos, 1e-6, True)
    for sched in ("dynamic", "hguided"):
        out, st, tr = run_payload(eng, ce.CE_KERNEL_NBODY_ACC, ce.ce_nbody_params(n, 1e-6, 1), [n], [256], [pos],
                                  (n, 4), np.float32, DEVS[devs], sched, mode="pinned")
        assert np.array_equal(out.view(np.uint32), ref.view(np.uint32)), sched


def test_blur_full_size_pinned(eng):
    w = h = 8192
    img = synth.blur_image(w, h)
    wt = ce.ce_gauss5_weights(1.0)
    ref = O.blur5(img, O.gauss5_weights(1.0))
    out, st, tr = run_payload(eng, ce.CE_KERNEL_BLUR5, ce.ce_blur5_params(w, h), [w, h], None, [img, wt], (h, w),
                              np.float32, BOTH, "hguided", mode="pinned")
    assert np.array_equal(out.view(np.uint32), ref.view(np.uint32)), diff_report(out, ref, tr)
    check_trace(tr, h, 2)


@pytest.mark.parametrize("w,h", [(1, 300), (31, 300), (32, 301), (40, 33), (63, 200), (64, 200), (65, 3), (513, 130)])
def test_block_and_tile_shapes_pinned(eng, w, h):
    """Widths around the wave's row of pixels that host memory takes, and blur
    tiles of every height that images of few tiles take."""
    p = synth.escape_region(w, h, -2.0, 0.6, -1.2, 1.2, 3000)
    ref = O.escape(p.w, p.h, *[float(v) for v in p.as_f32()], p.max_iter)
    img = synth.blur_image(w, h, seed=w + h)
    wt = ce.ce_gauss5_weights(1.0)
    blurred = O.blur5(img, O.gauss5_weights(1.0))
    for devs, sched in ((ce.CE_DEV_GPU, "static"), (ce.CE_DEV_GPU, "dynamic"), (BOTH, "hguided")):
        out, st, tr = run_payload(eng, ce.CE_KERNEL_ESCAPE, escape_params(p), [w, h], None, [], (h, w), np.uint32,
                                  devs, sched, mode="pinned")
        assert np.array_equal(out, ref), (sched, diff_report(out, ref, tr))
        out, st, tr = run_payload(eng, ce.CE_KERNEL_BLUR5, ce.ce_blur5_params(w, h), [w, h], None, [img, wt], (h, w),
                                  np.float32, devs, sched, mode="pinned")
        assert np.array_equal(out.view(np.uint32), blurred.view(np.uint32)), (sched, diff_report(out, blurred, tr))


@pytest.mark.parametrize("cap", [1024, 1025])
def test_escape_block_shapes_by_cap_pinned(eng, cap):
    w, h = 515, 130
    p = synth.escape_region(w, h, -2.0, 0.6, -1.2, 1.2, cap)
    ref = O.escape(p.w, p.h, *[float(v) for v in p.as_f32()], p.max_iter)
    for devs, sched in ((ce.CE_DEV_GPU, "static"), (ce.CE_DEV_GPU, "dynamic"), (BOTH, "hguided")):
        out, st, tr = run_payload(eng, ce.CE_KERNEL_ESCAPE, escape_params(p), [w, h], None, [], (h, w), np.uint32,
                                  devs, sched, mode="pinned")
        assert np.array_equal(out, ref), (sched, diff_report(out, ref, tr))
