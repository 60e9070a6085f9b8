"""Blur widths around a wave's 256 columns and a tile's 1024 at every alignment
of the rows, heights around the tile's rows, and image sizes on both sides of
the rule that picks them (192 and 512 tiles): the plain, direct and persistent
kernels and the serving kernel write every pixel, equal to the oracle's bit
for bit."""
import numpy as np
import pytest
import torch

import paper_1805_02755_amd as ce
from paper_1805_02755_amd import synth
from oracle import oracle as O

from gpu_util import DEV

pytestmark = pytest.mark.gpu
SIZES = [(1, 1), (3, 2), (5, 9), (255, 7), (256, 3), (257, 5), (258, 33), (259, 4), (260, 31), (511, 32), (512, 1),
         (513, 64), (769, 65), (1023, 18), (1024, 767), (1024, 769), (1025, 770), (1281, 131), (2049, 513), (4099, 409),
         (4096, 4095), (4097, 4100)]


@pytest.mark.parametrize("w,h", SIZES)
def test_every_kernel_every_pixel(w, h):
    img = synth.blur_image(w, h, seed=w * 7 + h) - np.float32(0.25)
    wt = ce.ce_gauss5_weights(1.0)
    ref = O.blur5(img, O.gauss5_weights(1.0)).view(np.uint32)
    prm = ce.ce_blur5_params(w, h)
    i_d, w_d = torch.from_numpy(img).to(DEV), torch.from_numpy(wt).to(DEV)
    guard = 64  # floats before and after the image that no kernel may touch
    buf = torch.full((w * h + 2 * guard,), float("nan"), device=DEV)
    out = buf[guard:guard + w * h]

    def check(name):
        got = buf.cpu().numpy()
        assert np.isnan(got[:guard]).all() and np.isnan(got[-guard:]).all(), name
        assert np.array_equal(got[guard:-guard].view(np.uint32).reshape(h, w), ref), name
        buf.fill_(float("nan"))
        torch.cuda.synchronize()

    torch.cuda.synchronize()
    ce.ce_bare_run(ce.CE_KERNEL_BLUR5, prm, [i_d, w_d], out)
    check("plain")
    with ce.Engine() as eng:
        eng.use(ce.CE_DEV_GPU, 0, 0)
        for name, sched in (("direct", dict(kind=ce.CE_SCHED_STATIC)),
                            ("persistent", dict(kind=ce.CE_SCHED_HGUIDED, power=[1], k=2, min_granules=[3])),
                            ("dynamic", dict(kind=ce.CE_SCHED_DYNAMIC, package_granules=max(1, h // 40)))):
            eng.work_items([w, h])
            eng.scheduler(**sched)
            eng.program_kernel(ce.CE_KERNEL_BLUR5, prm)
            eng.program_in(0, dev=i_d, nbytes=img.nbytes)
            eng.program_in(1, dev=w_d, nbytes=wt.nbytes)
            eng.program_out(0, dev=out, nbytes=img.nbytes)
            eng.run()
            check(name)
    if w * h < 100000:
        with ce.Server(4 << 20, keep_outputs=True, session_timeout_s=30.0) as srv:
            t = srv.submit(ce.CE_KERNEL_BLUR5, prm, i_d, w_d)
            srv.wait(t, 60.0)
            res = np.empty((h, w), np.float32)
            srv.copy_output(t, res)
            srv.drain(60.0)
        assert np.array_equal(res.view(np.uint32), ref), "serve"
