"""Batches whose packages are dealt in levels: every pixel is written, once per
run, for numbers of packages around the launch's workgroups and the levels'
sizes, one wide job, many tiny ones, and package sizes that do not divide the
tiles; the counter is left as the next run of the same graph needs it."""
import numpy as np
import pytest
import torch

import paper_1805_02755_amd as ce
from oracle import oracle as O

from gpu_util import DEV

pytestmark = pytest.mark.gpu

# (w, h) of the jobs
BATCHES = {
    "one_pixel": [(1, 1)],
    "one_row": [(5000, 1)],
    "one_column": [(1, 5000)],
    "tiny": [(3 + k % 11, 2 + k % 7) for k in range(700)],
    "uneven": [(16, 16), (1501, 1203), (17, 900), (33, 31), (640, 480), (1, 1)],
    "wide": [(2048, 2048)],
}


@pytest.mark.parametrize("rows,package", [(16, 1), (16, 2), (16, 3), (8, 7), (4, 32), (1, 1), (2, 100000)])
@pytest.mark.parametrize("name", sorted(BATCHES))
def test_every_pixel_in_every_run(name, rows, package):
    jobs = BATCHES[name]
    prm = [ce.ce_escape_params(w, h, -2.0, -1.5, np.float32(3.0 / w), np.float32(3.0 / h), 50 + k % 13)
           for k, (w, h) in enumerate(jobs)]
    sizes = [w * h for w, h in jobs]
    buf = torch.empty(sum(sizes), dtype=torch.int32, device=DEV)
    ref = np.concatenate([O.escape(p.w, p.h, p.x0, p.y0, p.dx, p.dy, p.max_iter).reshape(-1) for p in prm])
    b = ce.Batch()
    b.set_config(rows, package)
    for p, at, n in zip(prm, np.cumsum([0] + sizes), sizes):
        b.add_escape(p, buf[int(at):int(at) + n])
    for run in range(3):
        buf.fill_(-1)
        torch.cuda.synchronize()
        b.run()
        assert np.array_equal(buf.cpu().numpy().view(np.uint32), ref), run
    b.close()


@pytest.mark.parametrize("name,package", [("one_pixel", 1 << 20), ("uneven", 1 << 20), ("wide", 16383), ("wide", 16385)])
def test_a_package_longer_than_its_tiles_ends_with_them(name, package):
    """The parts of a package past the batch's last tile are not walked one by one
    (of 2^20 tiles, 4 million: 380 ms; a batch of these sizes takes 55 ms in one
    workgroup)."""
    jobs = BATCHES[name]
    outs = [torch.full((h, w), -1, dtype=torch.int32, device=DEV) for w, h in jobs]
    b = ce.Batch()
    b.set_config(16, package)
    prm = [ce.ce_escape_params(w, h, -2.0, -1.5, np.float32(3.0 / w), np.float32(3.0 / h), 64) for w, h in jobs]
    for p, o in zip(prm, outs):
        b.add_escape(p, o)
    torch.cuda.synchronize()
    for _ in range(3):
        b.run()
    assert b.stats().t_gpu_ms < 150.0
    for p, o in zip(prm, outs):
        assert np.array_equal(o.cpu().numpy().view(np.uint32), O.escape(p.w, p.h, p.x0, p.y0, p.dx, p.dy, p.max_iter))
    b.close()
