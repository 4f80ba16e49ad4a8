"""Captured calls follow the metric terms on the device.

A graph of an RK step, a residual or a reverse step is captured on an affine
mesh.  Replays after the metric terms were replaced (by a curved mesh's, and
with the per-element copies switched off) give what an eager call gives on
them: the same kernels on the same values in FP64, 1e-12 of the largest entry,
the bound between the kernel variants.  Eager work and synchronisations stand
between the replays.
"""
import sys

import numpy as np
import pytest

from paper_2605_28627_amd import inputs as I

pytestmark = pytest.mark.gpu
PI = np.pi


def _say(*a):
    print("[gpu-capture]", *a, flush=True)
    sys.stdout.flush()


CASES = [(7, 1, 1, 1), (5, 1, 1, 0), (4, 0, 1, 1), (3, 0, 1, 0), (3, 1, 0, 1)]   # N, nodes, form, physics


@pytest.mark.parametrize("case", CASES, ids=str)
def test_replay_after_the_metrics_changed(case):
    import torch
    from paper_2605_28627_amd.solver import DGSolver
    _say(case)
    N, nodes, form, physics = case
    cfg = dict(N=N, nodes=nodes, form=form, physics=physics, mu=0.02 if physics else 0.0)
    meshes = [I.box_mesh((3, 2, 2), (-PI,) * 3, (PI,) * 3, Ngeo=N, curved_amp=a, rotate_seed=6) for a in (0.0, 0.1)]
    s, curved = DGSolver(cfg, meshes[0], adjoint=True), DGSolver(cfg, meshes[1], adjoint=True)
    try:
        assert s.element_metric_count() == s.nElems and curved.element_metric_count() < s.nElems
        U0 = s.init_state(I.smooth_random_state(s.coords(), 81, amp=0.1))
        lam0 = s.to_device(np.random.default_rng(82).normal(size=s.state_shape))
        dt = 0.2 * s.timestep(U0, 0.9)
        U, dU, Ut, lam, lamd = (s.empty_state() for _ in range(5))

        def calls(x, U, dU, Ut, lam, lamd):
            x.rhs(U, Ut)
            x.adjoint_rk_step(U, lam, lamd, dt)
            x.rk_step(U, dU, dt, 1)

        def eager(x):
            a = [U0.clone(), torch.empty_like(U0), torch.empty_like(U0), lam0.clone(), torch.empty_like(U0)]
            calls(x, *a)
            return [v.cpu().numpy() for v in a[:4]]

        affine = eager(s)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            calls(s, U, dU, Ut, lam, lamd)

        def replay():
            U.copy_(U0)
            lam.copy_(lam0)
            for v in (dU, Ut, lamd):
                v.fill_(7.0)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            return [v.cpu().numpy() for v in (U, dU, Ut, lam)]

        def same(a, b):
            return max(np.abs(x - y).max() / np.abs(y).max() for x, y in zip(a, b))

        plane = s.metrics()[1:]
        err = [same(replay(), affine)]
        s.upload_metrics(*curved.metrics()[1:])
        err.append(same(replay(), eager(curved)))
        s.upload_metrics(*plane)
        err.append(same(replay(), affine))
        s.set_element_metrics(False)
        err.append(same(replay(), eager(s)))
    finally:
        s.close()
        curved.close()
    _say(case, err)
    assert max(err) < 1e-12
