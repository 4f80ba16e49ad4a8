"""Kernel variants that a rule on the mesh or the degree selects.

* Affine meshes: the split form's residual and the lifting run variants with
  uniform metric terms where every element is affine.  Against the general
  kernels (the same mesh with per-element metric terms switched off): the same
  operations, and for the lifting the factored gradient, so FP64 results agree
  to 1e-12 of each output's largest entry (the bound of the per-element metric
  terms).  With float fluxes a last-bit difference of an FP64 intermediate may
  move a float rounding (6e-8 of a flux; the residual is a difference of fluxes
  some 50 times its size): 5e-6.
* Sides with one normal: curved meshes with one plane layer of elements mix
  both kinds in one launch; the residual matches the oracle.
* N = 1 packs four elements into a wavefront: element counts that leave a
  wavefront partly empty, for every kernel, against the oracle (1e-12, as all
  residuals and transposed residuals).
"""
import sys

import numpy as np
import pytest

from paper_2605_28627_amd import inputs as I
from tests.helpers import rel_err_per_var

pytestmark = pytest.mark.gpu
PI = np.pi


def _say(*a):
    print("[gpu-variants]", *a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available()
    from paper_2605_28627_amd.solver import DGSolver
    return DGSolver


def _off(a, ref):
    """Largest relative error over the variables; one whose reference vanishes
    (a single periodic element: below 1e-12, rounding) counts absolutely."""
    scale = np.abs(ref).max(axis=tuple(range(1, ref.ndim)))
    err = np.abs(a - ref).max(axis=tuple(range(1, ref.ndim)))
    return (err / np.where(scale < 1e-12, 1.0, scale)).max()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("physics", [0, 1])
@pytest.mark.parametrize("nodes", [0, 1])
@pytest.mark.parametrize("N", range(1, 8))
def test_affine_variant_matches_general_kernels(S, N, nodes, physics, precision):
    _say("affine", N, nodes, physics, precision)
    mesh = I.box_mesh((3, 2, 3), (-PI,) * 3, (PI,) * 3, rotate_seed=5)
    s = S(dict(N=N, nodes=nodes, form=1, physics=physics, mu=1e-2 if physics else 0.0, precision=precision), mesh)
    try:
        assert s.element_metric_count() == mesh.nElems
        # (variations on both sides of the log means' series threshold)
        U0 = I.smooth_random_state(s.coords(), 71, amp=0.1)
        U0[:, : mesh.nElems // 2] = I.smooth_random_state(s.coords(), 71, amp=0.002)[:, : mesh.nElems // 2]
        dt = 0.2 * s.timestep(s.init_state(U0), 0.9)

        def run():
            U = s.init_state(U0)
            out = [s.rhs(U).cpu().numpy()]
            if physics:
                out.append(s.lift(U).cpu().numpy())
            dU = s.empty_state()
            s.rk_step(U, dU, dt, 2)
            return out + [dU.cpu().numpy(), U.cpu().numpy()]

        on = run()
        s.set_element_metrics(False)
        off = run()
    finally:
        s.close()
    for a, b in zip(on, off):
        assert np.isfinite(a).all()
        assert np.abs(a - b).max() <= (5e-6 if precision else 1e-12) * np.abs(b).max()


@pytest.mark.parametrize("case", [(7, 1, 1, 1), (4, 1, 0, 1), (3, 0, 0, 0), (5, 1, 1, 0)], ids=str)
def test_plane_and_curved_sides_in_one_launch(S, orc, case):
    """Random side orientations; the top layer of elements stays plane, the others are curved inside."""
    _say("mixed", case)
    N, nodes, form, physics = case
    mesh = I.box_mesh((2, 2, 3), (-PI,) * 3, (PI,) * 3, Ngeo=3, rotate_seed=9)
    low = np.arange(mesh.nElems) < 8
    z = mesh.X[2]
    bump = 0.1 * np.sin(1.5 * (z + PI)) * np.sin(mesh.X[0]) * np.sin(mesh.X[1])
    mesh.X[2][low] += np.where(z < PI / 3, bump, 0.0)[low]
    cfg = dict(N=N, nodes=nodes, form=form, physics=physics, mu=0.02 if physics else 0.0)
    o, s = orc.Oracle(cfg, mesh), S(cfg, mesh)
    try:
        assert 0 < s.element_metric_count() < mesh.nElems
        _, Ja, sJ, nv = s.metrics()
        _, J, Jo = o.geometry()
        n_affine = s.element_metric_count()
        # the oracle's metric terms on curved elements, the library's (same to rounding) on plane ones
        curved = np.array([np.ptp(sJ[e]) > 0 for e in range(mesh.nElems)])
        assert (~curved).sum() == n_affine
        U = I.smooth_random_state(o.coords(), 72, amp=0.2)
        R = s.rhs(s.init_state(U)).cpu().numpy()
    finally:
        s.close()
    ref = o.rhs(U)
    # the two sides' metric terms differ by rounding (bounded here by what they differ by)
    dm = np.abs(Ja - Jo).max() / np.abs(Jo).max()
    err = rel_err_per_var(R, ref)
    _say("mixed", case, err, "metric", dm)
    assert dm < 1e-12 and np.all(err < 1e-12 + 1e3 * dm), (err, dm)


@pytest.mark.parametrize("K", [(1, 1, 1), (2, 1, 1), (3, 1, 1), (3, 3, 1)], ids=str)
@pytest.mark.parametrize("nodes,form", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("physics", [0, 1])
def test_packed_elements(S, orc, K, nodes, form, physics):
    _say("packed", K, nodes, form, physics)
    mesh = I.box_mesh(K, (-PI,) * 3, (PI,) * 3, rotate_seed=4)
    cfg = dict(N=1, nodes=nodes, form=form, physics=physics, mu=0.02 if physics else 0.0)
    o, s = orc.Oracle(cfg, mesh), S(cfg, mesh, adjoint=True)
    f = S(dict(cfg, fv=1), mesh)
    of = orc.Oracle(dict(cfg, fv=1), mesh)
    try:
        _, J, Ja = o.geometry()
        for x in (s, f):
            x.upload_metrics(Ja, 1.0 / J, o.face_normals())
        U = I.smooth_random_state(o.coords(), 73, amp=0.1)
        Ug = s.init_state(U)
        assert _off(s.rhs(Ug).cpu().numpy(), o.rhs(U)) < 1e-12
        rng = np.random.default_rng(74)
        lam, d = rng.normal(size=U.shape), rng.normal(size=U.shape)
        out = s.adjoint_rhs(Ug, s.to_device(lam)).cpu().numpy()
        _, jd = o.rhs_jvp(U, d)
        assert abs((out * d).sum() - (lam * jd).sum()) < 1e-12 * np.abs(lam * jd).sum()
        dt = o.timestep(U, 0.9)
        s.rk_step(Ug, s.empty_state(), dt, 2)
        assert _off(Ug.cpu().numpy() - U, o.lserk(U, 2, dt) - U) < 1e-11
        mask = (np.arange(mesh.nElems) % 3 == 0).astype(np.int32)
        Uf = f.init_state(U)
        f.fv_switch(Uf, mask)
        Uo, _ = of.fv_switch(U, None, mask)
        assert _off(f.rhs(Uf).cpu().numpy(), of.rhs(Uo)) < 1e-12
    finally:
        s.close()
        f.close()


@pytest.mark.parametrize("physics", [0, 1])
@pytest.mark.parametrize("nodes", [0, 1])
@pytest.mark.parametrize("N", range(1, 8))
def test_affine_adjoint(S, orc, N, nodes, physics):
    """The split form's adjoint on an affine mesh, with the library's own
    (exactly constant) metric terms: against the oracle's tangent, whose terms
    differ by their rounding dm (the residual is a sum of n1 pairs per line,
    linear in Ja and 1/J, the viscous part quadratic in Ja: 20 dm covers it),
    and entry by entry against the kernels that read the node arrays."""
    _say("affine adjoint", N, nodes, physics)
    mesh = I.box_mesh((2, 2, 2), (-PI,) * 3, (PI,) * 3, rotate_seed=5)
    cfg = dict(N=N, nodes=nodes, form=1, physics=physics, mu=0.05 if physics else 0.0)
    o, s = orc.Oracle(cfg, mesh), S(cfg, mesh, adjoint=True)
    try:
        assert s.element_metric_count() == mesh.nElems
        _, Ja, sJ, nv = s.metrics()
        _, J, Jo = o.geometry()
        dm = max(np.abs(Ja.reshape(Jo.shape) - Jo).max() / np.abs(Jo).max(),
                 np.abs(sJ.reshape(J.shape) * J - 1.0).max(),
                 np.abs(nv.ravel() - o.face_normals().ravel()).max() / np.abs(nv).max())
        # (both branches of the log means; the Gauss split form's projected
        # traces stay positive at this amplitude)
        U0 = I.smooth_random_state(o.coords(), 75, amp=0.1)
        U0[:, : mesh.nElems // 2] = I.smooth_random_state(o.coords(), 75, amp=0.002)[:, : mesh.nElems // 2]
        rng = np.random.default_rng(76)
        lam, d = rng.normal(size=U0.shape), rng.normal(size=U0.shape)
        U = s.init_state(U0)
        dt = 0.2 * s.timestep(U, 0.9)

        def run():
            lamU, lamdU = s.to_device(lam), s.empty_state()
            out = s.adjoint_rhs(U, lamU).cpu().numpy()
            s.adjoint_rk_step(U, lamU, lamdU, dt)
            return out, lamU.cpu().numpy()

        on = run()
        s.set_element_metrics(False)
        off = run()
    finally:
        s.close()
    _, jd = o.rhs_jvp(U0, d)
    err = abs((on[0] * d).sum() - (lam * jd).sum()) / np.abs(lam * jd).sum()
    _say("affine adjoint", N, nodes, physics, "oracle", err, "metric", dm)
    assert dm < 1e-12 and err < 1e-12 + 20 * dm
    for a, b in zip(on, off):
        assert np.isfinite(a).all()
        assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()


@pytest.mark.parametrize("case", [(3, 0, 0, 0, 0, 0), (7, 1, 0, 1, 0, 0), (3, 0, 1, 1, 0, 0), (5, 1, 1, 0, 0, 0),
                                  (7, 1, 1, 1, 0, 0), (7, 1, 1, 1, 1, 0), (1, 0, 0, 0, 0, 1), (3, 1, 1, 1, 0, 1),
                                  (5, 0, 0, 0, 0, 1)], ids=str)
def test_register_contents_on_entry_are_ignored(S, case):
    """rk_step, rk_step_stages and the reverse step (its own register too) with
    a register of NaN give bitwise what they give with one of zeros."""
    import torch
    _say("register", case)
    N, nodes, form, physics, integrator, fv = case
    mesh = I.box_mesh((3, 2, 2), (-PI,) * 3, (PI,) * 3, rotate_seed=8)
    cfg = dict(N=N, nodes=nodes, form=form, physics=physics, mu=0.02 if physics else 0.0, integrator=integrator, fv=fv)
    s = S(cfg, mesh, adjoint=not fv)
    try:
        U0 = s.init_state(I.smooth_random_state(s.coords(), 77, amp=0.1))
        if fv:
            s.fv_switch(U0, (np.arange(mesh.nElems) % 2).astype(np.int32))
        dt = 0.2 * s.timestep(U0, 0.9)
        lam0 = s.to_device(np.random.default_rng(78).normal(size=s.state_shape))
        out = []
        for fill in (0.0, float("nan")):
            s.ws[: s.ws.numel() // 8 * 8].view(torch.float64).fill_(fill)   # (scratch: all of it is written before it is read)
            U, dU = U0.clone(), torch.full_like(U0, fill)
            s.rk_step(U, dU, dt, 2)
            res = [U, dU]
            if not fv:
                V, dV, Y = U0.clone(), torch.full_like(U0, fill), s.stage_buffer()
                s.rk_step_stages(V, dV, dt, Y)
                lam, lamd = lam0.clone(), torch.full_like(U0, fill)
                s.adjoint_rk_step(U0, lam, lamd, dt)
                res += [V, dV, Y, lam]
            out.append(res)
        for a, b in zip(*out):
            assert torch.isfinite(a).all() and torch.equal(a, b)
    finally:
        s.close()


@pytest.mark.parametrize("physics", [0, 1])
@pytest.mark.parametrize("curved,twopoint", [(0.0, 0), (0.1, 0), (0.1, 1)])
@pytest.mark.parametrize("N", [4, 5, 6])
def test_pair_exchange(S, orc, N, curved, twopoint, physics):
    """Lobatto split form on lines that straddle wavefronts: the residual hands
    each pair's second share over through LDS at every distance (N + 1 odd: none
    is met from both ends, N = 5: one is), the adjoint too for Chandrashekar's
    flux.  Element counts that leave work-items idle, random side orientations;
    oracle bounds as for all residuals, steps and transposed residuals."""
    _say("exchange", N, curved, twopoint, physics)
    mesh = I.box_mesh((2, 3, 2), (-PI,) * 3, (PI,) * 3, Ngeo=N if curved else 1, curved_amp=curved, rotate_seed=10)
    cfg = dict(N=N, nodes=1, form=1, physics=physics, mu=0.02 if physics else 0.0, twopoint=twopoint)
    o, s = orc.Oracle(cfg, mesh), S(cfg, mesh, adjoint=True)
    try:
        _, J, Ja = o.geometry()
        s.upload_metrics(Ja, 1.0 / J, o.face_normals())
        # (variations on both sides of the log means' series threshold)
        U = I.smooth_random_state(o.coords(), 91, amp=0.2)
        U[:, ::2] = I.smooth_random_state(o.coords(), 91, amp=0.002)[:, ::2]
        Ug = s.init_state(U)
        err = rel_err_per_var(s.rhs(Ug).cpu().numpy(), o.rhs(U))
        lam = np.random.default_rng(92).normal(size=U.shape)
        adj = _off(s.adjoint_rhs(Ug, s.to_device(lam)).cpu().numpy(), o.rhs_vjp(U, lam))
        dt = 0.5 * o.timestep(U, 0.9)
        s.rk_step(Ug, s.empty_state(), dt, 1)
        step = _off(Ug.cpu().numpy() - U, o.lserk(U, 1, dt) - U)
    finally:
        s.close()
    _say("exchange", N, curved, twopoint, physics, err.max(), adj, step)
    assert np.all(err < 1e-12) and adj < 1e-12 and step < 1e-11


@pytest.mark.parametrize("K", [(1, 1, 1), (3, 1, 1), (3, 3, 1)], ids=str)
@pytest.mark.parametrize("nodes,form", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("physics", [0, 1])
def test_packed_elements_steps(S, orc, K, nodes, form, physics):
    """N = 1, the kernels that test_packed_elements leaves out: the reverse step,
    and of FV contexts the step, the indicator and the switch with a register."""
    _say("packed steps", K, nodes, form, physics)
    mesh = I.box_mesh(K, (-PI,) * 3, (PI,) * 3, rotate_seed=4)
    cfg = dict(N=1, nodes=nodes, form=form, physics=physics, mu=0.02 if physics else 0.0)
    o, s = orc.Oracle(cfg, mesh), S(cfg, mesh, adjoint=True)
    of, f = orc.Oracle(dict(cfg, fv=1), mesh), S(dict(cfg, fv=1), mesh)
    try:
        _, J, Ja = o.geometry()
        for x in (s, f):
            x.upload_metrics(Ja, 1.0 / J, o.face_normals())
        U = I.smooth_random_state(o.coords(), 93, amp=0.1)
        rng = np.random.default_rng(94)
        lam, reg = rng.normal(size=U.shape), rng.normal(size=U.shape)
        dt = o.timestep(U, 0.9)
        lamU = s.to_device(lam)
        s.adjoint_rk_step(s.to_device(U), lamU, s.empty_state(), dt)
        assert _off(lamU.cpu().numpy(), o.lserk_adjoint(U, lam, 1, dt)) < 1e-12
        mask = (np.arange(mesh.nElems) % 3 == 0).astype(np.int32)
        Uf, dUf = f.init_state(U), f.to_device(reg)
        ind, ref = f.fv_indicator(Uf).cpu().numpy(), of.indicator(U)
        assert np.abs(ind - ref)[ref > -12].max(initial=0.0) < 1e-9
        f.fv_switch(Uf, mask, dU=dUf)
        Uo, dUo = of.fv_switch(U, reg, mask)
        assert _off(Uf.cpu().numpy(), Uo) < 1e-13 and _off(dUf.cpu().numpy(), dUo) < 1e-12
        f.rk_step(Uf, dUf, dt, 2)
        assert _off(Uf.cpu().numpy() - Uo, of.lserk(Uo, 2, dt) - Uo) < 1e-11
    finally:
        s.close()
        f.close()


@pytest.mark.parametrize("form,riemann,precision", [(0, 0, 0), (1, 0, 0), (1, 2, 0), (1, 0, 1)])
@pytest.mark.parametrize("nodes", [0, 1])
@pytest.mark.parametrize("N", range(1, 8))
def test_affine_variants_with_sutherland(S, N, nodes, form, riemann, precision):
    """Sutherland's law has lifting kernels of its own, and Roe's flux runs the
    general residual beside the affine lifting: on an affine mesh against the
    kernels that read the node arrays, with the bounds of
    test_affine_variant_matches_general_kernels (adjoint: 1e-12 too).  The RK
    register is left out: after a step it holds 1e-3 of the state, and last bits
    of the state between the stages move it by 3 to 6e-12 with either kernels."""
    _say("affine sutherland", N, nodes, form, riemann, precision)
    mesh = I.box_mesh((3, 2, 3), (-PI,) * 3, (PI,) * 3, rotate_seed=5)
    s = S(dict(N=N, nodes=nodes, form=form, physics=1, mu=1e-2, viscosity=1, Tref=1.0, Ts=0.4, riemann=riemann,
               precision=precision), mesh, adjoint=not precision)
    try:
        assert s.element_metric_count() == mesh.nElems
        U0 = s.init_state(I.smooth_random_state(s.coords(), 95, amp=0.1))
        lam = s.to_device(np.random.default_rng(96).normal(size=s.state_shape))
        dt = 0.2 * s.timestep(U0, 0.9)

        def run():
            out = [s.rhs(U0).cpu().numpy(), s.lift(U0).cpu().numpy()]
            U, dU = U0.clone(), s.empty_state()
            s.rk_step(U, dU, dt, 1)
            out.append(U.cpu().numpy())
            return out if precision else out + [s.adjoint_rhs(U0, lam).cpu().numpy()]

        on = run()
        s.set_element_metrics(False)
        off = run()
    finally:
        s.close()
    err = [np.abs(a - b).max() / np.abs(b).max() for a, b in zip(on, off)]
    _say("affine sutherland", N, nodes, form, riemann, precision, err)
    assert all(np.isfinite(a).all() for a in on) and max(err) <= (5e-6 if precision else 1e-12)
