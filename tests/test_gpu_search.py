"""GPU parity of the full Grover search (Sec. 5.1): G^{n_t} from HALL|0..0> with
n_t = floor((pi/4) sqrt(N)) through pk_evaluate_repeat (one graph of every pass).

  * noise-free, against the rotation closed form of the oracle (exact at any
    n_q): C_x = sin((2 n_t + 1) theta), the rest cos((2 n_t + 1) theta)/sqrt(N - 1);
    the normwise error is printed and held to a worst-case bound derived from the
    arithmetic (see ``_hall_bound``): errors of unitary iterations add up at most
    linearly, so n_t iterations stay within n_t times one iteration's bound;
  * a noisy iteration repeated, against the gate-by-gate oracle;
  * several marked items; reps = 1 equals pk_evaluate; a second replay of the graph.
Each test prints its case before touching the GPU.
"""

import sys

import numpy as np
import pytest

import oracle as O
from paper_0902_0699_amd import workload as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _pk():
    from paper_0902_0699_amd import paperkern as pk
    return pk


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _unit(prec):
    return 2.0 ** -53 if prec == "fp64" else 2.0 ** -24


def _hall_bound(nq, nt, prec):
    """Worst-case normwise error of n_t HALL-based iterations.  One iteration is
    2 n_q unnormalised butterfly levels (x + y, then x_new - 2 y: at most 2u of the
    output's norm per level), the Oracle and Inv signs (exact), a power-of-two scale
    (exact) and at most 4 more roundings (the odd 2^(-1/2), the readout): (2 n_q + 4) 2u.
    Each iteration is unitary, so its rounding error is carried by the later ones
    without growth: the errors of n_t iterations add to at most n_t times that, plus
    the rounding of the uniform input 2^(-n_q/2) (u for odd n_q)."""
    return nt * (2 * nq + 4) * 2 * _unit(prec) + _unit(prec)


def _diffusion_bound(nq, nt, prec):
    """Worst-case normwise error of n_t iterations of the diffusion variant: per
    iteration the FP64 mean of N terms (at most log2 N + 1 roundings of the sum's
    magnitude, in FP64) and 2 m - C (two roundings in the data's precision)."""
    return nt * (3 * _unit(prec) + (nq + 1) * 2.0 ** -53) + _unit(prec)


def _uniform(nq, dt=torch.complex128):
    return torch.full((1 << nq,), 2.0 ** (-nq / 2), dtype=dt, device="cuda")


@pytest.mark.parametrize("nq,prec", [(4, "fp64"), (10, "fp64"), (13, "fp64"), (16, "fp64"), (20, "fp64"),
                                     (12, "fp32"), (18, "fp32")])
def test_search_against_closed_form(nq, prec):
    pk = _pk()
    nt = pk.grover_iterations(nq)
    x = int(np.random.default_rng(nq).integers(0, 1 << nq))
    plan = pk.Plan({"nq": nq, "gates": W.grover_gates(), "marked": [x]}, prec=prec)
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    _say("search n_q=%d n_t=%d %s" % (nq, nt, prec))
    for _ in range(2):  # capture, then a replay of the same graph
        out, L, norm = pk.evaluate_repeat(plan, _uniform(nq, dt), nt)
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.complex128)
        want = O.grover_closed_form(nq, nt, x)
        err = float(np.linalg.norm(got - want))
        tol = _hall_bound(nq, nt, prec)
        _say("  normwise err %.3e (bound %.3e, %.1f%% of it; %.3e per iteration)  L %.12f (closed form %.12f)"
             % (err, tol, 100 * err / tol, err / nt, L.item(), abs(want[x]) ** 2))
        assert err <= tol
        # |L - L_ref| <= (|a| + |b|) |a - b| and |norm - 1| <= 2 err + err^2
        assert abs(L.item() - abs(want[x]) ** 2) <= 2.5 * tol and abs(norm.item() - 1.0) <= 2.5 * tol
    assert abs(want[x]) ** 2 > 0.9  # the search succeeds (Sec. 5.1)


@pytest.mark.parametrize("nq,prec,tile", [(12, "fp64", None), (20, "fp64", 12), (20, "fp64", None),
                                          (18, "fp32", None), (16, "fp64", 8)])
def test_persistent_launch_equals_launch_per_pass(nq, prec, tile, monkeypatch):
    """pk_evaluate_repeat runs one launch per pass; PK_REPEAT_PERSISTENT=1 runs every
    pass of every iteration in one persistent launch with grid barriers.  The same
    kernels run on the same tiles in the same order, so the states agree bit for
    bit."""
    pk = _pk()
    nt = pk.grover_iterations(nq)
    x = int(np.random.default_rng(nq + 7).integers(0, 1 << nq))
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    out = {}
    for mode in ("persistent", "per_pass"):
        monkeypatch.setenv("PK_REPEAT_PERSISTENT", "1" if mode == "persistent" else "0")
        plan = pk.Plan({"nq": nq, "gates": W.grover_gates((2, 3, 0.3, 0.4, 0.0)), "marked": [x]}, prec=prec)
        if tile:
            plan.set_tiling(tile, 4, 1)
        _say("repeat n_q=%d n_t=%d %s tile %s: %s" % (nq, nt, prec, tile, mode))
        for _ in range(2):  # capture, then a replay
            y, L, norm = pk.evaluate_repeat(plan, _uniform(nq, dt), nt)
        torch.cuda.synchronize()
        out[mode] = (y, L.item(), norm.item())
    assert torch.equal(out["persistent"][0], out["per_pass"][0])
    assert out["persistent"][1:] == out["per_pass"][1:]
    assert np.isfinite(out["persistent"][1])


def test_persistent_barrier_time_out_gives_nan(monkeypatch):
    """A grid barrier that is not complete within its bound gives up: forced here
    from the host with a zero wait bound (PK_BARRIER_SPIN_US=0), so workgroups
    that arrive before the last one stop waiting.  Every kernel still ends; L and
    the norm come out NaN instead of a hang or a silently wrong value."""
    pk = _pk()
    monkeypatch.setenv("PK_BARRIER_SPIN_US", "0")
    monkeypatch.setenv("PK_REPEAT_PERSISTENT", "1")
    nq = 20
    plan = pk.Plan({"nq": nq, "gates": W.grover_gates(), "marked": [5]})
    plan.set_tiling(12, 4, 1)
    _say("repeat with a zero barrier bound, n_q=%d" % nq)
    y, L, norm = pk.evaluate_repeat(plan, _uniform(nq), 50)
    torch.cuda.synchronize()
    assert np.isnan(L.item()) and np.isnan(norm.item())


def test_noisy_iteration_repeated_against_gate_by_gate_oracle():
    pk = _pk()
    nq, reps = 9, 7
    rng = np.random.default_rng(5)
    gates = W.grover_gates((3, 2, 1.2, 0.7, 0.0)) + [("D4", 1, 5, 0.3, 0.2, -0.1)]
    marked = [17, 300]
    psi = rng.standard_normal(1 << nq) + 1j * rng.standard_normal(1 << nq)
    psi /= np.linalg.norm(psi)
    plan = pk.Plan({"nq": nq, "gates": gates, "marked": marked})
    _say("noisy iteration x%d, n_q=%d" % (reps, nq))
    out, L, _ = pk.evaluate_repeat(plan, torch.from_numpy(psi).to("cuda"), reps)
    want = psi
    for _ in range(reps):
        want, Lw, _ = O.evaluate(nq, gates, marked, want)
    got = out.cpu().numpy()
    assert np.linalg.norm(got - want) <= 1e-12 * reps and abs(L.item() - Lw) <= 1e-12 * reps


@pytest.mark.parametrize("nq,reps,tiling,prec", [(14, 11, None, "fp64"), (15, 16, (9, 3, 1), "fp64"),
                                                  (16, 19, (12, 4, 1), "fp32"), (7, 9, None, "fp64")])
def test_fused_repeat_against_gate_by_gate_oracle(nq, reps, tiling, prec):
    """reps >= 8 applications of a list without angle parameters run 8 at a time as
    one fused schedule (reps mod 8 alone, first): every element against the oracle
    applying the list reps times; the launch count is the fused one."""
    pk = _pk()
    rng = np.random.default_rng(nq + reps)
    gates = [("H", 1), ("ONEOP", 3, O.PAULI_Y), ("CPHASE", 2, nq), ("HALL",), ("ORACLE",), ("INV",),
             ("CPHASEK", nq - 1, 1, 3), ("HALL",), ("H", nq)]
    marked = [int(rng.integers(0, 1 << nq)), 5]
    psi = rng.standard_normal(1 << nq) + 1j * rng.standard_normal(1 << nq)
    psi /= np.linalg.norm(psi)
    plan = pk.Plan({"nq": nq, "gates": gates, "marked": marked}, prec=prec)
    if tiling:
        plan.set_tiling(*tiling)
    launches = pk.repeat_launches(plan, reps)
    _say("fused repeat x%d n_q=%d %s %s: %d launches (%d unfused)" % (reps, nq, tiling, prec, launches,
                                                                    reps * plan.passes()))
    assert launches < reps * plan.passes() or plan.passes() == 1
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    out, L, norm = pk.evaluate_repeat(plan, torch.from_numpy(psi).to(dt).to("cuda"), reps)
    torch.cuda.synchronize()
    want = psi
    for _ in range(reps):
        want, Lw, nw = O.evaluate(nq, gates, marked, want)
    tol = (1e-12 if prec == "fp64" else 1e-5) * reps
    got = out.cpu().numpy().astype(np.complex128)
    assert np.linalg.norm(got - want) <= tol and abs(L.item() - Lw) <= tol and abs(norm.item() - nw) <= tol
    # a settings change rebuilds the fused schedule
    plan.set_tiling(8, 2, 1)
    out2, L2, _ = pk.evaluate_repeat(plan, torch.from_numpy(psi).to(dt).to("cuda"), reps)
    torch.cuda.synchronize()
    got2 = out2.cpu().numpy().astype(np.complex128)
    assert np.linalg.norm(got2 - want) <= tol and abs(L2.item() - Lw) <= tol


def test_repeat_once_equals_evaluate_and_rejects_bad_reps():
    pk = _pk()
    nq = 11
    plan = pk.Plan({"nq": nq, "gates": W.grover_gates((2, 4, 0.4, 0.5, 0.0)), "marked": [9]})
    x = _uniform(nq)
    _say("repeat once, n_q=%d" % nq)
    a, La, _ = pk.evaluate_repeat(plan, x, 1)
    b, Lb, _ = pk.evaluate(plan, x)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and La.item() == Lb.item()
    with pytest.raises(pk.PaperkernError):
        pk.evaluate_repeat(plan, x, 0)


# --------------------------------------------------------------------------- the diffusion variant


@pytest.mark.parametrize("nq,prec", [(3, "fp64"), (10, "fp64"), (16, "fp64"), (22, "fp64"), (14, "fp32"),
                                     (20, "fp32")])
def test_diffusion_variant_against_closed_form(nq, prec):
    pk = _pk()
    nt = pk.grover_iterations(nq)
    x = int(np.random.default_rng(nq + 1).integers(0, 1 << nq))
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    _say("diffusion variant n_q=%d n_t=%d %s" % (nq, nt, prec))
    out, L = pk.search_diffusion(nq, [x], nt, _uniform(nq, dt))
    torch.cuda.synchronize()
    want = O.grover_closed_form(nq, nt, x)
    err = float(np.linalg.norm(out.cpu().numpy().astype(np.complex128) - want))
    tol = _diffusion_bound(nq, nt, prec)
    _say("  normwise err %.3e (bound %.3e, %.1f%% of it)  L %.12f" % (err, tol, 100 * err / tol, L.item()))
    assert err <= tol and abs(L.item() - abs(want[x]) ** 2) <= 2.5 * tol


def test_diffusion_variant_equals_hall_form_with_several_marked():
    """From a random state with three marked items, the identity route and the
    HALL-based passes give the same state (and one step equals the gate-by-gate
    oracle)."""
    pk = _pk()
    nq, reps = 14, 9
    rng = np.random.default_rng(12)
    psi = rng.standard_normal(1 << nq) + 1j * rng.standard_normal(1 << nq)
    psi /= np.linalg.norm(psi)
    marked = [5, 999, (1 << nq) - 1]
    x = torch.from_numpy(psi).to("cuda")
    _say("diffusion variant vs HALL form, n_q=%d, %d marked" % (nq, len(marked)))
    a, La = pk.search_diffusion(nq, marked, reps, x)
    plan = pk.Plan({"nq": nq, "gates": W.grover_gates(), "marked": marked})
    b, Lb, _ = pk.evaluate_repeat(plan, x, reps)
    torch.cuda.synchronize()
    assert torch.linalg.vector_norm(a - b).item() <= 1e-12 * reps and abs(La.item() - Lb.item()) <= 1e-12 * reps
    one, L1 = pk.search_diffusion(nq, marked, 1, x)
    want, Lw, _ = O.evaluate(nq, W.grover_gates(), marked, psi)
    assert np.linalg.norm(one.cpu().numpy() - want) <= 1e-13 and abs(L1.item() - Lw) <= 1e-13
    # in place
    y = x.clone()
    pk.search_diffusion(nq, marked, reps, y, out=y)
    torch.cuda.synchronize()
    assert torch.linalg.vector_norm(y - a).item() == 0.0


def test_diffusion_variant_with_many_marks_in_one_block():
    """At n_q = 14 each block of the streaming pass owns 8 labels: marks 8..12 put
    five in one block (beyond the two a block keeps by value), 40 and 47 two in
    another; against the HALL-based passes and, for one step, the oracle."""
    pk = _pk()
    nq, reps = 14, 7
    rng = np.random.default_rng(21)
    psi = rng.standard_normal(1 << nq) + 1j * rng.standard_normal(1 << nq)
    psi /= np.linalg.norm(psi)
    marked = [8, 9, 10, 11, 12, 40, 47, 1000]
    x = torch.from_numpy(psi).to("cuda")
    _say("diffusion variant, %d marks, 5 in one block, n_q=%d" % (len(marked), nq))
    a, La = pk.search_diffusion(nq, marked, reps, x)
    plan = pk.Plan({"nq": nq, "gates": W.grover_gates(), "marked": marked})
    b, Lb, _ = pk.evaluate_repeat(plan, x, reps)
    torch.cuda.synchronize()
    assert torch.linalg.vector_norm(a - b).item() <= 1e-12 * reps and abs(La.item() - Lb.item()) <= 1e-12 * reps
    one, L1 = pk.search_diffusion(nq, marked, 1, x)
    want, Lw, _ = O.evaluate(nq, W.grover_gates(), marked, psi)
    assert np.linalg.norm(one.cpu().numpy() - want) <= 1e-13 and abs(L1.item() - Lw) <= 1e-13


def test_diffusion_variant_rejects_bad_arguments():
    pk = _pk()
    x = _uniform(6)
    for nq, marked, it in ((6, [64], 1), (6, [3, 3], 1), (6, [1], 0), (0, [0], 1)):
        with pytest.raises((pk.PaperkernError, ValueError)):
            pk.search_diffusion(nq, marked, it, x)


@pytest.mark.parametrize("nq,prec,gates", [(8, "fp64", "grover"), (13, "fp64", "grover"), (18, "fp64", "grover"),
                                           (18, "fp32", "grover"), (20, "fp32", "grover"), (20, "fp64", "qft")])
def test_persistent_launch_with_the_automatic_setting(nq, prec, gates, monkeypatch):
    """PK_REPEAT_PERSISTENT=1 is honoured where the library picks 3 register bits: with a
    zero wait bound L and the norm are NaN (more than one workgroup, so a barrier gave up),
    with the normal one the states equal the launch per pass bit for bit."""
    pk = _pk()
    reps = 7
    glist = [("QFT", 1, nq)] if gates == "qft" else W.grover_gates((2, 3, 0.3, 0.4, 0.0))
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    out = {}
    for mode, spin in (("persistent", "0"), ("persistent", None), ("per_pass", None)):
        monkeypatch.setenv("PK_REPEAT_PERSISTENT", "1" if mode == "persistent" else "0")
        if spin is None:
            monkeypatch.delenv("PK_BARRIER_SPIN_US", raising=False)
        else:
            monkeypatch.setenv("PK_BARRIER_SPIN_US", spin)
        plan = pk.Plan({"nq": nq, "gates": glist, "marked": [3]}, prec=prec)
        fwd = plan.describe()["instances"][0]["forward"]
        assert {p["rbits"] for p in fwd} == {3}
        _say("repeat n_q=%d %s %s: %s, bound %s" % (nq, prec, gates, mode, spin))
        y, L, norm = pk.evaluate_repeat(plan, _uniform(nq, dt), reps)
        torch.cuda.synchronize()
        if spin is None:
            out[mode] = (y, L.item(), norm.item())
        elif nq > fwd[0]["k"]:
            assert np.isnan(L.item()) and np.isnan(norm.item())
    assert torch.equal(out["persistent"][0], out["per_pass"][0])
    assert out["persistent"][1] == out["per_pass"][1]
    # the norm's terms may be contracted differently by the two kernels: n + 2 roundings
    u = 2.0 ** -53 if prec == "fp64" else 2.0 ** -24
    assert abs(out["persistent"][2] - out["per_pass"][2]) <= 4 * u + (1 << nq) * 2.0 ** -53
