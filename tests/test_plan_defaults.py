"""The library's own choice of tile and register bits for a single instance (CPU): the
schedule it leads to computes what the oracle and an explicit tiling compute.
"""

import numpy as np
import pytest

import oracle as O
from paper_0902_0699_amd import autotune as AT
from paper_0902_0699_amd import paperkern as pk
from paper_0902_0699_amd import workload as W
from schedule_emulator import run_backward, run_forward


def _gates(kind, nq, rng):
    a, b = 1, nq
    if kind == "hadamards":
        return W.grover_gates((max(1, nq // 2), 3, 0.7, 0.4, 0.0))
    if kind == "phases":
        return W.phase_circuit(rng, nq, 12) + [("D2", b, 0.2, 0.9, 0.1)]
    if kind == "qft":
        return [("H", nq), ("QFT", 1, nq - 1), ("ORACLE",)]
    u, _ = np.linalg.qr(rng.standard_normal((4, 4)) + 1j * rng.standard_normal((4, 4)))
    return [("HALL",), ("TWOOP", a, b, u), ("D4", b, a, 0.3, 0.5, -0.2), ("SWAP", 1, 2), ("CNOT", 2, a), ("INV",),
            ("HALL",)]


@pytest.mark.parametrize("kind", ["hadamards", "phases", "qft", "two_qubit"])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nq", [3, 9, 12, 13, 14, 15])
def test_automatic_schedule_matches_the_oracle(nq, prec, kind):
    rng = np.random.default_rng(nq)
    gates = _gates(kind, nq, rng)
    marked = [2, (1 << nq) - 1]
    prob = {"nq": nq, "gates": gates, "marked": marked}
    v = rng.standard_normal(1 << nq) + 1j * rng.standard_normal(1 << nq)
    psi = v / np.linalg.norm(v)
    want, Lw, _ = O.evaluate(nq, gates, marked, psi)
    plan = pk.Plan(prob, prec=prec)
    out, L = run_forward([prob], plan.describe(), 0, psi)
    np.testing.assert_allclose(out, want, rtol=0, atol=1e-12)
    assert abs(L - Lw) <= 1e-12
    if prec == "fp64":
        gpsi, gang = run_backward([prob], plan.describe(), 0, want, 0.5)
        wpsi, wang = O.adjoint_grad(nq, gates, marked, psi, 0.5)
        np.testing.assert_allclose(gpsi, wpsi, rtol=0, atol=1e-12)
        np.testing.assert_allclose(gang.reshape(-1), np.asarray(wang).reshape(-1), rtol=0, atol=1e-12)


@pytest.mark.parametrize("kind", ["hadamards", "phases", "qft", "two_qubit"])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nq", [1, 6, 12, 13, 16, 18, 19, 20, 21, 22, 23, 24, 25, 26])
def test_automatic_settings_stay_within_the_kernels(nq, prec, kind):
    """Tiles of at most 2^13, 3 to 5 register bits, at most 1024 threads, two-qubit gates
    with room for two pairs; setting either one restores the documented other."""
    if nq < 3 and kind != "hadamards":
        pytest.skip("needs three qubits")
    gates = _gates(kind, nq, np.random.default_rng(nq))
    plan = pk.Plan({"nq": nq, "gates": gates, "marked": [1]}, prec=prec)
    d = plan.describe()
    for p in d["instances"][0]["forward"]:
        assert p["k"] <= min(13, nq) and p["rbits"] in (3, 4, 5) and d["tile_bits"] - p["rbits"] <= 10
        assert kind != "two_qubit" or p["rbits"] == 4
    assert all(p["rbits"] == 4 and p["k"] <= 12 for p in d["instances"][0]["backward"])
    default = 4 if prec == "fp64" else 5
    plan.set_tiling(11, 4)
    assert {p["rbits"] for p in plan.describe()["instances"][0]["forward"]} == {default}
    plan = pk.Plan({"nq": nq, "gates": gates, "marked": [1]}, prec=prec)
    plan.set_launch(0, 0)
    d = plan.describe()
    assert d["tile_bits"] == 13 and {p["rbits"] for p in d["instances"][0]["forward"]} == {default}


def _mixed(kind, nq):
    """A Grover iteration with a few gates of another kind, or a list dense in them."""
    g = W.grover_gates((2, 2, 0.7, 0.4, 0.0))
    rng = np.random.default_rng(nq)
    u, _ = np.linalg.qr(rng.standard_normal((4, 4)) + 1j * rng.standard_normal((4, 4)))
    return {"one_phase": g + [("CPHASEK", 1, nq, 3)], "phase_inside": g[:3] + [("CPHASE", nq // 2, nq // 2 + 1)] + g[3:],
            "one_cnot": g + [("CNOT", 1, nq // 2)], "one_d4": g + [("D4", 2, nq - 2, 0.1, 0.2, 0.3)],
            "phases": W.phase_circuit(rng, nq, 12), "qft_half": [("QFT", 1, nq // 2)], "qft": [("QFT", 1, nq)],
            "brickwork": [("TWOOP", q, q + 1, u) for first in (1, 2) for q in range(first, nq, 2)],
            "qft_cnot": [("QFT", 1, nq), ("CNOT", 1, 2)]}[kind]


@pytest.mark.parametrize("kind", ["one_phase", "phase_inside", "one_cnot", "one_d4", "phases", "qft_half", "qft",
                                  "brickwork", "qft_cnot"])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nq", [14, 18, 19, 20, 21, 22, 23, 24, 25, 26, 27, 28, 29, 30])
def test_automatic_tiles_cost_no_passes(nq, prec, kind):
    """The chosen tiles take no more passes than 2^13 ones, but for half as many more at
    2^19 and 2^20 amplitudes with phases, and one more in FP32 from 2^23 to 2^27 with 4x4
    steps."""
    gates = _mixed(kind, nq)
    fours = kind in ("one_cnot", "one_d4", "brickwork", "qft_cnot")
    auto = pk.Plan({"nq": nq, "gates": gates, "marked": [1]}, prec=prec)
    big = pk.Plan({"nq": nq, "gates": gates, "marked": [1]}, prec=prec)
    big.set_launch(0, 4 if fours or prec == "fp64" else 5)
    big.set_tiling(13, 4)
    most = big.passes()
    if nq in (19, 20) and not fours:
        most = most * 3 // 2
    if prec == "fp32" and 23 <= nq <= 27 and fours:
        most += 1
    assert auto.passes() <= most


def test_automatic_registers_follow_the_share_of_phases():
    """FP32 2^13 tiles: 32 amplitudes a thread with few phases, 16 where most gates are;
    FP64 2^12 tiles from 2^27 on: 8 where that takes at most a quarter more exchanges than 16."""
    def rbits(nq, prec, gates):
        d = pk.Plan({"nq": nq, "gates": gates, "marked": []}, prec=prec).describe()
        return d["tile_bits"], {p["rbits"] for p in d["instances"][0]["forward"]}
    assert rbits(29, "fp32", _mixed("one_phase", 29)) == (13, {5})
    assert rbits(29, "fp32", _mixed("phases", 29)) == (13, {5})
    assert rbits(28, "fp32", _mixed("qft", 28)) == (13, {4})
    assert rbits(28, "fp64", [("QFT", 1, 8)]) == (12, {4})
    assert rbits(28, "fp64", [("QFT", 1, 10)]) == (12, {3})
    assert rbits(28, "fp64", [("QFT", 1, 14)]) == (12, {4})
    assert rbits(28, "fp64", [("QFT", 1, 20)]) == (12, {3})


def _used(plan):
    return plan.describe()["instances"][0]["used"]


def test_describe_reports_what_the_passes_use():
    """The library's overlapped loop and streaming where the caller set nothing, else the
    caller's settings; a batch's instances use neither."""
    prob = {"nq": 24, "gates": W.phase_circuit(np.random.default_rng(1), 24, 12), "marked": [1]}
    plan = pk.Plan(prob)
    n, nb = plan.passes(), len(_used(plan)["backward"])
    assert any(p["overlap"] == 1 for p in _used(plan)["forward"])
    assert all(p["overlap"] == 0 for p in plan.describe()["instances"][0]["forward"])
    plan.set_pass_overlap([0] * n)
    plan.set_pass_walk([4] * n + [16] * nb)
    assert all(p["overlap"] == 0 and p["walk"] == 4 for p in _used(plan)["forward"])
    assert all(p["walk"] == 16 for p in _used(plan)["backward"])
    big = pk.Plan({"nq": 30, "gates": W.grover_gates((2, 2, 0.4, 0.1, 0.2)), "marked": [1]})
    assert [p["stream"] for p in _used(big)["forward"]] == [0] * (big.passes() - 1) + [1]
    batch = pk.Plan([prob, dict(prob, nq=24)])
    for inst in batch.describe()["instances"]:
        assert all(p == {"walk": 0, "overlap": 0, "stream": 0} for p in inst["used"]["forward"] + inst["used"]["backward"])


class _NoTimer:
    def __init__(self, **_):
        pass

    def record(self):
        pass

    def elapsed_time(self, _):
        return 1.0


@pytest.mark.parametrize("walks", [None, 16])
def test_backward_walk_tuning_keeps_the_forward(walks, monkeypatch):
    """tune_backward_walk leaves the forward passes' walk and loop as they were, set by the
    caller or not (no kernel runs: the timing is replaced)."""
    import torch
    monkeypatch.setattr(torch.cuda, "Event", _NoTimer)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    monkeypatch.setattr(pk, "backward", lambda *a, **k: None)
    plan = pk.Plan({"nq": 30, "gates": W.grover_gates((2, 2, 0.4, 0.1, 0.2)), "marked": [1]})
    if walks:
        plan.set_pass_walk([walks] * plan.passes())
    before = _used(plan)["forward"]
    AT.tune_backward_walk(plan, None, None)
    assert _used(plan)["forward"] == before


@pytest.mark.parametrize("overlap", [True, False])
def test_walk_tuning_applies_a_loop_it_timed(overlap, monkeypatch):
    """tune_walk leaves every pass with a walk and a loop of the combinations that it timed:
    without `overlap` the plain loop, also where the library would overlap (the timing is
    replaced by one that favours the last combination)."""
    calls = []
    monkeypatch.setattr(pk, "time_passes", lambda plan, *_: calls.append(_used(plan)["forward"]) or
                        [100.0 - len(calls)] * plan.passes())
    plan = pk.Plan({"nq": 24, "gates": W.phase_circuit(np.random.default_rng(1), 24, 12), "marked": [1]})
    AT.tune_walk(plan, None, None, reps=1, walks=(0, 2), overlap=overlap)
    got = _used(plan)["forward"]
    assert got in calls and all(p["overlap"] == int(overlap) and p["walk"] == 2 for p in got)


@pytest.mark.parametrize("nq,prec", [(12, "fp64"), (14, "fp64"), (16, "fp32"), (18, "fp32"), (20, "fp64"), (24, "fp64")])
def test_tuning_can_keep_the_automatic_setting(nq, prec, monkeypatch):
    """The setting that the library chose is among those that tune times, and applying it
    gives the same schedule back (the timing is replaced by one that favours it)."""
    plan = pk.Plan({"nq": nq, "gates": W.grover_gates((2, 2, 0.4, 0.1, 0.2)), "marked": [1]}, prec=prec)
    own = plan.describe()["instances"]
    monkeypatch.setattr(AT, "_time", lambda *_: 1.0 if plan.describe()["instances"] == own else 2.0)
    best, table = AT.tune(plan, None, use_cache=False)
    assert plan.describe()["instances"] == own and table[0][1] == 1.0 and table[-1][1] == 2.0
    monkeypatch.setattr(AT, "_time", lambda *_: 1.0 if plan.describe()["instances"] != own else 2.0)
    AT.tune(plan, None, use_cache=False, cands=[dict(best, tile_bits=11, reg_bits=4)])
    assert plan.describe()["tile_bits"] == 11


@pytest.mark.parametrize("nq,prec", [(12, "fp64"), (24, "fp64"), (29, "fp64"), (30, "fp64"), (31, "fp32")])
def test_automatic_walk_is_strided(nq, prec):
    """No size has a tile walk of its own: strided until the caller sets one, and again
    after an empty list."""
    plan = pk.Plan({"nq": nq, "gates": W.grover_gates((2, 2, 0.4, 0.1, 0.2)), "marked": [1]}, prec=prec)
    for _ in range(2):
        assert all(p["walk"] == 0 for p in _used(plan)["forward"] + _used(plan)["backward"])
        plan.set_pass_walk([64] * plan.passes())
        plan.set_pass_walk([])


@pytest.mark.parametrize("kind,prec,nq,want", [
    ("hadamards", "fp64", 22, {0}), ("hadamards", "fp64", 24, {0}), ("hadamards", "fp64", 26, {1}),
    ("qft_half", "fp64", 22, {0}), ("qft_half", "fp32", 22, {1}), ("qft_half", "fp64", 25, {1}), ("phases", "fp64", 23, {1}), ("phases", "fp32", 24, {1}),
    ("brickwork", "fp64", 22, {1}), ("one_phase", "fp64", 24, {0}), ("one_phase", "fp32", 23, {0}),
    ("one_phase", "fp32", 25, {0, 1}), ("hadamards", "fp32", 26, {0}), ("small_tiles", "fp64", 26, {0})])
def test_automatic_loop_is_not_mixed_while_the_caches_hold_the_state(kind, prec, nq, want):
    """Every pass overlaps or none does, but for a list with a few phases from 2^13 tiles
    on, whose passes with phases do."""
    gates = W.grover_gates((2, 2, 0.7, 0.4, 0.0)) if kind in ("hadamards", "small_tiles") else _mixed(kind, nq)
    plan = pk.Plan({"nq": nq, "gates": gates, "marked": [1]}, prec=prec)
    if kind == "small_tiles":
        plan.set_tiling(12, 4)
    assert {p["overlap"] for p in _used(plan)["forward"]} == want


@pytest.mark.parametrize("kind", ["one_cnot", "one_d4", "brickwork", "hadamards"])
@pytest.mark.parametrize("prec,sizes", [("fp64", (17, 20)), ("fp32", (21, 22))])
def test_small_states_stream_by_their_size(prec, sizes, kind):
    """Whether the forward passes of a state about as large as the L2s stream follows from
    its size, whatever 4x4 steps it holds."""
    for nq in (sizes[0] - 1, *sizes, sizes[1] + 1):
        gates = W.grover_gates((2, 2, 0.7, 0.4, 0.0)) if kind == "hadamards" else _mixed(kind, nq)
        plan = pk.Plan({"nq": nq, "gates": gates, "marked": [1]}, prec=prec)
        assert {p["stream"] for p in _used(plan)["forward"]} == {int(nq in sizes)}


def test_a_repeat_that_cannot_fuse_is_planned_once():
    """A list whose eight applications take no fewer passes together than apart: the finding
    is kept, so later calls do not compile the eight again (the first does), until a setting
    changes the schedule."""
    import time
    plan = pk.Plan({"nq": 14, "gates": _mixed("brickwork", 14), "marked": [1]})

    def timed(calls):
        t = time.perf_counter()
        n = [pk.repeat_launches(plan, 40) for _ in range(calls)]
        return time.perf_counter() - t, set(n)

    first, n = timed(1)
    assert n == {40 * plan.passes()}  # nothing fused
    later, n = timed(20)
    assert n == {40 * plan.passes()} and later < first
    plan.set_tiling(13, 4)
    assert pk.repeat_launches(plan, 40) <= 40 * plan.passes()
