"""The two-pass step of 2D fields (row pass and axis-0 pass) on lattices that
the one-kernel step of small lattices does not take: kernel variants, storages,
restarts, two-stream steps, graph replays and repeatability, against the FP64
oracle and bit for bit against each other."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2511_22510_amd import workloads as W

pytestmark = pytest.mark.gpu

# relative error of the spectral state against the oracle (the bars of the
# workloads: 100-step trajectories)
TOL = {64: 1e-10, 32: 2e-4}


def _setd():
    from paper_2511_22510_amd import setd
    return setd


def _err(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _worst(g, o, R):
    return max(_err(g.get(r), o.get(r)) for r in range(R))


VARIANT_CASES = [
    W.model_b([128, 32], precision=64, realizations=1),
    W.kpz([128, 32], precision=64, realizations=2, ic_kind=1, ic_sigma=0.2),
    W.model_b([32, 128], precision=32, realizations=2),
    # five items: groups of 2, 4 and 8 end in a partial group
    W.model_b([128, 64], precision=32, realizations=5),
    W.model_a([16, 128], precision=64, order=2, realizations=5),
]


@pytest.mark.parametrize("variant", ["0,0,0", "1,1,1", "2,2,2", "3,3,3", "1,2,3", "3,0,1", "0,4,0", "2,5,3",
                                     "5,4,0", "14,1,1", "11,5,2", "15,0,3", "1,6,1", "0,9,2", "3,11,0",
                                     "1,12,1", "2,15,0"])
@pytest.mark.parametrize("history", [0, 1])
def test_every_real_variant_matches_oracle(variant, history, monkeypatch):
    """Each autotuner choice on real fields in both precisions, with either
    SETD2 storage, whole and partial item groups."""
    S = _setd()
    monkeypatch.setenv("SETD_VARIANT", variant)
    for p in VARIANT_CASES:
        p = dict(p, history_readback=history)
        g, o = S.Plan(p), O.Sim(p)
        assert int(g.info.passes_per_step) == 2
        for n in (1, 5, 6):
            g.step(n)
            o.step(n)
            assert _worst(g, o, p["realizations"]) <= TOL[p["precision"]], (p["nl"], p["n"], variant)
        g.close()


@pytest.mark.parametrize("p", [W.model_b([128, 64], realizations=5), W.kpz([64, 128], realizations=2, ic_kind=1, ic_sigma=0.2),
                               W.model_b([128, 32], precision=64, realizations=3, history_readback=1),
                               W.model_a([32, 128], precision=64, realizations=4)])
def test_real_fields_split_over_two_streams(p, monkeypatch):
    """Bitwise the trajectory of one stream, and the observables after it agree
    to the rounding of their FP64 atomic sums."""
    S = _setd()
    monkeypatch.setenv("SETD_VARIANT", "1,4,1")
    one = S.Plan(p)
    monkeypatch.setenv("SETD_SPLIT", "2")
    two = S.Plan(p)
    assert int(one.info.streams) == 1 and int(two.info.streams) == 2
    assert int(one.info.passes_per_step) == int(two.info.passes_per_step) == 2
    for n in (7, 1, 12):
        one.step(n)
        two.step(n)
        assert np.array_equal(one.get_all(), two.get_all())
    assert np.allclose(one.observe(S.OBS_WIDTH), two.observe(S.OBS_WIDTH), rtol=1e-12, atol=0)
    one.close()
    two.close()


@pytest.mark.parametrize("split", ["1", "2"])
@pytest.mark.parametrize("p", [W.model_b([128, 64], realizations=5),
                               W.kpz([32, 128], precision=64, realizations=3, ic_kind=1, ic_sigma=0.2)])
def test_graph_replays_of_two_pass_steps(p, split, monkeypatch):
    """Replays of a captured graph of 4 steps, with eager steps, field reads and
    observables between them, give bitwise the eager trajectory."""
    S = _setd()
    monkeypatch.setenv("SETD_VARIANT", "1,4,1")
    monkeypatch.setenv("SETD_SPLIT", split)
    monkeypatch.setenv("SETD_GRAPH", "0")
    eager = S.Plan(p)
    monkeypatch.setenv("SETD_GRAPH", "4")
    graph = S.Plan(p)
    assert int(eager.info.graph_steps) == 0 and int(graph.info.graph_steps) == 4
    for n in (8, 3, 4, 13, 1):
        eager.step(n)
        graph.step(n)
        assert np.array_equal(eager.get_all(), graph.get_all()), n
        assert np.allclose(eager.observe(S.OBS_WIDTH), graph.observe(S.OBS_WIDTH), rtol=1e-12, atol=0)
    eager.close()
    graph.close()


@pytest.mark.parametrize("kind,n", [("model_b", [128, 64]), ("kpz", [64, 128]), ("model_a", [128, 128])])
@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("history", [0, 1])
def test_set_state_and_step_index_on_two_passes(kind, n, prec, history):
    """A state set mid-run restarts its realization's history (F_{-1} = F_0),
    the other keeps its own; a set step index draws that step's noise; F_{n-1}
    is readable where it is stored."""
    S = _setd()
    p = getattr(W, kind)(n, precision=prec, realizations=2, order=2, history_readback=history, ic_kind=1, ic_sigma=0.1)
    g, o = S.Plan(p), O.Sim(p)
    assert int(g.info.passes_per_step) == 2

    def check(steps):
        for k in steps:
            g.step(k)
            o.step(k)
            assert _worst(g, o, 2) <= TOL[prec]
            if history:
                assert max(_err(g.history(r), o.get(r, which=1)) for r in range(2)) <= TOL[prec]

    check((1, 3))
    x = W.random_spectrum(p, 11, 0.05)
    g.set(1, x)
    o.set(1, x)
    check((1, 1, 5))
    g.set_step(1000)
    o.set_step(1000)
    check((1, 2))
    out = g.observe(S.OBS_STEP)
    assert out[0] == 1003 and out[1] == 0
    if not history:
        with pytest.raises(S.SetdError) as e:
            g.history(0)
        assert e.value.status == S.SETD_E_UNSUPPORTED
    g.close()


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("kind,n", [("kpz", [128, 64]), ("model_b", [64, 128])])
def test_carry_and_separate_storage_agree_on_two_passes(kind, n, prec):
    """The storages' trajectories agree to rounding, and reading phi from the
    carry plan leaves its trajectory bitwise unchanged."""
    S = _setd()
    base = getattr(W, kind)(n, precision=prec, realizations=2, ic_kind=1, ic_sigma=0.2)
    lean, sep, quiet = (S.Plan(dict(base, history_readback=h)) for h in (0, 1, 0))
    for _ in range(5):
        for g in (lean, sep, quiet):
            g.step(6)
        assert max(_err(lean.get(r), sep.get(r)) for r in range(2)) <= (1e-12 if prec == 64 else 2e-5)
    assert np.array_equal(quiet.get_all(), lean.get_all())
    for g in (lean, sep, quiet):
        g.close()


@pytest.mark.parametrize("kind,n,R,variant", [("cgl", [256, 512], 11, "1,12,1"), ("cgl", [512, 512], 8, "0,4,1"),
                                              ("model_b", [512, 256], 9, "1,12,1"), ("cgl", [256, 512], 11, "3,7,1")])
def test_large_double_precision_launches_repeat(kind, n, R, variant, monkeypatch):
    """FP64 SETD2 launches of more blocks than the chip holds at once, in calls
    of four and more steps, on one stream and in halves on two: the same bits
    in every run, and the oracle's trajectory (a few eps per transform stage and
    step)."""
    S = _setd()
    p = getattr(W, kind)(n, seed=77, realizations=R, precision=64, order=2)
    monkeypatch.setenv("SETD_VARIANT", variant)
    ref = None
    for split in ("1", "2", "2", "1", "2"):
        monkeypatch.setenv("SETD_SPLIT", split)
        g = S.Plan(p)
        assert int(g.info.streams) == int(split)
        g.step(4)
        a = g.get_all()
        g.step(5)
        b = g.get_all()
        g.close()
        if ref is None:
            ref = a, b
            for r in (0, R // 2, R - 1):
                o = O.Sim(p, r_first=r, r_count=1)
                o.step(4)
                assert _err(a[r], o.get(0)) <= 1e-12
        assert np.array_equal(a, ref[0]) and np.array_equal(b, ref[1])


@pytest.mark.parametrize("p", [W.model_a([512, 512], nl="none", order=2, precision=64, realizations=24, seed=5),
                               W.cgl([64, 64, 64], nl="none", precision=64, realizations=12, seed=6),
                               W.model_b([512, 256], nl="none", precision=32, realizations=40, seed=7)])
def test_large_linear_launches_repeat(p):
    """Linear plans advance by counting the blocks of their one pass: launches
    of many more blocks than the chip holds draw every mode's noise at the same
    step, the same bits in every run and the oracle's trajectory."""
    S = _setd()
    R, ref = p["realizations"], None
    for _ in range(4):
        g = S.Plan(p)
        g.step(1)
        g.step(5)
        a = g.get_all()
        out = g.observe(S.OBS_STEP)
        g.close()
        assert out[0] == 6 and out[1] == 0
        if ref is None:
            ref = a
            for r in (0, R // 2, R - 1):
                o = O.Sim(p, r_first=r, r_count=1)
                o.step(6)
                assert _err(a[r], o.get(0)) <= (1e-12 if p["precision"] == 64 else 2e-5)
        assert np.array_equal(a, ref)


@pytest.mark.parametrize("kind", ["cgl", "model_b"])
def test_long_double_precision_runs_repeat(kind, monkeypatch):
    """FP64 SETD2 steps on a full chip: the same bits after 3000 steps in every
    run, on one stream and in halves on two.  (With store data overwritten too
    early, one or more of a hundred calls of four such steps was wrong.)"""
    S = _setd()
    p = getattr(W, kind)([256, 1024], seed=77, realizations=11, precision=64, order=2)
    monkeypatch.setenv("SETD_VARIANT", "1,12,1")
    ref = None
    for split in ("2", "1", "2", "2"):
        monkeypatch.setenv("SETD_SPLIT", split)
        g = S.Plan(p)
        g.step(3000)
        a = g.get_all()
        g.close()
        ref = a if ref is None else ref
        assert np.isfinite(a.view(np.float64)).all()
        assert np.array_equal(a, ref)
