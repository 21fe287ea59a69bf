"""Kernels and dispatch branches of their own, at the sizes where they can go
wrong, against the FP64 oracle."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2511_22510_amd import workloads as W

pytestmark = pytest.mark.gpu


def _setd():
    from paper_2511_22510_amd import setd
    return setd


def _line(n, kind, **kw):
    if kind == "cgl":
        return W.cgl([n], **dict(dict(ic_sigma=0.3), **kw))
    return W.kpz([n], **dict(dict(ic_kind=1, ic_sigma=0.3, nu=1.0, lam=3.0, h=1e-3), **kw))


@pytest.mark.parametrize("n,kind,prec,R,dealias", [
    (8, "kpz", 64, 1, 1), (16, "cgl", 64, 5, 1), (32, "kpz", 32, 3, 0), (64, "cgl", 64, 2, 0), (64, "kpz", 64, 4, 1),
    (128, "kpz", 64, 7, 2), (128, "cgl", 32, 3, 2), (256, "kpz", 32, 9, 1), (512, "cgl", 64, 2, 1),
    (1024, "kpz", 64, 3, 0), (1024, "cgl", 32, 1, 1), (8, "kpz", 32, 4099, 1)])
def test_line_box_widths(n, kind, prec, R, dealias):
    """Every line length of the pairwise class sums (one wavefront per line:
    shorter and longer than a wavefront, more lines than wavefronts). The
    FP64 sums of both sides differ by rounding: w^2 is a difference of sums of
    about 2 N values, so 1e-10 relative covers FP64 states; an FP32 state is
    1e-6 off after a few steps, 2e-4 the bar of the workloads."""
    S = _setd()
    p = _line(n, kind, precision=prec, realizations=R, dealias=dealias, seed=7)
    g, o = S.Plan(p), O.Sim(p)
    g.step(3)
    o.step(3)
    a, b = g.box_width(), o.observe(O.OBS_BOXWIDTH)
    assert len(a) == len(b) == n.bit_length() - 1
    assert float(np.max(np.abs(a - b) / b)) <= (1e-10 if prec == 64 else 2e-4)
    g.close()


def _trajectory_error(g, o, R, steps):
    worst = 0.0
    for n in steps:
        g.step(n)
        o.step(n)
        for r in range(R):
            a, b = g.get(r), o.get(r)
            worst = max(worst, float(np.linalg.norm(a - b) / np.linalg.norm(b)))
    return worst


@pytest.mark.parametrize("n,R", [((32, 32, 32), 3), ((64, 32, 64), 2), ((32, 64, 128), 1), ((128, 128, 32), 1),
                                 ((32, 256, 64), 1), ((256, 32, 128), 1), ((64, 128, 256), 1)])
def test_two_pass_3d_step(n, R):
    """The 3D complex step with the axis-1 transform split between two passes,
    every axis length of its rule (1 to 8 x 32 along axis 1) and unequal axes:
    steps, the recovered state, a set state (restarted history) and a set step
    index follow the oracle to the FP32 bar of the workloads."""
    S = _setd()
    p = W.cgl(list(n), realizations=R, seed=11, ic_sigma=0.2)
    g, o = S.Plan(p), O.Sim(p)
    assert int(g.info.passes_per_step) == 2
    assert float(np.linalg.norm(g.get(0) - o.get(0)) / np.linalg.norm(o.get(0))) <= 2e-4
    assert _trajectory_error(g, o, R, (1, 2, 5)) <= 2e-4
    x = W.random_spectrum(p, 5, scale=float(np.sqrt(np.prod(n))))
    g.set(R - 1, x)
    o.set(R - 1, x)
    g.set_step(40)
    o.set_step(40)
    assert _trajectory_error(g, o, R, (1, 3)) <= 2e-4
    g.close()


@pytest.mark.parametrize("n,R", [((64, 64, 64), 6), ((32, 64, 128), 6), ((64, 128, 32), 9), ((128, 256, 32), 5),
                                 ((256, 64, 32), 3)])
def test_two_pass_3d_step_is_the_same_in_any_batch(n, R):
    """Launches that leave the chip idle take the lines of a block side by side
    and others in turn: a realization's bits do not depend on which."""
    S = _setd()
    one, many = S.Plan(W.cgl(list(n), seed=13, ic_sigma=0.3)), S.Plan(W.cgl(list(n), seed=13, ic_sigma=0.3, realizations=R))
    for _ in range(3):
        one.step(3)
        many.step(3)
        assert np.array_equal(one.get(0), many.get(0))
    one.close()
    many.close()


@pytest.mark.parametrize("n,kw", [((16, 32, 32), {}), ((32, 32, 512), {}), ((32, 32, 32), dict(precision=64)),
                                  ((32, 32, 32), dict(history_readback=1)), ((32, 32, 32), dict(order=1)),
                                  ((32, 32, 32), dict(dealias=0)), ((32, 32, 32), dict(noise_space=1))])
def test_general_3d_step_beside_the_rule(n, kw):
    """3D complex plans that the two-pass rule does not take keep the four
    passes and follow the oracle."""
    S = _setd()
    p = W.cgl(list(n), seed=12, ic_sigma=0.2, **kw)
    g, o = S.Plan(p), O.Sim(p)
    assert int(g.info.passes_per_step) == 4
    assert _trajectory_error(g, o, 1, (1, 3)) <= (1e-10 if p["precision"] == 64 else 2e-4)
    g.close()


@pytest.mark.parametrize("n", [(64, 64), (64, 32), (32, 64), (32, 32)])
@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("kind", ["a1", "b2", "kpz1", "kpz2", "b2h"])
def test_small_lattice_kernel(n, prec, kind):
    """Whole steps of 2D lattices of 32 and 64 points per axis in one kernel,
    each with SETD1, the SETD2 carry and the separate SETD2 storage: steps over
    several calls, a call of more steps than one launch takes (300), a set
    state (restarted history) and a set step index follow the oracle to the
    bars of the workloads."""
    S = _setd()
    kw = dict(precision=prec, realizations=2, seed=21, order=1 if kind.endswith("1") else 2,
              history_readback=1 if kind == "b2h" else 0)
    if kind.startswith("kpz"):
        p = W.kpz(list(n), ic_kind=1, ic_sigma=0.2, **kw)
    else:
        p = (W.model_a if kind[0] == "a" else W.model_b)(list(n), **kw)
    tol = 1e-10 if prec == 64 else 2e-4
    g, o = S.Plan(p), O.Sim(p)
    assert int(g.info.passes_per_step) == 1
    assert _trajectory_error(g, o, 2, (1, 2, 7)) <= tol
    x = W.random_spectrum(p, 5, 0.05)
    g.set(1, x)
    o.set(1, x)
    assert _trajectory_error(g, o, 2, (1, 4)) <= tol
    if kind == "b2h":
        assert float(np.linalg.norm(g.history(1) - o.get(1, which=1))) <= tol * float(np.linalg.norm(o.get(1, which=1)))
    g.set_step(1000)
    o.set_step(1000)
    assert _trajectory_error(g, o, 2, (3, 300)) <= (1e-9 if prec == 64 else 2e-4)
    out = g.observe(S.OBS_STEP)
    assert out[0] == 1303 and out[1] == 0
    g.close()


def test_small_lattice_jobs_take_their_own_steps():
    """Jobs of one small launch class with different step counts share the
    launches of a tick, each bitwise its solo run."""
    S = _setd()
    jobs = [(W.model_b([64, 64], realizations=3, seed=31), 40), (W.model_b([64, 64], realizations=1, seed=32), 7),
            (W.model_a([64, 64], order=2, precision=32, seed=33), 300)]
    srv = S.Server(64 << 20)
    ids = [srv.submit(p, k) for p, k in jobs]
    srv.drain()
    for j, (p, k) in zip(ids, jobs):
        solo = S.Plan(p)
        solo.step(k)
        for r in range(p["realizations"]):
            assert np.array_equal(srv.get(j, r), solo.get(r))
        solo.close()
    srv.close()


@pytest.mark.parametrize("p,M,calls", [
    (W.model_a([64], precision=64, realizations=2101, seed=41, dx=0.5), 64, (10, 53)),
    (W.model_a([8], precision=32, realizations=4099, seed=42, order=2), 8, (7,)),
    (W.cgl([32], precision=32, realizations=3, seed=43, ic_sigma=0.3), 512, (300, 211)),
    (W.model_b([32, 64], precision=64, realizations=3, seed=44), 16, (1, 14)),
    (W.model_a([64, 64], precision=32, realizations=2, seed=45, order=2, history_readback=1), 8, (7,)),
    (W.kpz([32, 32], precision=32, realizations=9, seed=46, ic_kind=1, ic_sigma=0.2), 32, (20, 20)),
])
def test_windows_recorded_by_the_step_kernels(p, M, calls):
    """Windows whose samples the line and small-lattice kernels store
    themselves, filled over several calls (the last one past its end, a window
    longer than a launch's 256 steps among them), and their sums over several
    realizations per block: C, chi and the FDT deviation against the oracle, to
    the bars of the workloads (the sums are means over thousands of values of
    both signs, compared to the largest one)."""
    S = _setd()
    p = dict(p, series_len=M)
    g, o = S.Plan(p), O.Sim(p)
    g.step(2)
    o.step(2)
    g.observe(S.OBS_SERIES_START)
    o.series_start(M)
    for n in calls:
        g.step(n)
        o.step(n)
    tol = 1e-10 if p["precision"] == 64 else 2e-4
    got = g.observe(S.OBS_SPECTRUM) if p["n"][0] == p["n"][-1] else None
    if got is not None:
        C, xr, xi, cnt = g.spectrum()
        oC, oxr, oxi, ocnt = o.spectrum()
        assert np.array_equal(cnt, ocnt)
        for a, b in ((C, oC), (xr, oxr), (xi, oxi)):
            assert float(np.max(np.abs(a - b))) <= tol * float(np.max(np.abs(b)))
    a, b = g.fdt(), o.fdt()
    assert abs(a[0] - b[0]) <= (1e-10 if p["precision"] == 64 else 1e-3) * b[0]
    assert abs(a[1] - b[1]) <= (1e-10 if p["precision"] == 64 else 1e-3) * b[0]
    for r in range(min(3, p["realizations"])):
        assert float(np.linalg.norm(g.get(r) - o.get(r))) <= tol * float(np.linalg.norm(o.get(r)))
    g.close()


@pytest.mark.parametrize("p", [
    W.cgl([128, 128, 128], seed=51), W.cgl([64, 64, 64], seed=52, realizations=2),
    W.cgl([64, 256, 128], seed=53), W.cgl([512, 512], seed=54, precision=64, dealias=0, history_readback=1),
    W.model_a([256, 128, 128], seed=55, precision=32), W.kpz([1024, 512], seed=56, ic_kind=1, ic_sigma=0.2),
    W.model_a([64, 512], seed=57, precision=64), W.cgl([1024], seed=58), W.model_a([8, 16], seed=59)])
def test_read_out_matches_the_device_unpack(p, monkeypatch):
    """The host read-out (planes scattered by several threads through a pinned
    buffer for large fields, the whole block on one thread for small ones)
    gives bitwise what the device unpacks for setd_run_noalloc: every lattice
    dimension, field type and dealiasing rule, removed modes zero over a
    buffer that was not.  (setd_run_noalloc steps with the default kernel
    variants, whose rounding differs from some tuned ones', so the plan does
    too.)"""
    S = _setd()
    monkeypatch.setenv("SETD_AUTOTUNE", "0")
    g = S.Plan(p)
    g.step(3)
    ref = S.run_noalloc(p, 3)
    import ctypes
    for r in range(p["realizations"]):
        buf = np.full(2 * g.nspec + 4, np.nan)
        S._check(g.lib, g.lib.setd_get_field(g.h, r, buf.ctypes.data_as(S._D), 2 * g.nspec))
        assert np.isnan(buf[2 * g.nspec:]).all()
        assert np.array_equal(buf[:2 * g.nspec].view(np.complex128).reshape(ref[r].shape), ref[r])
    if p.get("history_readback") and p["order"] == 2:
        assert np.isfinite(g.history(0)).all()
    g.close()


@pytest.mark.parametrize("n,large,model,order,precision,dealias", [
    (64, 16390, "model_a", 1, 32, 1), (64, 16390, "kpz", 2, 32, 2), (512, 2054, "model_b", 2, 32, 0),
    (512, 2054, "kpz", 2, 64, 1), (128, 8198, "model_a", 2, 64, 2)])
def test_lines_draw_in_a_second_wavefront_alike(n, large, model, order, precision, dealias):
    """A line's steps have the same bits whether its noise is drawn by a
    wavefront of its own (launches of at most 1024 line wavefronts) or not."""
    out = []
    for R in (4, large):
        pl = _setd().Plan(getattr(W, model)([n], seed=9, realizations=R, precision=precision, order=order,
                                            dealias=dealias, ic_kind=1, ic_sigma=0.2))
        pl.step(1)
        pl.step(2)
        pl.step(37)
        out.append([pl.get(r) for r in range(4)])
        pl.close()
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("n,R", [((256, 512), 11), ((512, 512), 8)])
def test_late_blocks_of_a_launch_take_the_same_step(n, R):
    """The row pass begins a step and the axis-0 pass only reads it: whichever
    blocks of a launch larger than the chip run last, every realization takes
    its first SETD2 step as the oracle does (a few eps per transform stage and
    step) and with the same bits each time."""
    S = _setd()
    p = W.cgl(list(n), seed=77, realizations=R, precision=64)
    g, o = S.Plan(p), O.Sim(p)
    assert _trajectory_error(g, o, R, (1, 2)) <= 1e-12
    a = g.get_all()
    g.close()
    for _ in range(3):
        g = S.Plan(p)
        g.step(1)
        g.step(2)
        assert np.array_equal(g.get_all(), a)
        g.close()


@pytest.mark.parametrize("variant", ["0,12,0", "1,12,0", "1,15,0"])
@pytest.mark.parametrize("kind", ["model_a", "model_b", "kpz"])
def test_one_column_axis_0_tiles(kind, variant, monkeypatch):
    """FP64 lines of 1024 rows have axis-0 tiles of a single column (the
    quarter-width variants), where the Hermitian column's state and SETD2 carry
    lie in lines of their own in LDS: the trajectory follows the oracle to the
    FP64 bar, with the carry alone and with both arrays stored."""
    S = _setd()
    monkeypatch.setenv("SETD_VARIANT", variant)
    for history in (0, 1):
        p = getattr(W, kind)([1024, 32], seed=31, realizations=2, precision=64, order=2, ic_kind=1, ic_sigma=0.2,
                             history_readback=history)
        g, o = S.Plan(p), O.Sim(p)
        assert _trajectory_error(g, o, 2, (1, 1, 4, 6)) <= 1e-10
        g.close()


@pytest.mark.parametrize("p,streams", [(W.model_b([64, 64], realizations=5), 2), (W.kpz([32, 64], realizations=2, ic_kind=1, ic_sigma=0.2), 2),
                                       (W.model_b([128, 32], realizations=5), 2), (W.model_a([64, 64], realizations=1), 1),
                                       (W.kpz([256], realizations=6, ic_kind=1, ic_sigma=0.2), 1), (W.cgl([64], realizations=3), 1)])
def test_reported_streams_are_those_of_the_steps(p, streams, monkeypatch):
    """With the split pinned, the record says two streams where the steps run
    in halves on two and one where they cannot; the bits do not depend on it,
    launches of 256 steps and a remainder included."""
    S = _setd()
    monkeypatch.setenv("SETD_VARIANT", "1,4,1")
    one = S.Plan(p)
    monkeypatch.setenv("SETD_SPLIT", "2")
    two = S.Plan(p)
    assert int(one.info.streams) == 1 and int(two.info.streams) == streams
    for n in (5, 3, 300):
        one.step(n)
        two.step(n)
        assert np.array_equal(one.get_all(), two.get_all())
    one.close()
    two.close()


@pytest.mark.parametrize("p,arrays", [(W.model_b([64, 32], realizations=3), 1), (W.kpz([64, 64], ic_kind=1), 2),
                                      (W.model_a([32, 64], order=2, precision=64, history_readback=1), 1)])
def test_bytes_of_a_small_lattice_launch(p, arrays):
    """A one-step launch of a small lattice reads and writes its axis-0
    intermediate (n_0 rows of the stored columns; KPZ two of them) and its
    state, with the separate SETD2 storage F_{n-1} too."""
    g = _setd().Plan(p)
    info = g.info
    n0, n1 = p["n"]
    kc = (n1 - 1) // 3 + 1
    modes = (2 * ((n0 - 1) // 3) + 1) * kc
    val = p["precision"] // 4 * p["realizations"]
    want = 2 * val * (arrays * n0 * kc + (2 if p.get("history_readback") else 1) * modes)
    assert list(info.pass_bytes) == [want, 0, 0, 0] and info.alg_bytes_per_step == want
    g.close()


@pytest.mark.parametrize("n,prec,dealias,kw", [(8, 64, 1, {}), (64, 32, 0, {}), (256, 64, 1, {}), (256, 32, 2, {}), (512, 64, 2, {}),
                                               (1024, 32, 1, {}), (1024, 64, 0, {}), (128, 64, 1, dict(nl="none")), (64, 32, 0, dict(nl="none", order=1))])
def test_open_window_leaves_complex_lines_alike(n, prec, dealias, kw):
    """Complex lines record an open window in an instantiation of their own: a
    trajectory has the same bits with and without the window, before, during and
    after it, and the window's correlations are the oracle's."""
    S = _setd()
    p = W.cgl([n], precision=prec, dealias=dealias, realizations=5, seed=61, ic_sigma=0.3, **kw)
    plain, rec = S.Plan(p), S.Plan(dict(p, series_len=8))
    for g in (plain, rec):
        g.step(3)
    rec.observe(S.OBS_SERIES_START)
    for k in (2, 1, 9, 4):
        plain.step(k)
        rec.step(k)
        assert np.array_equal(plain.get_all(), rec.get_all())
    o = O.Sim(p)
    o.step(3)
    o.series_start(8)
    o.step(16)
    C, xr, xi, cnt = rec.spectrum()
    oC, oxr, oxi, ocnt = o.spectrum()
    tol = 1e-10 if prec == 64 else 2e-4
    assert np.array_equal(cnt, ocnt)
    for a, b in ((C, oC), (xr, oxr), (xi, oxi)):
        assert float(np.max(np.abs(a - b))) <= tol * float(np.max(np.abs(b)))
    plain.close()
    rec.close()


@pytest.mark.parametrize("n,p", [(256, W.model_a([256], h=1e-3)), (1024, W.kpz([1024], h=1e-3)), (1024, W.cgl([1024], dealias=0)),
                                 (64, W.model_b([64], h=1e-4, dealias=2)), (1024, W.model_a([1024], nl="none", h=1e-3, order=2)),
                                 (512, W.cgl([512], nl="none"))])
def test_lines_keep_small_single_precision_states(n, p):
    """A line's state is held as it is stored: modes near the smallest normal
    single-precision numbers (1.2e-38) evolve with a float's relative precision
    (at most four roundings of 2^-24 a step), no bits lost to a scaled copy."""
    S = _setd()
    p = dict(p, precision=32, realizations=2, noise_D=0.0, ic_kind=0)
    g, o = S.Plan(p), O.Sim(p)
    rng = np.random.default_rng(5)
    shape = W.spectral_shape(p)
    for r in range(2):
        x = 3e-37 * np.exp(2j * np.pi * rng.random(shape)) * (1.0 + rng.random(shape))
        if not p["complex_field"]:
            x[0] = x[0].real
            x[-1] = x[-1].real
        x = x.astype(np.complex64).astype(np.complex128)
        g.set(r, x)
        o.set(r, x)
    steps = 12
    g.step(steps)
    o.step(steps)
    for r in range(2):
        a, b = g.get(r), o.get(r)
        m = np.abs(b) > 1e-37
        assert m.sum() > n // 8
        assert float(np.max(np.abs(a - b)[m] / np.abs(b)[m])) <= (4 * steps + 2) * 2.0 ** -24
    g.close()


@pytest.mark.parametrize("kind,kw", [("model_a", dict(nl="none", noise_space=1)), ("model_a", dict(nl="none", noise_space=1, dealias=0)),
                                     ("model_a", dict(nl="none")), ("cgl", dict(nl="none")), ("kpz", dict(noise_space=1))])
@pytest.mark.parametrize("prec", [64, 32])
def test_lines_of_two_wavefronts_in_any_block(kind, kw, prec):
    """Lines of 1024 sites take blocks of one or two lines by what their steps
    do and how many there are (one, a part and most of a wavefront per SIMD,
    more): a realization's bits do not depend on it, and follow the oracle.
    (Real lines pair realizations 2l and 2l + 1 in one transform, so the last of
    an odd count has other roundings: the first pair is compared.)"""
    S = _setd()
    out = []
    for R in (3, 511, 515, 1024, 1030):
        p = dict(getattr(W, kind)([1024], precision=prec, realizations=R, order=2, seed=71, ic_kind=1, ic_sigma=0.2), **kw)
        g = S.Plan(p)
        g.step(2)
        g.step(9)
        out.append([g.get(r) for r in range(2)])
        if R == 515:
            for r in (0, 513, 514):
                o = O.Sim(p, r_first=r, r_count=1)
                o.step(11)
                assert float(np.linalg.norm(g.get(r) - o.get(0))) <= (1e-10 if prec == 64 else 2e-4) * float(np.linalg.norm(o.get(0)))
        g.close()
    for b in out[1:]:
        for x, y in zip(out[0], b):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("n,prec,kind,limit", [((32, 32), 64, "model_b", 3072), ((32, 32), 32, "model_a", 5120), ((64, 32), 32, "kpz", 2048),
                                               ((32, 64), 32, "model_b", 3072), ((64, 64), 32, "model_b", None)])
def test_many_realizations_of_a_small_lattice_take_two_passes(n, prec, kind, limit):
    """Up to a number of realizations a small lattice steps in one kernel, above
    it (never at 64 x 64) in two passes: both follow the oracle, from the first
    realization to the last."""
    S = _setd()
    for R in ((limit, limit + 1) if limit else (6000,)):
        p = getattr(W, kind)(list(n), precision=prec, realizations=R, order=2, seed=81, ic_kind=1, ic_sigma=0.2)
        g = S.Plan(p)
        assert int(g.info.passes_per_step) == (2 if limit and R > limit else 1)
        g.step(1)
        g.step(6)
        for r in (0, R // 2, R - 1):
            o = O.Sim(p, r_first=r, r_count=1)
            o.step(7)
            assert float(np.linalg.norm(g.get(r) - o.get(0))) <= (1e-10 if prec == 64 else 2e-4) * float(np.linalg.norm(o.get(0)))
        g.close()


def test_small_lattice_jobs_keep_the_path_of_their_own_plan():
    """Jobs of one lattice whose plans take different paths (few and many
    realizations) run side by side in a server, each bitwise its solo run."""
    S = _setd()
    jobs = [(W.model_b([32, 32], realizations=3, seed=91), 60), (W.model_b([32, 32], realizations=5121, seed=92), 40),
            (W.model_b([32, 32], realizations=2, seed=93), 25)]
    srv = S.Server(512 << 20)
    ids = [srv.submit(p, k) for p, k in jobs]
    srv.drain()
    for j, (p, k) in zip(ids, jobs):
        solo = S.Plan(p)
        solo.step(k)
        for r in (0, p["realizations"] // 2, p["realizations"] - 1):
            assert np.array_equal(srv.get(j, r), solo.get(r))
        solo.close()
    srv.close()


SMALL_ROUTE = [(n, prec, kind, kw) for n, prec, kind, kw in [
    ((64, 64), 64, "kpz", {}), ((64, 64), 32, "model_b", {}), ((64, 64), 64, "model_a", dict(order=1)), ((32, 64), 64, "model_b", {}),
    ((64, 32), 32, "kpz", dict(history_readback=1)), ((32, 32), 32, "kpz", {}), ((32, 32), 64, "model_b", dict(history_readback=1)),
    ((32, 64), 32, "model_a", dict(order=1)), ((64, 32), 64, "kpz", dict(order=1)), ((64, 64), 32, "model_a", {}),
    ((32, 32), 32, "model_b", dict(order=1)), ((64, 64), 64, "model_b", dict(history_readback=1))]]


@pytest.mark.parametrize("n,prec,kind,kw", SMALL_ROUTE)
def test_small_lattice_calls_of_few_steps_have_the_same_bits(n, prec, kind, kw):
    """With many realizations a small lattice's calls of few steps take the two
    passes and longer ones the one kernel: a trajectory has the same bits
    however its steps are split over calls (a set state and a set step index
    among them), and those of a few realizations, which never take two passes."""
    S = _setd()
    kw = dict(dict(order=2), **kw)
    mk = lambda R: S.Plan(getattr(W, kind)(list(n), precision=prec, realizations=R, seed=95, ic_kind=1, ic_sigma=0.2, **kw))
    few, many, split = mk(3), mk(1500), mk(1500)
    x = W.random_spectrum(few.p, 5, 0.05)
    for part in range(3):
        few.step(14)
        many.step(14)
        for k in (1, 1, 2, 8, 1, 1):
            split.step(k)
        rs = (0, 1, 2)
        assert all(np.array_equal(few.get(r), many.get(r)) and np.array_equal(many.get(r), split.get(r)) for r in rs)
        assert all(np.array_equal(many.get(r), split.get(r)) for r in (700, 1499))
        for g in (few, many, split):
            if part == 0:
                g.set(1, x)
            else:
                g.set_step(500)
    for g in (few, many, split):
        g.close()


def test_threads_read_large_fields_of_one_plan():
    """Several host threads read the realizations of one plan at once (fields
    large enough to go through its pinned buffer): each gets its own."""
    from concurrent.futures import ThreadPoolExecutor
    g = _setd().Plan(W.cgl([128, 128, 128], realizations=6, seed=97, ic_sigma=0.3))
    g.step(2)
    want = [g.get(r) for r in range(6)]
    with ThreadPoolExecutor(6) as ex:
        for _ in range(4):
            got = list(ex.map(g.get, range(6)))
            assert all(np.array_equal(a, b) for a, b in zip(want, got))
    g.close()
