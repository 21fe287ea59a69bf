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
