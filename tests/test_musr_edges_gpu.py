"""Edges of the fit statistic's evaluation: runs of parameter sets and groups
of detectors at their limits, and counts and models outside the range of the
reciprocal-based terms (zero, negative, tiny, huge, not finite), whose terms
must be the ones written in the definition.

Tolerance 1e-12 relative against the exactly rounded oracle, as for the other
shapes (the terms are good to a few ulp and of one sign on average)."""

import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import musr_oracle as mo  # noqa: E402

pytestmark = pytest.mark.gpu


def dks():
    from paper_1509_07685_amd import dks as mod
    return mod


def params(n_det, seed, sets=1):
    g = np.random.default_rng(seed)
    p = np.empty((sets, 2 + 4 * n_det))
    p[:, 0], p[:, 1] = g.uniform(0.2, 0.5, sets), g.uniform(60.0, 120.0, sets)
    p[:, 2:] = np.stack([g.uniform(3, 5, (sets, n_det)), g.uniform(0.1, 0.5, (sets, n_det)),
                         g.uniform(0.1, 0.3, (sets, n_det)), g.uniform(0, 6.28, (sets, n_det))], 2).reshape(sets, -1)
    return p


@pytest.mark.parametrize("stat", ["chisq", "mle"])
@pytest.mark.parametrize("n_det,n_bins,sets", [(1, 1, 2), (4, 255, 8), (5, 257, 9), (16, 256, 17), (17, 300, 3),
                                               (20, 140_000, 40), (32, 1000, 133)])
def test_runs_and_groups(n_det, n_bins, sets, stat):
    d = np.random.default_rng(n_bins).poisson(3.0, (n_det, n_bins)).astype(np.float64)
    dt = 7.0 / n_bins
    P = params(n_det, n_det + sets, sets)
    fit = dks().MusrFit(torch.from_numpy(d).cuda(), dt, max_sets=sets)
    got = fit.eval_batch(stat, torch.from_numpy(P).cuda()).cpu().numpy()
    for k in sorted({0, sets // 2, sets - 1}):
        ref = mo.evaluate(stat, d, P[k], dt)
        assert abs(got[k] - ref) <= 1e-12 * abs(ref), k
        assert abs(fit(stat, P[k]) - ref) <= 1e-12 * abs(ref), k


@pytest.mark.parametrize("stat", ["chisq", "mle"])
@pytest.mark.parametrize("what", [0.0, -2.0, 5e-310, 1e-300, 1e300, math.inf, -math.inf, math.nan, "N0", "Nneg"])
def test_terms_out_of_range_follow_the_definition(what, stat):
    n_det, n_bins = 6, 300
    dt = 7.0 / n_bins
    d = np.random.default_rng(8).poisson(3.0, (n_det, n_bins)).astype(np.float64)
    p = params(n_det, 9)[0]
    if what == "N0":            # a detector whose model is 0 in every bin
        p[2 + 4 * 2:2 + 4 * 2 + 3] = 0.0
    elif what == "Nneg":        # ... and one whose model is negative
        p[2 + 4 * 2:2 + 4 * 2 + 3] = (-1.0, 0.0, 0.0)
    else:
        d[2, 5] = d[5, 299] = what
    with np.errstate(all="ignore"):
        t = mo.chisq_terms(d, mo.model(p, n_det, n_bins, dt)) if stat == "chisq" else \
            mo.mle_terms(d, mo.model(p, n_det, n_bins, dt))
        ref = float(np.sum(t))
    fit = dks().MusrFit(torch.from_numpy(d).cuda(), dt, max_sets=3)
    got = [fit(stat, p)] + fit.eval_batch(stat, torch.from_numpy(np.tile(p, (3, 1))).cuda()).cpu().tolist()
    for v in got:
        if math.isnan(ref) or math.isinf(ref):
            assert (math.isnan(v) and math.isnan(ref)) or v == ref
        else:
            assert abs(v - ref) <= 1e-12 * abs(ref)
