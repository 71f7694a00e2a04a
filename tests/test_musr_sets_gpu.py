"""A parameter set's value has the same bits whichever call evaluates it: alone
with the parameters by value, alone in a batch, in a batch of any size and
place.  The counts include some outside the fast terms' range (negative, and
for the likelihood a tiny one: its chi-square term would be all of the sum),
because the choice between the two forms of a term must not depend on the
launch either."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def dks():
    from paper_1509_07685_amd import dks as mod
    return mod


@pytest.mark.parametrize("stat", ["chisq", "mle"])
@pytest.mark.parametrize("n_det,n_bins", [(1, 300), (3, 70_000), (6, 5000), (16, 777), (18, 6256), (24, 40_000),
                                          (32, 4096), (16, 66_000)])
def test_same_bits_in_every_call(n_det, n_bins, stat):
    sets = 40
    g = np.random.default_rng(n_det + n_bins)
    d = g.poisson(3.0, (n_det, n_bins)).astype(np.float64)
    d[n_det // 2, 7], d[n_det - 1, n_bins - 1], d[0, 100] = -3.0, 1e-300 if stat == "mle" else -1.0, 0.25
    P = np.empty((sets, 2 + 4 * n_det))
    P[:, 0], P[:, 1] = g.uniform(0.2, 0.5, sets), g.uniform(60.0, 120.0, sets)
    P[:, 2:] = np.stack([g.uniform(3, 5, (sets, n_det)), g.uniform(0.1, 0.5, (sets, n_det)),
                         g.uniform(0.1, 0.3, (sets, n_det)), g.uniform(-7, 7, (sets, n_det))], 2).reshape(sets, -1)
    dev = torch.from_numpy(P).cuda()
    fit = dks().MusrFit(torch.from_numpy(d).cuda(), 8.0 / n_bins, max_sets=sets)
    every = fit.eval_batch(stat, dev).cpu().numpy()
    assert np.isfinite(every).all()
    for first, count in ((0, 1), (1, 2), (3, 5), (11, 9), (20, 17), (7, 33)):
        part = fit.eval_batch(stat, dev[first:first + count].contiguous()).cpu().numpy()
        assert np.array_equal(part, every[first:first + count]), (first, count)
    few = dks().MusrFit(torch.from_numpy(d).cuda(), 8.0 / n_bins)
    for k in (0, 13, 39):
        assert fit(stat, P[k]) == few(stat, P[k]) == every[k], k
