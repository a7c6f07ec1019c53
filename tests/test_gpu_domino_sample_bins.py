"""Samples taken inside the launches into bins of many sizes, against the
oracle's counts: runs of sites that end with a bin's column, its row, a word or
the row of sites, bins summed in LDS and bins too many for it, one bin for the
whole diamond."""
import pytest

import oracle
from gpu_helpers import need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bin_", [1, 2, 3, 5, 16, 31, 32, 33, 64, 127, 1 << 30])
@pytest.mark.parametrize("n", [1, 5, 32, 33, 64, 100, 127, 128])
def test_bins(n, bin_):
    tl = need_gpu()
    say("domino samples n=%d bin=%d" % (n, bin_))
    s = tl.Sampler(tl.domain(tl.TL_DOMINO, n=n), tl.weights(tl.TL_W_UNIFORM), 7 + n,
                   tl.options(obs_every=2, obs_bin=bin_))
    o = oracle.DominoOracle(n, oracle.table_from_ratios(oracle.domino_ratios(), False), seed=7 + n, obs_every=2,
                            bin_=bin_)
    for k in (5, 40):
        s.sweep(k)
        o.sweep(k)
        obs = s.observables()
        assert obs["samples"] == int(o.samples[0])
        assert (obs["bin_sum"].reshape(-1) == o.bin_sum).all(), "after %d sweeps" % o.t
