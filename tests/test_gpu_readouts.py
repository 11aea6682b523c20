"""Initial counts, counts and histograms at the sizes where their kernels
change: replicas below and past one sweep of the histogram's workgroups,
molecules at the edges of a draw's words, bins at every size of the division
that a multiplication stands for."""

import numpy as np
import pytest
import torch  # its HIP runtime is the one the library is to use

import paper_2412_16613_amd as bwg
from oracle import ssa
from workloads import frank_network, paper_network

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 31, 1025])
@pytest.mark.parametrize("n_tot", [1, 15, 16, 17, 63, 64, 65, 128, 200])
def test_multinomial_start(n_tot, M):
    ens = bwg.Ensemble(bwg.Network(paper_network(n_tot)), M, seed=3, net_id=9)
    ens.init(("multinomial",))
    np.testing.assert_array_equal(ens.read_counts().cpu().numpy(),
                                  ssa.init_multinomial(3, 9, 0, M, n_tot))
    events, real = ens.read_events()
    assert (events.cpu().numpy() == 0).all() and (real.cpu().numpy() == 0).all()


@pytest.mark.parametrize("n_tot,M", [(2, 511), (61, 513), (61, 512 * 512 + 77), (1024, 4000),
                                     (16383, 3000)])
def test_histogram_bins(n_tot, M):
    ens = bwg.Ensemble(bwg.Network(paper_network(n_tot)), M, seed=1, net_id=2)
    ens.init(("multinomial",)).step(min(50 * n_tot, 50000))
    counts = ens.read_counts().cpu().numpy()
    assert (counts.sum(axis=1) == n_tot).all()
    for n_bins in (1, 7, 256, 16384):
        np.testing.assert_array_equal(ens.histogram(n_bins).cpu().numpy(),
                                      ssa.ee_histogram(counts, n_tot, n_bins).astype(np.int64))


@pytest.mark.parametrize("M", [1, 64, 4097])
def test_all_of_one_kind(M):
    # every replica in the last bin, and in the first
    for c, b in (((61, 0, 0), 6), ((0, 61, 0), 0)):
        ens = bwg.Ensemble(bwg.Network(frank_network(61, k0=0.05)), M, seed=1, net_id=2)
        ens.init(("fixed", c))
        h = ens.histogram(7).cpu().numpy()
        assert h[b] == M and h.sum() == M
        events, _ = ens.read_events()
        assert (events.cpu().numpy() == 0).all()
