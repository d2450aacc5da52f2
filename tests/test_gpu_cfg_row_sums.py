"""Configuration rows at the edges of the sums' chunks (64 atoms, 16 lanes, 4
configurations a block): each equals the sum of its atoms' rows.  A sum of n
FP64 terms in any order is off by at most n 2^-53 sum|x|, n <= 321 here (the
sum it is compared with likewise)."""
import numpy as np
import pytest

from paper_2304_13144_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[1], [64], [16, 48, 64], [1, 15, 16, 17, 0, 63, 64, 65], [128, 129, 2, 200, 321, 7]])
def test_rows_of_configurations_are_sums(sizes):
    r = np.random.default_rng(len(sizes))
    lat, cell = synth.lattice("bcc", 3.3, (6, 6, 6))
    cfgs = [synth.Config(lat[np.sort(r.permutation(len(lat))[:n])] + r.normal(0.0, 0.1, (n, 3)), np.zeros(n, np.int32),
                         cell) for n in sizes]
    m = api.Model.create(8, 1, 2.0, 5.0)
    m.set_params(synth.theta_normal(1, 1, m.info["n_lin"], m.info["n_rad"]))
    b = api.Batch(cfgs)
    nb = api.Neighbors().build(m, b, max_nbrs=80)
    for mode in ("full", "linear"):
        rows = api.b_rows(m, b, nb, np.arange(sum(sizes)), mode).cpu().numpy()
        got = api.cfg_rows(m, b, nb, "fp64", mode + "_cfg").cpu().numpy()
        ends = np.cumsum(sizes)
        for c, n in enumerate(sizes):
            part = rows[ends[c] - n:ends[c]]
            bound = 321 * 2.0 ** -53 * np.abs(part).sum(0)
            assert np.all(np.abs(got[c] - part.sum(0)) <= 2 * bound), (c, n)
