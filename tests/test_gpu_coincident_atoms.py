"""Two atoms in one place: the neighbor build reports them, and an evaluation that
is made all the same counts their pair as it counts any other in the energy and
in the rows (equal to the oracle's, FP64 bar 1e-10 of the largest), while their
forces, which have no direction, are not numbers in either precision."""
import numpy as np
import pytest

from oracle import mtp as om
from oracle import neighbors as onb
from paper_2304_13144_amd import api, synth

pytestmark = pytest.mark.gpu
R_CUT = 5.0


@pytest.mark.parametrize("lanes", ["2", "4", "8"])
@pytest.mark.parametrize("level,n_types", [(8, 1), (16, 2)])
def test_pair_at_distance_zero(monkeypatch, level, n_types, lanes):
    monkeypatch.setenv("MTP_LANES", lanes)
    r = np.random.default_rng([level, 9])
    pos, cell = synth.lattice("bcc", 3.3, (4, 4, 4))
    pos = pos + r.normal(0.0, 0.1, pos.shape)
    pos[7] = pos[30]
    c = synth.Config(pos, r.integers(0, n_types, len(pos)).astype(np.int32), cell)
    pot = om.Potential(level, n_types, 2.0, R_CUT)
    theta = 0.05 * synth.theta_normal(1, n_types, pot.n_lin, pot.n_rad)   # (FP32 holds the products at r = 0)
    m = api.Model.create(level, n_types, 2.0, R_CUT)
    m.set_params(theta)
    keep = m.kept_columns()
    m.set_active_set("full", np.eye(len(keep)))
    b = api.Batch([c])
    nb = api.Neighbors().build(m, b, max_nbrs=96, check_status=False)
    with pytest.raises(api.MtpError) as e:
        nb.status()
    assert e.value.status == "MTP_E_OVERLAP"
    pairs = onb.neighbors(c.pos, c.cell, c.pbc, R_CUT)
    E = om.energy_forces_stress(pot, theta, c.pos, c.types, c.cell, pairs)[0]
    rows = om.b_rows(pot, theta, c.pos, c.types, c.cell, pairs)[:, keep]
    ev = api.evaluate(m, b, nb, "fp64", "full")
    gr = api.grade(m, b, nb, "fp64", "full", rows=True)
    scale = np.abs(rows).max()
    assert np.abs(gr["rows"].cpu().numpy() - rows).max() <= 1e-10 * scale
    for g in (ev["gamma"], gr["gamma"]):   # the active set is the identity
        assert np.abs(g.cpu().numpy() - np.abs(rows).max(axis=1)).max() <= 1e-10 * scale
    for p in ("fp64", "mixed"):
        out = api.energy_forces_stress(m, b, nb, p)
        bar = 1e-10 if p == "fp64" else 1e-4
        assert abs(float(out["energy"][0]) - E) <= bar * np.abs(out["site_e"].cpu().numpy()).max()
        for F in (out["forces"], api.evaluate(m, b, nb, p, "full")["forces"]):
            bad = np.isnan(F.cpu().numpy()).any(axis=1)
            assert np.array_equal(np.flatnonzero(bad), [7, 30]), p
