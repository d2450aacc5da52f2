"""Atoms hundreds of cells away from theirs: the neighbor build reports that their
image shifts do not fit, and the lists it made all the same have the neighbors
in the order they have with every atom at home (grouped by species), and give
its forces.  An image of 700 cells of 12 A rounds a position by 2^-40 A, far
less than the 1e-8 of the largest force that is asked for."""
import numpy as np
import pytest

from paper_2304_13144_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_types", [1, 2, 3, 4])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("reps", [(4, 4, 4), (13, 14, 15)])   # the one-launch build and the general one
def test_lists_of_far_images(n_types, axis, reps):
    r = np.random.default_rng([n_types, axis])
    pos, cell = synth.lattice("bcc", 3.3, reps)
    pos = (pos + r.normal(0.0, 0.1, pos.shape)) % np.diag(cell)
    types = r.integers(0, n_types, len(pos)).astype(np.int32)
    far = pos.copy()
    far[::2, axis] += np.rint(r.uniform(-700, 700, len(far[::2]))) * cell[axis, axis]
    m = api.Model.create(8, n_types, 2.0, 5.0)
    m.set_params(synth.theta_normal(1, n_types, m.info["n_lin"], m.info["n_rad"]))
    seen = []
    for x in (pos, far):
        b = api.Batch([synth.Config(x, types, cell)])
        nb = api.Neighbors().build(m, b, max_nbrs=64, check_status=False)
        if x is far:
            with pytest.raises(api.MtpError) as e:
                nb.status()
            assert e.value.status == "MTP_E_INVAL" and "image shift" in str(e.value)
        count, j, _ = (t.cpu().numpy() for t in nb.export(b))
        F = api.energy_forces_stress(m, b, nb)["forces"].cpu().numpy()
        seen.append((count, [j[i, :count[i]] for i in range(len(x))], F))
    assert np.array_equal(seen[0][0], seen[1][0])
    for a, b in zip(seen[0][1], seen[1][1]):
        assert np.array_equal(a, b)
    assert np.abs(seen[0][2] - seen[1][2]).max() <= 1e-8 * np.abs(seen[0][2]).max()
