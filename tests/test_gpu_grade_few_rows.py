"""The FP64 grade product at the row counts where its blocks change (16, 32 and
64 rows): the same products in the same order whatever the block, so the
grades of a prefix of the rows are bitwise those of all rows, and they match
a plain product to 1e-12 of the sums' absolute terms."""
import numpy as np
import pytest
import torch

from paper_2304_13144_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("level,n_types,mode", [(8, 1, "full"), (16, 2, "linear"), (16, 2, "full")])
def test_prefixes_of_rows_grade_the_same(level, n_types, mode):
    m = api.Model.create(level, n_types, 2.0, 5.0)
    mm = m.m(mode)
    r = np.random.default_rng([level, 7])
    A = r.normal(size=(mm, mm)) + 3.0 * np.eye(mm)
    m.set_active_set(mode, A)
    Ai = m.get_active_set(mode)[1].cpu().numpy()
    N = 8193                                   # 64-row blocks
    rows = r.normal(size=(N, mm))
    cm = torch.zeros(api.row_stride(mm), N, dtype=torch.float64, device="cuda")
    cm[:mm] = torch.from_numpy(rows.T.copy()).cuda()
    full = {k: v.cpu().numpy() for k, v in api.grade_rows(m, cm, "fp64", mode).items()}
    C = np.abs(rows @ Ai)
    bound = 1e-12 * (np.abs(rows) @ np.abs(Ai)).max(axis=1)
    assert np.all(np.abs(full["gamma"] - C.max(axis=1)) <= bound)
    assert np.all(C.max(axis=1) - C[np.arange(N), full["argmax"]] <= bound)
    for n in (1, 15, 16, 17, 33, 4095, 4096, 4097, 8191, 8192):   # 16-row blocks, 32-row blocks from 4,097
        part = api.grade_rows(m, cm[:, :n].contiguous(), "fp64", mode)
        assert np.array_equal(part["gamma"].cpu().numpy(), full["gamma"][:n]), n
        assert np.array_equal(part["argmax"].cpu().numpy(), full["argmax"][:n]), n
