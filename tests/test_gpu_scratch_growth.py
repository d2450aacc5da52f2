"""A call that is no larger than one made before finds its scratch in place: it is
captured without an eager run of its own, which fails if the library allocates
(allocating under capture is an error; outside of it, growing would free what a
captured graph still points to).  Replays equal the eager call that follows."""
import numpy as np
import pytest
import torch

from paper_2304_13144_amd import api, synth

pytestmark = pytest.mark.gpu


def _model(level, n_types):
    m = api.Model.create(level, n_types, 2.0, 5.0)
    m.set_params(synth.theta_normal(1, n_types, m.info["n_lin"], m.info["n_rad"]))
    k = m.m("full")
    m.set_active_set("full", np.eye(k) + 0.1 * np.random.default_rng(k).normal(size=(k, k)) / np.sqrt(k))
    return m


def _lists(m, n, n_types, seed):
    """n atoms of a displaced BCC cell with vacancies, and their lists."""
    r = np.random.default_rng([n, seed])
    reps = int(np.ceil((n / 2) ** (1 / 3)))
    pos, cell = synth.lattice("bcc", 3.3, (reps, reps, reps))
    pos = pos[np.sort(r.permutation(len(pos))[:n])] + r.normal(0.0, 0.1, (n, 3))
    b = api.Batch([synth.Config(pos, r.integers(0, n_types, n).astype(np.int32), cell)])
    return b, api.Neighbors().build(m, b, max_nbrs=64)


def _buffers(b):
    f = lambda t, *shape: torch.zeros(shape, dtype=t, device=b.device)
    return {"energy": f(torch.float64, 1), "forces": f(torch.float64, b.n_atoms, 3),
            "stress": f(torch.float64, 1, 3, 3), "site_e": f(torch.float64, b.n_atoms),
            "gamma": f(torch.float64, b.n_atoms), "argmax": f(torch.int32, b.n_atoms),
            "sel_idx": f(torch.int32, b.n_atoms), "sel_count": f(torch.int32, 1)}


def _capture_and_check(call, out):
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    eager = None
    for _ in range(3):
        for t in out.values():
            t.zero_()
        g.replay()
        torch.cuda.synchronize()
        got = {k: t.clone() for k, t in out.items()}
        if eager is None:
            call()
            torch.cuda.synchronize()
            eager = {k: t.clone() for k, t in out.items()}
        for k in out:
            assert torch.equal(got[k], eager[k]), k


# the preselection's counts: per 64 rows above 8,192, per 32 and per 16 rows below
@pytest.mark.parametrize("n_large,n", [(10000, 8192), (10000, 4096), (8193, 8190)])
def test_preselection_counts(n_large, n):
    m = _model(8, 1)
    large, small = _lists(m, n_large, 1, 1), _lists(m, n, 1, 2)
    api.evaluate(m, *large, "fp64", "full", gamma_save=2.0)
    out = _buffers(small[0])
    _capture_and_check(lambda: api.evaluate(m, *small, "fp64", "full", out=out, gamma_save=2.0), out)
    assert 0 < int(out["sel_count"].item())


# rows padded to whole blocks of 64: 80 mixed rows of 256 columns hold fewer words than 100 of 224 in FP64, and
# 27 FULL rows of 224 columns fewer than 64 LINEAR ones of 96, though padded they are more
@pytest.mark.parametrize("first,then", [((100, "fp64", "full"), (80, "mixed", "full")),
                                        ((64, "fp64", "linear"), (27, "fp64", "full"))])
def test_padded_rows(first, then):
    m = _model(16, 2)
    k = m.m("linear")
    m.set_active_set("linear", np.eye(k))
    large, small = _lists(m, first[0], 2, 1), _lists(m, then[0], 2, 2)
    api.evaluate(m, *large, first[1], first[2], gamma_save=2.0)
    out = _buffers(small[0])
    _capture_and_check(lambda: api.evaluate(m, *small, then[1], then[2], out=out, gamma_save=2.0), out)


def _backward_captured(level, first, then):
    m = _model(level, 2)
    large, small = _lists(m, first[0], 2, 1), _lists(m, then[0], 2, 2)
    g = [[torch.from_numpy(np.random.default_rng(3).normal(size=s)).cuda() for s in ((1,), (b.n_atoms, 3), (1, 3, 3))]
         for b, _ in (large, small)]
    api.efs_backward(m, *large, *g[0], first[1])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = api.efs_backward(m, *small, *g[1], then[1])
    for _ in range(3):
        got.zero_()
        graph.replay()
        torch.cuda.synchronize()
        seen = got.clone()
        assert torch.equal(seen, api.efs_backward(m, *small, *g[1], then[1]))


def test_padded_gradient_columns():   # half the neighborhoods in twice the bytes
    _backward_captured(8, (64, "mixed"), (32, "fp64"))


def test_partial_gradients():   # one chunk of 4,096 neighborhoods, then two in half the bytes each
    _backward_captured(8, (4096, "fp64"), (8192, "mixed"))
