"""Candidate lists by groups of bins: the neighbour sets equal the oracle's bit for bit where
the group walk has edges (stencils that wrap onto themselves, runs cut by the cell's end, more
atoms or records than a wave holds, atoms of several lattice images, images far away)."""
import numpy as np
import pytest

from gpu_cases import sort_entries

pytestmark = pytest.mark.gpu


def _structure(kind, seed):
    rng = np.random.default_rng(seed)
    L = dict(thin=(2.9, 17.0, 6.1), long=(5.7, 5.9, 61.0)).get(kind, (12.0, 11.0, 13.5))
    h = np.diag(L) + np.array([[0, 0, 0], [0.7, 0, 0], [-0.5, 0.9, 0]])
    if kind == "cluster":  # one bin with more atoms than a wave, a stage that overflows
        a = rng.normal(0.0, 0.8, (600, 3)) + np.array([6.0, 5.5, 6.5])
        pos = np.concatenate([a, rng.random((100, 3)) @ h])
    else:  # dense: the half-width stencil
        g = np.stack(np.meshgrid(*[np.arange(max(2, int(v / 1.05))) for v in L], indexing="ij"), -1).reshape(-1, 3)
        pos = (g / (g.max(0) + 1)) @ h + rng.normal(0.0, 0.08, g.shape)
    if kind == "images":  # neighbours written in different lattice images
        pos = pos + rng.integers(-3, 4, pos.shape) @ h
    if kind == "far":
        pos = pos + np.array([6.0, -5.0, 0.0]) @ h
    return pos, h


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("kind", ["plain", "thin", "long", "images", "far", "cluster"])
def test_group_candidates_give_the_exact_sets(kind, fp64):
    import oracle
    import torch
    from paper_2510_16721_amd import cfneb
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    pos, h = _structure(kind, 3)
    p = cfneb.default_params(cfneb.CFNEB_LJ, n_images=3, max_images=3, force_fp64=int(fp64), lj_sigma=0.4,
                             nbr_cap=700 if kind == "cluster" else 200)
    band = cfneb.Band(p, pos, h, pos + 0.01, h @ (np.eye(3) * 1.003))
    for k in range(3):
        img = band.image(k)
        cnt, ent = band.neighbours(k)
        ref = oracle.nlist(img["R"], img["h"], 2.5)
        assert [int(c) for c in cnt] == [len(r) for r in ref]
        for i in range(len(pos)):
            np.testing.assert_array_equal(sort_entries(ent[i]), ref[i])
