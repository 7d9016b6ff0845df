"""Carbon atoms with more than four bonds where a block takes more than 64 items (8 blocks, 80
items each): atoms that were crowded in the evaluation before and are not any more, in the same
late items as atoms that are now.  The same bits as a block per tile and as a band that never
had the earlier coordinates, and the oracle's values."""
import numpy as np
import pytest

from gpu_cases import TOL_F, oracle_params_like

pytestmark = pytest.mark.gpu

NX, NY, NZ, A, IMAGES, BLOCKS = 16, 16, 8, 3.566, 12, 8  # 16,384 atoms: 64 items an image


def _diamond():
    fcc = np.array([[0.0, 0.0, 0.0], [0.0, 0.5, 0.5], [0.5, 0.0, 0.5], [0.5, 0.5, 0.0]])
    g = np.stack(np.meshgrid(np.arange(NX), np.arange(NY), np.arange(NZ), indexing="ij"), -1).reshape(-1, 1, 3)
    return ((g + np.concatenate([fcc, fcc + 0.25])) * A).reshape(-1, 3), np.diag([NX * A, NY * A, NZ * A])


def _crowd(pos, h, centres):
    """The atoms within 3.1 of each centre drawn a quarter of the way to it (the twelve second
    neighbours to 1.89, inside the cutoff); returns the positions and which atoms moved."""
    out, moved = pos.copy(), np.zeros(len(pos), bool)
    L = np.diag(h)
    for c in centres:
        d = pos - pos[c]
        d -= np.round(d / L) * L
        near = np.linalg.norm(d, axis=1) < 3.1
        out[near] -= 0.25 * d[near]
        moved |= near
    return out, moved


def _late_waves(atoms_per_image):
    """(block, wave) of every late item (from a block's 64th on) that holds one of the atoms."""
    tiles = NX * NY * NZ * 8 // 256
    chunk = tiles * (IMAGES - 2) // BLOCKS
    found = set()
    for k, atoms in enumerate(atoms_per_image):
        for i in atoms:
            item = k * tiles + i // 256
            if item % chunk >= 63:
                found.add((item // chunk, i % 256 // 64, item))
    return found


@pytest.mark.parametrize("fp64", [False, True])
def test_late_items(fp64, monkeypatch):
    import oracle
    import torch
    from paper_2510_16721_amd import cfneb
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    pos, h = _diamond()
    n, M = len(pos), IMAGES
    rng = np.random.default_rng(3)
    centres = [rng.choice(n, 48, replace=False) for _ in range(M - 2)]
    before = [_crowd(pos, h, c[:24])[0] for c in centres]
    now = [_crowd(pos, h, c[24:]) for c in centres]
    # the case itself: a wave with an item crowded now and another crowded only before, both late
    was, is_ = (_late_waves([c[s] for c in centres]) for s in (slice(0, 24), slice(24, 48)))
    left = {(b, w) for b, w, q in was if (b, w, q) not in is_}
    assert left & {(b, w) for b, w, _ in is_}

    p = cfneb.default_params(cfneb.CFNEB_TERSOFF_C, force_fp64=int(fp64), n_images=M, max_images=M, nbr_cap=32)

    def band(grid, states):
        monkeypatch.setenv("CFNEB_FORCE_GRID", grid)
        g = cfneb.Band(p, pos, h, pos + 0.01, h)
        assert g.step(1, 1e30)[2]  # an evaluation without a move
        monkeypatch.delenv("CFNEB_FORCE_GRID")
        for images in states:
            st = g.get_state()
            X = st["X"]
            X[1:-1, :n] = images
            g.set_state(X, st["v"], st["dt"], st["alpha"], st["n_pos"], st["fresh"], st["step"], st["ci"])
            assert g.step(1, 1e30)[2]
        out = [g.image(k) for k in range(1, M - 1)]
        g.close()
        return out

    images = [x for x, _ in now]
    got = band(str(BLOCKS), [before, images])
    for other in (band("tile", [before, images]), band("tile", [images])):
        for a, b in zip(got, other):
            assert a["E"] == b["E"]
            np.testing.assert_array_equal(a["V"], b["V"])
            np.testing.assert_array_equal(a["F"], b["F"])
    for k in (1, 9):
        img, (_, moved) = got[k], now[k]
        E, _, F, V = oracle.evaluate(oracle_params_like("ts"), img["R"], img["h"])
        # FP64: rounding of some n^2 terms; FP32: 2^-24 on the bond lengths, amplified by the
        # exponents' l1 r < 8 and summed over an atom's bonds, against the largest value
        tol = 1e-11 if fp64 else 2e-5
        assert abs(img["E"] - E) <= tol * abs(E)
        assert np.abs(img["V"] - V).max() <= tol * np.abs(V).max()
        assert np.abs(img["F"] - F).max() <= tol * np.abs(F).max()
        # the ordinary atoms against their own scale
        far = _far(pos, h, moved)
        assert far.any() and np.abs(img["F"] - F)[far].max() <= TOL_F * (1e-6 if fp64 else 1.0)


def _far(pos, h, moved):
    """Atoms at least two cutoffs from every moved one."""
    from scipy.spatial import cKDTree
    L = np.diag(h)
    s = np.mod(pos, L)
    d, _ = cKDTree(s[moved], boxsize=L).query(s)
    return d > 4.5
