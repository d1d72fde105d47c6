"""Neighbour lists over cell grids where the candidate search can go wrong:
one, two, three and more cells per axis in every mix, runs of cells cut by the
box, empty cells, cells of more atoms than a batch of 64-atom blocks, and more
atoms of a type than a wave's worth of blocks in the row order.  Lists are
compared with the oracle's bit for bit."""
import sys

import numpy as np
import pytest

from paper_2005_00223_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _spread(n, box, rng, dmin=0.9):
    """n atoms on a jittered grid of spacing >= dmin inside box."""
    k = np.maximum(1, np.floor(np.asarray(box) / 1.5)).astype(int)
    g = np.stack(np.meshgrid(*[np.arange(q) for q in k], indexing="ij"), -1).reshape(-1, 3)
    assert len(g) >= n
    h = np.asarray(box) / k
    return (g[rng.permutation(len(g))[:n]] + 0.5 + rng.uniform(-0.2, 0.2, size=(n, 3))) * h


# box (cutoff 4.5), atoms, the part of the box they fill
CASES = [((9.1, 9.1, 9.1), 60, 1.0), ((9.1, 13.6, 22.9), 300, 1.0), ((13.6, 13.6, 13.6), 250, 1.0),
         ((32.0, 9.2, 18.1), 240, 0.6), ((46.0, 14.0, 13.7), 1, 1.0), ((32.0, 27.5, 36.0), 480, 0.45),
         ((60.0, 62.0, 61.0), 17000, 1.0),
         # both sides of the one-workgroup preparation: halves of 1,024 atoms, 2,048 atoms, 4,096 cells
         ((20.0, 20.0, 20.0), 1023, 1.0), ((20.0, 20.0, 20.0), 1025, 1.0), ((21.0, 24.0, 22.0), 2048, 1.0),
         ((21.0, 24.0, 22.0), 2049, 1.0), ((72.1, 72.1, 72.1), 1500, 1.0), ((77.0, 72.1, 72.1), 1500, 1.0)]


@pytest.mark.parametrize("box,n,part", CASES)
def test_lists(box, n, part):
    from oracle import oracle as O
    from paper_2005_00223_amd.model import DPModel
    rng = np.random.default_rng(n)
    x = _spread(n, np.asarray(box) * part, rng)
    x = (x + rng.uniform(0, 1, size=3) * box) % box
    t = rng.integers(0, 2, size=n).astype(np.int32)
    spec = synth.random_model(2, 4.5, 2.0, (96, 96), fit=(32,), seed=3)
    print(f"[lists] box {box}, {n} atoms", flush=True)
    sys.stdout.flush()
    m = DPModel(synth.pack_blob(spec), "fp64")
    m.compute(x, t, np.asarray(box))
    nl, nr = m.nlist(n, spec.nnei, 2)
    onl, onr, _ = O.Oracle(synth.pack_blob(spec)).nlist(x, t, np.asarray(box))
    assert np.array_equal(np.asarray(nr.cpu() if hasattr(nr, "cpu") else nr), onr)
    assert np.array_equal(np.asarray(nl.cpu() if hasattr(nl, "cpu") else nl), onl)


def test_small_bricks_sum_to_the_whole():
    """Rows for the first atoms only, cells for all (compute_local of small
    bricks, ghosts included): the bricks' energies, forces and virials sum to the
    whole system's.  FP64 bars of the whole-box test."""
    from paper_2005_00223_amd.model import DPModel
    rng = np.random.default_rng(5)
    box = np.array([27.0, 14.0, 13.7])
    x = _spread(600, box, rng)
    t = rng.integers(0, 2, size=600).astype(np.int32)
    spec = synth.random_model(2, 4.5, 2.0, (96, 96), fit=(32,), seed=3)
    m = DPModel(synth.pack_blob(spec), "fp64")
    e0, f0, v0 = m.compute(x, t, box)
    e0, v0 = float(e0), v0.cpu().numpy()
    f0 = f0.clone()
    ftot, etot, vtot = torch.zeros((600, 3), dtype=torch.float64, device="cuda"), 0.0, 0.0
    for b in range(2):
        sh = synth.brick_share(x, t, box, (2, 1, 1), (b, 0, 0), spec.rcut)
        print(f"[lists] brick {b}: {sh['n_local']} of {len(sh['types'])}", flush=True)
        e, f, v = m.compute_local(sh["coords"], sh["types"], sh["box"], sh["n_local"])
        m.scatter_add_forces(sh["index"], f, ftot)
        etot += float(e)
        vtot = vtot + v.cpu().numpy()
    assert float((ftot - f0).abs().max()) <= 1e-9
    assert abs(etot - e0) <= 1e-10 * abs(e0)
    assert np.abs(vtot - v0).max() <= 1e-10 * np.abs(v0).max()
