"""The embedding nets' piecewise expansions (double kernels: FP64; float
kernels: FP32 and FP16) where they can go wrong: distances on both sides of every
piece boundary, neighbour counts at the edges of the 16- and 64-neighbour
chunks, several pieces in one atom's list, pairs beyond the range (the layer
kernels then evaluate the frame), in single evaluations and in MD.

Bars, set before the first run.  FP64: the parity bars of the FP64 tests
(energy 1e-10 relative, forces 1e-9 eV/A) with forces relative to the
largest where close pairs make them large.  FP32 against the
oracle on the weights its kernels hold: 2^-12 of the largest force and
virial component and of the summed |E_i| -- the 1 - t^2 of the fitting net's
saturated tanh, which close pairs bring, costs FP32 up to 1.3e-4
(measured with the layer kernels on dimers)."""
import copy
import sys

import numpy as np
import pytest

from paper_2005_00223_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _held(spec, prec):
    """The weights the kernels of a precision hold, in FP64."""
    q = copy.deepcopy(spec)
    f32 = lambda w: np.asarray(w, dtype=np.float32).astype(np.float64)
    for t in range(spec.ntypes):
        for u in range(spec.ntypes):
            for l in range(len(spec.emb)):
                W = spec.emb_W[t][u][l]
                if prec != "fp64":
                    q.emb_W[t][u][l] = f32(W)
                    q.emb_b[t][u][l] = f32(spec.emb_b[t][u][l])
        for l in range(len(spec.fit) + 1):
            W = spec.fit_W[t][l]
            if prec != "fp64":
                q.fit_W[t][l] = f32(W)
                q.fit_b[t][l] = f32(spec.fit_b[t][l])
    return q


def _check(spec, x, t, box, prec, tag):
    from oracle import oracle as O
    from paper_2005_00223_amd.model import DPModel
    m = DPModel(synth.pack_blob(spec), prec)
    m.compute(x, t, box, keep_intermediates=True)
    e, f, v = m.compute(x, t, box, keep_intermediates=True)
    r = O.Oracle(synth.pack_blob(_held(spec, prec))).eval(x, t, box)
    f, v = f.cpu().numpy(), v.cpu().numpy()
    fmax = max(1.0, float(np.abs(r["force"]).max()))
    vmax = max(1.0, float(np.abs(r["virial"]).max()))
    emax = max(1.0, float(np.abs(r["atom_e"]).sum()))
    df, de, dv = np.abs(f - r["force"]).max() / fmax, abs(float(e) - r["energy"]) / emax, \
        np.abs(v - r["virial"]).max() / vmax
    say(f"  {tag} {prec}: F {df:.2e} of {fmax:.3g}, E {de:.2e}, V {dv:.2e} of {vmax:.3g}")
    bar = {"fp64": (1e-9, 1e-10, 1e-9), "fp32": (2.0 ** -12,) * 3}[prec]
    assert df <= bar[0] and de <= bar[1] and dv <= bar[2]


# r = 1/s below the switch radius: s on and beside the boundaries of the
# halved intervals of [0, 8], out to the cutoff
RADII = sorted({r for s in (0.125, 0.25, 0.5, 0.75, 1.0, 1.25, 1.5, 2.0, 2.5, 3.0, 4.0, 6.0, 7.5)
                for r in (1.0 / s, (1.0 - 1e-9) / s, (1.0 + 1e-9) / s)} | {2.9, 4.4, 5.999, 6.0, 6.001})


def test_dimers_across_the_pieces():
    """One dimer per radius, far from each other, O-O, O-H and H-H in turn."""
    spec = synth.random_model(2, 6.0, 8.5e-1, (46, 92), seed=5, out_scale=-8.0, desc_norm=2.0)
    spec.rcut_smth = 5.0
    rng = np.random.default_rng(3)
    x, t = [], []
    n = int(np.ceil(len(RADII) ** (1 / 3)))
    for k, r in enumerate(RADII):
        c = 16.0 * np.array([k % n, k // n % n, k // n // n]) + 4.0
        d = rng.normal(size=3)
        x += [c, c + r * d / np.linalg.norm(d)]
        t += [(0, 0), (0, 1), (1, 1)][k % 3]
    say(f"[expand] {len(RADII)} dimers")
    _check(spec, np.array(x), np.array(t, dtype=np.int32), np.full(3, 16.0 * n), "fp64", "dimers")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("count", [1, 15, 16, 17, 63, 64, 65, 127, 129, 200])
def test_neighbour_counts(count, prec):
    """A cluster of count + 1 atoms, every one the others' neighbour, with
    distances from 0.6 A on: several pieces in each list."""
    spec = synth.random_model(1, 7.0, 3.0, (256,), seed=6, out_scale=-20.0, desc_norm=8.0)
    rng = np.random.default_rng(count)
    g = np.stack(np.meshgrid(*[np.arange(6)] * 3, indexing="ij"), -1).reshape(-1, 3)
    g = g[np.argsort(((g - 2.5) ** 2).sum(1), kind="stable")][:count + 1]
    x = 0.85 * g + rng.uniform(-0.1, 0.1, size=g.shape) + 8.0
    say(f"[expand] cluster of {count + 1}")
    _check(spec, x, np.zeros(count + 1, dtype=np.int32), np.full(3, 22.0), prec, f"count {count}")


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
def test_pair_beyond_the_range(prec):
    """Two atoms 0.1 A apart in an ordinary crystal (s = 10, beyond every
    expansion): the frame is evaluated by the layers; the next frame,
    without that pair, on the same model again by the expansions."""
    x, t, box = synth.fcc_copper(5, 3.634, 0.05, seed=9)
    spec = synth.copper_model(1)
    far = x.copy()
    far[1] = far[0] + [0.1, 0.0, 0.0]
    say("[expand] pair at 0.1 A")
    if prec == "fp64":
        _check(spec, far, t, box, prec, "far")
    from paper_2005_00223_amd.model import DPModel
    m = DPModel(synth.pack_blob(spec), prec)
    e0, f0, v0 = m.compute(x, t, box)
    m.compute(far, t, box)
    st = m.stats()
    assert st["evaluations"] == 2
    e1, f1, v1 = m.compute(x, t, box)
    assert abs(float(e0) - float(e1)) <= 1e-12 * abs(float(e0))
    assert float((f0 - f1).abs().max()) <= 1e-11 and float((v0 - v1).abs().max()) <= 1e-9
    # the two halves, the far pair in the forward
    m.energy(far, t, box)
    f2, v2 = m.energy_backward(1.0)
    e3, f3, v3 = m.compute(far, t, box)
    s = float(f3.abs().max())
    assert float((f2 - f3).abs().max()) <= 1e-10 * s


def test_md_through_the_range():
    """An NVE run in which two atoms meet: fired at each other they pass
    0.125 A, where the run changes to the layer kernels and goes on; the
    trajectory is the oracle's Verlet run.  Bar: 1e-7 A and relative in the
    velocities (FP64 rounding, amplified by the stiff encounter)."""
    from oracle import oracle as O
    from paper_2005_00223_amd.model import DPModel
    spec = synth.copper_model(1)
    x = np.array([[9.0, 9.0, 9.0], [9.63, 9.05, 9.0], [13.0, 10.0, 8.0]])
    v = np.array([[0.2, 0.0, 0.0], [-0.2, 0.0, 0.0], [0.0, 0.0, 0.0]])
    t, box, nst = np.zeros(3, dtype=np.int32), np.full(3, 21.0), 12
    ora = O.Oracle(synth.pack_blob(spec))
    seen = [ora.verlet(x, v, t, box, [63.546], 0.25, k, every=0)[0] for k in range(nst + 1)]
    dist = [float(np.linalg.norm(y[0] - y[1])) for y in seen]
    xo, vo, tho = ora.verlet(x, v, t, box, [63.546], 0.25, nst, every=4)
    m = DPModel(synth.pack_blob(spec), "fp64")
    xg, vg = torch.tensor(x, device="cuda"), torch.tensor(v, device="cuda")
    th = m.md_run(xg, vg, t, box, [63.546], 0.25, nst, skin=1.0, thermo_every=4).cpu().numpy()
    say(f"[expand] MD: distances {dist[0]:.3f} .. {min(dist):.3f} .. {dist[-1]:.3f} A, x {np.abs(xg.cpu().numpy() - xo).max():.2e}, "
        f"v {np.abs(vg.cpu().numpy() - vo).max():.2e}")
    assert dist[0] > 0.5 and min(dist) < 0.125 and dist[-1] > 0.3
    assert np.abs(xg.cpu().numpy() - xo).max() <= 1e-7
    assert np.abs(vg.cpu().numpy() - vo).max() <= 1e-7 * max(1.0, np.abs(vo).max())
    assert np.abs(th[:, 1:5] - tho[:, 1:5]).max() <= 1e-6 * np.abs(tho[:, 1:5]).max()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("order", ["lattice", "shuffled"])
@pytest.mark.parametrize("reps", [(4, 2, 1), (4, 3, 1)])
def test_merged_scatter(reps, order, prec):
    """Forces merged in the workgroups' LDS tables (4,000 and 6,000 atoms, the
    smallest that are): neighbours shared by consecutive rows, and rows in
    random order, whose neighbours overflow the table.  The system is a cell
    of 500 repeated, so every copy has the oracle's forces of the cell."""
    from oracle import oracle as O
    from paper_2005_00223_amd.model import DPModel
    x, t, box = synth.fcc_copper(5, 3.634, 0.1, seed=4)
    spec = synth.copper_model(1)
    r = O.Oracle(synth.pack_blob(_held(spec, prec))).eval(x, t, box)
    copies = np.stack(np.meshgrid(*[np.arange(k) for k in reps], indexing="ij"), -1).reshape(-1, 3)
    X = (x[None] + copies[:, None] * box).reshape(-1, 3)
    n = len(X)
    p = np.random.default_rng(1).permutation(n) if order == "shuffled" else np.arange(n)
    say(f"[expand] merged scatter {n} {order} {prec}")
    m = DPModel(synth.pack_blob(spec), prec)
    e, f, v = m.compute(X[p], np.tile(t, len(copies))[p], box * np.array(reps))
    want = np.tile(r["force"], (len(copies), 1))[p]
    fmax, vmax = max(1.0, np.abs(want).max()), max(1.0, np.abs(r["virial"]).max())
    df = np.abs(f.cpu().numpy() - want).max() / fmax
    de = abs(float(e) / len(copies) - r["energy"]) / np.abs(r["atom_e"]).sum()
    dv = np.abs(v.cpu().numpy() / len(copies) - r["virial"]).max() / vmax
    say(f"  F {df:.2e}, E {de:.2e}, V {dv:.2e}")
    bar = {"fp64": (1e-9, 1e-10, 1e-9), "fp32": (2.0 ** -12,) * 3}[prec]
    assert df <= bar[0] and de <= bar[1] and dv <= bar[2]
