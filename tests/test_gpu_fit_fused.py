"""The fused FP64 / FP32 fitting-net kernels on both sides of their dispatch:
16, 32 and 64 rows a workgroup forward, 16 and 32 rows and the row-wave kernel
backward, type blocks that end inside a tile, hidden widths of one tile up to
sixteen, with and without the skip, fewer than 16 columns of D.

A large system is a small periodic cell repeated, so every copy of an atom has
the energy and force that the oracle gives for the cell.

Bars, set before the first run: FP64 1e-9 of the largest force and virial
component and 1e-10 of the summed |E_i| (the parity bars); FP32 2^-12 of the
same, against the oracle on the weights rounded to FP32."""
import copy
import sys

import numpy as np
import pytest

from paper_2005_00223_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CELL = 187  # atoms: 143 of type 0, 44 of type 1


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _held(spec, prec):
    """The weights the kernels of a precision hold, in FP64."""
    q = copy.deepcopy(spec)
    if prec == "fp32":
        f32 = lambda w: np.asarray(w, dtype=np.float32).astype(np.float64)
        for t in range(spec.ntypes):
            for u in range(spec.ntypes):
                for l in range(len(spec.emb)):
                    q.emb_W[t][u][l] = f32(spec.emb_W[t][u][l])
                    q.emb_b[t][u][l] = f32(spec.emb_b[t][u][l])
            for l in range(len(spec.fit) + 1):
                q.fit_W[t][l] = f32(spec.fit_W[t][l])
                q.fit_b[t][l] = f32(spec.fit_b[t][l])
    return q


def _cell():
    rng = np.random.default_rng(11)
    g = np.stack(np.meshgrid(*[np.arange(6)] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = 2.2 * rng.permutation(g)[:CELL] + rng.uniform(-0.3, 0.3, size=(CELL, 3)) + 1.1
    return x % 13.2, (np.arange(CELL) >= 143).astype(np.int32), np.full(3, 13.2)


# hidden widths, M2, repeats of the cell
CASES = [((240, 240, 240), 16, (1, 1, 1)),     # 187 atoms: 16 rows, layer 0 spread over workgroups
         ((240, 240), 7, (1, 1, 1)),           # ... D too narrow to hold what the spread passes on
         ((240, 240, 240), 16, (4, 4, 1)),     # 2,992: 16 rows, one kernel a pass
         ((240, 240, 240), 16, (5, 5, 1)),     # 4,675: 32 rows
         ((240, 240, 240), 16, (10, 7, 1)),    # 13,090: 64 rows (FP64) and the row-wave backward
         ((240,), 7, (10, 7, 1)),              # ... of one layer, fewer columns of D
         ((256, 256), 16, (10, 7, 1)),         # the widest, not row-wave
         ((16, 64, 64, 48), 12, (1, 1, 1)),    # waves without a column tile, no skip, skip
         ((16, 64, 64, 48), 12, (5, 5, 1))]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("fit,M2,reps", CASES)
def test_fit_fused(fit, M2, reps, prec):
    from oracle import oracle as O
    from paper_2005_00223_amd.model import DPModel
    spec = synth.random_model(2, 4.5, 2.0, (64, 64), M2=M2, fit=fit, seed=21, out_scale=-8.0, desc_norm=2.0)
    x, t, box = _cell()
    r = O.Oracle(synth.pack_blob(_held(spec, prec))).eval(x, t, box)
    copies = np.stack(np.meshgrid(*[np.arange(k) for k in reps], indexing="ij"), -1).reshape(-1, 3)
    X = (x[None] + copies[:, None] * box).reshape(-1, 3)
    T = np.tile(t, len(copies))
    perm = np.random.default_rng(2).permutation(len(X))
    print(f"[fit] {fit} M2 {M2} {prec}: {len(X)} atoms", flush=True)
    sys.stdout.flush()
    m = DPModel(synth.pack_blob(spec), prec)
    e, f, v = m.compute(X[perm], T[perm], box * np.array(reps))
    want = np.tile(r["force"], (len(copies), 1))[perm]
    fmax, vmax = np.abs(r["force"]).max(), np.abs(r["virial"]).max()
    df = np.abs(f.cpu().numpy() - want).max() / fmax
    de = abs(float(e) / len(copies) - r["energy"]) / np.abs(r["atom_e"]).sum()
    dv = np.abs(v.cpu().numpy() / len(copies) - r["virial"]).max() / vmax
    print(f"  F {df:.2e} of {fmax:.3g}, E {de:.2e}, V {dv:.2e} of {vmax:.3g}", flush=True)
    bar = {"fp64": (1e-9, 1e-10, 1e-9), "fp32": (2.0 ** -12,) * 3}[prec]
    assert df <= bar[0] and de <= bar[1] and dv <= bar[2]


@pytest.mark.parametrize("prec", ["fp16"])
@pytest.mark.parametrize("fit", [(240, 240, 240), (240,)])
@pytest.mark.parametrize("reps", [(7, 7, 1), (16, 10, 1)])
def test_fit_mix_sizes(reps, fit, prec):
    """16-bit fitting net: 16 rows a workgroup (187 atoms, which the tests of
    the precisions compare with the oracle) against 32 (9,163) and 64 forward
    and the row-wave backward (29,920).  The products are the same in the same
    order; the sums over tiles and rows of D are FP32 in another: 2^-16 of the
    largest force and of the summed |E_i|."""
    from paper_2005_00223_amd.model import DPModel
    spec = synth.random_model(2, 4.5, 2.0, (64, 64), fit=fit, seed=21, out_scale=-8.0, desc_norm=2.0)
    x, t, box = _cell()
    m = DPModel(synth.pack_blob(spec), prec)
    e1, f1, v1 = m.compute(x, t, box, keep_intermediates=True)
    e1, f1, v1 = float(e1), f1.cpu().numpy(), v1.cpu().numpy()
    scale = np.abs(m.intermediates(CELL, 100, 16, spec.nnei, ("atom_e",))["atom_e"].cpu().numpy()).sum()
    copies = np.stack(np.meshgrid(*[np.arange(k) for k in reps], indexing="ij"), -1).reshape(-1, 3)
    X = (x[None] + copies[:, None] * box).reshape(-1, 3)
    perm = np.random.default_rng(2).permutation(len(X))
    print(f"[fit] {fit} {prec}: {len(X)} atoms", flush=True)
    sys.stdout.flush()
    e, f, v = m.compute(X[perm], np.tile(t, len(copies))[perm], box * np.array(reps))
    want = np.tile(f1, (len(copies), 1))[perm]
    df = np.abs(f.cpu().numpy() - want).max() / np.abs(f1).max()
    de = abs(float(e) / len(copies) - e1) / scale
    dv = np.abs(v.cpu().numpy() / len(copies) - v1).max() / np.abs(v1).max()
    print(f"  F {df:.2e}, E {de:.2e}, V {dv:.2e}", flush=True)
    assert max(df, de, dv) <= 2.0 ** -16
