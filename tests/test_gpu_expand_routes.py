"""Routes of an evaluation around the net expansions: which buffers they
borrow, when the layers take over, and what a judge's two net sets share.

Bars, set before the first run: FP64 1e-9 of the largest force and virial
component and 1e-10 of the summed |E_i| (the parity bars); FP32 2^-12 of the
same against the oracle on the weights rounded to FP32."""
import copy
import sys

import numpy as np
import pytest

from paper_2005_00223_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BARS = {"fp64": (1e-9, 1e-10, 1e-9), "fp32": (2.0 ** -12,) * 3}


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _model(spec, prec):
    from paper_2005_00223_amd.model import DPModel
    return DPModel(synth.pack_blob(spec), prec)


def _held(spec, prec):
    """The weights the kernels of a precision hold, in FP64."""
    q = copy.deepcopy(spec)
    if prec == "fp32":
        f32 = lambda w: np.asarray(w, dtype=np.float32).astype(np.float64)
        for t in range(spec.ntypes):
            for u in range(spec.ntypes):
                q.emb_W[t][u] = [f32(w) for w in spec.emb_W[t][u]]
                q.emb_b[t][u] = [f32(w) for w in spec.emb_b[t][u]]
            q.fit_W[t] = [f32(w) for w in spec.fit_W[t]]
            q.fit_b[t] = [f32(w) for w in spec.fit_b[t]]
    return q


def _oracle(spec, x, t, box, prec="fp64"):
    from oracle import oracle as O
    return O.Oracle(synth.pack_blob(_held(spec, prec))).eval(x, t, box)


def _compare(out, r, prec, tag, copies=1, order=None):
    """(E, F, V) of `copies` periodic repeats, atoms in `order`, against the
    oracle's result r of one cell."""
    e, f, v = out
    want = np.tile(r["force"], (copies, 1))
    if order is not None:
        want = want[order]
    fmax, vmax = max(1.0, np.abs(want).max()), max(1.0, np.abs(r["virial"]).max())
    df = np.abs(f.cpu().numpy() - want).max() / fmax
    de = abs(float(e) / copies - r["energy"]) / max(1.0, np.abs(r["atom_e"]).sum())
    dv = np.abs(v.cpu().numpy() / copies - r["virial"]).max() / vmax
    say(f"  {tag} {prec}: F {df:.2e} of {fmax:.3g}, E {de:.2e}, V {dv:.2e} of {vmax:.3g}")
    assert df <= BARS[prec][0] and de <= BARS[prec][1] and dv <= BARS[prec][2]


def _cell(ntypes=2, n=187):
    """n atoms on a jittered grid in a box of 13.2 A, the first three quarters
    of type 0."""
    rng = np.random.default_rng(11)
    g = np.stack(np.meshgrid(*[np.arange(6)] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = 2.2 * rng.permutation(g)[:n] + rng.uniform(-0.3, 0.3, size=(n, 3)) + 1.1
    t = np.arange(n) * ntypes // n if ntypes > 2 else (np.arange(n) >= n * 143 // 187)
    return x % 13.2, t.astype(np.int32), np.full(3, 13.2)


def _repeat(x, t, box, reps, seed=2):
    copies = np.stack(np.meshgrid(*[np.arange(k) for k in reps], indexing="ij"), -1).reshape(-1, 3)
    X = (x[None] + copies[:, None] * box).reshape(-1, 3)
    order = np.random.default_rng(seed).permutation(len(X))
    return X[order], np.tile(t, len(copies))[order], box * np.array(reps), len(copies), order


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("fit", [(16,), (240, 240, 240)])
@pytest.mark.parametrize("M2", [1, 2, 3])
def test_fewer_columns_than_components(M2, fit, prec):
    """D of one to three columns: dE/dT, which takes dE/dD's place in the fused
    fitting kernels, is then the larger of the two."""
    spec = synth.random_model(2, 4.5, 2.0, (64, 64), M2=M2, fit=fit, seed=21, out_scale=-8.0, desc_norm=2.0)
    x, t, box = _cell()
    r = _oracle(spec, x, t, box, prec)
    X, T, B, copies, order = _repeat(x, t, box, (5, 5, 1))
    say(f"[routes] M2 {M2}, fitting {fit}, {prec}: {len(X)} atoms")
    _compare(_model(spec, prec).compute(X, T, B), r, prec, f"M2 {M2}", copies, order)


def _rough_copper(scale=24.0):
    """The copper model with first embedding layers too steep for an
    expansion in any precision: its layers are evaluated."""
    spec = synth.copper_model(1)
    for row in spec.emb_W:
        for W in row:
            W[0] = W[0] * scale
    return spec


def _md(m, w, nsteps, prec):
    t = w["types"]
    x = torch.tensor(w["coords"], dtype=torch.float64, device="cuda")
    v = torch.tensor(synth.maxwell_boltzmann(w["masses"][t], 300.0, w["vseed"]), dtype=torch.float64, device="cuda")
    return m.md_run(x, v, t, w["box"], w["masses"], 0.2, nsteps, skin=0.3, thermo_every=10).cpu().numpy()


# judge over all atoms, and over a cube confirmed by all
@pytest.mark.parametrize("name,side", [("cu_cells5", 0.0), ("cu_cells9", 10.0)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_judge_of_a_teacher_without_expansion(prec, name, side):
    """A student on an expansion judged by a teacher on its layers: a student
    with zero outputs (no forces) is rejected at step 0 with the RMS of the
    teacher's forces, and the run is the teacher's from there on; a kept
    student's RMSE is that of the two nets' own evaluations.  RMSE within 1e-6
    relative (atomics' order); trajectories 1e-9 (FP32 1e-7: a last bit of an
    s may round otherwise)."""
    w = synth.workload(name)
    teacher = _rough_copper()
    n = len(w["types"])
    mt = _model(teacher, prec)
    _, ft, _ = mt.compute(w["coords"], w["types"], w["box"])
    r = _oracle(teacher, w["coords"], w["types"], w["box"], prec)
    df = np.abs(ft.cpu().numpy() - r["force"]).max() / np.abs(r["force"]).max()
    say(f"[routes] judge {name} {prec}: teacher F {df:.2e}")
    assert df <= BARS[prec][0]
    want = _md(mt, w, 20, prec)
    P = synth.random_student_params(teacher, 31)
    zero = P.copy()
    zero[:, -33 * teacher.M1:] = 0.0
    for params, keep in ((zero, False), (P, True)):
        m = _model(teacher, prec)
        m.student_set_model(synth.pack_blob(synth.student_spec(teacher, params)))
        m.student_use(True)
        _, fs, _ = m.compute(w["coords"], w["types"], w["box"])
        expect = float(((fs - ft) ** 2).sum(1).mean().sqrt())
        m.student_judge(20, 1e6 if keep else 1e-3, sample_side=0.0 if keep else side)
        th = _md(m, w, 0 if keep else 20, prec)
        st = m.stats()
        say(f"  keep={keep}: RMSE {st['last_judge_rmse']:.9e} over {st['judge_atoms']}, expected {expect:.9e}")
        assert abs(st["last_judge_rmse"] - expect) <= 1e-6 * expect
        assert st["judge_atoms"] == n and st["teacher_fallbacks"] == (0 if keep else 1)
        if not keep:
            tol = 1e-9 if prec == "fp64" else 1e-7
            np.testing.assert_allclose(th, want, rtol=tol, atol=tol)


# ---------------------------------------------------------------------------
# the layers in place of the expansions: pairs beyond the range of s (closer
# than 1/32 A for these nets), more than twelve pieces in one atom's list
# ---------------------------------------------------------------------------
BOX = np.array([44.0, 21.0, 21.0])
CRYSTAL = 108


def _frame(kind):
    """3^3 cells of copper at one end of the box, a cluster at the other, more
    than a cutoff away: a pair at 0.05 A (on the expansions), a pair at 0.02 A
    (beyond them), or an atom with neighbours in 9 or
    in 20 pieces of the double tables (none beyond them)."""
    far, _, _ = synth.fcc_copper(3, 3.634, 0.05, seed=9)
    rng = np.random.default_rng(4)
    d = rng.normal(size=(40, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    r = {"in": [0.05], "pair": [0.02], "few": np.geomspace(0.25, 1.9, 10), "many": np.geomspace(0.06, 1.9, 40)}[kind]
    c = np.array([30.0, 10.0, 10.0])
    x = np.concatenate([far + 2.0, [c], c + d[:len(r)] * np.asarray(r)[:, None]])
    return x, np.zeros(len(x), dtype=np.int32), BOX


def _crystal_energies(m, kind):
    """E_i of the crystal's atoms, whose surroundings do not depend on the
    cluster: bit for bit the same on one route, in the last bits not on the
    other (which is how the tests see the route)."""
    x, t, box = _frame(kind)
    out = m.compute(x, t, box, keep_intermediates=True)
    e = m.intermediates(len(x), 100, 16, 512, ("atom_e",))["atom_e"].cpu().numpy()
    return out, e[:CRYSTAL]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
def test_layers_take_over(prec):
    spec = synth.copper_model(1)
    m = _model(spec, prec)
    _, e0 = _crystal_energies(m, "in")
    for kind, layers in (("pair", True), ("few", False), ("many", True), ("in", False)):
        if prec != "fp64" and kind == "many":
            continue  # the float tables have fewer pieces than an atom holds
        out, e = _crystal_energies(m, kind)
        same = np.array_equal(e, e0)
        say(f"[routes] {kind} {prec}: same route as the first frame {same}, E_i {np.abs(e - e0).max():.2e}")
        assert same == (not layers)
        assert np.abs(e - e0).max() <= {"fp64": 1e-11, "fp32": 2e-4, "fp16": 2e-4}[prec] * np.abs(e0).max()
        x, t, box = _frame(kind)
        if prec == "fp64":
            _compare(out, _oracle(spec, x, t, box), prec, kind)
        # the other entry points agree: both halves, centres first, no allocation
        s = max(1.0, float(out[1].abs().max()))
        tol = {"fp64": 1e-10, "fp32": 1e-6, "fp16": 1e-6}[prec]
        m.energy(x, t, box)
        f, v = m.energy_backward(2.0)
        assert float((f - 2.0 * out[1]).abs().max()) <= tol * s
        el, fl, vl = m.compute_local(x, t, box, len(x))
        assert abs(float(el) - float(out[0])) <= tol * abs(float(out[0])) and float((fl - out[1]).abs().max()) <= tol * s


def test_far_pair_among_the_centres_or_the_ghosts():
    """Rank share: the far pair's atoms as centres, or as ghosts only, where no
    centre meets it (the crystal alone has centres) and the expansions stay."""
    spec = synth.copper_model(1)
    m = _model(spec, "fp64")
    x, t, box = _frame("pair")
    r = _oracle(spec, x, t, box)
    for n_local in (CRYSTAL, CRYSTAL + 1):
        e, f, v = m.compute_local(x, t, box, n_local)
        want = r["atom_e"][:n_local].sum()
        say(f"[routes] local {n_local}: E {abs(float(e) - want):.2e}")
        assert abs(float(e) - want) <= 1e-10 * np.abs(r["atom_e"]).sum()
        assert np.abs(f[:CRYSTAL].cpu().numpy() - r["force"][:CRYSTAL]).max() <= 1e-9


@pytest.mark.parametrize("thermo", [1, 4, 12])
def test_md_passes_beyond_the_range(thermo):
    """Two atoms fired at each other come within 0.01 A at step 7 and part
    again.  The run restarts at that step (its later steps count twice) and
    follows the oracle's Verlet run: 1e-7 A, and relative in the velocities
    and energies 1e-6 (FP64 rounding amplified by the stiff encounter)."""
    from oracle import oracle as O
    spec = synth.copper_model(1)
    x = np.array([[9.0, 9.0, 9.0], [9.69, 9.005, 9.0], [13.0, 10.0, 8.0]])
    v = np.array([[0.2, 0.0, 0.0], [-0.2, 0.0, 0.0], [0.0, 0.0, 0.0]])
    t, box, nst = np.zeros(3, dtype=np.int32), np.full(3, 21.0), 12
    ora = O.Oracle(synth.pack_blob(spec))
    dist = []
    for k in range(nst + 1):
        y = ora.verlet(x, v, t, box, [63.546], 0.25, k, every=0)[0]
        dist.append(float(np.linalg.norm(y[0] - y[1])))
    assert min(dist) < 0.02 and int(np.argmin(dist)) == 7 and dist[0] > 0.5 and dist[-1] > 0.3
    xo, vo, tho = ora.verlet(x, v, t, box, [63.546], 0.25, nst, every=thermo)
    m = _model(spec, "fp64")
    xg, vg = torch.tensor(x, device="cuda"), torch.tensor(v, device="cuda")
    th = m.md_run(xg, vg, t, box, [63.546], 0.25, nst, skin=1.0, thermo_every=thermo).cpu().numpy()
    dx, dv = np.abs(xg.cpu().numpy() - xo).max(), np.abs(vg.cpu().numpy() - vo).max()
    ev = m.stats()["evaluations"]
    say(f"[routes] MD past {min(dist):.3f} A: x {dx:.2e}, v {dv:.2e}, {ev} evaluations")
    assert ev == nst + -(-7 // thermo) * thermo - 7  # the steps from 7 to the next check, once more
    assert dx <= 1e-7 and dv <= 1e-7 * max(1.0, np.abs(vo).max())
    assert np.abs(th[:, 1:5] - tho[:, 1:5]).max() <= 1e-6 * np.abs(tho[:, 1:5]).max()


def test_md_starts_beyond_the_range():
    """The first frame already holds the far pair (a run of no steps too)."""
    from oracle import oracle as O
    spec = synth.copper_model(1)
    x = np.array([[9.0, 9.0, 9.0], [9.015, 9.0, 9.005], [13.0, 10.0, 8.0]])
    t, box = np.zeros(3, dtype=np.int32), np.full(3, 21.0)
    ora = O.Oracle(synth.pack_blob(spec))
    for nst in (0, 2):
        xo, vo, tho = ora.verlet(x, 0 * x, t, box, [63.546], 0.01, nst, every=1)
        m = _model(spec, "fp64")
        xg, vg, fg = (torch.tensor(a, device="cuda") for a in (x, 0 * x, 0 * x))
        th = m.md_run(xg, vg, t, box, [63.546], 0.01, nst, skin=1.0, thermo_every=1, forces=fg).cpu().numpy()
        r = ora.eval(xo, t, box)
        df = np.abs(fg.cpu().numpy() - r["force"]).max() / np.abs(r["force"]).max()
        say(f"[routes] MD from a far pair, {nst} steps: F {df:.2e}, x {np.abs(xg.cpu().numpy() - xo).max():.2e}")
        assert np.abs(xg.cpu().numpy() - xo).max() <= 1e-9 and df <= 1e-7
        assert np.abs(th[:, 1:5] - tho[:, 1:5]).max() <= 1e-8 * np.abs(tho[:, 1:5]).max()


# ---------------------------------------------------------------------------
# change of precision
# ---------------------------------------------------------------------------
def test_precision_changes_with_a_student():
    """Through every precision and back, teacher and student: energies bit for
    bit those of a context that was loaded in that precision, forces but for
    the atomics' order."""
    w = synth.workload("water192")
    spec = w["spec"]
    sblob = synth.pack_blob(synth.student_spec(spec, synth.random_student_params(spec, 12)))

    def both(m):
        out = []
        for use in (False, True):
            m.student_use(use)
            e, f, _ = m.compute(w["coords"], w["types"], w["box"])
            out.append((float(e), f.cpu().numpy()))
        return out

    want = {}
    for prec in ("fp64", "fp32", "fp16", "bf16"):
        fresh = _model(spec, prec)
        fresh.student_set_model(sblob)
        fresh.student_table(False)
        want[prec] = both(fresh)
    m = _model(spec, "fp64")
    m.student_set_model(sblob)
    m.student_table(False)
    for prec in ("fp32", "fp64", "bf16", "fp64", "fp16", "fp32", "bf16", "fp16", "fp64"):
        m.set_precision(prec)
        for (e, f), (e0, f0) in zip(both(m), want[prec]):
            say(f"[routes] to {prec}: E {abs(e - e0):.1e}, F {np.abs(f - f0).max():.1e}")
            assert e == e0 and np.abs(f - f0).max() <= 1e-11


def test_precision_change_lays_nothing_out_twice():
    """FP64 to FP32 and back once both have been used: the tables are there.
    (Laying the water nets' out takes 20 ms and more.)"""
    import time
    m = _model(synth.workload("water192")["spec"], "fp64")
    m.set_precision("fp32")
    took = []
    for k in range(10):
        t0 = time.perf_counter()
        m.set_precision("fp32" if k & 1 else "fp64")
        took.append(time.perf_counter() - t0)
    say(f"[routes] change of precision {min(took) * 1e3:.3f} .. {max(took) * 1e3:.3f} ms")
    assert sorted(took)[5] <= 2e-3


# ---------------------------------------------------------------------------
# workspaces
# ---------------------------------------------------------------------------
def test_only_users_of_expansions_carry_their_buffers():
    """Device memory of an evaluation of 12,288 water atoms: BF16, whose nets
    have no expansion, takes 6 KB an atom less than FP16, whose nets have (of
    the same layout otherwise)."""
    import gc
    w = synth.workload("water12288")
    took = {}
    gc.collect()  # no context of an earlier test is freed in between
    for prec in ("bf16", "fp16"):
        m = _model(w["spec"], prec)
        x, t = torch.tensor(w["coords"], device="cuda"), torch.tensor(w["types"], device="cuda")
        m.compute(x[:192], t[:192], w["box"])  # what is not the workspace
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        m.compute(x, t, w["box"])
        torch.cuda.synchronize()
        took[prec] = free - torch.cuda.mem_get_info()[0]
        del m
    say(f"[routes] workspace bf16 {took['bf16'] / 2**20:.0f} MiB, fp16 {took['fp16'] / 2**20:.0f} MiB")
    assert took["fp16"] - took["bf16"] >= 5000 * 12288


def test_noalloc_route_is_the_calls_own():
    """No-allocation calls: a system too large to have the expansions' buffers
    beside its own leaves none of its route to the small one after it, whose
    energy is bit for bit that of a context's first call.  FP16, where the two
    routes differ in digits that a sum of energies shows (bars of the FP16 tests:
    2^-14 of the energy, force RMSE 1e-3 eV/A)."""
    from paper_2005_00223_amd import _lib as L

    def run(ctx, x, t, box):
        xd, td = torch.tensor(x, device="cuda"), torch.tensor(t, device="cuda")
        e, f, v = (torch.zeros(k, dtype=torch.float64, device="cuda") for k in (1, 3 * len(x), 9))
        L.dp_compute_noalloc(ctx, len(x), xd.data_ptr(), td.data_ptr(), [box[0], 0, 0, 0, box[1], 0, 0, 0, box[2]],
                             e.data_ptr(), f.data_ptr(), v.data_ptr())
        torch.cuda.synchronize()
        return e.item(), f.cpu().numpy().reshape(-1, 3)

    small = synth.workload("water192")
    blob = synth.pack_blob(small["spec"])
    bx, bt, bbox = synth.water_system(19, 19 * 3.105, 0.1, seed=6)
    out = []
    for first in (None, (bx, bt, bbox)):
        ctx = L.dp_create(0, torch.cuda.current_stream().cuda_stream)
        L.dp_set_model(ctx, blob, L.PRECISION["fp16"])
        if first:
            eb, fb = run(ctx, *first)
            m = _model(small["spec"], "fp16")
            e0, f0, _ = m.compute(*first)
            rmse = np.sqrt(((fb - f0.cpu().numpy()) ** 2).sum(1).mean())
            say(f"[routes] noalloc {len(bt)} atoms: E {abs(eb / float(e0) - 1):.1e}, F RMSE {rmse:.1e}")
            assert 0.0 < abs(eb / float(e0) - 1) <= 2.0 ** -14 and rmse <= 1e-3
        out.append(run(ctx, small["coords"], small["types"], small["box"]))
        L.dp_destroy(ctx)
    (e1, f1), (e2, f2) = out
    say(f"[routes] noalloc water192 first / after the large one: E {abs(e1 - e2):.1e}, F {np.abs(f1 - f2).max():.1e}")
    assert e1 == e2 and np.abs(f1 - f2).max() <= 1e-12


# ---------------------------------------------------------------------------
# MD: from the layers back to the expansions
# ---------------------------------------------------------------------------
def test_md_returns_to_the_expansions():
    """Two pairs meet in turn, at steps 7 and 15 (checks every 4 steps): each
    restarts the run, so between them it was back on the expansions.  Step 8
    and step 16 count twice; the trajectory is the oracle's."""
    from oracle import oracle as O
    spec = synth.copper_model(1)
    x = np.array([[9.0, 9.0, 9.0], [9.69, 9.005, 9.0], [13.0, 10.0, 8.0], [30.0, 9.0, 9.0], [31.5, 9.005, 9.0]])
    v = np.array([[0.2, 0.0, 0.0], [-0.2, 0.0, 0.0], [0.0, 0.0, 0.0], [0.2, 0.0, 0.0], [-0.2, 0.0, 0.0]])
    t, box, nst = np.zeros(5, dtype=np.int32), np.array([44.0, 21.0, 21.0]), 20
    ora = O.Oracle(synth.pack_blob(spec))
    near = []
    for k in range(nst + 1):
        y = ora.verlet(x, v, t, box, [63.546], 0.25, k, every=0)[0]
        near.append(min(np.linalg.norm(y[0] - y[1]), np.linalg.norm(y[3] - y[4])))
    assert [k for k in range(nst + 1) if near[k] < 1.0 / 32.0] == [7, 15]
    xo, vo, tho = ora.verlet(x, v, t, box, [63.546], 0.25, nst, every=4)
    m = _model(spec, "fp64")
    xg, vg = torch.tensor(x, device="cuda"), torch.tensor(v, device="cuda")
    th = m.md_run(xg, vg, t, box, [63.546], 0.25, nst, skin=1.0, thermo_every=4).cpu().numpy()
    dx, dv, ev = np.abs(xg.cpu().numpy() - xo).max(), np.abs(vg.cpu().numpy() - vo).max(), m.stats()["evaluations"]
    say(f"[routes] MD, two meetings: x {dx:.2e}, v {dv:.2e}, {ev} evaluations")
    assert ev == nst + 2
    assert dx <= 1e-7 and dv <= 1e-7 * max(1.0, np.abs(vo).max())
    assert np.abs(th[:, 1:5] - tho[:, 1:5]).max() <= 1e-6 * np.abs(tho[:, 1:5]).max()


@pytest.mark.parametrize("thermo", [1, 3])
def test_md_of_a_pair_that_stays_beyond_the_range(thermo):
    """A pair that stays at 0.016 A: the returns to the expansions fail, ever
    more rarely, and the run goes on by the layers."""
    from oracle import oracle as O
    spec = synth.copper_model(1)
    x = np.array([[9.0, 9.0, 9.0], [9.015, 9.0, 9.005], [13.0, 10.0, 8.0]])
    t, box, nst = np.zeros(3, dtype=np.int32), np.full(3, 21.0), 24
    ora = O.Oracle(synth.pack_blob(spec))
    xo, vo, tho = ora.verlet(x, 0 * x, t, box, [63.546], 0.002, nst, every=thermo)
    assert np.linalg.norm(xo[0] - xo[1]) < 1.0 / 32.0
    m = _model(spec, "fp64")
    xg, vg = (torch.tensor(a, device="cuda") for a in (x, 0 * x))
    th = m.md_run(xg, vg, t, box, [63.546], 0.002, nst, skin=1.0, thermo_every=thermo).cpu().numpy()
    dx = np.abs(xg.cpu().numpy() - xo).max()
    say(f"[routes] MD at 0.016 A: x {dx:.2e}, {m.stats()['evaluations']} evaluations")
    assert dx <= 1e-9
    assert np.abs(th[:, 1:5] - tho[:, 1:5]).max() <= 1e-8 * np.abs(tho[:, 1:5]).max()


# ---------------------------------------------------------------------------
# expansions in company they had not been seen in
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("reps", [(1, 1, 1), (5, 5, 1)])
@pytest.mark.parametrize("fit,M2", [((40,), 16), ((120, 240), 16), ((24, 24, 24), 5), ((272, 272), 16)])
def test_layer_fitting_nets_behind_expansions(fit, M2, reps, prec):
    """Fitting nets the fused kernels do not take (a width that is not a
    multiple of 16 or above 256, a doubling skip): D and dE/dD in memory between
    the expansions and the layer GEMMs."""
    spec = synth.random_model(2, 4.5, 2.0, (64, 64), M2=M2, fit=fit, seed=22, out_scale=-8.0, desc_norm=2.0)
    x, t, box = _cell()
    r = _oracle(spec, x, t, box, prec)
    X, T, B, copies, order = _repeat(x, t, box, reps)
    say(f"[routes] fitting {fit}, M2 {M2}, {prec}: {len(X)} atoms")
    _compare(_model(spec, prec).compute(X, T, B), r, prec, f"{fit}", copies, order)


@pytest.mark.parametrize("ntypes,prec", [(3, "fp64"), (4, "fp64"), (4, "fp32"), (6, "fp32"), (8, "fp32")])
@pytest.mark.parametrize("reps", [(1, 1, 1), (5, 5, 1)])
def test_many_types(ntypes, prec, reps):
    """Three types in double, four and six in float on expansions (tests of the
    tables say which have them), four in double and eight in float by the layers."""
    spec = synth.random_model(ntypes, 4.5, 2.0, (32,) * ntypes, seed=5, out_scale=-8.0, desc_norm=2.0)
    x, t, box = _cell(ntypes)
    r = _oracle(spec, x, t, box, prec)
    X, T, B, copies, order = _repeat(x, t, box, reps)
    say(f"[routes] {ntypes} types, {prec}: {len(X)} atoms")
    _compare(_model(spec, prec).compute(X, T, B), r, prec, f"{ntypes} types", copies, order)


# bars of the FP16 tests' kernel arithmetic, against the oracle on the weights
# the kernels hold: 2^-14, here of the largest force and virial component and of
# the summed |E_i|
FP16_BAR = 2.0 ** -14


@pytest.mark.parametrize("order", ["lattice", "shuffled"])
def test_merged_scatter_fp16(order):
    """4,000 atoms in FP16, forces merged in LDS: copies of a cell of 500."""
    from oracle import oracle as O
    from oracle import student as S
    x, t, box = synth.fcc_copper(5, 3.634, 0.1, seed=4)
    spec = synth.copper_model(1)
    r = O.Oracle(synth.pack_blob(S.round_spec16(spec, 0))).eval(x, t, box)
    X, T, B, copies, p = _repeat(x, t, box, (4, 2, 1), seed=1)
    if order == "lattice":
        back = np.argsort(p)
        X, T, p = X[back], T[back], np.arange(len(p))
    e, f, v = _model(spec, "fp16").compute(X, T, B)
    want = np.tile(r["force"], (copies, 1))[p]
    df = np.abs(f.cpu().numpy() - want).max() / np.abs(want).max()
    de = abs(float(e) / copies - r["energy"]) / np.abs(r["atom_e"]).sum()
    dv = np.abs(v.cpu().numpy() / copies - r["virial"]).max() / np.abs(r["virial"]).max()
    say(f"[routes] merged scatter fp16 {order}: F {df:.2e}, E {de:.2e}, V {dv:.2e}")
    assert max(df, de, dv) <= FP16_BAR


@pytest.mark.parametrize("count", [1, 15, 16, 17, 63, 64, 65, 127, 129, 200])
def test_neighbour_counts_fp16(count):
    """A cluster of count + 1 atoms, every one the others' neighbour, several
    pieces in each list; a first fitting layer scaled down so that its tanh does
    not saturate (1 - t^2 of a saturated one loses the digits that this test
    looks at).  Forces and energy; the virial of a cluster is a small difference."""
    from oracle import oracle as O
    from oracle import student as S
    spec = synth.random_model(1, 7.0, 3.0, (256,), seed=6, out_scale=-20.0, desc_norm=8.0 + count / 2.0)
    spec.fit_W[0][0] = spec.fit_W[0][0] * 0.1
    rng = np.random.default_rng(count)
    g = np.stack(np.meshgrid(*[np.arange(6)] * 3, indexing="ij"), -1).reshape(-1, 3)
    g = g[np.argsort(((g - 2.5) ** 2).sum(1), kind="stable")][:count + 1]
    x = 0.85 * g + rng.uniform(-0.1, 0.1, size=g.shape) + 8.0
    t, box = np.zeros(count + 1, dtype=np.int32), np.full(3, 22.0)
    r = O.Oracle(synth.pack_blob(S.round_spec16(spec, 0))).eval(x, t, box)
    e, f, _ = _model(spec, "fp16").compute(x, t, box)
    df = np.abs(f.cpu().numpy() - r["force"]).max() / np.abs(r["force"]).max()
    de = abs(float(e) - r["energy"]) / np.abs(r["atom_e"]).sum()
    say(f"[routes] fp16 cluster of {count + 1}: F {df:.2e}, E {de:.2e}")
    assert max(df, de) <= FP16_BAR


def test_judge_meets_a_far_pair():
    """FP16: the student's layers take a pair at 0.02 A, the judging teacher's
    expansions do not; the run starts again on the layers and the RMSE is that
    of the two nets' own evaluations (1e-6 relative: atomics' order)."""
    x, t, box = _frame("pair")
    spec = synth.copper_model(1)
    m = _model(spec, "fp16")
    m.student_set_model(synth.pack_blob(synth.student_spec(spec, synth.random_student_params(spec, 31))))
    m.student_table(False)
    _, ft, _ = m.compute(x, t, box)
    m.student_use(True)
    _, fs, _ = m.compute(x, t, box)
    expect = float(((fs - ft) ** 2).sum(1).mean().sqrt())
    m.student_judge(20, 1e9)
    xg = torch.tensor(x, device="cuda")
    m.md_run(xg, torch.zeros_like(xg), t, box, [63.546], 1e-3, 0, skin=0.5, thermo_every=1)
    st = m.stats()
    say(f"[routes] judge with a far pair: RMSE {st['last_judge_rmse']:.9e}, expected {expect:.9e}")
    assert abs(st["last_judge_rmse"] - expect) <= 1e-6 * expect and st["teacher_fallbacks"] == 0
