"""Host side of the embedding nets' expansions: the tables against the nets
themselves in extended precision, over the whole range of s.

Bars, set before the first run.  Double: a sum of 16 Chebyshev terms in double,
each of them at most about the largest feature (slope): 2^-49 of it.  Float
tables, summed in double here: the last two coefficients of 2^-25 each and the
rounding of twelve coefficients to float: 2^-21."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2005_00223_amd import build, synth

HERE = os.path.dirname(os.path.abspath(__file__))
PMAX, KP = 32, 16


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("native") / "expand_host.so")
    subprocess.run([build.hipcc(), "-x", "hip", "--offload-host-only", "-O3", "-std=c++17", "-fPIC", "-shared",
                    "-I", build.CSRC, os.path.join(HERE, "native", "expand_host.cpp"),
                    os.path.join(build.CSRC, "expand.cpp"), "-o", so], check=True, capture_output=True)
    return ctypes.CDLL(so)


def _tables(lib, spec, f64):
    nets, w = spec.ntypes ** 2, np.array((1,) + tuple(spec.emb), dtype=np.int32)
    wt = np.concatenate([np.asarray(a, dtype=np.float64).ravel() for t in range(spec.ntypes)
                         for u in range(spec.ntypes)
                         for pair in zip(spec.emb_W[t][u], spec.emb_b[t][u]) for a in pair])
    if not f64:
        wt = wt.astype(np.float32).astype(np.float64)
    M1p = (spec.M1 + 15) // 16 * 16
    P, smax = ctypes.c_int(), ctypes.c_double()
    lo, mid, ih, C = (np.zeros(nets * PMAX * k) for k in (1, 1, 1, 2 * KP * M1p))
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    if not lib.expand_host(spec.ntypes, len(spec.emb), ptr(w), int(spec.emb_out_linear), ptr(wt), int(f64),
                           ctypes.byref(P), ctypes.byref(smax), ptr(lo), ptr(mid), ptr(ih), ptr(C)):
        return None
    n = nets * P.value
    return dict(smax=smax.value, lo=lo[:n].reshape(nets, -1), mid=mid[:n].reshape(nets, -1),
                ih=ih[:n].reshape(nets, -1), C=C[:n * 2 * KP * M1p].reshape(nets, P.value, 2, KP, M1p))


def _net(spec, t, u, s, dt):
    """G and dG/ds of net (t, u) in the real type dt."""
    h = s.astype(dt)[:, None]
    hd = np.ones_like(h)
    for k, (W, b) in enumerate(zip(spec.emb_W[t][u], spec.emb_b[t][u])):
        z, zd = h @ np.asarray(W).astype(dt) + np.asarray(b).astype(dt), hd @ np.asarray(W).astype(dt)
        if not (spec.emb_out_linear and k + 1 == len(spec.emb)):
            z = np.tanh(z)
            zd = zd * (1 - z * z)
            if z.shape[1] == h.shape[1]:
                z, zd = z + h, zd + hd
            elif z.shape[1] == 2 * h.shape[1]:
                z, zd = z + np.concatenate([h, h], 1), zd + np.concatenate([hd, hd], 1)
        h, hd = z, zd
    return h, hd


def _sum(tab, net, s, M1):
    """G and dG/ds by the expansion, in double."""
    p = np.searchsorted(tab["lo"][net], s, side="right") - 1
    x = ((s - tab["mid"][net][p]) * tab["ih"][net][p])[:, None]
    C = tab["C"][net][p]
    out = []
    for w in range(2):
        t0, t1 = np.ones_like(x), x
        g = C[:, w, 0] + x * C[:, w, 1]
        for k in range(2, KP):
            t0, t1 = t1, 2 * x * t1 - t0
            g = g + t1 * C[:, w, k]
        out.append(g[:, :M1])
    return out


def _models():
    return {"copper": synth.copper_model(1), "water": synth.water_model(0),
            "three types": synth.random_model(3, 6.0, 2.0, (20, 20, 20), seed=5),
            "128 wide": synth.random_model(1, 8.0, 2.0, (64,), emb=(128, 128, 128), seed=2)}


@pytest.mark.parametrize("f64", [True, False])
@pytest.mark.parametrize("name", ["copper", "water", "three types", "128 wide"])
def test_tables_against_the_nets(lib, name, f64):
    spec = _models()[name]
    tab = _tables(lib, spec, f64)
    assert tab is not None and tab["smax"] >= 12.0
    bar = 2.0 ** -49 if f64 else 2.0 ** -21
    ref = spec
    if not f64:
        ref = synth.random_model(spec.ntypes, 6.0, 2.0, spec.sel, emb=spec.emb, seed=spec.seed)
        f32 = lambda v: np.asarray(v, dtype=np.float32).astype(np.float64)
        ref.emb_W = [[[f32(W) for W in ws] for ws in row] for row in spec.emb_W]
        ref.emb_b = [[[f32(b) for b in bs] for bs in row] for row in spec.emb_b]
        tab = dict(tab, C=f32(tab["C"]))
    rng = np.random.default_rng(1)
    for t in range(spec.ntypes):
        for u in range(spec.ntypes):
            for a, b in ((0.0, 1.0), (1.0, 8.0), (8.0, tab["smax"])):
                s = rng.uniform(a, b, 800)
                want, got = _net(ref, t, u, s, np.longdouble), _sum(tab, t * spec.ntypes + u, s, spec.M1)
                e = [float(np.abs(g - w).max() / np.abs(w).max()) for g, w in zip(got, want)]
                print(f"{name} ({t},{u}) s {a:g}..{b:g}: G {e[0]:.1e}, dG {e[1]:.1e}")
                assert max(e) <= bar, (t, u, a, b, e)


def _steeper(spec, f):
    for row in spec.emb_W:
        for W in row:
            W[0] = W[0] * f
    return spec


# model, has a double table, has a float table: nets that put an atom's ordinary
# neighbours (beyond 1 A) in more than eight pieces have none
RANGE = [(lambda: synth.random_model(3, 6.0, 2.0, (20,) * 3, seed=5), True, True),
         (lambda: synth.random_model(4, 6.0, 2.0, (20,) * 4, seed=5), False, True),
         (lambda: synth.random_model(8, 6.0, 2.0, (20,) * 8, seed=5), False, False),
         (lambda: _steeper(synth.copper_model(1), 4.0), False, True),
         (lambda: _steeper(synth.copper_model(1), 24.0), False, False)]


@pytest.mark.parametrize("which", range(len(RANGE)))
def test_which_nets_have_tables(lib, which):
    make, f64, f32 = RANGE[which]
    assert (_tables(lib, make(), True) is not None) == f64
    assert (_tables(lib, make(), False) is not None) == f32
