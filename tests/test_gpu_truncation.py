"""The truncation kernels at the edges of their blockings, against the oracle.

Decaying boundary spectra (a product state plus a Gaussian PEPS) take every branch of the
truncation step: the Gram eigenproblem, and the refinement of the kept subspace wherever a kept
eigenvalue falls below 1e-6 of the largest.  The bounds are those of the float64 path: 1e-10
relative on ln|W|, 1e-9 on E and on the log-derivatives.
"""
import json
import os

import numpy as np
import pytest

import oracle as O
from paper_1806_03761_amd.workloads import Lattice, make_random, make_workload

pytestmark = pytest.mark.gpu


def _weak(lat, batch, seed, eps):
    A, S = make_random(lat, batch, seed)
    A = eps * A
    A[:, :, 0, 0, 0, 0] += np.random.default_rng(seed).uniform(0.5, 1.5, size=(lat.N, 2))
    return A, S


def _peps():
    import torch
    from paper_1806_03761_amd import peps
    assert torch.cuda.is_available()
    return peps


def _dev(*xs):
    import torch
    return [torch.from_numpy(x).to("cuda:0") for x in xs]


# (Lx, Ly, D, Dc): one per register blocking of the refinement, with kept counts on both sides
# of a wave's 16 columns and orders that do and do not fill their 16-row chunks
@pytest.mark.parametrize("shape", [(5, 4, 2, 4), (6, 4, 3, 7), (5, 5, 4, 16), (5, 4, 4, 17), (5, 4, 5, 25),
                                   (5, 4, 6, 36), (4, 4, 7, 43), (4, 4, 8, 33), (3, 4, 16, 32)])
@pytest.mark.parametrize("eps", [0.3, 0.02])
def test_truncation_of_decaying_spectra(shape, eps):
    Lx, Ly, D, Dc = shape
    lat = Lattice(Lx, Ly, D, Dc)
    A, S = _weak(lat, 2, 60 + D, eps)
    la, sg, e, d, fl = (t.cpu().numpy() for t in _peps().evaluate(*_dev(A, S), lat, "f64", grad_mode=1))
    for b in range(len(S)):
        la_o, sg_o, e_o, d_o, fl_o = O.full_path_one(A, lat, S[b])
        assert fl[b] == 0 and fl_o == 0 and sg[b] == sg_o
        assert abs(la[b] - la_o) <= 1e-10 * max(1, abs(la_o)), (shape, b, la[b], la_o)
        assert abs(e[b] - e_o) <= 1e-9 * max(1, abs(e_o)), (shape, b, e[b], e_o)
        assert np.linalg.norm(d[b] - d_o) <= 1e-9 * np.linalg.norm(d_o), (shape, b)


# batches on both sides of every change of the eigenvalue kernel's launch shape (points per
# eigenvalue, matrices per block, one launch or two): each sample equals its own single call
# bit for bit
@pytest.mark.parametrize("shape,batch", [((4, 4, 2, 4), 3000), ((5, 4, 4, 16), 1500), ((5, 4, 4, 16), 5000),
                                         ((4, 4, 5, 25), 600), ((4, 3, 6, 36), 300)])
def test_truncation_independent_of_the_batch(shape, batch):
    Lx, Ly, D, Dc = shape
    lat = Lattice(Lx, Ly, D, Dc)
    A, S = make_random(lat, batch, 70 + D)
    peps = _peps()
    Ad, Sd = _dev(A, S)
    la, sg, fl = peps.log_amplitude(Ad, Sd, lat)
    for b in (0, 1, 63, batch // 2, batch - 1):
        l1, s1, f1 = peps.log_amplitude(Ad, Sd[b:b + 1].contiguous(), lat)
        assert int(f1[0]) == int(fl[b]) == 0 and int(s1[0]) == int(sg[b])
        assert float(l1[0]) == float(la[b])


# column tensors at the row counts where the blocked R factor changes its blocking (128-row tiles
# of its eight waves, 16-column panels above 1408 rows, row blocks above 2048) and at column
# counts that leave a part of a 32- or 16-column panel; more columns than rows in the first row
@pytest.mark.parametrize("shape", [(8, 5, 5, 21), (8, 5, 5, 25), (8, 5, 6, 33), (8, 5, 6, 36), (6, 5, 7, 43),
                                   (6, 4, 7, 49), (7, 4, 8, 64), (4, 3, 9, 50), (4, 3, 12, 20), (4, 3, 16, 17),
                                   (4, 4, 16, 32)])
def test_blocked_r_factor(shape):
    Lx, Ly, D, Dc = shape
    lat = Lattice(Lx, Ly, D, Dc)
    A, S = make_random(lat, 2, 80 + D)
    la, sg, fl = (t.cpu().numpy() for t in _peps().log_amplitude(*_dev(A, S), lat, "f64"))
    la_o, sg_o, fl_o = O.log_amplitude(A, lat, S)
    assert not fl.any() and not np.any(fl_o) and np.array_equal(sg, sg_o)
    assert np.all(np.abs(la - la_o) <= 1e-10 * np.maximum(1, np.abs(la_o)))


# the float64 products computed from registers (the untuned choice) against the LDS-staged
# kernel (tile 4), which sum every output alike: equal bits over odd legs and bonds (a K that 4
# does not divide, split indices of 2 to 7, ragged edges of every block shape), with scattered
# operands and samples a power of two apart, and both boundary methods
@pytest.mark.parametrize("case", [(4, 4, 2, 3, 5, 0), (5, 4, 3, 7, 33, 0), (4, 5, 5, 17, 9, 0),
                                  (4, 3, 7, 19, 2, 0), (4, 5, 3, 9, 300, 2),
                                  (5, 4, 6, 30, 7, 1), (4, 4, 2, 1, 700, 0),
                                  (4, 4, 8, 16, 3, 0), (4, 3, 16, 12, 2, 1)])
def test_register_products_equal_staged(case, tmp_path):
    Lx, Ly, D, Dc, batch, sweeps = case
    p, lat = _peps(), Lattice(Lx, Ly, D, Dc)
    A, S = make_random(lat, batch, 300 + D)
    Ad, Sd = _dev(A, S)
    keys, saved, path = [], str(tmp_path / "saved.txt"), str(tmp_path / "t.txt")
    p.tune_save(saved)
    p.set_truncation(sweeps)
    try:
        base = [t.cpu().numpy() for t in p.evaluate(Ad, Sd, lat, "f64", grad_mode=3)]
        p.autotune(Ad, Sd, lat, "f64")
        p.tune_save(path)
        keys = [ln.split()[0] for ln in open(path) if ln.strip() and not ln.startswith("#")]
        with open(path, "w") as f:
            f.writelines(f"{k} 4\n" for k in keys)
        p.tune_load(path)
        got = [t.cpu().numpy() for t in p.evaluate(Ad, Sd, lat, "f64", grad_mode=3)]
    finally:
        with open(path, "w") as f:
            f.writelines(f"{k} 0\n" for k in keys)
        p.tune_load(path)
        p.tune_load(saved)
        p.set_truncation(0)
    assert keys
    for x, y in zip(got, base):
        assert np.array_equal(x, y)


# the fused float64 sandwich steps against their GEMM form, both of which sum every output in
# one order: one workgroup per sample (rescaling in the kernel) and several, a last block of
# fewer free bond values, legs of 1 at the edges, bonds up to the last that one workgroup's
# scratch holds and past it, and legs beyond the fused form
@pytest.mark.parametrize("case", [(3, 3, 2, 2, 1), (4, 4, 2, 5, 700), (5, 4, 3, 9, 37), (4, 5, 3, 23, 9),
                                  (5, 5, 4, 13, 33), (6, 4, 4, 16, 5), (4, 4, 4, 33, 6), (4, 4, 4, 64, 3),
                                  (4, 3, 5, 20, 4), (2, 4, 4, 16, 6), (4, 2, 3, 9, 6)])
def test_fused_float64_steps_equal_products(case):
    Lx, Ly, D, Dc, batch = case
    p, lat = _peps(), Lattice(Lx, Ly, D, Dc)
    A, S = make_random(lat, batch, 500 + D)
    Ad, Sd = _dev(A, S)
    base = [t.cpu().numpy() for t in p.evaluate(Ad, Sd, lat, "f64", grad_mode=1)]
    p.set_fused_steps(False)
    try:
        got = [t.cpu().numpy() for t in p.evaluate(Ad, Sd, lat, "f64", grad_mode=1)]
    finally:
        p.set_fused_steps(True)
    for x, y in zip(got, base):
        assert np.array_equal(x, y, equal_nan=True)


# site factorisations of the variational compression at the edges of their register blockings
# (256 x 40, 512 x 32 and 512 x 64; n = 8, 16, 32 and 40 are whole slots of eight waves)
@pytest.mark.parametrize("case", [(4, 4, 7, 36), (4, 4, 7, 37), (4, 4, 8, 32), (4, 4, 10, 30), (4, 4, 12, 33),
                                  (4, 4, 13, 20), (4, 4, 5, 8), (4, 4, 4, 9)])
def test_register_site_factorisations(case):
    Lx, Ly, D, Dc = case
    p, lat = _peps(), Lattice(Lx, Ly, D, Dc)
    A, S = _weak(lat, 2, 900 + D, 0.3 / D ** 2)
    p.set_truncation(1)
    try:
        la, sg, fl = (t.cpu().numpy() for t in p.log_amplitude(*_dev(A, S), lat, "f64"))
    finally:
        p.set_truncation(0)
    assert not fl.any()
    for b in range(len(S)):
        la_o, sg_o, fl_o = O.log_amplitude_one(A, lat, S[b], 1)
        assert fl_o == 0 and int(sg[b]) == int(sg_o)
        assert abs(la[b] - la_o) <= 1e-10 * max(1.0, abs(la_o))


# rescaling and overlap of partials around the 8192 entries where 1024 threads take over: two-row
# partials of 36 36 6 6 entries, of 15 15 6 6 = 8100, 16 16 6 6 and 13 13 7 7 = 8281, against the oracle
@pytest.mark.parametrize("case", [(4, 4, 6, 36), (4, 4, 6, 15), (4, 4, 6, 16), (4, 4, 7, 13)])
def test_long_partials(case):
    Lx, Ly, D, Dc = case
    lat = Lattice(Lx, Ly, D, Dc)
    A, S = _weak(lat, 2, 950 + D, 0.3 / D ** 2)
    la, sg, e, g, fl = (t.cpu().numpy() for t in _peps().evaluate(*_dev(A, S), lat, "f64", grad_mode=1))
    assert not fl.any()
    for b in range(len(S)):
        la_o, sg_o, e_o, d_o, fl_o = O.full_path_one(A, lat, S[b])
        assert fl_o == 0 and int(sg[b]) == int(sg_o)
        assert abs(la[b] - la_o) <= 1e-10 * max(1.0, abs(la_o))
        assert abs(e[b] - e_o) <= 1e-9 * max(1.0, abs(e_o))
        assert np.linalg.norm(g[b] - d_o) <= 1e-9 * np.linalg.norm(d_o)


# ln|W| is exact under scalings of the site tensors, far beyond the squares of doubles: a leading
# bond index between two columns made negligible (zero, or `s` of the others) or carried by its
# neighbour (s on one side, 1 / s on the other: the state is unchanged), the left half of the lattice
# s per site against 1 / s in the right, and all sites small.  Column tensors with R by register
# panels, R from the small kernels, and centres tridiagonalised in memory (order 320).
@pytest.mark.parametrize("shape", [(6, 5, 6, 36), (6, 5, 4, 16), (6, 4, 8, 40)])
@pytest.mark.parametrize("kind,s", [("drop", 0.0), ("drop", 1e-40), ("drop", 1e-100), ("carry", 1e-40),
                                    ("carry", 1e-100), ("carry", 1e-150), ("halves", 1e-30), ("all", 1e-20)])
def test_scaled_site_tensors(shape, kind, s):
    Lx, Ly, D, Dc = shape
    lat = Lattice(Lx, Ly, D, Dc)
    A, S = make_random(lat, 1, 990 + D)
    A = A.reshape(Ly, Lx, 2, D, D, D, D)   # legs left, up, right, down
    B, shift = A.copy(), 0.0
    if kind in ("drop", "carry"):
        B[:, 2, :, :, :, 0] *= s
        if kind == "carry":
            B[:, 3, :, 0] *= 1.0 / s
    elif kind == "halves":
        B[:, :Lx // 2] *= s
        B[:, Lx // 2:] *= 1.0 / s
    else:
        B *= s
        shift = lat.N * np.log(s)
    A, B = (x.reshape(lat.N, 2, D, D, D, D) for x in (A, B))
    la, sg, fl = (t.cpu().numpy() for t in _peps().log_amplitude(*_dev(B, S), lat, "f64"))
    la_o, sg_o, fl_o = O.log_amplitude_one(B if kind == "drop" else A, lat, S[0])
    assert fl_o == 0 and fl[0] == 0 and int(sg[0]) == int(sg_o)
    assert abs(la[0] - shift - la_o) <= 1e-10 * max(1.0, abs(la_o), abs(shift)), (la[0], shift, la_o)


# The headline lattice.  A few configurations in a thousand magnify rounding by more than 1e5 (their W
# is small by cancellation: the share above a deviation x falls as 1/x), so ln|W| is held to values in
# extended precision, the most sensitive five of the workload's first 1024 and two ordinary ones,
# within ten times the oracle's own largest deviation from them ...
def test_amplitudes_against_extended_precision():
    with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "extended_16x16_D6_Dc36.json")) as f:
        g = json.load(f)["samples"]
    lat, A, S, _ = make_workload("16x16_D6_Dc36")
    la, _, fl = (t.cpu().numpy() for t in _peps().log_amplitude(*_dev(A, S[[r["index"] for r in g]]), lat, "f64"))
    assert not fl.any()
    for r, x in zip(g, la):
        assert abs(x - r["log_abs"]) <= max(1e-10 * abs(r["log_abs"]), 10 * max(r["oracle_off"])), (r["index"], x)


# ... and over 512 configurations to itself under a compensated scaling of the sites, which a LAPACK
# sweep moves by 1e-10 (median) and, by the 1/x tail, by more than 1e-6 in one of 1e4
def test_amplitude_noise_over_many_configurations():
    lat, A, S, _ = make_workload("16x16_D6_Dc36", 512)
    f = np.random.default_rng(41).uniform(0.5, 2.0, size=lat.N)
    p = _peps()
    la, _, fl = (t.cpu().numpy() for t in p.log_amplitude(*_dev(A, S), lat, "f64"))
    lb, _, fb = (t.cpu().numpy() for t in p.log_amplitude(*_dev(A * f[:, None, None, None, None, None], S), lat, "f64"))
    d = np.abs(lb - np.log(f).sum() - la)
    assert not fl.any() and not fb.any()
    assert np.median(d) <= 1e-9 and np.mean(d > 1e-6) <= 0.01, (np.median(d), np.sort(d)[-8:])


# products of one size whose operands are scattered or not (backward and forward site products at
# legs of 16) are timed apart, and a table saved without the distinction still serves both
def test_tuning_tells_scattered_products_apart(tmp_path):
    p, lat = _peps(), Lattice(4, 4, 16, 12)
    A, S = make_random(lat, 2, 316)
    Ad, Sd = _dev(A, S)
    keys, saved, path = [], str(tmp_path / "saved.txt"), str(tmp_path / "t.txt")

    def load(table):
        with open(path, "w") as f:
            f.writelines(f"{k} {t}\n" for k, t in table.items())
        p.tune_load(path)

    p.tune_save(saved)
    base = [t.cpu().numpy() for t in p.evaluate(Ad, Sd, lat, "f64", grad_mode=3)]
    try:
        p.autotune(Ad, Sd, lat, "f64")
        p.tune_save(path)
        keys = [ln.split()[0] for ln in open(path) if ln.strip() and not ln.startswith("#")]
        tuned = [t.cpu().numpy() for t in p.evaluate(Ad, Sd, lat, "f64", grad_mode=3)]
        load({k: 4 for k in keys if not k.endswith(",8")})
        plain = [t.cpu().numpy() for t in p.evaluate(Ad, Sd, lat, "f64", grad_mode=3)]
    finally:
        load({k: 0 for k in keys})
        p.tune_load(saved)
    apart = [k for k in keys if k.endswith(",8")]
    assert apart and all(k.split(",")[4] == "0" for k in apart)
    for x, y, z in zip(base, tuned, plain):
        assert np.array_equal(x, y) and np.array_equal(x, z)


# the lower boundary sweep beside the upper one against the two in turn on one stream (as they run
# while launches are timed): equal bits, over several chunks, on the default stream and on another,
# twice on each, with work of the caller before and after
@pytest.mark.parametrize("case", [(4, 4, 2, 4, 300, 0), (7, 5, 3, 10, 37, 0), (8, 8, 4, 16, 24, 0), (5, 6, 6, 20, 9, 0),
                                  (6, 6, 4, 16, 17, 1), (5, 5, 6, 20, 5, 2)])
def test_sweeps_side_by_side_equal_sweeps_in_turn(case):
    import torch
    Lx, Ly, D, Dc, batch, sweeps = case
    p, lat = _peps(), Lattice(Lx, Ly, D, Dc)
    A, S = _weak(lat, batch, 700 + D, 0.3)
    Ad, Sd = _dev(A, S)
    other = torch.cuda.Stream()
    limit = p.workspace_bytes(lat, max(1, batch // 3))

    def call():
        return [t.clone() for m in (1, 3) for t in p.evaluate(Ad * 1.0, Sd, lat, "f64", grad_mode=m)]

    p.set_truncation(sweeps)
    p.set_workspace_limit(limit)
    try:
        p.profile_enable(("qr",))
        turn = call()
        p.profile_enable(())
        got = [call(), call()]
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            got += [call(), call()]
        other.synchronize()
    finally:
        p.profile_enable(())
        p.set_workspace_limit(0)
        p.set_truncation(0)
    assert not turn[4].any()
    for g in got:
        for x, y in zip(g, turn):
            assert torch.equal(x, y)
