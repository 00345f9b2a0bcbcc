"""GPU eigensolvers (Lanczos ground state, lowest-k with locking) against the oracle.

Bars: FP64 path within 1e-10 of the oracle eigenvalue, FP32-mixed path (FP32
vectors and H.v, FP64 reductions and refinement) within 1e-6, both relative to
max(|E|, 1) (a zero-energy sector makes a pure relative error meaningless).
"""
import json
import os

import numpy as np
import pytest

import oracle as orc
from gpu_common import build, generic_model, generic_terms, gpu_ed, sector
from paper_1004_3354_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"
GOLD = os.path.join(os.path.dirname(__file__), "golden", "oracle_e0.json")
TOL = {0: 1e-10, 1: 1e-6}


def _v0(D, prec, seed=11):
    ed = gpu_ed()
    v = torch.empty(D, dtype=torch.float64 if prec == 0 else torch.float32, device=DEV)
    ed.fill_random(v, seed, 1)
    return v


def _rel(a, b):
    return abs(a - b) / max(1.0, abs(b))


def _golden(key, sec):
    if not os.path.exists(GOLD):
        pytest.skip("oracle golden values not generated")
    g = json.load(open(GOLD))["entries"]
    if key not in g or sec not in g[key]["sectors"]:
        pytest.skip("no oracle golden value for %s %s" % (key, sec))
    return g[key]["sectors"][sec]["evals"]


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_config0_hv_then_100_step_lanczos(prec):
    ed = gpu_ed()
    phys, sectors = wl.config(0)
    b, H = build(phys, 4, 4, prec)
    sec = sector(phys, 4, 4)
    ev = np.linalg.eigvalsh(sec.dense())
    v0 = _v0(b.D, prec, wl.start_vector_seed(0))
    E, info = H.lanczos_ground(v0, ed.options(max_iter=100, max_basis=100, tol=1e-14), allow_noconv=True)
    assert info["iters"] <= 100
    assert _rel(E, ev[0]) <= TOL[prec], (E, ev[0])
    assert E >= ev[0] - 1e-12 * max(1, abs(ev[0]))   # Rayleigh quotient is variational


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("name,phys,nn", [
    ("kan9_45", wl.kanamori(3, 2, 2.3, 0.4, seed=3), (4, 5)),
    ("hub3x3_45", wl.hubbard(3, 3, 1.0, 4.0), (4, 5)),
    ("aim8_26", wl.aim(7, 2.0, -1.0, seed=8), (2, 6)),
], ids=["kan9_45", "hub3x3_45", "aim8_26"])
def test_ground_state_small(name, phys, nn, prec):
    ed = gpu_ed()
    b, H = build(phys, *nn, prec)
    sec = sector(phys, *nn)
    e_ref = orc.lowest_k(sec, 1, tol=1e-14)[0]
    psi = torch.empty(b.D, dtype=torch.float64 if prec == 0 else torch.float32, device=DEV)
    E, info = H.lanczos_ground(_v0(b.D, prec), ed.options(tol=1e-10 if prec == 0 else 1e-7), psi=psi)
    assert info["converged"] == 1
    assert _rel(E, e_ref) <= TOL[prec], (E, e_ref)
    # the returned vector is normalised and is an eigenvector to the reported residual
    p = psi.double().cpu().numpy()
    assert abs(np.linalg.norm(p) - 1.0) < (1e-12 if prec == 0 else 1e-6)
    r = np.linalg.norm(sec.spmv(p) - E * p)
    assert r <= max(10 * info["residual"], 1e-9)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("max_basis", [120, 12], ids=["basis120", "basis12_restarts"])
@pytest.mark.parametrize("name,phys,nn", [
    ("kan9_45", wl.kanamori(3, 2, 2.3, 0.4, seed=3), (4, 5)),
    ("hub3x3_45", wl.hubbard(3, 3, 1.0, 4.0), (4, 5)),
], ids=["kan9_45", "hub3x3_45"])
def test_ground_state_single_read_projections(name, phys, nn, max_basis, prec):
    """reorth = 3: both Gram-Schmidt projections from one read of the basis
    (second-pass coefficients through the Gram matrix) reach the oracle E0 to
    the same tolerance as two full passes, also across restarts."""
    ed = gpu_ed()
    b, H = build(phys, *nn, prec)
    sec = sector(phys, *nn)
    e_ref = orc.lowest_k(sec, 1, tol=1e-14)[0]
    psi = torch.empty(b.D, dtype=torch.float64 if prec == 0 else torch.float32, device=DEV)
    E, info = H.lanczos_ground(_v0(b.D, prec), ed.options(tol=1e-10 if prec == 0 else 1e-7, reorth=3,
                                                           max_basis=max_basis, max_iter=3000), psi=psi)
    assert info["converged"] == 1
    assert _rel(E, e_ref) <= TOL[prec], (E, e_ref)
    if max_basis == 12:
        assert info["restarts"] > 0
    p = psi.double().cpu().numpy()
    r = np.linalg.norm(sec.spmv(p) - E * p)
    assert r <= max(10 * info["residual"], 1e-9)


@pytest.mark.parametrize("reorth", [2, 3], ids=["cgs2", "single_read"])
@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("name,phys,nn", [
    ("kan9_45", wl.kanamori(3, 2, 2.3, 0.4, seed=3), (4, 5)),
    ("hub3x3_45", wl.hubbard(3, 3, 1.0, 4.0), (4, 5)),
    ("aim8_26", wl.aim(7, 2.0, -1.0, seed=8), (2, 6)),
], ids=["kan9_45", "hub3x3_45", "aim8_26"])
def test_ground_state_implicit_restart(name, phys, nn, prec, reorth):
    """keep = k: exact-shift implicit restarts keep k vectors; the result is the
    oracle E0 and takes fewer steps than restarting from the Ritz vector alone."""
    ed = gpu_ed()
    b, H = build(phys, *nn, prec)
    sec = sector(phys, *nn)
    e_ref = orc.lowest_k(sec, 1, tol=1e-14)[0]
    tol = 1e-10 if prec == 0 else 1e-7
    v0 = _v0(b.D, prec)
    psi = torch.empty(b.D, dtype=torch.float64 if prec == 0 else torch.float32, device=DEV)
    E, info = H.lanczos_ground(v0, ed.options(tol=tol, reorth=reorth, max_basis=14, keep=6, max_iter=4000),
                               psi=psi)
    assert info["converged"] == 1 and info["restarts"] > 0, info
    assert _rel(E, e_ref) <= TOL[prec], (E, e_ref, info)
    p = psi.double().cpu().numpy()
    r = np.linalg.norm(sec.spmv(p) - E * p)
    assert r <= max(10 * info["residual"], 1e-9)
    _, i0 = H.lanczos_ground(v0, ed.options(tol=tol, reorth=reorth, max_basis=14, keep=0, max_iter=4000))
    assert info["iters"] <= i0["iters"], (info, i0)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_single_read_projections_match_cgs2(prec):
    """Same start vector, same Krylov space: the two orthogonalisation forms
    give the same E0 and about the same number of steps."""
    ed = gpu_ed()
    phys, _ = wl.config(3)
    b, H = build(phys, 6, 6, prec)
    v0 = _v0(b.D, prec)
    tol = 1e-10 if prec == 0 else 1e-7
    E2, i2 = H.lanczos_ground(v0, ed.options(tol=tol, reorth=2, max_basis=80))
    E3, i3 = H.lanczos_ground(v0, ed.options(tol=tol, reorth=3, max_basis=80))
    assert _rel(E3, E2) <= (1e-11 if prec == 0 else 1e-7), (E2, E3)
    assert abs(i3["iters"] - i2["iters"]) <= max(8, i2["iters"] // 10), (i2, i3)


def test_generic_model_ground_state():
    ed = gpu_ed()
    p = generic_model(9, 4)
    b = ed.Basis(9, 4, 5)
    H = ed.Hamiltonian(p, b, ed.ED_FP64)
    sec = orc.Sector(9, 4, 5, generic_terms(p))
    e_ref = orc.lowest_k(sec, 1, tol=1e-14)[0]
    E, info = H.lanczos_ground(_v0(b.D, 0), ed.options(tol=1e-11))
    assert _rel(E, e_ref) <= 1e-10


@pytest.mark.parametrize("keep", [0, 10], ids=["ritz_restart", "implicit_restart"])
@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("name,phys,nn,k", [
    ("kanatom_bath", wl.kanamori(3, 1, 2.3, 0.4, seed=2), (3, 3), 8),
    ("hub2x3", wl.hubbard(3, 2, 1.0, 4.0), (3, 3), 6),
    ("kan9_32", wl.kanamori(3, 2, 2.3, 0.4, seed=6), (3, 2), 5),
    ("kan9_32_k24", wl.kanamori(3, 2, 2.3, 0.4, seed=6), (3, 2), 24),
], ids=["kanatom_bath", "hub2x3", "kan9_32", "kan9_32_k24"])
def test_lowest_k_with_multiplicity(name, phys, nn, k, prec, keep):
    ed = gpu_ed()
    b, H = build(phys, *nn, prec)
    sec = sector(phys, *nn)
    ev = np.linalg.eigvalsh(sec.dense())[:k]
    evecs = torch.empty((k, b.D), dtype=torch.float64 if prec == 0 else torch.float32, device=DEV)
    mb = 60 if keep == 0 else 30
    got, infos = H.lowest(k, _v0(b.D, prec), ed.options(tol=1e-10 if prec == 0 else 1e-7, max_basis=mb, keep=keep,
                                                        max_iter=20000), evecs=evecs)
    if keep:
        assert sum(i["restarts"] for i in infos) > 0
    tol = 1e-9 if prec == 0 else 1e-6
    np.testing.assert_allclose(np.sort(got), ev, atol=tol * max(1.0, abs(ev[0])))
    V = evecs.double().cpu().numpy()
    G = V @ V.T
    assert np.max(np.abs(G - np.eye(k))) < (1e-8 if prec == 0 else 1e-4)


def test_breakdown_exact_eigenvector_start():
    ed = gpu_ed()
    phys = wl.hubbard(3, 2, 1.0, 4.0)
    b, H = build(phys, 2, 2, 0)
    sec = sector(phys, 2, 2)
    w, V = np.linalg.eigh(sec.dense())
    v0 = torch.from_numpy(V[:, 0].copy()).to(DEV)
    E, info = H.lanczos_ground(v0, ed.options(tol=1e-12))
    assert info["converged"] == 1 and info["iters"] <= 2
    assert _rel(E, w[0]) <= 1e-12


def test_dimension_one_sector():
    ed = gpu_ed()
    phys = wl.config(3)[0]
    b, H = build(phys, 12, 0, 0)
    sec = sector(phys, 12, 0)
    E, info = H.lanczos_ground(_v0(1, 0), ed.options())
    assert abs(E - sec.dense()[0, 0]) < 1e-12


def test_bit_reproducible():
    ed = gpu_ed()
    phys = wl.kanamori(3, 2, 2.3, 0.4, seed=3)
    b, H = build(phys, 4, 4, 1)
    v0 = _v0(b.D, 1)
    E1, _ = H.lanczos_ground(v0, ed.options(tol=1e-7))
    E2, _ = H.lanczos_ground(v0, ed.options(tol=1e-7))
    assert E1 == E2


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("nn", ["6,6", "5,7", "3,9", "0,1", "12,11"])
def test_config3_sectors_vs_golden(nn, prec):
    ed = gpu_ed()
    phys, _ = wl.config(3)
    a, c = (int(v) for v in nn.split(","))
    e_ref = _golden("cfg3", nn)[0]
    b, H = build(phys, a, c, prec)
    E, info = H.lanczos_ground(_v0(b.D, prec), ed.options(tol=1e-10 if prec == 0 else 1e-7))
    assert _rel(E, e_ref) <= TOL[prec], (E, e_ref, info)


@pytest.mark.parametrize("solver", [(2, 100, 0), (3, 100, 0), (3, 24, 12)],
                         ids=["cgs2", "single_read", "single_read_implicit_restart"])
@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("jp", [True, False], ids=["jp_on", "jp_off"])
def test_config2_full_size_vs_golden(jp, prec, solver):
    ed = gpu_ed()
    reorth, m, keep = solver
    phys, sectors = wl.config(2, jprime=jp)
    e_ref = _golden("cfg2" if jp else "cfg2_jp_off", "7,7")[0]
    b, H = build(phys, 7, 7, prec)
    E, info = H.lanczos_ground(_v0(b.D, prec, wl.start_vector_seed(2)),
                               ed.options(tol=1e-10 if prec == 0 else 1e-7, max_basis=m, reorth=reorth, keep=keep))
    assert _rel(E, e_ref) <= TOL[prec], (E, e_ref, info)


def test_config2_lowest_3_fp32_vs_golden():
    ed = gpu_ed()
    phys, sectors = wl.config(2)
    ev = _golden("cfg2", "7,7")
    b, H = build(phys, 7, 7, 1)
    got, infos = H.lowest(3, _v0(b.D, 1, wl.start_vector_seed(2)), ed.options(tol=1e-7, max_basis=80))
    for g, r in zip(np.sort(got), ev[:3]):
        assert _rel(g, r) <= 1e-6, (got, ev)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_lowest_more_continues_from_converged_levels(prec):
    """ed_arnoldi_lowest_more on top of 4 levels gives the same 10 lowest as the
    dense spectrum, with the first 4 vectors left untouched."""
    ed = gpu_ed()
    phys, nn = wl.kanamori(3, 2, 2.3, 0.4, seed=6), (3, 2)
    b, H = build(phys, *nn, prec)
    ev = np.linalg.eigvalsh(sector(phys, *nn).dense())[:10]
    dt = torch.float64 if prec == 0 else torch.float32
    o = ed.options(tol=1e-10 if prec == 0 else 1e-7, max_basis=30, keep=10, max_iter=20000)
    e4 = torch.empty((4, b.D), dtype=dt, device=DEV)
    E4, _ = H.lowest(4, _v0(b.D, prec), o, evecs=e4)
    e10 = torch.empty((10, b.D), dtype=dt, device=DEV)
    e10[:4].copy_(e4)
    E10, infos = H.lowest_more(4, 10, E4, _v0(b.D, prec), e10, o)
    assert len(infos) == 6
    assert torch.equal(e10[:4], e4)
    tol = 1e-9 if prec == 0 else 1e-6
    np.testing.assert_allclose(np.sort(E10), ev, atol=tol * max(1.0, abs(ev[0])))
    V = e10.double().cpu().numpy()
    assert np.max(np.abs(V @ V.T - np.eye(10))) < (1e-8 if prec == 0 else 1e-4)
    with pytest.raises(ed.EDError):
        H.lowest_more(10, 10, E10, _v0(b.D, prec), e10, o)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("ns,nn,basis,keep", [
    (3, (1, 1), 9, 0),        # D = 9: one ragged group of elements
    (7, (3, 2), 40, 8),       # D = 735: one workgroup, ragged end
    (8, (4, 4), 120, 0),      # D = 4900: coefficients from the partial sums, vectors split over the waves
    (9, (5, 4), 33, 8),       # D = 15,876: the most partial sums an update adds up itself
    (10, (5, 4), 34, 0),      # D = 52,920: finished coefficients, vectors split over the waves
    (11, (6, 5), 35, 8),      # D = 213,444: a wave's own elements
], ids=["d9", "d735", "d4900", "d15876", "d52920", "d213444"])
def test_two_pass_reorthogonalisation_sizes(ns, nn, basis, keep, prec):
    """reorth = 2 at the sizes where its kernels change their split: the two
    lowest levels (the second one deflated, so the vector tables start with a
    locked vector) against the oracle."""
    ed = gpu_ed()
    phys = wl.aim(ns - 1, 2.0, -1.0, seed=40 + ns)
    b, H = build(phys, *nn, prec)
    e_ref = orc.lowest_k(sector(phys, *nn), 2, tol=1e-13)
    E, info = H.lowest(2, _v0(b.D, prec, 5), ed.options(tol=1e-10 if prec == 0 else 1e-7, reorth=2, max_basis=basis,
                                                        keep=keep, max_iter=3000))
    assert all(i["converged"] == 1 for i in info)
    for a, r in zip(E, e_ref):
        assert _rel(a, r) <= TOL[prec], (E, e_ref)


@pytest.mark.parametrize("basis,keep,check,reorth", [
    (20, 6, 1, 2),      # a step queued after every check, restarts in between
    (21, 0, 4, 3),      # restarts from the Ritz vector, the basis full between two checks
    (40, 8, 1000, 3),   # checks only when the basis is full: nothing queued ahead but after the first
], ids=["each", "ritz", "full"])
def test_solves_sharing_a_handle(basis, keep, check, reorth):
    """Two solves at once on one handle, of which one at a time holds the pinned
    words (the other copies through pageable memory), against the same solve
    alone: every number is the same, and the levels are the oracle's."""
    import threading

    ed = gpu_ed()
    phys = wl.aim(7, 2.0, -1.0, seed=23)
    b, H = build(phys, 4, 3, 0)
    v0 = _v0(b.D, 0, 4)
    o = ed.options(tol=1e-10, reorth=reorth, max_basis=basis, keep=keep, check_every=check, max_iter=3000, refine=0)
    E1, i1 = H.lowest(2, v0, o)
    for a, r in zip(E1, orc.lowest_k(sector(phys, 4, 3), 2, tol=1e-13)):
        assert _rel(a, r) <= TOL[0], E1
    start, got = threading.Barrier(2), [[], []]
    torch.cuda.synchronize()

    def work(t):
        with torch.cuda.stream(torch.cuda.Stream()):
            start.wait(timeout=60)
            for _ in range(4):
                got[t].append(H.lowest(2, v0, o))

    pool = [threading.Thread(target=work, args=(t,)) for t in range(2)]
    for t in pool:
        t.start()
    for t in pool:
        t.join()
    for runs in got:
        assert len(runs) == 4
        for E, i in runs:
            assert list(E) == list(E1)
            for x, y in zip(i, i1):
                assert (x["iters"], x["restarts"], x["residual"], x["traffic"]) == (
                    y["iters"], y["restarts"], y["residual"], y["traffic"])


@pytest.mark.parametrize("m,reorth", [(1, 3), (2, 3), (3, 3), (5, 3), (6, 3), (44, 3), (100, 3), (301, 0)])
def test_tridiagonal_lowest_eigenpair(m, reorth):
    """The device eigensolve of T_m against numpy: theta to the rounding of T,
    the residual estimate |beta_m s_m| to that of the eigenvector's last
    component (301 three-term steps hold several copies of the lowest value:
    theta only)."""
    ed = gpu_ed()
    phys = wl.aim(7, 2.0, -1.0, seed=21)
    b, H = build(phys, 4, 4, 0)
    v0 = _v0(b.D, 0, 9)
    a, be, _ = H.lanczos_tridiag(v0, m, ed.options(reorth=reorth))
    assert len(a) == m
    E, info = H.lanczos_ground(v0, ed.options(max_iter=m, max_basis=max(m, 2), check_every=1000, tol=1e-200, refine=0,
                                              reorth=reorth), allow_noconv=True)
    assert info["iters"] == m
    w, z = np.linalg.eigh(np.diag(a) + np.diag(be[:m - 1], 1) + np.diag(be[:m - 1], -1))
    eps, nrm = 2.0 ** -52, np.max(np.abs(w))
    assert abs(E - w[0]) <= 16 * eps * nrm, (E, w[0])
    if reorth == 3:
        gap = w[1] - w[0] if m > 1 else nrm
        assert abs(info["residual"] - abs(be[m - 1] * z[-1, 0])) <= 64 * eps * nrm / gap * be[m - 1]


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("name", ["aim8", "kan9"])
def test_handle_shared_by_solves_and_rayleigh_quotients(name, prec):
    """A new handle used by four threads at once, each on a stream of its own: two
    solves with the FP64 Rayleigh quotient (refine), Rayleigh quotients of a given
    vector, and products.  Everything equals the same call alone on that handle, so
    neither the first calls' tuning and work lists nor the reduction buffer are
    shared without order."""
    import threading

    ed = gpu_ed()
    phys, nn = (wl.aim(7, 2.0, -1.0, seed=29), (4, 4)) if name == "aim8" else (wl.kanamori(3, 2, 2.3, 0.4, seed=3), (4, 5))
    b, H = build(phys, *nn, prec)
    v0, x = _v0(b.D, prec, 4), _v0(b.D, prec, 8)
    ys = [torch.empty_like(x) for _ in range(5)]
    o = ed.options(tol=1e-10 if prec == 0 else 1e-7, reorth=2, max_basis=30, keep=8, max_iter=3000, refine=1)
    start, got, errs = threading.Barrier(4), [[] for _ in range(4)], []
    torch.cuda.synchronize()

    def work(t):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                start.wait(timeout=60)
                for i in range(4):
                    if t < 2:
                        E, info = H.lanczos_ground(v0, o)
                        got[t].append((E, info["residual"], info["rq_fp64"], info["iters"]))
                    elif t == 2:
                        got[t].extend(H.rayleigh(x) for _ in range(8))
                    else:
                        H.apply(x, ys[i])
                torch.cuda.current_stream().synchronize()
        except Exception as e:  # reported by the main thread
            errs.append(e)

    pool = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in pool:
        t.start()
    for t in pool:
        t.join()
    assert not errs, errs
    E, info = H.lanczos_ground(v0, o)
    alone = (E, info["residual"], info["rq_fp64"], info["iters"])
    assert got[0] == [alone] * 4 and got[1] == [alone] * 4
    assert got[2] == [H.rayleigh(x)] * 32
    H.apply(x, ys[4])
    torch.cuda.synchronize()
    for y in ys[:4]:
        assert torch.equal(y, ys[4])
    e_ref = orc.lowest_k(sector(phys, *nn), 1, tol=1e-13)[0]
    assert _rel(E, e_ref) <= TOL[prec]


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("name,k,tol,reorth,basis,keep", [
    ("aim8", 1, 1e-10, 2, 120, 0), ("aim8", 1, 1e-10, 3, 120, 0), ("aim8", 5, 1e-3, 2, 120, 0),
    ("kan9", 1, 1e-10, 2, 24, 8), ("kan9", 1, 1e-10, 3, 24, 8), ("kan9", 6, 1e-4, 2, 20, 6), ("hub6", 3, 1e-10, 2, 120, 0),
], ids=["two", "gram", "two-locked", "two-restarts", "gram-restarts", "two-locked-restarts", "two-small"])
def test_device_basis_is_orthogonal(name, k, tol, reorth, basis, keep, prec):
    """max |<v_i, v_j>| of the stored vectors that a solve leaves in its workspace, and
    against the locked ones (some locked at a loose tolerance, so that the products
    have a component on them).  A vector is rounded once when it is stored and once
    more when a restart combines it (2 u each, u the unit roundoff of the storage), and
    the FP64 sums leave 64 eps of |H v| over the smallest beta.  reorth = 2 projects
    once on two vectors and once on all, reorth = 3 twice on all."""
    ed = gpu_ed()
    phys, nn = {"aim8": (wl.aim(7, 2.0, -1.0, seed=5), (4, 4)), "kan9": (wl.kanamori(3, 2, 2.3, 0.4, seed=3), (4, 5)),
                "hub6": (wl.hubbard(3, 2, 1.0, 4.0), (3, 3))}[name]
    b, H = build(phys, *nn, prec)
    o = ed.options(tol=tol if prec == 0 else max(tol, 1e-7), reorth=reorth, max_basis=basis, keep=keep, max_iter=3000,
                   layout=1)
    dt, elem = (torch.float64, 8) if prec == 0 else (torch.float32, 4)
    ws = torch.zeros(H.workspace_bytes(o, k), dtype=torch.uint8, device=DEV)
    _, info = H.lowest(k, _v0(b.D, prec, 5), o, ws=ws)
    steps, restarts = info[-1]["iters"], info[-1]["restarts"]
    assert (restarts > 0) == (keep > 0)
    last = keep + steps - basis - (restarts - 1) * (basis - keep) if restarts else steps   # S_0 .. S_last
    size = (b.D * elem + 255) // 256 * 256   # slots of the basis, then of the locked vectors
    S = [ws[i * size:i * size + b.D * elem].view(dt) for i in list(range(last + 1)) + [basis + 1 + e for e in range(k - 1)]]
    y = torch.empty(b.D, dtype=dt, device=DEV)
    hv = 0.0
    for v in S[:last]:
        H.apply(v.clone(), y)
        hv = max(hv, float(y.double().norm() / v.double().norm()))
    beta = min(float(v.double().norm()) for v in S[(keep if restarts else 0) + 1:last + 1])
    V = torch.stack([v.double() for v in S])
    V /= V.norm(dim=1, keepdim=True)
    G = (V @ V.T).abs().fill_diagonal_(0.0)
    unit = 2.0 ** -53 if prec == 0 else 2.0 ** -24
    assert float(G[:last + 1].max()) <= 4 * unit + 64 * 2.0 ** -52 * hv / beta


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("reorth", [0, 1, 2, 3])
@pytest.mark.parametrize("nn", [(3, 6), (4, 6), (4, 7), (5, 7)], ids=["2.3e6", "6.8e6", "8.8e6", "1.9e7"])
def test_step_relation_where_the_vector_kernels_split(nn, reorth, prec):
    """Every step obeys H v_j = beta_{j-1} v_{j-1} + alpha_j v_j + beta_j v_{j+1} on the
    stored vectors, and they are orthogonal, at sizes on both sides of the vector
    kernels' rules: two and four whole passes of the workgroups and beyond (8.4e6),
    groups of vectors side by side or in turn (32 MiB a vector), 8 or 16 vectors per
    group (1.7e7 FP32), partial sums finished by their own kernel.  A stored vector
    and a product are rounded once each (u of |H v|), each of the projections on the
    older vectors is of the size of that rounding, and the FP64 sums leave 64 eps."""
    ed = gpu_ed()
    phys = wl.kanamori(3, 4, 2.3, 0.4, seed=3)
    b, H = build(phys, *nn, prec)
    m, dt, elem = 20, (torch.float64, torch.float32)[prec], (8, 4)[prec]
    o = ed.options(reorth=reorth, layout=1)
    ws = torch.zeros(H.tridiag_workspace_bytes(m, o), dtype=torch.uint8, device=DEV)
    al, be, _ = H.lanczos_tridiag(_v0(b.D, prec, 5), m, o, ws=ws)
    assert len(al) == m
    size = (b.D * elem + 255) // 256 * 256
    ring = 3 if reorth == 0 else m + 1      # the three-term recurrence keeps three vectors

    def vec(i):
        v = ws[(i % ring) * size:(i % ring) * size + b.D * elem].view(dt)
        return v, v.double() / v.double().norm()

    unit, y = (2.0 ** -53, 2.0 ** -24)[prec], torch.empty(b.D, dtype=dt, device=DEV)
    for j in range(m - 1 if reorth == 0 else 1, m):
        raw, v = vec(j)
        H.apply(raw.clone(), y)
        hv = y.double() / raw.double().norm()
        scale = float(hv.norm())
        hv -= al[j] * v + be[j - 1] * vec(j - 1)[1]
        hv -= be[j] * vec(j + 1)[1]
        bound = (m + 8) * unit * scale + 64 * 2.0 ** -52 * scale
        assert float(hv.norm()) <= bound, (j, float(hv.norm()), bound)
        for i in range(j - 1 if reorth == 0 else 0, j + 1):
            d = float((vec(i)[1] * vec(j + 1)[1]).sum().abs())
            assert d <= 4 * unit + 64 * 2.0 ** -52 * scale / be[j], (i, j, d)
