"""Edges of the kernels' size rules: the sizes where a launch shape, a tile or a
class of rows changes, against the CPU oracle."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_2606_26760_amd as hq
import workloads as W
from tests.gpu_helpers import (gpu_rows_as_tuples, log, oracle_for, oracle_rows_as_tuples, row_bound,
                               solver_for)

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _elapsed(f, repeats=9):
    """Median time of f in ms."""
    f()
    times = []
    for _ in range(repeats):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        f()
        t1.record()
        t1.synchronize()
        times.append(t0.elapsed_time(t1))
    return sorted(times)[repeats // 2]


@pytest.mark.parametrize("ndet", [1, 5, 8192, 8193])
def test_sigma_either_side_of_the_small_set_rule(ndet):
    """One wave per row up to 8,192 rows, teams with staging above: widths that
    are padded and that are not, both precisions, both orders, X and S one
    element off 16-byte alignment, and the bits of the entry point that
    allocates nothing."""
    ints, a, b, cfg = W.config_inputs(1, ndet=ndet)
    log(f"sigma at {ndet} rows")
    s = solver_for(ints, a, b, cfg.na, cfg.nb)
    o = oracle_for(ints, a, b, cfg.na, cfg.nb)
    rows = np.unique(np.linspace(0, ndet - 1, 300).astype(np.int64))
    perm = s.permutation().cpu().numpy()
    _, r = oracle_rows_as_tuples(o, rows)
    for k in (1, 3, 8, 16):
        X = W.random_block(ndet, k, 900 + k)
        for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 2e-6)):
            Xd = torch.from_numpy(X).to(dtype).cuda()
            Xr = Xd.double().cpu().numpy()
            ref, bound = o.sigma_rows(Xr, rows), row_bound(r, Xr, k)
            flat = torch.empty(ndet * k + 1, dtype=dtype, device="cuda")
            odd = flat[1:].view(ndet, k)
            odd.copy_(Xd)
            out = torch.empty(ndet * k + 1, dtype=dtype, device="cuda")[1:].view(ndet, k)
            S = s.sigma(Xd)
            products = [S, s.sigma(odd, out=out), s.sigma_noalloc(Xd, torch.empty_like(Xd))]
            sorted_S = s.sigma(Xd[torch.from_numpy(perm).long().cuda()].contiguous(), sorted_order=True)
            back = torch.empty_like(S)
            back[torch.from_numpy(perm).long().cuda()] = sorted_S
            for P in products + [back]:
                err = np.abs(P.double().cpu().numpy()[rows] - ref)
                assert np.all(err <= tol * bound + 1e-300), (k, dtype)
            assert torch.equal(products[2], S)


@pytest.mark.parametrize("ndet", [5, 400, 8192, 8193])
def test_caller_order_sigma_into_its_own_input(ndet):
    """A caller-order product written over X, or over rows shifted against it, is
    the product of X as it was: the rows come through a copy at every size."""
    ints, a, b, cfg = W.config_inputs(1, ndet=ndet)
    log(f"sigma over its own input at {ndet} rows")
    s = solver_for(ints, a, b, cfg.na, cfg.nb)
    o = oracle_for(ints, a, b, cfg.na, cfg.nb)
    rows = np.unique(np.linspace(0, ndet - 1, 300).astype(np.int64))
    _, r = oracle_rows_as_tuples(o, rows)
    for k in (1, 3, 8, 16):
        X = W.random_block(ndet, k, 700 + k)
        for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 2e-6)):
            Xd = torch.from_numpy(X).to(dtype).cuda()
            Xr = Xd.double().cpu().numpy()
            ref, bound = o.sigma_rows(Xr, rows), row_bound(r, Xr, k)
            for product in (s.sigma, s.sigma_noalloc):
                for shift in (0, 4):
                    buf = torch.zeros((ndet + shift) * k, dtype=dtype, device="cuda")
                    src, dst = buf[:ndet * k].view(ndet, k), buf[shift * k:].view(ndet, k)
                    src.copy_(Xd)
                    product(src, out=dst)
                    err = np.abs(dst.double().cpu().numpy()[rows] - ref)
                    assert np.all(err <= tol * bound + 1e-300), (k, dtype, shift)


@pytest.mark.parametrize("norb,na,nb,ndet", [(1, 1, 0, 1), (2, 1, 1, 4), (9, 4, 5, 63), (16, 8, 8, 65), (16, 7, 5, 3001),
                                             (17, 6, 5, 2500)])
def test_rdm12_either_side_of_the_table_rule(norb, na, nb, ndet):
    """Class tables in LDS up to 16 orbitals, global copies above: uneven spins,
    row counts around a wave, the smallest orbital counts."""
    log(f"rdm12 norb {norb}, {ndet} determinants")
    ints = W.gen_integrals(norb, 3, -2.0, -0.5, 77)
    if ndet >= 64:
        a, b = W.sample_determinants(norb, na, nb, ndet, 0.4, 0.1, 78)
    else:
        a, b = W.sample_determinants(norb, na, nb, ndet, 0.4, 0.0, 78)
    s = solver_for(ints, a, b, na, nb)
    o = oracle_for(ints, a, b, na, nb)
    c = np.random.default_rng(5).standard_normal(ndet)
    c /= np.linalg.norm(c)
    for order in (False, True):
        x = torch.from_numpy(c).cuda()
        if order:
            x = x[s.permutation().long()].contiguous()
        d1, d2 = (t.cpu().numpy() for t in s.rdm12(x, sorted_order=order))
        r1, r2 = o.rdm12(c)
        # sums of at most ndet * couplings products of two coefficients
        assert np.abs(d1 - r1).max() <= 1e-12 * max(1.0, np.abs(r1).max())
        assert np.abs(d2 - r2).max() <= 1e-12 * max(1.0, np.abs(r2).max())


def _pt2_set(kind):
    rng = np.random.default_rng(21)
    if kind == "many strings":   # more distinct beta strings than the member tables hold: the scan
        norb, na, nb = 18, 9, 9
        a, b = W.sample_determinants(norb, na, nb, 60_000, 0.4, 1.0, 22)
        assert len(np.unique(b)) > 32 * 1024
    elif kind == "large group":  # one alpha group of 3,432 members, next to small ones
        norb, na, nb = 14, 7, 7
        sb = W.fci_strings(norb, nb)
        ra, rb = W.sample_determinants(norb, na, nb, 1500, 0.4, 0.0, 23)
        keep = ra != (1 << na) - 1
        a = np.concatenate([np.full(len(sb), (1 << na) - 1, dtype=np.uint64), ra[keep]])
        b = np.concatenate([sb, rb[keep]])
    else:                        # more than 64 moves per spin
        norb, na, nb = 20, 5, 10
        a, b = W.sample_determinants(norb, na, nb, 3000, 0.3, 0.0, 24)
    order = rng.permutation(len(a))
    return norb, na, nb, a[order], b[order]


@pytest.mark.parametrize("kind", ["many strings", "large group", "many moves"])
def test_pt2_table_and_scan_paths(kind):
    """Candidates in runs of 1, 63, 64, 65 and more that share an alpha string
    (tile edges), members and repeats among them, in shuffled order; a malformed
    candidate gives NaN for itself only."""
    norb, na, nb, a, b = _pt2_set(kind)
    log(f"pt2 {kind}: norb {norb}, {len(a)} determinants")
    ints = W.gen_integrals(norb, 2, -2.0, -0.5, 88)
    s = solver_for(ints, a, b, na, nb)
    o = oracle_for(ints, a, b, na, nb)
    rng = np.random.default_rng(25)
    c = rng.standard_normal(len(a))
    ref = np.uint64((1 << na) - 1)
    single = ref ^ np.uint64(1) ^ np.uint64(1 << na)
    far = ref ^ np.uint64(3) ^ np.uint64(3 << na)
    betas = np.unique(b)
    ca, cb = [a[:20]], [b[:20]]
    for alpha, n in ((ref, 65), (single, 64), (far, 63), (np.uint64(ref << np.uint64(norb - na)), 1), (a[3], 130)):
        ca.append(np.full(n, alpha, dtype=np.uint64))
        cb.append(betas[rng.integers(0, len(betas), n)])
    ca, cb = np.concatenate(ca), np.concatenate(cb)
    order = rng.permutation(len(ca))
    ca, cb = ca[order], cb[order]
    e0 = float(o.pt2(c, 0.0, a[:200], b[:200])[1].min()) - 0.5
    cd = torch.from_numpy(c).cuda()
    num, hxx, score = (t.cpu().numpy() for t in s.pt2(cd, e0, ca, cb))
    rn, rh, rs, absnum = o.pt2(c, e0, ca, cb, with_scale=True)
    assert np.all(np.abs(num - rn) <= 1e-12 * absnum + 1e-300)
    assert np.all(np.abs(hxx - rh) <= 1e-12 * np.abs(rh).max())
    assert np.array_equal(score, num * num / np.abs(e0 - hxx))
    bad_a = ca.copy()
    bad_a[7] ^= np.uint64(1 << (norb - 1)) if not (int(bad_a[7]) >> (norb - 1)) & 1 else np.uint64(1)
    with pytest.raises(hq.HinqsError) as ei:
        s.pt2(cd, e0, bad_a, cb)
    assert ei.value.name == "BAD_OCCUPATION"


def test_pt2_path_follows_the_candidates(monkeypatch):
    """One candidate, lists spread over thousands of alpha strings and lists that share a
    few: both paths against the oracle, and the path taken is the faster of the two
    where they are far apart (measured apart by 2 or more, bound halfway)."""
    ints, a, b, cfg = W.config_inputs(2, ndet=100_000)
    log("pt2 of sparse and dense lists, 1e5 determinants")
    s = solver_for(ints, a, b, cfg.na, cfg.nb)
    o = oracle_for(ints, a, b, cfg.na, cfg.nb)
    rng = np.random.default_rng(61)
    c = rng.standard_normal(len(a))
    c /= np.linalg.norm(c)
    cd = torch.from_numpy(c).cuda()
    sa, sb = W.fci_strings(cfg.norb, cfg.na), W.fci_strings(cfg.norb, cfg.nb)
    e0 = -1000.0
    for nalpha, n in ((1, 1), (len(sa), 300), (len(sa), 30_000), (40, 12_000)):
        pick = sa[rng.permutation(len(sa))[:nalpha]]
        ca, cb = pick[rng.integers(0, nalpha, n)], sb[rng.integers(0, len(sb), n)]
        at = rng.permutation(n)[:400]
        rn, rh, _, absnum = o.pt2(c, e0, ca[at], cb[at], with_scale=True)
        da, db = (torch.from_numpy(x.astype(np.int64)).cuda() for x in (ca, cb))
        ms = {}
        for path in ("0", "1", ""):
            monkeypatch.setenv("HINQS_PT2_TABLES", path)
            num, hxx, score = (t.cpu().numpy() for t in s.pt2(cd, e0, da, db))
            assert np.all(np.abs(num[at] - rn) <= 1e-12 * absnum + 1e-300)
            assert np.all(np.abs(hxx[at] - rh) <= 1e-12 * np.abs(rh).max())
            assert np.array_equal(score, num * num / np.abs(e0 - hxx))
            ms[path] = _elapsed(lambda: s.pt2(cd, e0, da, db))
        log(f"  {n} candidates, {nalpha} alpha strings: scan {ms['0']:.3f} tables {ms['1']:.3f} chosen {ms['']:.3f} ms")
        assert ms[""] <= 1.5 * min(ms["0"], ms["1"])


@pytest.mark.parametrize("per_lane", [False, True])
@pytest.mark.parametrize("ndet", [1, 2, 31, 33, 63, 64, 65, 255, 1025])
def test_couplings_both_enumerators(ndet, per_lane, monkeypatch):
    """One wave per row and one row per lane (asked for through its group
    lookup limit) list the same couplings as the oracle, at row counts around a
    wave, a scan step and a workgroup, with groups of one row to whole ones."""
    if per_lane:
        monkeypatch.setenv("HINQS_CONNECT_LOOKUP_MIN", "1000000")
    log(f"couplings of {ndet} rows, per lane {per_lane}")
    ints = W.gen_integrals(9, 3, -2.0, -0.5, 31)
    a, b = W.sample_determinants(9, 4, 5, ndet, 0.6, 0.2, 32 + ndet)
    s = solver_for(ints, a, b, 4, 5)
    o = oracle_for(ints, a, b, 4, 5)
    rows = np.arange(ndet)
    ref, _ = oracle_rows_as_tuples(o, rows)
    got = gpu_rows_as_tuples(s, rows)
    for i in rows:
        assert got[int(i)] == ref[int(i)], i


@pytest.mark.parametrize("ndet", [65_536, 65_537])
def test_sigma_either_side_of_the_enumerator_rule(ndet):
    ints, a, b, cfg = W.config_inputs(3, ndet=ndet)
    log(f"couplings and sigma at {ndet} rows")
    s = solver_for(ints, a, b, cfg.na, cfg.nb)
    o = oracle_for(ints, a, b, cfg.na, cfg.nb)
    rows = np.random.default_rng(3).choice(ndet, 200, replace=False)
    X = W.random_block(ndet, 2, 4)
    _, r = oracle_rows_as_tuples(o, rows)
    err = np.abs(s.sigma(torch.from_numpy(X).cuda()).cpu().numpy()[rows] - o.sigma_rows(X, rows))
    assert np.all(err <= 1e-12 * row_bound(r, X, 2) + 1e-300)
    rowptr = s.connectivity()[0].cpu().numpy()
    assert np.array_equal(np.diff(rowptr)[rows], np.diff(r["rowptr"]) - 1)


@pytest.mark.parametrize("n", [2, 511, 513, 8192, 8193, 70_001, (1 << 23) + 5])
def test_ranking_at_the_sizes_of_the_sorts(n):
    """One workgroup in LDS, small tiles, large tiles: stable, ties by index."""
    log(f"top_k of {n} values")
    v = torch.from_numpy(np.random.default_rng(n).integers(-40, 40, n).astype(np.float64)).cuda()
    v[n // 2:] *= 1.5
    ints, a, b, cfg = W.config_inputs(0)
    s = solver_for(ints, a, b, cfg.na, cfg.nb)
    for largest in (False, True):
        ref = torch.sort(v, stable=True, descending=largest).indices.int()
        assert torch.equal(s.top_k(v, n, largest=largest), ref)


@pytest.mark.parametrize("block,max_space,threads", [(1, 3, "1024"), (1, 7, "256"), (2, 10, "512"), (4, 20, "256"),
                                                     (8, 48, "1024"), (8, 56, "512"), (16, 64, "1024"),
                                                     (16, 64, "256")])
def test_batch_subspaces_of_every_size(block, max_space, threads, monkeypatch):
    """Sets from the smallest that the subspace allows up to 301 rows together:
    subspaces of odd and of even size, full ones with columns that drop out,
    and chunks of fewer rows than a wave.  A dense eigenvalue lies within the residual's
    norm (tol) of each value, which is at most the lowest diagonal element."""
    monkeypatch.setenv("HINQS_BATCH_RR_THREADS", threads)
    ints = W.gen_integrals(9, 3, -2.0, -0.5, 31)
    s, ref = hq.Hinqs(), []
    for n in sorted({max_space, max_space + 1, 31, 47, 64, 65, 129, 301}):
        if n < max_space:
            continue
        a, b = W.sample_determinants(9, 4, 5, n, 0.4, 0.0, 32 + n)
        s.batch_add(ints.h, ints.eri, ints.e_core, a, b, 4, 5)
        o = oracle_for(ints, a, b, 4, 5)
        ref.append((o.spectrum(n), o.diag().min()))
    log(f"batch block {block}, max_space {max_space}, {threads} threads")
    e, _, info = s.batch_lowest_eigenpair(block=block, max_space=max_space, tol=1e-9, max_iter=600)
    assert info["converged"]
    for x, (spectrum, dmin) in zip(e, ref):
        slack = 1e-12 * np.abs(spectrum).max()
        assert np.abs(spectrum - x).min() <= 1e-9 + slack and x <= dmin + slack, (x, spectrum[:4], dmin)


@pytest.mark.parametrize("block,max_space", [(1, 3), (2, 7), (4, 12), (8, 24), (8, 48), (8, 60), (16, 96)])
@pytest.mark.parametrize("ndet", [63, 64, 65, 1025])
def test_solver_subspaces_and_row_tiles(ndet, block, max_space):
    """Rows around a tile of the tall products, subspaces up to and past 48
    columns, restarts after every and after many steps.  A dense eigenvalue
    lies within the residual's norm (tol) of the result, which is at most the
    lowest diagonal element, and the vector's residual is the one reported."""
    log(f"solver {ndet} rows, block {block}, max_space {max_space}")
    ints = W.gen_integrals(9, 3, -2.0, -0.5, 41)
    a, b = W.sample_determinants(9, 4, 5, ndet, 0.4, 0.0, 42 + ndet)
    s, o = solver_for(ints, a, b, 4, 5), oracle_for(ints, a, b, 4, 5)
    e, c, st = s.lowest_eigenpair(block=block, max_space=max_space, tol=1e-9, max_iter=2000)
    assert st["converged"]
    w, c = o.spectrum(ndet), c.cpu().numpy()
    slack = 1e-12 * np.abs(w).max()
    assert np.abs(w - e).min() <= 1e-9 + slack and e <= o.diag().min() + slack
    assert abs(np.linalg.norm(c) - 1.0) <= 1e-12
    assert np.linalg.norm(o.dense() @ c - e * c) <= 1e-9 + 100 * slack


@pytest.mark.parametrize("evict", ["none", "first", "last", "every other"])
@pytest.mark.parametrize("n_old", [31, 32, 33, 64, 65, 1027])
def test_update_at_word_and_wave_edges(n_old, evict):
    """Kept-row bits around a word and a wave, rows shorter and longer than the
    entries in flight, appended rows that fill the last wave and that do not:
    the couplings, their values and the products of a fresh build."""
    log(f"update of {n_old} rows, evict {evict}")
    ints = W.gen_integrals(9, 3, -2.0, -0.5, 51)
    a, b = W.sample_determinants(9, 4, 5, n_old + 38, 0.6, 0.2, 52 + n_old)
    ev = {"none": [], "first": [0], "last": [n_old - 1], "every other": list(range(0, n_old, 2))}[evict]
    s = solver_for(ints, a[:n_old], b[:n_old], 4, 5)
    s.update_determinants(a[n_old:], b[n_old:], evict=np.array(ev, np.int32) if ev else None)
    keep = np.setdiff1d(np.arange(n_old), ev)
    na, nb = np.concatenate([a[keep], a[n_old:]]), np.concatenate([b[keep], b[n_old:]])
    f = solver_for(ints, na, nb, 4, 5)
    rows = np.arange(len(na))
    assert gpu_rows_as_tuples(s, rows) == gpu_rows_as_tuples(f, rows)
    X = W.random_block(len(na), 3, 53)
    o = oracle_for(ints, na, nb, 4, 5)
    bound = row_bound(oracle_rows_as_tuples(o, rows)[1], X, 3)
    for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 2e-6)):
        Xd = torch.from_numpy(X).to(dtype).cuda()
        ref = o.sigma_rows(Xd.double().cpu().numpy(), rows)
        assert np.all(np.abs(s.sigma(Xd).double().cpu().numpy() - ref) <= tol * bound + 1e-300)


@pytest.mark.parametrize("ndet", [32_767, 32_768, 32_771])
def test_couplings_either_side_of_the_rows_per_wave_rule(ndet):
    """One row or four per wave: runs of rows with one alpha string that begin
    and end inside a wave, and a last wave with fewer rows."""
    ints, a, b, cfg = W.config_inputs(3, ndet=ndet)
    log(f"couplings at {ndet} rows")
    s = solver_for(ints, a, b, cfg.na, cfg.nb)
    o = oracle_for(ints, a, b, cfg.na, cfg.nb)
    last = s.permutation().cpu().numpy()[-5:].astype(np.int64)
    rows = np.unique(np.concatenate([np.random.default_rng(5).choice(ndet, 300, replace=False), last]))
    ref, _ = oracle_rows_as_tuples(o, rows)
    assert gpu_rows_as_tuples(s, rows) == ref


@pytest.mark.parametrize("team,unr", [(8, 2), (8, 8), (16, 4), (32, 2), (32, 8), (64, 4), (64, 8)])
@pytest.mark.parametrize("ndet", [8193, 9001])
def test_sigma_lanes_and_steps(ndet, team, unr, monkeypatch):
    """Lanes that fetch their own coupling and hand it to their group: every
    width, one to eight lanes per coupling, rows that end anywhere in a step,
    rows written in sorted and in caller order, padded and not, with fixed
    strides and with counters."""
    ints, a, b, cfg = W.config_inputs(1, ndet=ndet)
    log(f"sigma at {ndet} rows, team {team}, {unr} gathers in flight")
    for name, v in (("TEAM", team), ("UNR", unr), ("OCC", 4)):
        monkeypatch.setenv("HINQS_SIGMA_" + name, str(v))
    s = solver_for(ints, a, b, cfg.na, cfg.nb)
    o = oracle_for(ints, a, b, cfg.na, cfg.nb)
    rows = np.unique(np.linspace(0, ndet - 1, 250).astype(np.int64))
    perm = torch.from_numpy(s.permutation().cpu().numpy()).long().cuda()
    _, r = oracle_rows_as_tuples(o, rows)
    for k in (1, 2, 3, 4, 8, 11, 16):
        X = W.random_block(ndet, k, 950 + k)
        for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 2e-6)):
            Xd = torch.from_numpy(X).to(dtype).cuda()
            Xr = Xd.double().cpu().numpy()
            ref, bound = o.sigma_rows(Xr, rows), row_bound(r, Xr, k)
            for run in ("0", "3"):
                monkeypatch.setenv("HINQS_SIGMA_RUN", run)
                S = s.sigma(Xd)
                back = torch.empty_like(S)
                back[perm] = s.sigma(Xd[perm].contiguous(), sorted_order=True)
                for P in (S, back):
                    err = np.abs(P.double().cpu().numpy()[rows] - ref)
                    assert np.all(err <= tol * bound + 1e-300), (k, dtype, run)


def test_default_shape_of_a_large_set_with_short_rows(monkeypatch):
    """1e7 rows of 13.5 couplings take as few lanes per row as those of a small set: the
    untuned product against teams of 8 and 16 lanes in time (32 and 64 lanes take 1.7
    to 4 times as long, bound at 1.4) and in value, and one row against the oracle."""
    rng = np.random.default_rng(71)
    norb, ne, n = 19, 9, 10_000_000
    st = W.fci_strings(norb, ne)
    key = np.unique(rng.integers(0, len(st) ** 2, n + n // 100))
    key = rng.permutation(key)[:n]
    a, b = st[key // len(st)], st[key % len(st)]
    log(f"sigma of {n} rows, norb {norb}")
    ints = W.gen_integrals(norb, 1, -2.0, -0.5, 72)
    s = solver_for(ints, a, b, ne, ne)
    perm = s.permutation().long()
    for k in (1, 8):
        g = torch.Generator(device="cuda")
        g.manual_seed(k)
        X = torch.randn((n, k), dtype=torch.float64, device="cuda", generator=g)
        out, ref, ms = torch.empty_like(X), torch.empty_like(X), {}
        ms["default"] = _elapsed(lambda: s.sigma(X, out=out, sorted_order=True))
        for team in ("8", "16"):
            monkeypatch.setenv("HINQS_SIGMA_TEAM", team)
            monkeypatch.setenv("HINQS_SIGMA_RUN", "0")
            ms[team] = _elapsed(lambda: s.sigma(X, out=ref, sorted_order=True))
            assert float((out - ref).abs().max()) <= 1e-12 * float(ref.abs().max())
        monkeypatch.delenv("HINQS_SIGMA_TEAM")
        monkeypatch.delenv("HINQS_SIGMA_RUN")
        log(f"  k {k}: " + ", ".join(f"{t} {v:.3f} ms" for t, v in ms.items()))
        assert ms["default"] <= 1.4 * min(ms["8"], ms["16"])
    # the determinants at most two electrons from one of them
    i = int(perm[n // 2])
    near = np.flatnonzero(np.bitwise_count(a ^ a[i]).astype(int) + np.bitwise_count(b ^ b[i]) <= 4)
    assert 2 <= len(near) <= 200
    sub = oracle_for(ints, a[near], b[near], ne, ne)
    x = np.random.default_rng(73).standard_normal(n)
    got = float(s.sigma(torch.from_numpy(x).cuda())[i])
    at = int(np.flatnonzero(near == i)[0])
    want = float(sub.sigma_rows(x[near][:, None], np.array([at]))[0, 0])
    _, r = oracle_rows_as_tuples(sub, np.array([at]))
    assert abs(got - want) <= 1e-12 * row_bound(r, x[near][:, None], 1)[0, 0]


def test_tuned_small_batch_runs_the_untuned_chunks(monkeypatch):
    """A batch too small for 256 chunks of the tuner's smallest size is cut finer whether it
    was tuned or not: with the threads and the product's shape held, both solves sum
    in the same order, so energies and vectors are equal in every bit."""
    for name, v in (("SIGMA_TEAM", 16), ("SIGMA_UNR", 4), ("SIGMA_OCC", 4), ("BATCH_RR_THREADS", 1024)):
        monkeypatch.setenv("HINQS_" + name, str(v))
    results = []
    for tune in (False, True):
        s = hq.Hinqs()
        for i in (18, 29, 40, 51):
            ints, a, b, spec = W.batch_instance(i, 0.1)
            s.batch_add(ints.h, ints.eri, ints.e_core, a, b, spec["na"], spec["nb"])
        e, c, info = s.batch_lowest_eigenpair(tol=1e-9, autotune=tune)
        log(f"batch, tuned {tune}: {info['stats']['iterations']} iterations, {info['stats']['ms_iterations']:.2f} ms")
        assert (info["stats"]["ms_tune"] > 0.0) == tune
        results.append((e, c))
    assert np.array_equal(results[0][0], results[1][0]) and torch.equal(results[0][1], results[1][1])


_TUNED_CHILD = """
import sys
import numpy as np, torch
import paper_2606_26760_amd as hq
import workloads as W
ndet = int(sys.argv[1])
ints, a, b, cfg = W.config_inputs(1, ndet=ndet)
s = hq.Hinqs()
s.set_integrals(ints.h, ints.eri, ints.e_core)
s.set_determinants(a, b, cfg.na, cfg.nb)
X = torch.from_numpy(W.random_block(ndet, 8, 5)).cuda()
before = s.sigma(X)
shape, ms = s.autotune(8, hq.HINQS_FP64)
print("shape", *shape[:3], ms, int(torch.equal(before, s.sigma(X))), flush=True)
"""


def _tuned_child(path, ndet=3001):
    """One process that reads the plans of ``path``: (team, unroll, workgroups), ms of the
    plan, and whether a caller-order product kept its bits."""
    env = dict(os.environ, HINQS_TUNE_CACHE=str(path), PYTHONPATH=ROOT)
    for name in [n for n in env if n.startswith("HINQS_SIGMA_")]:
        del env[name]
    r = subprocess.run([sys.executable, "-c", _TUNED_CHILD, str(ndet)], cwd=ROOT, env=env, capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, r.stderr
    f = r.stdout.split("shape", 1)[1].split()
    return tuple(int(x) for x in f[:3]), float(f[3]), f[4] == "1"


def test_tuned_shape_leaves_staged_products_of_small_sets_alone(tmp_path):
    """A team shape tuned for a small set serves the products it was timed on (sorted,
    aligned); a caller-order one keeps the launch that needs no staging, bit for bit."""
    log("a plan with a team shape for 3,001 rows")
    plans = tmp_path / "plans"
    _tuned_child(plans)
    key = plans.read_text().split()[0]
    plans.write_text(f"{key} 16 4 4 0 0.125\n")
    shape, ms, same = _tuned_child(plans)
    assert shape == (16, 4, 4) and ms == 0.125
    assert same


def test_plans_of_other_kernels_and_of_the_other_size_class_are_not_used(tmp_path):
    """A plan saved under a key without the kernels' version is tuned again, and so is a set
    of 8,193 rows after one of 8,192, which runs another kernel."""
    log("plans without a version; plans of 8,192 and 8,193 rows")
    plans = tmp_path / "plans"
    _tuned_child(plans)
    key = plans.read_text().split()[0]
    old = "|".join(p for p in key.split("|") if not p.startswith("v")).replace("|s", "|d")
    plans.write_text(f"{old} 16 4 4 1 0.125\n")
    assert _tuned_child(plans)[1] != 0.125
    times = []
    for ndet in (8192, 8193):
        ints, a, b, cfg = W.config_inputs(1, ndet=ndet)
        times.append(solver_for(ints, a, b, cfg.na, cfg.nb).autotune(4, hq.HINQS_FP32)[1])
    assert times[0] != times[1]


@pytest.mark.parametrize("path", ["0", "1"])
@pytest.mark.parametrize("n", [200, 700])
def test_pt2_malformed_candidates_are_nan_alone(n, path, monkeypatch):
    """Wrong counts and bits at or above norb, alone in a tile and among others that share
    their strings: those outputs are NaN, every other one is that of the clean list."""
    norb, na, nb, a, b = _pt2_set("large group")
    log(f"pt2 with malformed candidates, {n} candidates, path {path}")
    monkeypatch.setenv("HINQS_PT2_TABLES", path)
    ints = W.gen_integrals(norb, 2, -2.0, -0.5, 88)
    s = solver_for(ints, a, b, na, nb)
    rng = np.random.default_rng(62)
    cd = torch.from_numpy(rng.standard_normal(len(a))).cuda()
    ua, ub = np.unique(a), np.unique(b)
    ca, cb = ua[rng.integers(0, 6, n)], ub[rng.integers(0, len(ub), n)]
    clean = [t.cpu().numpy() for t in s.pt2(cd, -1000.0, ca, cb)]
    bad = rng.permutation(n)[:n // 10]
    xa, xb = ca.copy(), cb.copy()
    for i, at in enumerate(bad):
        if i % 4 == 0:
            xa[at] ^= np.uint64(1)                         # one electron more or less
        elif i % 4 == 1:
            xb[at] ^= np.uint64(1)
        elif i % 4 == 2:
            xa[at] |= np.uint64(1 << norb)
        else:
            xb[at] |= np.uint64(1 << 40)
    da, db = (torch.from_numpy(x.view(np.int64)).cuda() for x in (xa, xb))
    out = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(3)]
    rc = s._lib.hinqs_pt2(s._h, s._ptr(cd), -1000.0, n, s._ptr(da), s._ptr(db), *[s._ptr(t) for t in out], 0)
    assert rc != 0
    with pytest.raises(hq.HinqsError) as ei:
        s._check(rc)
    assert ei.value.name == "BAD_OCCUPATION"
    good = np.setdiff1d(np.arange(n), bad)
    for got, ref in zip(out, clean):
        got = got.cpu().numpy()
        assert np.all(np.isnan(got[bad])) and np.array_equal(got[good], ref[good])


@pytest.mark.parametrize("block,max_space", [(4, 24), (8, 48), (8, 60), (16, 96)])
@pytest.mark.parametrize("ndet", [65, 1025])
def test_solver_finds_the_lowest_state(ndet, block, max_space):
    """With four or more roots followed, the state found is the lowest one: the residual's
    norm (tol) bounds its distance from the dense spectrum's first value."""
    log(f"lowest state of {ndet} rows, block {block}, max_space {max_space}")
    ints = W.gen_integrals(9, 3, -2.0, -0.5, 41)
    a, b = W.sample_determinants(9, 4, 5, ndet, 0.4, 0.0, 42 + ndet)
    s, o = solver_for(ints, a, b, 4, 5), oracle_for(ints, a, b, 4, 5)
    for mixed in (False, True):
        e, _, st = s.lowest_eigenpair(block=block, max_space=max_space, tol=1e-9, max_iter=2000, mixed=mixed)
        w = o.spectrum(ndet)
        assert st["converged"] and abs(e - w[0]) <= 1e-9 + 1e-12 * np.abs(w).max(), (e, w[:4])


@pytest.mark.parametrize("block,max_space", [(4, 24), (8, 48), (8, 56), (16, 64)])
def test_batch_finds_the_lowest_states(block, max_space):
    log(f"lowest states of a batch, block {block}, max_space {max_space}")
    ints = W.gen_integrals(9, 3, -2.0, -0.5, 31)
    s, ref = hq.Hinqs(), []
    for n in (65, 129, 301, 1025):
        a, b = W.sample_determinants(9, 4, 5, n, 0.4, 0.0, 32 + n)
        s.batch_add(ints.h, ints.eri, ints.e_core, a, b, 4, 5)
        ref.append(oracle_for(ints, a, b, 4, 5).spectrum(n))
    e, _, info = s.batch_lowest_eigenpair(block=block, max_space=max_space, tol=1e-9, max_iter=600)
    assert info["converged"]
    for x, w in zip(e, ref):
        assert abs(x - w[0]) <= 1e-9 + 1e-12 * np.abs(w).max(), (x, w[:4])


class _PoolUpTo(hq.TorchAllocator):
    """PyTorch's pool; requests above ``limit`` bytes get nothing."""

    def __init__(self):
        super().__init__(0, torch.cuda.current_stream(0).cuda_stream)
        self.limit, self.refused = 1 << 62, 0

    def alloc(self, nbytes):
        if nbytes > self.limit:
            self.refused += 1
            return 0
        return super().alloc(nbytes)


@pytest.mark.parametrize("refused_from", [0, 16_384])
def test_pt2_without_memory_for_its_tables_scans(refused_from, monkeypatch):
    """The member tables (214 KB) and the tile lists are memory that the scan does not need:
    when the allocator has none for both, or for the tables alone, the scan's results come
    back bit for bit."""
    ints, a, b, cfg = W.config_inputs(3, ndet=60_000)
    log(f"pt2 with requests above {refused_from} bytes refused")
    pool = _PoolUpTo()
    s = hq.Hinqs(allocator=pool)
    s.set_integrals(ints.h, ints.eri, ints.e_core)
    s.set_determinants(a, b, cfg.na, cfg.nb)
    rng = np.random.default_rng(81)
    cd = torch.from_numpy(rng.standard_normal(len(a))).cuda()
    ca, cb = a[:600][rng.integers(0, 600, 1200)], b[rng.integers(0, len(b), 1200)]
    monkeypatch.setenv("HINQS_PT2_TABLES", "0")
    ref = s.pt2(cd, -1000.0, ca, cb)
    monkeypatch.setenv("HINQS_PT2_TABLES", "1")
    pool.limit = refused_from
    got = s.pt2(cd, -1000.0, ca, cb)
    assert pool.refused > 0
    for x, y in zip(got, ref):
        assert torch.equal(x, y)
    pool.limit = 1 << 62
    for x, y in list(zip(s.pt2(cd, -1000.0, ca, cb), ref))[:2]:
        assert float((x - y).abs().max()) <= 1e-12 * float(y.abs().max())
