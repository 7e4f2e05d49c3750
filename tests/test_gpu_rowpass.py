"""The row passes (the fused pass with u~ and finished stars kept in LDS or in registers until a
round of rows ends, aprod 1 and the star-ordered aprod 2 by themselves) at the sizes where they
can go wrong, through the C ABI against the oracle: rows that end inside a wave step, a wave's
share and a round; stars that span several waves and blocks; one row per star; more stars in a
round than it has slots; stars without rows; the register form with and without its exchange
area; several rounds per block; instrumental columns beyond the fused pass and beyond LDS; enough
rows for the knot-by-knot copy of the attitude unknowns.

Tolerances: rounding-order differences of a product stay within 1e-13 of its largest entry where
a column sums up to about 1e5 terms, 1e-12 beyond; LSQR iterates after three steps within 1e-10
relative (the bounds of the other parity tests)."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import assert_close_scaled, cuda, host, open_system, oracle_system, rel
from paper_2212_11675_amd import gsr

pytestmark = pytest.mark.gpu


def _runs(counts, n_dfa, n_instr, seed):
    """A system whose star k has counts[k] rows."""
    counts = np.asarray(counts, dtype=np.int64)
    m = int(counts.sum())
    shape = synth.Shape(1, m, m, n_dfa, n_instr, seed=seed)
    out = synth.rows(shape, 0, m)
    out["star"] = np.repeat(np.arange(counts.size, dtype=np.int32), counts)
    out["dims"] = dict(n_rows=m, n_stars=int(counts.size), n_dfa=n_dfa, n_instr=n_instr, n_glob=1)
    return out


LONG = [3, 5000, 1, 1, 20000, 7, 16, 16, 300, 40000, 2]
CROWD = [40000] + [1] * 30000  # far more stars than the mean in the second half
GAPS = [0, 17, 0, 0, 5, 1, 0] * 900
CASES = {
    "one_row": ([1], 9, 12),
    "tile_edge_17": ([10, 7], 9, 12),
    "wave_edge": ([16] * 4096 + [1], 50, 40),
    "wave_edge_under": ([16] * 4095 + [15], 50, 40),
    "long_stars": (LONG, 40, 60),
    "one_row_per_star": ([1] * 70001, 40, 60),
    "crowded_slots": (CROWD, 40, 60),
    "gaps": (GAPS, 30, 40),
    "two_rounds_lds": ([23] * 27000 + [500, 1], 300, 8400),
    "reg_exchange_long": (LONG + [25] * 6000, 40, 10100),
    "reg_exchange_gaps": (GAPS * 2, 40, 10100),
    "reg_no_exchange": (LONG + [25] * 2000 + GAPS, 40, 10200),
    "reg_two_rounds": ([37] * 57000 + [3, 41], 300, 10100),
    # so many stars that two rounds of the LDS form would be short ones: the register form with a
    # narrow instrumental section
    "reg_narrow": ([1] * 1000000, 50, 12),
    "wide": (LONG + [25] * 2000 + GAPS, 40, 11000),
    "beyond_lds": (LONG + [25] * 2000 + GAPS, 40, 21000),
}


@pytest.mark.parametrize("name", CASES)
def test_iterates_of_every_form_match_the_oracle(name):
    counts, n_dfa, n_instr = CASES[name]
    print(f"[row pass] {name}", flush=True)
    sysd = _runs(counts, n_dfa, n_instr, seed=171)
    S = oracle_system(sysd)
    h, _ = open_system(sysd, allow_empty_cols=True, build_f32=True)
    rng = np.random.default_rng(172)
    b = rng.standard_normal(S.m)
    x = torch.empty(S.n, dtype=torch.float64, device="cuda")
    it = 3 if S.m > 100 else 1  # a handful of rows is solved exactly after a few steps
    info = gsr.gsr_lsqr_solve(h, cuda(b), x, gsr.solve_opts(itnlim=it, fixed_iters=True))
    assert info["fused"] == int(n_instr <= 10239)
    xo, io = S.lsqr(b, itnlim=it, fixed=True)
    assert info["itn"] == io["itn"] == it
    assert rel(host(x), xo) <= 1e-10
    # binary32 coefficients, one inner solve
    S32 = S.with_vals(sysd["vals"].astype(np.float32).astype(np.float64))
    gsr.gsr_lsqr_solve(h, cuda(b), x, gsr.solve_opts(itnlim=it, fixed_iters=True,
                                                     precision=gsr.GSR_F32V, max_refine=1))
    assert rel(host(x), S32.lsqr(b, itnlim=it, fixed=True)[0]) <= 1e-10
    # the transposed recurrence of the adjoint solve, in the space of the rows
    g = rng.standard_normal(S.n)
    mu = torch.empty(S.m, dtype=torch.float64, device="cuda")
    lam = torch.empty(S.n, dtype=torch.float64, device="cuda")
    gsr.gsr_lsqr_solve_adjoint(h, cuda(g), mu, lam, gsr.solve_opts(itnlim=it, fixed_iters=True))
    assert rel(host(mu), S.lsqr_transposed(g, itnlim=it, fixed=True)[0]) <= 1e-10
    h.close()


@pytest.mark.parametrize("name", CASES)
def test_products_of_every_form_match_the_oracle(name):
    counts, n_dfa, n_instr = CASES[name]
    print(f"[row products] {name}", flush=True)
    sysd = _runs(counts, n_dfa, n_instr, seed=173)
    S = oracle_system(sysd)
    S32 = S.with_vals(sysd["vals"].astype(np.float32).astype(np.float64))
    h, _ = open_system(sysd, allow_empty_cols=True, build_f32=True)
    rng = np.random.default_rng(174)
    tol = 1e-13 if S.m < 200000 else 1e-12
    x, y0 = rng.standard_normal(S.n), rng.standard_normal(S.m)
    y, x0 = rng.standard_normal(S.m), rng.standard_normal(S.n)
    for a1, a2, ref in ((gsr.gsr_aprod1, gsr.gsr_aprod2, S),
                        (gsr.gsr_aprod1_f32v, gsr.gsr_aprod2_f32v, S32)):
        yd, xd = cuda(y0), cuda(x0)
        a1(h, cuda(x), yd)
        assert_close_scaled(host(yd), ref.aprod1(x, y0), tol)
        a2(h, cuda(y), xd)
        assert_close_scaled(host(xd), ref.aprod2(y, x0), tol)
    r = torch.empty(S.m, dtype=torch.float64, device="cuda")
    gsr.gsr_residual(h, cuda(y0), cuda(x), r)
    assert_close_scaled(host(r), S.residual(y0, x), tol)
    p = torch.empty(S.n, dtype=torch.float64, device="cuda")
    gsr.gsr_precond(h, p)
    np.testing.assert_allclose(host(p), S.colnorm(), rtol=1e-12, atol=0)
    h.close()


@pytest.mark.parametrize("itnlim", [15, 16, 17, 32])
def test_steps_at_the_ends_of_a_replayed_sequence(itnlim):
    """The scalar steps are taken by the kernels that follow them, the last one of a replayed
    sequence (16 iterations) by a kernel of its own: solves that stop around its end.  Two replays
    of the same handle; attitude buckets narrower than a row's knots (n_dfa 4) and wider."""
    for n_dfa in (4, 60):
        sysd = _runs([7, 1, 12, 30, 3] * 60, n_dfa, 40, seed=175)
        S = oracle_system(sysd)
        h, _ = open_system(sysd, allow_empty_cols=True)
        rng = np.random.default_rng(176)
        x = torch.empty(S.n, dtype=torch.float64, device="cuda")
        mu = torch.empty(S.m, dtype=torch.float64, device="cuda")
        o = gsr.solve_opts(itnlim=itnlim, fixed_iters=True)
        for _ in range(2):
            b, g = rng.standard_normal(S.m), rng.standard_normal(S.n)
            assert gsr.gsr_lsqr_solve(h, cuda(b), x, o)["itn"] == itnlim
            assert rel(host(x), S.lsqr(b, itnlim=itnlim, fixed=True)[0]) <= 1e-10
            lam = torch.empty(S.n, dtype=torch.float64, device="cuda")
            gsr.gsr_lsqr_solve_adjoint(h, cuda(g), mu, lam, o)
            assert rel(host(mu), S.lsqr_transposed(g, itnlim=itnlim, fixed=True)[0]) <= 1e-10
        h.close()


@pytest.mark.parametrize("k,n_instr", [(1, 40), (2, 40), (4, 60), (8, 40), (8, 1100)])
def test_batched_row_pass_matches_the_oracle(k, n_instr):
    """The batched row and attitude passes at their edges: the runs of stars above as systems of
    one batch (stars past the last slot of a round, stars without rows, rows that end inside a
    wave step, a system of one row), attitude runs that begin and end inside a block of 32 rows
    (n_dfa 40) and runs of thousands of rows (n_dfa 4), the unknowns of the instrumental columns
    staged in LDS and (n_instr 1,100 with 8 right-hand sides) read from the operand."""
    print(f"[batch row pass] k={k} n_instr={n_instr}", flush=True)
    runs = [([1], 4), (CROWD, 40), ([10, 7], 9), (GAPS, 4), ([1] * 5003, 3000), (LONG, 40),
            ([16] * 300 + [15], 50)]
    systems = [_runs(c, n_dfa, n_instr, seed=180 + i) for i, (c, n_dfa) in enumerate(runs)]
    dims = [gsr.make_dims(s["dims"]["n_rows"], s["dims"]["n_stars"], s["dims"]["n_dfa"],
                          s["dims"]["n_instr"]) for s in systems]
    ro = np.concatenate([[0], np.cumsum([s["dims"]["n_rows"] for s in systems])])
    dev = {key: torch.from_numpy(np.concatenate([s[key] for s in systems])).to("cuda:0")
           for key in ("vals", "star", "att", "instr")}
    b = gsr.gsr_batch_setup(dims, ro.tolist(), dev["vals"], dev["star"], dev["att"], dev["instr"],
                            k, allow_empty_cols=True)
    rhs = np.random.default_rng(190).standard_normal((b.m, k))
    for iters in (1, 3):
        x = torch.empty(b.n * k, dtype=torch.float64, device="cuda")
        gsr.gsr_batch_solve(b, cuda(rhs.ravel()), x, gsr.solve_opts(itnlim=iters, fixed_iters=True))
        xg = host(x).reshape(b.n, k)
        for i, sysd in enumerate(systems):
            if iters > 1 and sysd["dims"]["n_rows"] < 100:
                continue  # solved exactly before that
            S = oracle_system(sysd)
            c0, c1 = b.col_offset[i], b.col_offset[i + 1]
            for j in range(k):
                xo, _ = S.lsqr(rhs[ro[i]:ro[i + 1], j], itnlim=iters, fixed=True)
                assert rel(xg[c0:c1, j], xo) <= 1e-10, (i, j, iters)
    b.close()


def test_batched_row_pass_with_the_widest_instrumental_section():
    """The most instrumental columns that a batch with 8 right-hand sides takes, one row per star:
    the sums leave room for fewer star slots than one wave step of a block needs."""
    k, n_instr = 8, 1279
    print(f"[batch row pass, widest] k={k} n_instr={n_instr}", flush=True)
    systems = [_runs([1] * m, 30, n_instr, seed=195 + i) for i, m in enumerate((1501, 4100))]
    dims = [gsr.make_dims(s["dims"]["n_rows"], s["dims"]["n_stars"], s["dims"]["n_dfa"],
                          s["dims"]["n_instr"]) for s in systems]
    ro = np.concatenate([[0], np.cumsum([s["dims"]["n_rows"] for s in systems])])
    dev = {key: torch.from_numpy(np.concatenate([s[key] for s in systems])).to("cuda:0")
           for key in ("vals", "star", "att", "instr")}
    b = gsr.gsr_batch_setup(dims, ro.tolist(), dev["vals"], dev["star"], dev["att"], dev["instr"],
                            k, allow_empty_cols=True)
    rhs = np.random.default_rng(197).standard_normal((b.m, k))
    x = torch.empty(b.n * k, dtype=torch.float64, device="cuda")
    gsr.gsr_batch_solve(b, cuda(rhs.ravel()), x, gsr.solve_opts(itnlim=2, fixed_iters=True))
    xg = host(x).reshape(b.n, k)
    for i, sysd in enumerate(systems):
        S = oracle_system(sysd)
        for j in range(k):
            xo, _ = S.lsqr(rhs[ro[i]:ro[i + 1], j], itnlim=2, fixed=True)
            assert rel(xg[b.col_offset[i]:b.col_offset[i + 1], j], xo) <= 1e-10, (i, j)
    b.close()
