"""Systems near the limit of the device memory: what setup needs at its peak and what it can do
without.  The rest of the memory is held by one allocation meanwhile; results are compared with
those of a handle opened with all of it free (products to 1e-12 of the largest entry, iterates to
1e-10: other orders of summation)."""
import contextlib

import pytest
import torch

from gpu_util import assert_close_scaled, host, rel
from paper_2212_11675_amd import gsr

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _system(stars, per, n_dfa, n_instr, seed):
    """`stars` stars of `per` rows each, made on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    m = stars * per
    star = torch.arange(stars, dtype=torch.int32, device="cuda").repeat_interleave(per)
    att = torch.randint(0, n_dfa - 3, (m,), dtype=torch.int32, device="cuda", generator=g)
    step = n_instr // 6
    instr = torch.randint(0, step, (m, 6), dtype=torch.int32, device="cuda", generator=g)
    instr += step * torch.arange(6, dtype=torch.int32, device="cuda")
    vals = torch.randn(24 * m, dtype=torch.float64, device="cuda", generator=g)
    dims = gsr.make_dims(m, stars, n_dfa, n_instr)
    return dims, (vals, star, att, instr.reshape(-1).contiguous())


def _free():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


@contextlib.contextmanager
def _room(nbytes):
    """All free device memory but `nbytes` held (in a few pieces: the free memory reported grows
    by half a GiB once most of it is taken)."""
    held = []
    for _ in range(4):
        more = (_free() - nbytes) // (2 * MIB) * (2 * MIB)
        if more > 0:
            held.append(torch.empty(more, dtype=torch.uint8, device="cuda"))
    print(f"[memory] room {_free() / MIB:.0f} MiB of {nbytes / MIB:.0f}", flush=True)
    try:
        yield
    finally:
        held.clear()
        torch.cuda.empty_cache()


def _compare(h, ref, with_f32):
    """Products, solves and the adjoint solve of two handles on the same system."""
    g = torch.Generator(device="cuda").manual_seed(5)

    def vec(n):
        return torch.randn(n, dtype=torch.float64, device="cuda", generator=g)

    x, y = vec(h.n), vec(h.m)
    forms = [(gsr.gsr_aprod1, gsr.gsr_aprod2)]
    if with_f32:
        forms.append((gsr.gsr_aprod1_f32v, gsr.gsr_aprod2_f32v))
    for a1, a2 in forms:
        out = []
        for k in (h, ref):
            ax, aty = torch.zeros_like(y), torch.zeros_like(x)
            a1(k, x, ax)
            a2(k, y, aty)
            out.append((host(ax), host(aty)))
        assert_close_scaled(out[0][0], out[1][0], 1e-12)
        assert_close_scaled(out[0][1], out[1][1], 1e-12)
    res, pre = [], []
    for k in (h, ref):
        r, p = torch.empty_like(y), torch.empty_like(x)
        gsr.gsr_residual(k, y, x, r)
        gsr.gsr_precond(k, p)
        res.append(host(r))
        pre.append(host(p))
    assert_close_scaled(res[0], res[1], 1e-12)
    assert_close_scaled(pre[0], pre[1], 1e-12)
    precisions = [gsr.GSR_F64] + ([gsr.GSR_F32V] if with_f32 else [])
    for precision in precisions:
        o = gsr.solve_opts(itnlim=17, fixed_iters=True, precision=precision, max_refine=2)
        xs = []
        for k in (h, ref):
            xk = torch.empty_like(x)
            gsr.gsr_lsqr_solve(k, y, xk, o)
            xs.append(host(xk))
        assert rel(xs[0], xs[1]) <= 1e-10
    o = gsr.solve_opts(itnlim=3, fixed_iters=True)
    mus = []
    for k in (h, ref):
        mu, lam = torch.empty_like(y), torch.empty_like(x)
        gsr.gsr_lsqr_solve_adjoint(k, x, mu, lam, o)
        mus.append(host(mu))
    assert rel(mus[0], mus[1]) <= 1e-10


def test_setup_needs_no_more_than_the_handle_keeps():
    """The sort of the attitude copy (240 MB of keys and buffers for 6e6 rows) is over before the
    row tiles (1.3 GB) are allocated: setup fits where the finished handle does."""
    dims, arrays = _system(300_000, 20, 3000, 1200, seed=301)
    before = _free()
    h = gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True)
    kept = before - _free()
    h.close()
    print(f"[memory] handle {kept / MIB:.0f} MiB", flush=True)
    with _room(kept + 64 * MIB):
        h = gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True)
    ref = gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True)
    _compare(h, ref, with_f32=False)
    h.close()
    ref.close()


def test_one_residual_vector_where_the_second_does_not_fit():
    """The forward solves' second u~ is left out when the memory ends before it; the row pass then
    works in place."""
    dims, arrays = _system(300_000, 20, 3000, 1200, seed=302)
    before = _free()
    ref = gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True, build_f32=True)
    kept = before - _free()
    ref.close()
    one = 8 * dims.n_rows
    print(f"[memory] handle {kept / MIB:.0f} MiB, one u~ {one / MIB:.0f}", flush=True)
    with _room(kept - one - one // 2):  # neither the binary32 form's nor the binary64 form's
        h = gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True, build_f32=True)
    ref = gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True, build_f32=True)
    _compare(h, ref, with_f32=True)
    h.close()
    ref.close()


@pytest.mark.parametrize("n_instr", [11_000, 21_000])  # instrumental sums in LDS and beyond it
def test_unfused_system_whose_row_tiles_do_not_fit(n_instr):
    """Products and solves from the caller's arrays, binary64 and binary32, with new values too."""
    dims, arrays = _system(300_000, 20, 3000, n_instr, seed=303)
    before = _free()
    ref = gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True, build_f32=True)
    kept = before - _free()
    ref.close()
    short = 224 * dims.n_rows + 100 * MIB  # what stays holds neither of the two tile arrays
    print(f"[memory] handle {kept / MIB:.0f} MiB, {short / MIB:.0f} short", flush=True)
    with _room(kept - short):
        h = gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True, build_f32=True)
    ref = gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True, build_f32=True)
    _compare(h, ref, with_f32=True)
    new = torch.randn_like(arrays[0])
    for k in (h, ref):
        gsr.gsr_update_values(k, new)
    _compare(h, ref, with_f32=True)
    h.close()
    ref.close()


def test_a_failed_setup_leaves_no_error_behind():
    """The status says that the memory ended; the runtime's last error is clear again, and the
    caller's next launch is fine."""
    dims, arrays = _system(300_000, 20, 3000, 1200, seed=305)
    with _room(600 * MIB):
        with pytest.raises(gsr.GsrError):  # in the attitude copy's arrays or its sort
            gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True)
        assert float(torch.ones(8, device="cuda").sum()) == 8.0
    h = gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True)
    h.close()


def test_constraint_rows_whose_workspace_does_not_fit():
    """After the error the handle is the one without constraint rows, its workspaces in place."""
    dims, arrays = _system(100_000, 20, 3000, 1200, seed=304)
    h = gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True, build_f32=True)
    ref = gsr.gsr_lsqr_setup(dims, *arrays, allow_empty_cols=True, build_f32=True)
    n_con = 40_000_000  # rows without entries: 320 MB for their sums, as much for every u~
    con = (torch.zeros(n_con + 1, dtype=torch.int64, device="cuda"),
           torch.zeros(0, dtype=torch.int64, device="cuda"),
           torch.zeros(0, dtype=torch.float64, device="cuda"))
    with _room(400 * MIB):
        with pytest.raises(gsr.GsrError) as e:
            gsr.gsr_set_constraints(h, *con)
    assert "GSR_E_NOMEM" in str(e.value)
    assert h.m == dims.n_rows
    _compare(h, ref, with_f32=True)
    b = torch.randn(h.m, dtype=torch.float64, device="cuda")
    x = torch.empty(h.n, dtype=torch.float64, device="cuda")
    want = torch.empty_like(x)
    buf = gsr.solve_info_buffer()
    for precision in (gsr.GSR_F64, gsr.GSR_F32V):
        o = gsr.solve_opts(itnlim=5, fixed_iters=True, precision=precision, max_refine=1)
        gsr.gsr_lsqr_solve_async(h, b, x, buf, o)
        gsr.gsr_lsqr_solve(ref, b, want, o)
        assert rel(host(x), host(want)) <= 1e-10
    h.close()
    ref.close()
