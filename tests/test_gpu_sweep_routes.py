"""Solves through the two routes of a half-sweep (pair_rows = 0: a launch per colour; default: tiles where they apply),
with every way of sharing the SpMV with the last sweep.  Each route does the same operations in the same order, so the
iterates must agree bit for bit (tolerance zero)."""
import pytest

from paper_2507_11512_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hp():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2507_11512_amd import hpgmx
    return hpgmx


def uniform(dims, seed):
    import torch
    return torch.from_numpy(inputs.uniform(dims, seed)).to("cuda", torch.float64)


def solves(hp, dims, modes, solve, **kw):
    """{(mode, route): result of solve(P)} for the colour launches and the default."""
    out = {}
    for mode in modes:
        for route, lay in (("colours", {"pair_rows": 0}), ("tiles", {})):
            P = hp.Problem(dims, beta=0.5, layout={"spmv_in_sweep": mode, **lay}, **kw)
            try:
                out[mode, route] = solve(P)
            finally:
                P.close()
    return out


def same(a, b):
    import torch
    return torch.equal(a[0], b[0]) and a[1] == b[1]


@pytest.mark.parametrize("sweep", ["forward", "backward", "symmetric"])
@pytest.mark.parametrize("precision,cols", [("mxp", "int32"), ("fp64", "int32"), ("fp16", "int32"), ("bf16", "int32"),
                                            ("fp16-mg", "int32"), ("bf16-mg", "int32"), ("mxp", "offset16"),
                                            ("fp64", "offset16"), ("bf16-mg", "offset16")])
@pytest.mark.parametrize("dims,levels,post", [((32, 24, 40), 3, 1), ((20, 24, 14), 2, 2)])
def test_spmv_modes(hp, sweep, precision, cols, dims, levels, post):
    """The colour launches that write their rows (1) or partial sums (2) of w against the SpMV that forms them alone
    (0, 3), and all of them against the tiled solve."""
    b = uniform(dims, 11)

    def solve(P):
        x, st = P.solve(b, tol=1e-9, max_iters=60, precision=precision)
        return x, (st.iters, st.final_rel_res)
    out = solves(hp, dims, (0, 1, 2, 3), solve, levels=levels, post=post, sweep=sweep, cols=cols)
    for a, c in ((0, 1), (2, 3)):
        assert same(out[a, "colours"], out[c, "colours"]), (a, c)
    for mode in (0, 1, 2, 3):
        assert same(out[mode, "colours"], out[mode, "tiles"]), mode


@pytest.mark.parametrize("sweep", ["forward", "backward", "symmetric"])
@pytest.mark.parametrize("precision", ["mxp", "fp64", "fp16"])
@pytest.mark.parametrize("nrhs", [2, 3, 8])
def test_batched_spmv_modes(hp, sweep, precision, nrhs):
    import torch
    dims = (16, 24, 20)
    B = torch.stack([uniform(dims, 20 + j) for j in range(nrhs)])

    def solve(P):
        X, st = P.solve_batched(B, tol=1e-9, max_iters=60, precision=precision)
        return X, [(s.iters, s.final_rel_res) for s in st]
    out = solves(hp, dims, (0, 1, 2, 3), solve, levels=3, sweep=sweep)
    assert same(out[0, "colours"], out[1, "colours"]) and same(out[2, "colours"], out[3, "colours"])
    for mode in (0, 1, 2, 3):
        assert same(out[mode, "colours"], out[mode, "tiles"]), mode


@pytest.mark.parametrize("dims,precision", [((144, 128, 120), "mxp"), ((160, 160, 160), "mxp"), ((144, 128, 120), "bf16-mg")])
def test_tiled_level_beyond_one_spmv_launch(hp, dims, precision):
    """Levels in tiles of more than 2^21 rows: the split sums of their SpMV take a launch per colour."""
    b = uniform(dims, 12)

    def solve(P):
        x, st = P.solve(b, tol=0.0, restart=6, max_iters=6, precision=precision)
        return x, (st.iters, st.final_rel_res)
    out = solves(hp, dims, (2, 3), solve, levels=3)
    assert all(same(out[2, "colours"], o) for o in out.values())


def equal_but_nan(a, b):
    import torch
    return torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(), b.nan_to_num())


@pytest.mark.parametrize("dtype,nrhs", [(0, 1), (1, 1), (4, 1), (5, 1), (0, 2), (1, 3), (1, 8), (3, 4)])
@pytest.mark.parametrize("dims", [(24, 20, 16), (14, 18, 10)])
def test_not_finite_in_batches_and_starts(hp, dtype, nrhs, dims):
    """Infinities and NaN in one right-hand side, and in the values a sweep starts from, spread as they do through the
    colour launches, and not to the right-hand side that shares a lane."""
    import torch
    vt = {0: torch.float64, 4: torch.float16, 5: torch.bfloat16}.get(dtype, torch.float32)
    n = dims[0] * dims[1] * dims[2]
    for sweep in ("forward", "backward", "symmetric"):
        Ps = [hp.Problem(dims, beta=0.3, levels=2, sweep=sweep, layout=lay) for lay in (None, {"pair_rows": 0})]
        code = {"forward": hp.GS_FORWARD, "backward": hp.GS_BACKWARD, "symmetric": hp.GS_SYMMETRIC}[sweep]
        try:
            for at, v in ((0, "inf"), (n // 2 + 1, "nan"), (n // 2, "-inf"), (n - 1, "nan")):
                r = torch.stack([uniform(dims, 30 + j).to(vt) for j in range(nrhs)])
                bad = r.clone()
                bad[nrhs // 2, at] = float(v)

                def run(P):
                    out = [torch.zeros_like(r), bad.clone(), r.clone()]
                    if nrhs == 1:
                        hp.vcycle(P.h, dtype, bad[0], out[0][0])
                        hp.smooth(P.h, 0, dtype, code, r[0], out[1][0])
                        hp.smooth(P.h, 0, dtype, code, bad[0], out[2][0])
                    else:
                        hp.vcycle_batched(P.h, dtype, bad, out[0])
                        hp.smooth_batched(P.h, 0, dtype, code, r, out[1])
                        hp.smooth_batched(P.h, 0, dtype, code, bad, out[2])
                    return out
                for a, b in zip(*(run(P) for P in Ps)):
                    assert equal_but_nan(a, b), (sweep, at, v)
                    for j in range(nrhs):
                        assert j == nrhs // 2 or a[j].isfinite().all()
        finally:
            for P in Ps:
                P.close()
