"""Half-sweeps run as one launch (tiles of whole x-lines with halo rows relaxed redundantly) against the colour
launches: the same operations in the same order, so the results must agree bit for bit (tolerance zero).  A handle
with pair_rows = 0 runs every colour as its own launch."""
import numpy as np
import pytest

from paper_2507_11512_amd import inputs

pytestmark = pytest.mark.gpu

VEC = {0: "float64", 4: "float16", 5: "bfloat16"}


@pytest.fixture(scope="module")
def hp():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2507_11512_amd import hpgmx
    return hpgmx


def vec(dims, seed, dtype):
    import torch
    return torch.from_numpy(inputs.uniform(dims, seed)).to("cuda", getattr(torch, VEC.get(dtype, "float32")))


def pair(hp, dims, **kw):
    return [hp.Problem(dims, beta=0.3, layout=lay, **kw) for lay in (None, {"pair_rows": 0})]


def launches(hp, P, call):
    """Number of launches `call` enqueues on P's stream (which must not be the default one), by capturing it."""
    import ctypes as C
    import torch
    stream, graph, n = C.c_void_p(P.stream.cuda_stream), C.c_void_p(), C.c_size_t()
    call()  # what a first call allocates and works out
    torch.cuda.synchronize()
    assert hp.lib.hipStreamBeginCapture(stream, 1) == 0  # 1: thread-local
    try:
        call()
    finally:
        assert hp.lib.hipStreamEndCapture(stream, C.byref(graph)) == 0
    assert hp.lib.hipGraphGetNodes(graph, None, C.byref(n)) == 0 and hp.lib.hipGraphDestroy(graph) == 0
    return n.value


# tile edges: one cell, fewer cells than a tile, odd extents in each direction, several tiles with a remainder, tiles
# of several row chunks, the largest level (2^22 rows; in FP64 beyond its largest), long and short x-lines
DIMS = [(2, 2, 2), (3, 5, 4), (13, 9, 7), (2, 34, 3), (64, 3, 2), (37, 26, 51), (50, 38, 26), (100, 102, 102), (131, 70, 99),
        (128, 256, 128)]


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("dtype", [0, 1, 2, 3, 4, 5])
def test_smooth(hp, dims, dtype):
    import torch
    Ps = pair(hp, dims, levels=1)
    try:
        r = vec(dims, 41, dtype)
        for sweep in (0, 1, 2):
            for zero in (True, False):
                zs = [vec(dims, 42, dtype) for _ in Ps]
                for P, z in zip(Ps, zs):
                    hp.smooth(P.h, 0, dtype, sweep, r, z, zero_guess=zero)
                assert torch.equal(zs[0], zs[1]), (sweep, zero)
    finally:
        for P in Ps:
            P.close()


@pytest.mark.parametrize("dims,levels,pre,post,coarsest", [((16, 16, 16), 3, 1, 1, 1), ((24, 20, 28), 3, 1, 1, 1),
                                                           ((50, 38, 26), 2, 2, 1, 1), ((48, 8, 40), 3, 1, 2, 3),
                                                           ((32, 24, 16), 3, 2, 2, 1), ((16, 16, 16), 2, 0, 1, 1),
                                                           ((16, 16, 16), 2, 1, 0, 0), ((192, 160, 128), 4, 1, 1, 1)])
@pytest.mark.parametrize("dtype,cols", [(0, "int32"), (1, "int32"), (1, "offset16"), (2, "int32"), (5, "int32")])
def test_vcycle(hp, dims, levels, pre, post, coarsest, dtype, cols):
    """Restriction and prolongation ride on the sweeps; every sweep kind, several sweeps per level."""
    import torch
    for sweep in ("forward", "backward", "symmetric"):
        Ps = pair(hp, dims, levels=levels, pre=pre, post=post, coarsest=coarsest, sweep=sweep, cols=cols)
        try:
            r = vec(dims, 43, dtype)
            zs = [torch.full_like(r, float("nan")) for _ in Ps]
            for P, z in zip(Ps, zs):
                hp.vcycle(P.h, dtype, r, z)
            assert torch.isfinite(zs[0]).all() and torch.equal(zs[0], zs[1]), sweep
        finally:
            for P in Ps:
                P.close()


@pytest.mark.parametrize("dtype", [0, 1, 4])
def test_not_finite(hp, dtype):
    """Infinities and NaN spread as they do through the colour launches (padded and skipped slots add nothing)."""
    import torch
    dims = (24, 20, 16)
    for sweep in ("forward", "backward", "symmetric"):
        Ps = pair(hp, dims, levels=3, sweep=sweep)
        try:
            for at, v in ((0, "inf"), (3001, "nan"), (3000, "-inf"), (24 * 20 * 16 - 1, "nan")):
                r = vec(dims, 50, dtype)
                r[at] = float(v)
                zs = [torch.zeros_like(r) for _ in Ps]
                for P, z in zip(Ps, zs):
                    hp.vcycle(P.h, dtype, r, z)
                assert torch.equal(zs[0].isnan(), zs[1].isnan()), (sweep, at)
                assert torch.equal(zs[0].nan_to_num(), zs[1].nan_to_num()), (sweep, at)
        finally:
            for P in Ps:
                P.close()


@pytest.mark.parametrize("dtype,nrhs,extents", [(0, 1, range(128, 240, 12)), (1, 1, range(256, 480, 24)),
                                                 (5, 1, range(512, 960, 48)), (1, 8, range(24, 72, 4)),
                                                 (0, 4, range(24, 72, 4))])
def test_widest_lines(hp, dtype, nrhs, extents):
    """Around the widest x-lines whose tiles fit the LDS: the forms of a sweep need different amounts of it (the
    backward restriction most), and a level runs in tiles only if all of them fit."""
    import torch
    for nx in extents:
        dims = (nx, 8, 12)
        for sweep in ("forward", "backward", "symmetric"):
            Ps = pair(hp, dims, levels=2, sweep=sweep)
            try:
                r = torch.stack([vec(dims, 70 + j, dtype) for j in range(nrhs)])
                zs = [torch.full_like(r, float("nan")) for _ in Ps]
                for P, z in zip(Ps, zs):
                    if nrhs == 1:
                        hp.vcycle(P.h, dtype, r[0], z[0])
                    else:
                        hp.vcycle_batched(P.h, dtype, r, z)
                assert torch.isfinite(zs[0]).all() and torch.equal(zs[0], zs[1]), (nx, sweep)
            finally:
                for P in Ps:
                    P.close()


# interleaved right-hand sides: levels below and above what a workgroup can hold, odd extents
@pytest.mark.parametrize("dims,levels", [((16, 12, 20), 3), ((40, 48, 56), 2), ((37, 26, 51), 1), ((64, 40, 48), 3),
                                         ((112, 88, 72), 4)])
@pytest.mark.parametrize("nrhs", [2, 3, 8])
@pytest.mark.parametrize("dtype", [0, 1, 3])
def test_batched(hp, dims, levels, nrhs, dtype):
    import torch
    for sweep in ("forward", "backward", "symmetric"):
        Ps = pair(hp, dims, levels=levels, sweep=sweep)
        try:
            r = torch.stack([vec(dims, 60 + j, dtype) for j in range(nrhs)])
            zs = [torch.full_like(r, float("nan")) for _ in Ps]
            for P, z in zip(Ps, zs):
                hp.vcycle_batched(P.h, dtype, r, z)
            assert torch.isfinite(zs[0]).all() and torch.equal(zs[0], zs[1]), sweep
            code = {"forward": hp.GS_FORWARD, "backward": hp.GS_BACKWARD, "symmetric": hp.GS_SYMMETRIC}[sweep]
            for zero in (True, False):
                for P, z in zip(Ps, zs):
                    z.copy_(r)
                    hp.smooth_batched(P.h, 0, dtype, code, r, z, zero_guess=zero)
                assert torch.equal(zs[0], zs[1]), (sweep, zero)
        finally:
            for P in Ps:
                P.close()


@pytest.mark.parametrize("bound", [False, True])
def test_solve_in_bound_workspace(hp, bound):
    """The second vectors of the tiled sweeps come out of a workspace of the advertised size; replayed graphs and
    launches from the host give the same iterates."""
    import torch
    dims = (40, 24, 32)
    out = []
    for graph in (False, True):
        ws = None
        if bound:
            h = hp.setup_problem(*dims, beta=0.3)
            ws = torch.empty(hp.workspace_bytes(h, levels=3, restart=30, dtype_mask=3), dtype=torch.uint8, device="cuda")
            hp.destroy(h)
        P = hp.Problem(dims, beta=0.3, levels=3, sweep="symmetric", workspace=ws)
        b = P.rhs_from_x(vec(dims, 44, 0))
        for _ in range(3):
            x, st = P.solve(b, tol=1e-11, precision="mxp", graph=graph)
            assert st.converged
            out.append(x.cpu().numpy())
        P.close()
    assert all(np.array_equal(out[0], o) for o in out[1:])
    ref = inputs.uniform(dims, 44)
    assert np.linalg.norm(out[0] - ref) <= 1e-8 * np.linalg.norm(ref)


def test_workspace_without_second_vectors(hp):
    """The tiled sweeps take no memory of their own: a workspace that holds what the colour launches need holds every
    call, in the order that takes the single-precision vectors first, and gives the iterates of owned memory."""
    import torch
    dims, mask = (48, 40, 32), 0x3F
    size = []
    for lay in ({}, {"pair_rows": 0}):
        h = hp.setup_problem(*dims, beta=0.3)
        hp.set_layout(h, **lay)
        size.append(hp.workspace_bytes(h, levels=3, restart=30, dtype_mask=mask) +
                    hp.workspace_bytes_batched(h, 4, levels=3, restart=30, dtype_mask=0xF))
        hp.destroy(h)
    assert size[0] == size[1]
    ws = torch.empty(size[1], dtype=torch.uint8, device="cuda")
    Ps = [hp.Problem(dims, beta=0.3, levels=3, sweep="symmetric", workspace=w) for w in (None, ws)]
    try:
        out = [[], []]
        for P, o in zip(Ps, out):
            b = P.rhs_from_x(vec(dims, 44, 0))
            B = torch.stack([b, 2 * b, b.flip(0)])
            for dtype in (1, 0, 4, 5):
                z = torch.zeros_like(vec(dims, 45, dtype))
                hp.vcycle(P.h, dtype, vec(dims, 45, dtype), z)
                o.append(z)
            for dtype in (1, 0):
                R = B.to(getattr(torch, VEC.get(dtype, "float32")))
                Z = torch.zeros_like(R)
                hp.vcycle_batched(P.h, dtype, R, Z)
                o.append(Z)
            for precision in ("mxp", "fp64", "fp16", "bf16", "fp16-mg", "bf16-mg"):
                o.append(P.solve(b, tol=1e-9, precision=precision)[0])
            for precision in ("mxp", "fp64", "fp16", "bf16"):
                o.append(P.solve_batched(B, tol=1e-9, precision=precision)[0])
        assert all(torch.equal(a, c) for a, c in zip(*out))
    finally:
        for P in Ps:
            P.close()


def test_tuning_table_keeps_the_dispatch(hp):
    """A table of tile shapes that is read back and set on another handle, or set by hand, leaves the sweeps in tiles:
    as many launches as without a table, fewer than a launch per colour."""
    import torch
    dims, nrhs = (32, 32, 32), 4
    r = torch.stack([vec(dims, 80 + j, 1) for j in range(nrhs)])
    Ps = [hp.Problem(dims, levels=3, stream=torch.cuda.Stream(), layout=lay) for lay in (None, None, {"pair_rows": 0})]
    try:
        def count(P):
            z = torch.zeros_like(r)
            return (launches(hp, P, lambda: hp.vcycle_batched(P.h, 1, r, z)),
                    launches(hp, P, lambda: hp.smooth_batched(P.h, 0, 1, hp.GS_FORWARD, r, z)))
        plain, colours = count(Ps[0]), count(Ps[2])
        assert plain[0] < colours[0] - 20 and plain[1] == colours[1] - 7
        table = hp.batch_autotune(Ps[0].h, nrhs, 1)["rhs_per_lane"]
        assert count(Ps[0]) == plain
        hp.batch_set_tuning(Ps[1].h, nrhs, 1, table)
        assert hp.batch_get_tuning(Ps[1].h, nrhs, 1)["rhs_per_lane"] == table and count(Ps[1]) == plain
        hp.batch_set_tuning(Ps[1].h, nrhs, 1, 1)
        assert count(Ps[1]) == plain
    finally:
        for P in Ps:
            P.close()


@pytest.mark.parametrize("dims,levels", [((16, 16, 16), 3), ((24, 20, 16), 3), ((14, 18, 10), 2)])
@pytest.mark.parametrize("nrhs", [2, 3, 8])
@pytest.mark.parametrize("dtype", [0, 1, 3])
def test_colour_launches_every_tile_shape(hp, dims, levels, nrhs, dtype):
    """The batched colour launches in every tile shape against the tiled sweeps."""
    import torch
    K = 2 if nrhs <= 2 else 4 if nrhs <= 4 else 8
    for sweep in ("forward", "backward", "symmetric"):
        P, Q = pair(hp, dims, levels=levels, sweep=sweep)
        try:
            r = torch.stack([vec(dims, 90 + j, dtype) for j in range(nrhs)])
            code = {"forward": hp.GS_FORWARD, "backward": hp.GS_BACKWARD, "symmetric": hp.GS_SYMMETRIC}[sweep]

            def results(H):
                out = [torch.full_like(r, float("nan")), torch.full_like(r, float("nan")), r.clone()]
                hp.vcycle_batched(H.h, dtype, r, out[0])
                hp.smooth_batched(H.h, 0, dtype, code, r, out[1], zero_guess=True)
                hp.smooth_batched(H.h, 0, dtype, code, r, out[2])
                return out
            ref = results(P)
            for R in (1, 2, 4, 8):
                if R > K:
                    continue
                hp.batch_set_tuning(Q.h, nrhs, dtype, R)
                assert all(torch.equal(a, b) for a, b in zip(results(Q), ref)), (sweep, R)
        finally:
            P.close()
            Q.close()


@pytest.mark.parametrize("dims,dtype,nrhs,sweep,cycle,alone", [
    ((160, 160, 160), 1, 1, "forward", True, True), ((256, 128, 120), 1, 1, "forward", True, True),
    ((400, 100, 104), 1, 1, "forward", False, True), ((440, 96, 96), 1, 1, "symmetric", False, True),
    ((440, 64, 64), 1, 1, "backward", False, True), ((112, 112, 112), 0, 1, "forward", True, True),
    ((220, 80, 88), 0, 1, "forward", False, False), ((200, 60, 60), 0, 1, "backward", False, True),
    ((160, 160, 160), 4, 1, "forward", True, True), ((640, 80, 80), 5, 1, "forward", False, True),
    ((900, 16, 16), 5, 1, "symmetric", False, False), ((256, 128, 120), 2, 1, "forward", True, True),
    ((400, 100, 104), 2, 1, "backward", False, True), ((96, 96, 96), 1, 2, "symmetric", True, True),
    ((220, 48, 48), 1, 2, "forward", False, False), ((110, 48, 48), 1, 4, "symmetric", False, False),
    ((48, 64, 64), 1, 8, "backward", False, True), ((80, 80, 80), 0, 2, "forward", True, True)])
def test_long_lines_keep_the_colour_launches(hp, dims, dtype, nrhs, sweep, cycle, alone):
    """Levels where half-sweeps in tiles were measured slower, because a tile of whole x-lines leaves room for few
    cells in y and z, take a launch per colour: in a V-cycle (`cycle`: level 0 runs in tiles), or for a sweep by
    itself from given values (`alone`), where tiles pay further."""
    import torch
    P = hp.Problem(dims, levels=2, sweep=sweep, stream=torch.cuda.Stream())
    code = {"forward": hp.GS_FORWARD, "backward": hp.GS_BACKWARD, "symmetric": hp.GS_SYMMETRIC}[sweep]
    half = 2 if sweep == "symmetric" else 1
    try:
        r = torch.zeros((nrhs, P.N), device="cuda", dtype=getattr(torch, VEC.get(dtype, "float32")))
        z = torch.zeros_like(r)
        if nrhs == 1:
            n = [launches(hp, P, f) for f in (lambda: hp.smooth(P.h, 0, dtype, code, r[0], z[0]),
                                              lambda: hp.vcycle(P.h, dtype, r[0], z[0]))]
        else:
            n = [launches(hp, P, f) for f in (lambda: hp.smooth_batched(P.h, 0, dtype, code, r, z),
                                              lambda: hp.vcycle_batched(P.h, dtype, r, z))]
        assert n[0] - 3 == (half if alone else 8 * half - half // 2)  # beside two permutations in and one out
        # beside a permutation each way, level 0 in tiles takes a launch per half-sweep (level 1 up to eight)
        assert (n[1] - 2 <= 2 * half + 8 * half) == cycle, n[1]
    finally:
        P.close()


def test_handles_on_two_threads(hp):
    """Two threads with a handle each, whose tiles take different amounts of LDS in the same kernel: the limit that a
    launch asks for is the kernel's, so each must leave it high enough for the other."""
    import threading

    import torch
    shapes = [(320, 64, 48), (200, 152, 104)]
    Ps = [hp.Problem(d, levels=2, stream=torch.cuda.Stream()) for d in shapes]
    rs = [vec(d, 95, 1) for d in shapes]
    refs = [torch.empty_like(r) for r in rs]
    for P, r, z in zip(Ps, rs, refs):
        hp.vcycle(P.h, 1, r, z)
    torch.cuda.synchronize()
    bad = []

    def work(P, r, ref):
        try:
            z = torch.empty_like(r)
            for _ in range(200):
                hp.vcycle(P.h, 1, r, z)
            P.stream.synchronize()
            if not torch.equal(z, ref):
                bad.append("result")
        except Exception as e:
            bad.append(e)
    threads = [threading.Thread(target=work, args=a) for a in zip(Ps, rs, refs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for P in Ps:
        P.close()
    assert not bad, bad


@pytest.mark.parametrize("sweep", ["forward", "backward", "symmetric"])
@pytest.mark.parametrize("nrhs", [1, 3])
def test_profile_times_the_launches_of_the_solve(hp, sweep, nrhs):
    """A profiled solve makes the launches of any other where level 0 runs in tiles: every level counts one per
    half-sweep, with the restriction and the prolongation in it, and the byte model prices them as such."""
    import torch

    import bench
    from paper_2507_11512_amd import perfmodel as pm
    dims, V, half = (32, 48, 40), 31, 2 if sweep == "symmetric" else 1
    cfg = pm.Config(dims=dims, levels=3, sweep=bench.SWEEP_CODE[sweep])
    for lay, tiles in ((None, True), ({"pair_rows": 0}, False)):
        P = hp.Problem(dims, levels=3, sweep=sweep, layout=lay)
        try:
            b = P.rhs_from_x(vec(dims, 96, 0))
            B = torch.stack([b, 2 * b, b.flip(0)])
            kw = dict(tol=0.0, restart=30, max_iters=30)
            x = [P.solve(b, profile=p, **kw)[0] if nrhs == 1 else P.solve_batched(B, profile=p, **kw)[0]
                 for p in (False, True)]
            assert torch.equal(x[0], x[1])
            n = {(k, l): hp.profile_get(P.h, k, l)[1] for l in range(3)
                 for k in (hp.K_GS, hp.K_GS_ZERO, hp.K_RESTRICT, hp.K_PROLONG)}
            assert bench.tiled_levels(hp, P.h, cfg, [30]) == ({0, 1, 2} if tiles else set())
            T = bench.kernel_bytes_table(cfg, [30], 1, hp, pm, tiled={0, 1, 2} if tiles else ())
            for l in range(3):
                if tiles:
                    assert n[hp.K_GS_ZERO, l] == V and n[hp.K_GS, l] == V * (2 * half - 1 if l < 2 else half - 1)
                    assert n[hp.K_RESTRICT, l] == n[hp.K_PROLONG, l] == 0
                for k in (hp.K_GS, hp.K_GS_ZERO, hp.K_RESTRICT, hp.K_PROLONG):
                    assert (T.get((k, l), 0) > 0) == (n[k, l] > 0)
        finally:
            P.close()


@pytest.mark.parametrize("dims,dtype,nrhs", [((64, 64, 64), 1, 1), ((320, 64, 48), 1, 1), ((96, 80, 64), 0, 1),
                                             ((40, 48, 56), 1, 3)])
def test_captured_cycle(hp, dims, dtype, nrhs):
    """A program that captures a V-cycle: replays on new inputs, with the program's own work between them."""
    import torch
    P = hp.Problem(dims, levels=3, stream=torch.cuda.Stream())
    try:
        rs = [torch.stack([vec(dims, 97 + 5 * i + j, dtype) for j in range(nrhs)]) for i in range(3)]
        r, z = rs[0].clone(), torch.zeros_like(rs[0])

        def cycle():
            if nrhs == 1:
                hp.vcycle(P.h, dtype, r[0], z[0])
            else:
                hp.vcycle_batched(P.h, dtype, r, z)
        torch.cuda.synchronize()
        refs = []
        for x in rs:
            r.copy_(x)
            torch.cuda.synchronize()
            cycle()
            torch.cuda.synchronize()
            refs.append(z.clone())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=P.stream):
            cycle()
        for _ in range(2):
            for x, ref in zip(rs, refs):
                r.copy_(x)
                z.zero_()
                torch.cuda.synchronize()
                g.replay()
                torch.cuda.synchronize()
                assert torch.equal(z, ref)
                assert torch.equal((2 * x).sum(), (x + x).sum())  # other work between the replays
    finally:
        P.close()
