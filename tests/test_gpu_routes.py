"""Which launches a plan takes: the plane passes (both transforms of a z-plane
by one workgroup) or a pass each along x and y, the plane-range depths of the
marches, and the tuner's y tile.  The fields of each route are compared with
the FP64 oracle, as in the other parity tests."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2204_08834_amd import inputs  # noqa: E402

PER, NEU, DIR = 0, 1, 2
EPS = 2.0 ** -52


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_08834_amd import poisson
    poisson.lib()
    return poisson


def _kappa(shape, sp, bc_z):
    """Condition number of the operator periodic in x and y."""
    lo, hi = [], 0.0
    for n, h, per in ((shape[0], sp[0], True), (shape[1], sp[1], True), (shape[2], sp[2], bc_z == PER)):
        if n == 1:
            continue
        m = np.arange(n) + (1 if not per and bc_z == DIR else 0)
        lam = 4 / h ** 2 * np.sin(np.pi * m / (n if per else 2 * n)) ** 2
        lo.append(lam[lam > 0].min())
        hi += lam.max()
    return hi / min(lo)


def _check(orc, P, nx, ny, nz, bc, precision, route, **kw):
    sp = (1.0 / nx, 1.0 / nx, 1.0 / nx)
    f = inputs.uniform_velocity_rhs(nx, ny, nz, nx * sp[0], ny * sp[1], nz * sp[2], bc, 29)
    rhs = torch.from_numpy(f).cuda()
    print(f"[routes] {nx}x{ny}x{nz} bc {bc} {precision} {route}", flush=True)
    with P.Plan(nx, ny, nz, *sp, bc, precision, bc_x=kw.get("bc_x", PER), bc_y=kw.get("bc_y", PER)) as plan:
        assert f" xy={route} " in plan.describe()
        out, st = plan.solve(rhs, torch.full_like(rhs, float("nan")))
        torch.cuda.synchronize()
    p = out.cpu().numpy()
    if precision == "fp64":
        ref = orc.solve(f, *sp, bc, **kw)
        err = np.linalg.norm(p - ref) / np.linalg.norm(ref)
        assert err <= max(1e-12, 4 * _kappa((nx, ny, nz), sp, bc) * EPS), err
    else:
        res, _ = orc.residual(f, p, *sp, bc, **kw)
        assert st["status"] == 0 and res <= 1e-10, res


# the largest planes of each precision with enough of them, the smallest, and
# what has no plane pass: more values than fit, a length without a class, walls
ROUTES = [
    ("fp64", 24, 2, 3, "plane"), ("fp64", 128, 128, 48, "plane"), ("fp64", 256, 64, 48, "plane"),
    ("fp64", 24, 512, 3, "plane"), ("fp64", 32, 512, 2, "plane"), ("fp32_refine", 192, 96, 64, "plane"),
    ("fp32_refine", 256, 128, 64, "plane"), ("fp32_refine", 128, 128, 2, "plane"),
    ("fp64", 256, 128, 4, "separate"), ("fp64", 384, 8, 4, "separate"),
    ("fp32_refine", 256, 256, 3, "separate"),
    # few of the largest planes
    ("fp64", 256, 64, 47, "separate"), ("fp64", 128, 128, 2, "separate"),
    ("fp32_refine", 192, 96, 63, "separate"), ("fp32_refine", 256, 128, 2, "separate"),
]


@pytest.mark.parametrize("case", ROUTES, ids=["-".join(map(str, c)) for c in ROUTES])
def test_transform_route(orc, case):
    precision, nx, ny, nz, route = case
    _check(orc, _gpu(), nx, ny, nz, NEU, precision, route)


def test_walls_along_y_take_separate_passes(orc):
    _check(orc, _gpu(), 64, 32, 6, NEU, "fp64", "separate", bc_y=NEU)


@pytest.mark.parametrize("shape", [(128, 128, 12), (256, 64, 12), (64, 256, 12), (32, 512, 12)])
def test_route_by_planes_in_flight_keeps_fp64_fields(shape):
    """A batch with enough planes takes the plane passes where one of its
    problems alone takes the separate ones: the same FP64 field bitwise."""
    P = _gpu()
    nx, ny, nz = shape
    spec = dict(nx=nx, ny=ny, nz=nz, dx=1.0 / nx, dy=1.0 / nx, dz=1.0 / nx, bc_z=NEU)
    print(f"[routes] batch of 4 {nx}x{ny}x{nz}", flush=True)
    rhs = [torch.from_numpy(inputs.random_rhs(nx, ny, nz, seed=60 + i)).cuda() for i in range(4)]
    outs = [torch.full_like(r, float("nan")) for r in rhs]
    bp = P.BatchPlan([spec] * 4, "fp64")
    assert " xy=plane " in bp.describe()
    bp.solve(rhs, outs)
    torch.cuda.synchronize()
    bp.close()
    route = "plane" if nx == 32 else "separate"
    with P.Plan(nx, ny, nz, 1.0 / nx, 1.0 / nx, 1.0 / nx, NEU, "fp64") as plan:
        assert f" xy={route} " in plan.describe()
        for r, o in zip(rhs, outs):
            q, _ = plan.solve(r, torch.full_like(r, float("nan")))
            torch.cuda.synchronize()
            assert torch.equal(q, o)


def test_plane_lists_of_deep_and_shallow_shapes(orc):
    """Small deep planes and large shallow ones in one batch, enough of both
    for a launch of their own, and shapes that share theirs: the oracle's
    field, FP64 with every problem bitwise as its single plan solves it."""
    P = _gpu()
    shapes = [(64, 64, 96)] * 6 + [(128, 128, 16)] * 8 + [(48, 24, 30), (96, 32, 9)]
    sp = [(1.0 / s[0],) * 3 for s in shapes]
    fs = [inputs.random_rhs(*s, seed=80 + i) for i, s in enumerate(shapes)]
    rhs = [torch.from_numpy(f).cuda() for f in fs]
    specs = [dict(nx=s[0], ny=s[1], nz=s[2], dx=h[0], dy=h[1], dz=h[2], bc_z=NEU)
             for s, h in zip(shapes, sp)]
    for precision in ("fp64", "fp32_refine"):
        print(f"[routes] deep and shallow planes {precision}", flush=True)
        bp = P.BatchPlan(specs, precision)
        assert "schedule=list" in bp.describe() and bp.describe().count("xy=plane") == 4
        outs = [torch.full_like(r, float("nan")) for r in rhs]
        bp.solve(rhs, outs)
        torch.cuda.synchronize()
        bp.close()
        for i in (0, 6, 13, 14, 15):
            if precision == "fp32_refine":
                res, _ = orc.residual(fs[i], outs[i].cpu().numpy(), *sp[i], NEU)
                assert res <= 1e-10, (i, res)
                continue
            with P.Plan(*shapes[i], *sp[i], NEU, precision) as plan:
                q, _ = plan.solve(rhs[i], torch.full_like(rhs[i], float("nan")))
                torch.cuda.synchronize()
            assert torch.equal(q, outs[i]), i


def test_residual_depth_fits_one_problem_only(monkeypatch):
    """An exact residual depth is chosen for a plan of one problem; the shapes
    of a batch keep the plain depth, halved by the problems of the launch."""
    P = _gpu()
    for v in ("POISSON_MARCH_PLANES", "POISSON_AUTOTUNE", "POISSON_TUNE_CACHE"):
        monkeypatch.delenv(v, raising=False)
    specs = [dict(nx=n, ny=n, nz=nz, dx=1.0 / n, dy=1.0 / n, dz=1.0 / n, bc_z=NEU)
             for n, nz in ((64, 66), (128, 62), (96, 50))]
    bp = P.BatchPlan(specs, "fp32_refine")
    assert bp.describe().count("march_planes=8 ") == 3, bp.describe()
    bp.close()
    for s in specs:
        with P.Plan(**s, precision="fp32_refine") as plan:
            assert "march_planes=8 " not in plan.describe(), plan.describe()
        one = P.BatchPlan([s], "fp32_refine")  # a batch of one is one problem
        assert "march_planes=8 " not in one.describe()
        one.close()


@pytest.mark.parametrize("planes", [4, 11])
def test_exact_depth_from_the_environment_reaches_the_divergence(planes, monkeypatch):
    """POISSON_MARCH_PLANES sets the depth of the projection's divergence march
    too, exact depths included: its partial sums number one per y-row block and
    range of planes (the sum pass reads 32 bytes of each).  4 planes are halved
    for a small grid, to one."""
    P = _gpu()
    nx, ny, nz = 64, 64, 44
    sums = {}
    for k in (planes, nz):
        monkeypatch.setenv("POISSON_MARCH_PLANES", str(k))
        u, v, w = (torch.from_numpy(inputs.random_rhs(nx, ny, nz, seed=90 + i)).cuda() for i in range(3))
        print(f"[routes] projection {nx}x{ny}x{nz} depth {k}", flush=True)
        with P.Plan(nx, ny, nz, 1.0 / nx, 1.0 / nx, 1.0 / nx, NEU, "fp32") as plan:
            plan.set_timing(True)
            plan.project(u, v, w)
            torch.cuda.synchronize()
            sums[k] = plan.timing()["sum_partials"]["bytes_per_launch"] / 32
    ranges = {4: nz, 11: 4}[planes]
    assert sums[planes] == ranges * sums[nz], sums


def test_y_tile_is_tuned_where_planes_fit(tmp_path, monkeypatch):
    """The corrections and the projection of a plane-sized problem run the
    forward y pass: the tuner picks its tile by timing, whatever tile the plan
    was created with (eight forced starts are not all recorded as chosen)."""
    P = _gpu()
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("POISSON_TUNE_CACHE", str(cache))
    nx, ny, nz = 64, 128, 64
    forced, chosen = [], []
    for v in (0, 1, 2, 3) * 2:
        monkeypatch.setenv("POISSON_Y_VARIANT", str(v))
        with P.Plan(nx, ny, nz, 1.0 / nx, 1.0 / nx, 1.0 / nx, NEU, "fp32_refine") as plan:
            assert " xy=plane " in plan.describe()
            plan.autotune(force=True)
        line = next(ln for ln in cache.read_text().splitlines()
                    if ln.startswith(f"f32 {nx} {ny} {nz} 001 "))
        forced.append(v)
        chosen.append(int(line.split(":")[1].split()[1]))
    print("[routes] y tiles", chosen, flush=True)
    assert all(0 <= c <= 3 for c in chosen) and chosen != forced


def test_zero_mode_block_keeps_tiles_on_their_dies(monkeypatch):
    """The workgroup of the zero wavenumber must not shift the z solve's tiles
    to other dies than those whose L2 holds (and will be asked for) their
    columns: the inverse y pass after a z solve with a zero mode takes what it
    takes after one without (Dirichlet walls along x; the y pass is the same
    kernel on the same sizes).  One leading block more, and not eight, made it
    1.9 times as long at this size, where the spectrum fits the eight L2s."""
    P = _gpu()
    monkeypatch.setenv("POISSON_BLOCK_ORDER", "forward")
    monkeypatch.setenv("POISSON_Y_VARIANT", "1")
    nx, ny, nz = 512, 128, 32
    f = torch.from_numpy(inputs.random_rhs(nx, ny, nz, seed=3)).cuda()
    out = torch.empty_like(f)
    best = {}
    for bc_x in (NEU, DIR):
        with P.Plan(nx, ny, nz, 1.0 / nx, 1.0 / nx, 1.0 / nx, NEU, "fp64", bc_x=bc_x) as plan:
            plan.set_timing(True)
            times = []
            for _ in range(8):
                plan.reset_timing()
                for _ in range(10):
                    plan.solve_async(f, out)
                torch.cuda.synchronize()
                t = plan.timing()["y_inv_f64"]
                times.append(t["total_ms"] / t["launches"])
            best[bc_x] = min(times)
    print(f"[routes] y inverse after z, us: {1e3 * best[NEU]:.1f} with a zero mode, "
          f"{1e3 * best[DIR]:.1f} without", flush=True)
    assert best[NEU] <= 1.25 * best[DIR], best


def test_mixed_batches_of_few_planes_take_separate_passes():
    """Plane groups beside others, fewer than 512 planes or less than a third of
    the points: every shape takes the separate passes, with the FP64 fields of the
    single plans bitwise.  512 planes of a third of the points, few planes of few
    values, and FP64 rows of 32 keep the plane passes."""
    P = _gpu()

    def batch(shapes, precision):
        return P.BatchPlan([dict(nx=s[0], ny=s[1], nz=s[2], dx=1.0 / s[0], dy=1.0 / s[0],
                                 dz=1.0 / s[0], bc_z=NEU) for s in shapes], precision)

    other = (256, 256, 4)
    for shapes, precision, planes in (
            ([(64, 64, 40), other], "fp64", 0), ([(64, 64, 40), other], "fp32_refine", 1),
            ([(96, 64, 40), other], "fp32_refine", 0), ([(96, 64, 40), (64, 64, 9), other], "fp32", 2),
            ([(64, 64, 128)] * 4 + [other], "fp64", 1), ([(64, 64, 127)] * 4 + [other], "fp64", 0),
            ([(64, 64, 128)] * 4 + [(256, 256, 70)], "fp64", 0),
            ([(64, 48, 9), (24, 24, 5), (256, 256, 1)], "fp64", 0),
            ([(64, 48, 14), (24, 24, 5), (256, 256, 1)], "fp64", 2),
            ([(64, 64, 9), (48, 24, 9)], "fp64", 2),
            ([(64, 64, 9), (32, 16, 4), other], "fp64", 2),
            ([(64, 64, 9), (32, 16, 4), other], "fp32", 2)):
        bp = batch(shapes, precision)
        assert bp.describe().count(" xy=plane ") == planes, (shapes, precision, bp.describe())
        bp.close()
    for precision in ("fp64", "fp32", "fp32_refine"):
        shapes = [(96, 64, 40), (128, 96, 7), other]
        print(f"[routes] mixed batch {precision}", flush=True)
        rhs = [torch.from_numpy(inputs.random_rhs(*s, seed=70 + i)).cuda()
               for i, s in enumerate(shapes)]
        outs = [torch.full_like(r, float("nan")) for r in rhs]
        bp = batch(shapes, precision)
        assert bp.describe().count(" xy=plane ") == 0
        bp.solve(rhs, outs)
        torch.cuda.synchronize()
        bp.close()
        for s, r, o in zip(shapes, rhs, outs):
            with P.Plan(*s, *((1.0 / s[0],) * 3), NEU, precision) as plan:
                assert (" xy=plane " in plan.describe()) == (s != other)
                q, _ = plan.solve(r, torch.full_like(r, float("nan")))
                torch.cuda.synchronize()
            if precision == "fp32_refine":
                assert float((q - o).abs().max()) <= 1e-14 * float(q.abs().max()), s
            else:
                assert torch.equal(q, o), (s, precision)


def test_large_fp32_planes_keep_the_route_of_their_own_plan():
    """256x128 (16 values per thread, two routes that round differently): 32
    planes are separate in a single plan and so in a batch of four; 192x96, whose
    routes give the same bits, goes by the planes of the batch."""
    P = _gpu()
    for nx, ny, nz, route in ((256, 128, 32, "separate"), (192, 96, 32, "plane")):
        spec = dict(nx=nx, ny=ny, nz=nz, dx=1.0 / nx, dy=1.0 / nx, dz=1.0 / nx, bc_z=NEU)
        print(f"[routes] four of {nx}x{ny}x{nz} fp32", flush=True)
        rhs = [torch.from_numpy(inputs.random_rhs(nx, ny, nz, seed=50 + i)).cuda() for i in range(4)]
        outs = [torch.full_like(r, float("nan")) for r in rhs]
        bp = P.BatchPlan([spec] * 4, "fp32")
        assert f" xy={route} " in bp.describe()
        bp.solve(rhs, outs)
        torch.cuda.synchronize()
        bp.close()
        with P.Plan(**spec, precision="fp32") as plan:
            assert " xy=separate " in plan.describe()
            for r, o in zip(rhs, outs):
                q, _ = plan.solve(r, torch.full_like(r, float("nan")))
                torch.cuda.synchronize()
                assert torch.equal(q, o)


@pytest.mark.parametrize("precision,nx", [("fp64", n) for n in (24, 32, 48, 64, 96, 128, 192, 256)]
                         + [("fp32", n) for n in (96, 128, 192)])
def test_routes_give_the_same_bits(precision, nx):
    """Plane passes against separate ones (which per-pass timing runs), every
    plane size of FP64 and the FP32 row lengths whose route a batch may choose: the
    same bits but for FP64 rows of 32 and 24x384, whose routes are never mixed."""
    P = _gpu()
    cap, many = (8192, 6144) if precision == "fp64" else (16384, 8192)
    for ny in (2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512):
        if nx // 2 * ny > cap:
            continue
        nz = 64 if nx // 2 * ny > many else 3
        f = torch.from_numpy(inputs.random_rhs(nx, ny, nz, seed=ny)).cuda()
        with P.Plan(nx, ny, nz, 1.0 / nx, 1.0 / ny, 1.0 / nz, NEU, precision) as plan:
            assert " xy=plane " in plan.describe(), (nx, ny, nz)
            a, _ = plan.solve(f, torch.full_like(f, float("nan")))
            plan.set_timing(True)
            b, _ = plan.solve(f, torch.full_like(f, float("nan")))
            torch.cuda.synchronize()
        if precision == "fp64" and (nx == 32 or (nx, ny) == (24, 384)):
            assert torch.allclose(a, b, rtol=0, atol=1e-12 * float(b.abs().max())), (nx, ny)
        else:
            assert torch.equal(a, b), (nx, ny)
