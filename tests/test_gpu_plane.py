"""Plane passes (k_plane.hip: both transforms of a z-plane by one workgroup)
at the edges of their range: the fewest rows, lengths with a factor 3 along x
and y, rows that leave threads of the last wavefront idle, the largest planes
(8192 complex values per plane in FP64 with 1024 threads, 16384 in FP32 with
16 values per thread), and batches whose work list mixes plane sizes.

Against the FP64 oracle: FP64 to max(1e-12, 4 kappa eps) as in the other
parity tests, FP32 + refinement to an oracle residual of 1e-10 (the stopping
rule).  With per-pass timing the same plan runs the separate passes: both
give the oracle's field."""
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
    lo, hi = [], 0.0
    for n, h, per in ((shape[0], sp[0], True), (shape[1], sp[1], True), (shape[2], sp[2], bc_z == PER)):
        if n == 1:
            continue
        m = np.arange(n) + (1 if not per and bc_z == DIR else 0)
        lam = 4 / h ** 2 * np.sin(np.pi * m / (n if per else 2 * n)) ** 2
        lo.append(lam[lam > 0].min())
        hi += lam.max()
    return hi / min(lo)


# nx, ny, nz, bc_z
CASES = [(24, 2, 5, NEU), (32, 3, 7, DIR), (48, 6, 4, PER), (64, 48, 3, NEU), (96, 96, 5, NEU),
         (192, 24, 6, PER), (128, 128, 2, NEU), (256, 64, 3, DIR), (24, 512, 2, NEU),
         (256, 128, 3, NEU), (192, 128, 2, NEU)]


@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}x{c[1]}x{c[2]}_{'pnd'[c[3]]}" for c in CASES])
def test_plane_passes_match_oracle(orc, case, precision):
    P = _gpu()
    nx, ny, nz, bc = case
    sp = (1.0 / nx, 1.0 / nx, 1.0 / nx)
    f = inputs.uniform_velocity_rhs(nx, ny, nz, nx * sp[0], ny * sp[1], nz * sp[2], bc, 17)
    ref = orc.solve(f, *sp, bc)
    bound = max(1e-12, 4 * _kappa((nx, ny, nz), sp, bc) * EPS)
    print(f"[plane] {case} {precision}", flush=True)
    rhs = torch.from_numpy(f).cuda()
    for timing in (False, True):
        with P.Plan(nx, ny, nz, *sp, bc, precision) as plan:
            plan.set_timing(timing)
            out, st = plan.solve(rhs, torch.full_like(rhs, float("nan")))
            torch.cuda.synchronize()
        p = out.cpu().numpy()
        if precision == "fp64":
            err = np.linalg.norm(p - ref) / np.linalg.norm(ref)
            assert err <= bound, (timing, err)
        else:
            res, _ = orc.residual(f, p, *sp, bc)
            assert st["status"] == 0 and res <= 1e-10, (timing, res)


@pytest.mark.parametrize("mode", ["host", "graph"])
def test_plane_lists_of_mixed_sizes(orc, mode):
    """A batch whose plane lists hold every thread count, one shape with 16
    values per thread and one without plane passes."""
    P = _gpu()
    shapes = [(24, 4, 6), (64, 64, 5), (128, 128, 3), (256, 128, 2), (512, 8, 4)]
    probs = [(nx, ny, nz, b) for nx, ny, nz in shapes for b in range(2)]
    fs = [inputs.uniform_velocity_rhs(nx, ny, nz, 1.0, ny / nx, nz / nx, NEU, 40 + b)
          for nx, ny, nz, b in probs]
    specs = [dict(nx=nx, ny=ny, nz=nz, dx=1.0 / nx, dy=1.0 / nx, dz=1.0 / nx, bc_z=NEU)
             for nx, ny, nz, _ in probs]
    bp = P.BatchPlan(specs, "fp32_refine")
    bp.set_graph(mode)
    rhs = [torch.from_numpy(f).cuda() for f in fs]
    outs = [torch.full_like(r, float("nan")) for r in rhs]
    for _ in range(2):
        rc, st = bp.solve(rhs, outs, check=False)
        torch.cuda.synchronize()
        assert rc == 0, st
        for f, o, s in zip(fs, outs, specs):
            res, _ = orc.residual(f, o.cpu().numpy(), s["dx"], s["dy"], s["dz"], NEU)
            assert res <= 1e-10, (s, res)
    bp.close()
