"""y transforms of the lengths that take a radix of 12 or 16 (384, 768, 1024,
2048), each beside a ragged tile of x-wavenumbers, forward and inverse, with
the tile widths of the launch variants: against the FP64 oracle, to
max(1e-12, 4 kappa eps) in FP64 and an oracle residual of 1e-10 under FP32 +
refinement (as the other parity tests)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2204_08834_amd import inputs  # noqa: E402


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
@pytest.mark.parametrize("ny", [384, 768, 1024, 2048])
def test_long_y_matches_oracle(orc, ny, precision, variant, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_08834_amd import poisson as P
    nx, nz, h = 48 if precision == "fp64" else 96, 3, 1.0 / 64
    print(f"[radix] {nx}x{ny}x{nz} {precision} variant {variant}", flush=True)
    monkeypatch.setenv("POISSON_Y_VARIANT", str(variant))
    f = inputs.uniform_velocity_rhs(nx, ny, nz, nx * h, ny * h, nz * h, 1, 23)
    ref = orc.solve(f, h, h, h, 1)
    rhs = torch.from_numpy(f).cuda()
    with P.Plan(nx, ny, nz, h, h, h, 1, precision) as plan:
        plan.set_timing(True)  # separate passes also where planes fit one workgroup
        out, st = plan.solve(rhs, torch.full_like(rhs, float("nan")))
        torch.cuda.synchronize()
    p = out.cpu().numpy()
    if precision == "fp64":
        kappa = 12.0 / (4 * np.sin(np.pi / ny) ** 2)
        err = np.linalg.norm(p - ref) / np.linalg.norm(ref)
        assert err <= max(1e-12, 4 * kappa * 2.0 ** -52), err
    else:
        res, _ = orc.residual(f, p, h, h, h, 1)
        assert st["status"] == 0 and res <= 1e-10, res


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("bc_y", [1, 2])
@pytest.mark.parametrize("ny", [384, 768, 1024])
def test_long_wall_y_matches_oracle(orc, ny, bc_y, variant, monkeypatch):
    """The same lengths between walls along y (both forward variants)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_08834_amd import poisson as P
    nx, nz, h = 24, 3, 1.0 / 64
    monkeypatch.setenv("POISSON_Y_VARIANT", str(variant))
    f = inputs.random_rhs(nx, ny, nz, seed=ny + bc_y)
    ref = orc.solve(f, h, h, h, 1, bc_y=bc_y)
    res_ref, _ = orc.residual(f, ref, h, h, h, 1, bc_y=bc_y)
    kappa = 12.0 / (4 * np.sin(np.pi / (2 * ny)) ** 2)
    rhs = torch.from_numpy(f).cuda()
    for precision in ("fp64", "fp32_refine"):
        print(f"[radix] {nx}x{ny}x{nz} walls {bc_y} {precision} variant {variant}", flush=True)
        rtol = max(1e-10, 10 * res_ref)
        with P.Plan(nx, ny, nz, h, h, h, 1, precision, rtol=rtol, bc_y=bc_y) as plan:
            out, st = plan.solve(rhs, torch.full_like(rhs, float("nan")))
            torch.cuda.synchronize()
        p = out.cpu().numpy()
        if precision == "fp64":
            err = np.linalg.norm(p - ref) / np.linalg.norm(ref)
            assert err <= max(1e-12, 4 * kappa * 2.0 ** -52), err
        else:
            res, _ = orc.residual(f, p, h, h, h, 1, bc_y=bc_y)
            assert st["status"] == 0 and res <= rtol, res
