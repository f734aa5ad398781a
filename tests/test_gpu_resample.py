"""The maps between species grids where their kernel splits its work differently: one thread
per pencil with many pencils, several with few, on the smallest and the largest grid.  Every
node equals its result alone bit for bit; one node against the oracle.

Tolerances: relative L-inf over each (node, species), 1e-12 for FP64 and 1e-5 for FP32 plans,
as in the other parity tests."""
import numpy as np
import pytest

from oracle import grids as G
from oracle import spectral as OS
from synth import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,precision,batch", [(16, "f64", 1), (16, "f32", 300), (24, "f64", 130), (64, "f32", 2)])
def test_maps_between_grids(N, precision, batch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1903_03056_amd import CollisionPlan
    print(f"[case] resample N={N} {precision} batch {batch}", flush=True)
    masses, Ls, M, nrho, omega = (1.0, 2.0), (6.0, 4.5), 6, 2, 0.74
    plan = CollisionPlan(masses, N, Ls, M, nrho, omega=omega, precision=precision)
    few = I.draw_bimaxwellian_batch(np.random.default_rng(91), min(batch, 3), 2, N, Ls, masses)
    ft = torch.tensor(few, dtype=plan.dtype, device="cuda")[torch.arange(batch) % len(few)].contiguous()
    Q = plan.collide(ft)
    for b in sorted({0, batch - 1}):
        assert torch.equal(plan.collide(ft[b:b + 1].contiguous())[0], Q[b]), b
    # without the memory that spreads a small call's directions
    per = (plan.workspace_bytes(4000) - plan.workspace_bytes(3000)) // 1000
    tight = torch.empty(per + 12 * 256, dtype=torch.uint8, device="cuda")
    assert torch.equal(plan.collide(ft[:1].contiguous(), workspace=tight)[0], Q[0])
    ref = G.collide(ft[0].double().cpu().numpy(), OS.vhs_problem(masses, omega, max(Ls), N, M, nrho), Ls).reshape(2, -1)
    got = Q[0].double().cpu().numpy().reshape(ref.shape)
    err = float(np.max(np.abs(got - ref).max(1) / np.abs(ref).max(1)))
    print(f"relative L-inf {err:.3e}", flush=True)
    assert err <= (1e-12 if precision == "f64" else 1e-5)
