"""The radial sums where their work is shared differently: the VSS sum with one, two, three
or four nodes per thread (by the number of nodes), two or four output slots, one to four
chunks; the VHS sum with a ragged number of radial points over the threads that share an
element.  Every node equals its result alone bit for bit; one node against the oracle.

Tolerances: relative L-inf over each (node, species), 1e-12 for FP64 and 1e-5 for FP32 plans,
as in the other parity tests."""
import numpy as np
import pytest

from oracle import params as P
from oracle import spectral as OS
from synth import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,nrho,alpha,masses,precision,batch", [
    (16, 3, 1.4, (1.0, 2.0), "f32", 90), (16, 3, 1.4, (1.0, 2.0, 4.0), "f32", 230), (16, 3, 1.4, (1.0, 2.0), "f64", 45),
    (32, 2, 1.4, (1.0, 2.0), "f32", 23), (32, 2, 1.4, (1.0, 2.0), "f32", 183), (24, 2, 1.4, (1.0, 2.0), "f32", 3),
    (24, 1, 1.0, (1.0, 2.0), "f32", 2), (24, 5, 1.0, (1.0,), "f64", 3), (64, 9, 1.0, (1.0,), "f32", 2)])
def test_shared_radial_sums(N, nrho, alpha, masses, precision, batch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1903_03056_amd import CollisionPlan, vss_kernel
    print(f"[case] radial N={N} nrho={nrho} alpha={alpha} s={len(masses)} {precision} batch {batch}", flush=True)
    L, M, omega = 6.0, 6, 0.74
    plan = CollisionPlan(masses, N, L, M, nrho, kernel=vss_kernel(masses, omega, alpha), precision=precision)
    few = I.draw_bimaxwellian_batch(np.random.default_rng(81), 5, len(masses), N, L, masses, noise=1e-2)
    ft = torch.tensor(few, dtype=plan.dtype, device="cuda")[torch.arange(batch) % 5].contiguous()
    Q = plan.collide(ft)
    alone = plan.collide(ft[:1].contiguous())
    for b in sorted({0, 5, (batch - 1) // 5 * 5} & set(range(batch))):
        assert torch.equal(Q[b], alone[0]), b
    last = plan.collide(ft[batch - 1:].contiguous())
    assert torch.equal(Q[batch - 1], last[0])
    C = [[(omega, alpha, P.vss_prefactor(mi, mj, omega, alpha)) for mj in masses] for mi in masses]
    prob = OS.Problem(masses=masses, L=L, N=N, M=M, nrho=nrho, kernel=C)
    ref = OS.collide(ft[batch - 1].double().cpu().numpy(), prob).reshape(len(masses), -1)
    got = Q[batch - 1].double().cpu().numpy().reshape(ref.shape)
    err = float(np.max(np.abs(got - ref).max(1) / np.abs(ref).max(1)))
    print(f"relative L-inf {err:.3e}", flush=True)
    assert err <= (1e-12 if precision == "f64" else 1e-5)
