"""How the gain's work items are dealt to the chip: whole nodes per XCD for every eight
nodes, the items of the last nb % 8 nodes over all XCDs; in small calls one workgroup per direction (N = 16 here up to 53
nodes, N = 24 up to 35).  At the edges of those rules every node's result is its result alone,
bit for bit, and the oracle's; so it is where the workspace has no room for the split.

Tolerances: relative L-inf over each (node, species) against the FP64 oracle, 1e-12 for
FP64 and 1e-5 for FP32 plans, as in the other parity tests."""
import numpy as np
import pytest

from oracle import spectral as OS
from synth import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,precision", [(16, "f64"), (24, "f32"), (32, "f32")])
@pytest.mark.parametrize("batch", [1, 7, 8, 9, 39, 45])
def test_every_node_at_the_edges_of_the_dealing(N, precision, batch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1903_03056_amd import CollisionPlan
    print(f"[case] gain items N={N} {precision} batch {batch}", flush=True)
    masses, L, M, nrho = (1.0, 2.0), 6.0, 6, 3
    plan = CollisionPlan(masses, N, L, M, nrho, omega=0.74, precision=precision)
    f = I.draw_bimaxwellian_batch(np.random.default_rng(61), batch, 2, N, L, masses, noise=1e-2)
    ft = torch.tensor(f, dtype=plan.dtype, device="cuda")
    Q = plan.collide(ft)
    for b in range(batch):
        assert torch.equal(plan.collide(ft[b:b + 1].contiguous())[0], Q[b]), b
    if batch == 7:
        # per node and alignment only, without what the split asks for beyond that
        per = (plan.workspace_bytes(2000) - plan.workspace_bytes(1000)) // 1000
        tight = torch.empty(per * batch + 1024, dtype=torch.uint8, device="cuda")
        assert tight.numel() <= plan.workspace_bytes(batch)
        assert torch.equal(plan.collide(ft, workspace=tight), Q)
    ref = OS.collide(ft[batch - 1].double().cpu().numpy(), OS.vhs_problem(masses, 0.74, L, N, M, nrho))
    got = Q[batch - 1].double().cpu().numpy()
    err = float(np.max(np.abs(got - ref).reshape(2, -1).max(1) / np.abs(ref).reshape(2, -1).max(1)))
    print(f"relative L-inf {err:.3e}", flush=True)
    assert err <= (1e-12 if precision == "f64" else 1e-5)


@pytest.mark.parametrize("N,precision,tile,s,M,nrho,batches", [
    (16, "f64", None, 2, 6, 3, (53, 54)), (24, "f32", (3, 1), 1, 12, 12, (17, 18)),
    (24, "f64", None, 1, 12, 12, (4, 5, 8, 9)), (32, "f64", None, 1, 12, 16, (3, 4, 5, 7)),
    (32, "f64", None, 2, 12, 16, (1, 2)), (32, "f32", (2, 1), 1, 24, 16, (5, 6, 9, 11)),
    (32, "f32", (4, 2), 2, 12, 16, (3,)), (16, "f32", (2, 1), 3, 12, 4, (5,)), (24, "f32", (3, 4), 2, 6, 4, (3,))])
def test_split_calls_equal_whole_ones(N, precision, tile, s, M, nrho, batches):
    """On both sides of the limits, with whole rounds of one workgroup per CU between them: with
    room for the split and without it, and a node in a batch and alone, bit for bit."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1903_03056_amd import CollisionPlan
    masses, L = (1.0, 2.0, 4.0)[:s], 6.0
    plan = CollisionPlan(masses, N, L, M, nrho, omega=0.74, precision=precision, tile=tile)
    f = I.draw_bimaxwellian_batch(np.random.default_rng(67), max(batches), s, N, L, masses, noise=1e-2)
    ft = torch.tensor(f, dtype=plan.dtype, device="cuda")
    for batch in batches:
        print(f"[case] split N={N} {precision} {tile} s={s} M={M} batch {batch}", flush=True)
        Q = plan.collide(ft[:batch])
        least = plan.workspace_bytes(batch) - plan.spread_bytes(batch)
        assert torch.equal(plan.collide(ft[:batch], workspace=torch.empty(least, dtype=torch.uint8, device="cuda")), Q)
        for b in (0, batch - 1):
            assert torch.equal(plan.collide(ft[b:b + 1].contiguous())[0], Q[b]), b


@pytest.mark.parametrize("N,precision,alpha,s,M", [
    (64, "f32", 1.0, 1, 6), (64, "f64", 1.0, 1, 6), (64, "f64", 1.0, 1, 12), (32, "f64", 1.0, 2, 6), (24, "f64", 1.0, 2, 6),
    (24, "f64", 1.0, 2, 12), (16, "f64", 1.4, 2, 6), (16, "f64", 1.4, 2, 12), (24, "f32", 1.4, 1, 12)])
def test_x_transforms_kept_or_not(N, precision, alpha, s, M):
    """Plans whose directions mostly share a sigma_x (M = 12) keep x-transforms in whole items,
    those with more fresh directions (M = 6) do not: both against the oracle."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import params as P
    from paper_1903_03056_amd import CollisionPlan, vss_kernel
    print(f"[case] kept x-transforms N={N} {precision} alpha={alpha} s={s} M={M}", flush=True)
    masses, L, nrho, omega = (1.0, 2.0)[:s], 6.0, 2, 0.74
    plan = CollisionPlan(masses, N, L, M, nrho, kernel=vss_kernel(masses, omega, alpha), precision=precision)
    f = I.draw_bimaxwellian_batch(np.random.default_rng(71), 2, s, N, L, masses, noise=1e-2)
    ft = torch.tensor(f, dtype=plan.dtype, device="cuda")
    least = plan.workspace_bytes(2) - plan.spread_bytes(2)    # no room to split
    Q = plan.collide(ft, workspace=torch.empty(least, dtype=torch.uint8, device="cuda"))
    assert torch.equal(plan.collide(ft), Q)
    C = [[(omega, alpha, P.vss_prefactor(mi, mj, omega, alpha)) for mj in masses] for mi in masses]
    ref = OS.collide(ft[1].double().cpu().numpy(), OS.Problem(masses=masses, L=L, N=N, M=M, nrho=nrho, kernel=C))
    got = Q[1].double().cpu().numpy()
    err = float(np.max(np.abs(got - ref).reshape(s, -1).max(1) / np.abs(ref).reshape(s, -1).max(1)))
    print(f"relative L-inf {err:.3e}", flush=True)
    assert err <= (1e-12 if precision == "f64" else 1e-5)


def test_whole_fp64_items_at_n32():
    """FP64 at N = 32 past the split (480 items): every node equals its result alone, which is
    split, bit for bit, and the oracle's."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1903_03056_amd import CollisionPlan
    masses, N, L, M, nrho, batch = (1.0, 2.0), 32, 6.0, 12, 8, 5
    print(f"[case] whole items N={N} f64 M={M} batch {batch}", flush=True)
    plan = CollisionPlan(masses, N, L, M, nrho, omega=0.74, precision="f64")
    f = I.draw_bimaxwellian_batch(np.random.default_rng(73), batch, 2, N, L, masses, noise=1e-2)
    ft = torch.tensor(f, device="cuda")
    Q = plan.collide(ft)
    for b in range(batch):
        assert torch.equal(plan.collide(ft[b:b + 1].contiguous())[0], Q[b]), b
    prob = OS.vhs_problem(masses, 0.74, L, N, M, nrho)
    for b in (0, batch - 1):
        ref = OS.collide(f[b], prob)
        err = float(np.max(np.abs(Q[b].cpu().numpy() - ref).reshape(2, -1).max(1) / np.abs(ref).reshape(2, -1).max(1)))
        print(f"relative L-inf {err:.3e}", flush=True)
        assert err <= 1e-12
