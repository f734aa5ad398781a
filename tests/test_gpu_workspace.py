"""What a workspace has to hold: the part of its size with which small calls spread over the
chip is optional in every entry point, and the rest grows with the batch, so that a workspace
of a larger batch serves every smaller one.  Results are the same bit for bit either way."""
import numpy as np
import pytest

from synth import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MASSES, L = (1.0, 2.0), 6.0


def _plan(N, M=12, nrho=4, precision="f32", masses=MASSES, L=L, **kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1903_03056_amd import CollisionPlan
    return CollisionPlan(masses, N, L, M, nrho, omega=0.74, precision=precision, **kw)


def _state(plan, batch, seed=41):
    f = I.draw_bimaxwellian_batch(np.random.default_rng(seed), batch, plan.s, plan.N, plan.L_species, plan.masses,
                                  noise=1e-2)
    return torch.tensor(f, dtype=plan.dtype, device="cuda")


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda")


def _per_node(plan):
    """Bytes per node of a large call, which has no optional part."""
    return (plan.workspace_bytes(20000) - plan.workspace_bytes(10000)) // 10000


def _group_bytes(plans, batches):
    """The bytes that a group's calls need, each plan's share a multiple of 256."""
    return sum((_per_node(p) * b + 1024 + 255) // 256 * 256 for p, b in zip(plans, batches))


@pytest.mark.parametrize("N,M,nrho,precision,masses,L", [
    (16, 12, 8, "f32", MASSES, 6.0), (24, 12, 12, "f32", (1.0, 2.0, 4.0), 6.0), (16, 6, 4, "f64", (1.0,), 6.0),
    (16, 12, 5, "f32", MASSES, (6.0, 4.0)), (32, 12, 16, "f32", MASSES, 6.0)])
def test_sizes_grow_with_the_batch(N, M, nrho, precision, masses, L):
    print(f"[case] workspace sizes N={N} M={M} {precision} s={len(masses)} L={L}", flush=True)
    plan = _plan(N, M, nrho, precision, masses, L)
    for size in (plan.workspace_bytes, plan.relax_workspace_bytes):
        sizes = [size(b) for b in range(1, 200)]
        assert sizes == sorted(sizes)
    assert plan.spread_bytes(10000) == 0
    # the rest: per node and alignment, and at least what the plain path needs for one node
    need = [plan.workspace_bytes(b) - plan.spread_bytes(b) for b in range(1, 200)]
    fixed = need[-1] - 199 * _per_node(plan)
    assert 0 < fixed <= 12 * 256
    assert need == [max(need[0], _per_node(plan) * b + fixed) for b in range(1, 200)]


def test_group_takes_a_workspace_without_the_optional_part():
    print("[case] group workspaces", flush=True)
    from paper_1903_03056_amd import CollisionGroup
    from paper_1903_03056_amd._lib import DgfsError
    plans = [_plan(24), _plan(16), _plan(16, nrho=3)]
    batches = (3, 5, 2)
    group = CollisionGroup(plans)
    fs = [_state(p, b) for p, b in zip(plans, batches)]
    want = [p.collide(f) for p, f in zip(plans, fs)]
    assert all(p.spread_bytes(b) > 0 for p, b in zip(plans, batches))
    need, full = _group_bytes(plans, batches), group.workspace_bytes(batches)
    # none of the optional part, a part of it, all of it, and the size for a larger batch
    for n in (need, need + plans[0].spread_bytes(3) + 256, full, _group_bytes(plans, (90, 90, 90))):
        print(f"[step] {n} bytes", flush=True)
        ws = _bytes(n)
        for q, w in zip(group.collide(fs, workspace=ws), want):
            assert torch.equal(q, w)
        graph, outs = group.capture(fs, workspace=ws)
        for _ in range(2):
            for q in outs:
                q.zero_()
            torch.cuda.synchronize()
            graph.launch()
            graph.stream.synchronize()
            assert all(torch.equal(q, w) for q, w in zip(outs, want))
    with pytest.raises(DgfsError):
        group.collide(fs, workspace=_bytes(need - 256))


@pytest.mark.parametrize("scheme", ["euler", "ssprk2"])
def test_slab_takes_a_workspace_without_the_optional_part(scheme):
    print(f"[case] slab workspaces {scheme}", flush=True)
    from paper_1903_03056_amd import Slab
    from paper_1903_03056_amd._lib import DgfsError
    plan = _plan(16)
    wall = [dict(kind="wall", u=(0.0, u, 0.0), T=1.0) for u in (-0.3, 0.3)]
    slab = Slab(plan, 0.0, 1.0, 4, 3, *wall)
    f = _state(plan, 12)
    full, spread = slab.workspace_bytes(scheme), plan.spread_bytes(12)
    assert spread > 0
    want = slab.step(f.clone(), 2e-4, 2, scheme=scheme)
    assert torch.equal(slab.step(f.clone(), 2e-4, 2, scheme=scheme, workspace=_bytes(full - spread)), want)
    with pytest.raises(DgfsError):
        slab.step(f.clone(), 2e-4, 1, scheme=scheme, workspace=_bytes(full - spread - 256))
    # a slab without collisions has no optional part
    free = Slab(plan, 0.0, 1.0, 4, 3, *wall, collide=False)
    free.step(f.clone(), 2e-4, 1, scheme=scheme, workspace=_bytes(free.workspace_bytes(scheme)))


@pytest.mark.parametrize("N,M,nrho,precision,masses,batch,tile", [
    (32, 24, 16, "f64", (1.0,), 3, None),          # 302 MB of terms: two groups of radial points
    (24, 24, 12, "f32", (1.0,), 17, None),         # 271 MB: two groups
    (32, 24, 1, "f32", (1.0,), 85, (4, 2)),        # 267 MB for the one point: the most that fit
    (32, 24, 1, "f32", (1.0,), 86, (4, 2))])       # one node more: no split
def test_the_optional_part_is_bounded(N, M, nrho, precision, masses, batch, tile):
    print(f"[case] spread bytes N={N} M={M} nrho={nrho} {precision} batch {batch}", flush=True)
    plan = _plan(N, M, nrho, precision, masses, tile=tile)
    assert max(plan.spread_bytes(b) for b in range(1, 400)) <= 256 << 20
    assert plan.spread_bytes(1) > 0
    f = _state(plan, min(batch, 3))[torch.arange(batch) % 3].contiguous()
    need = plan.workspace_bytes(batch) - plan.spread_bytes(batch)
    Q = plan.collide(f, workspace=_bytes(need + (256 << 20)))
    assert torch.equal(plan.collide(f, workspace=_bytes(need)), Q)
    assert torch.isfinite(Q).all() and float(Q.abs().max()) > 0


@pytest.mark.parametrize("case", ["vhs", "grids", "vss", "dealiased", "matrix", "pairs", "relax"])
@pytest.mark.parametrize("nodes", [1, 3])
def test_slices_give_the_same_results(case, nodes):
    """A workspace of `nodes` nodes without the optional part makes a batch of 7 run in slices
    (the last one ragged for 3 nodes); one with it runs some slices split and others not."""
    from paper_1903_03056_amd import vss_kernel
    print(f"[case] slices {case} of {nodes}", flush=True)
    if case == "grids":
        plan = _plan(16, nrho=4, masses=(1.0, 20.0), L=(6.0, 2.0))
    elif case == "vss":
        plan = _plan(16, nrho=4, kernel=vss_kernel(MASSES, 0.74, 1.4))
    elif case == "matrix":
        plan = _plan(32, nrho=3)
    else:
        plan = _plan(16, nrho=4, dealias=case == "dealiased")
    f = _state(plan, 7)
    if case == "relax":
        one = plan.relax_workspace_bytes(nodes) - plan.spread_bytes(nodes)
        # the stage states of the whole batch, and the collide workspace of `nodes` nodes
        states = 2 * ((7 - nodes) * plan.s * plan.N ** 3 * 4)
        want = plan.relax(f.clone(), 0.01, 2)
        run = lambda n: plan.relax(f.clone(), 0.01, 2, workspace=_bytes(states + n))
        per = (plan.relax_workspace_bytes(20000) - plan.relax_workspace_bytes(10000)) // 10000 \
            - 2 * plan.s * plan.N ** 3 * 4
    else:
        pairs = case == "pairs"
        # the size counts the pair-resolved form's slots; a pass without them takes less
        need = plan.workspace_bytes(nodes) - plan.spread_bytes(nodes)
        per = _per_node(plan)
        per_sum = (plan.relax_workspace_bytes(20000) - plan.relax_workspace_bytes(10000)) // 10000 \
            - 2 * plan.s * plan.N ** 3 * 4
        slack = plan.workspace_bytes(20000) - 20000 * per
        one = need if pairs else per_sum * nodes + slack
        per = per if pairs else per_sum
        want = plan.collide(f, pairs=pairs)
        run = lambda n: plan.collide(f, pairs=pairs, workspace=_bytes(n))
    assert one < per * (nodes + 1)          # at most `nodes` nodes in a pass
    assert torch.equal(run(one), want)
    # room for the split's terms of fewer nodes than a slice has, and a little more
    for extra in (plan.spread_bytes(1), per // 2, per + plan.spread_bytes(nodes) // 2):
        assert torch.equal(run(one + extra), want)
