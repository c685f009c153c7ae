"""Plan steps of more block partials than the merge reads directly: the fold in between, at
the first size that has one, at row counts around whole groups of 64 partials, and through
every launch that merges (plain, allocation-free, with the next bounds in either launch, a
serving batch).  Costs do not depend on the fold; U*, weights and statistics are checked in
float64 from the returned costs, U* to the parity bar of the repository's oracle tests."""
import numpy as np
import pytest

from synth import workload as W
from tests.gpu_helpers import U_ATOL

pytestmark = pytest.mark.gpu

# H = 64: 4 rollouts per partial, so 6145 rollouts are 1537 partials, the first folded ones
# (25 groups, the last of one row); 6400 and 6401 end a group of 64 and begin one.
CASES = [(6144, 64), (6145, 64), (6400, 64), (6401, 64), (12345, 40), (70001, 3)]


def _check(S, out, noise, U_bar, lam):
    S = S.astype(np.float64)
    e = np.exp(-(S - S.min()) / lam)
    w = e / e.sum()
    U = U_bar.astype(np.float64) + np.tensordot(w, noise.astype(np.float64), axes=1)
    # One float32 rounding of a cost moves its weight by |S| 2^-24 / lambda, relatively.
    rel = 1e-5 + 4 * np.abs(S).max() * 2.0 ** -24 / lam
    if "weights" in out:
        np.testing.assert_allclose(out["weights"], w, rtol=rel, atol=1e-9)
    np.testing.assert_allclose(out["stats"][:3], [S.min(), e.sum(), 1 / (w * w).sum()], rtol=rel)
    # The same change of every weight bounds the change of U*.
    tol = U_ATOL + rel * np.tensordot(w, np.abs(noise - U[None] + U_bar[None]), axes=1)
    assert np.all(np.abs(out["U"] - U) <= tol), float(np.abs(out["U"] - U).max())


@pytest.mark.parametrize("K,H", CASES)
def test_folded_steps(K, H):
    import torch

    from paper_2512_22575_amd import smpc as S
    inp = W.make_inputs(7, K=K, H=H, dt=0.02, n=32, voxel=0.05, n_boxes=4, n_spheres=4)
    dev = torch.device("cuda:0")
    grid = torch.from_numpy(inp.grid).to(dev)
    noise = torch.from_numpy(inp.noise).to(dev)
    U_in = torch.from_numpy(inp.U_bar).to(dev)
    planner = S.Planner(inp.robot, device=0)
    cells = S.smpc_grid_coarse_cells(32, 32, 32)
    stream = torch.cuda.current_stream(dev).cuda_stream
    table, other = torch.empty(cells, device=dev), torch.empty(cells, device=dev)
    assert S.smpc_grid_coarse_min(grid, S.GRID_F32, table.data_ptr(), stream) == S.SMPC_OK
    results = {}
    for how in ("plain", "noalloc", "bounds beside rollouts", "bounds beside merge"):
        if how == "noalloc" and S.smpc_plan_workspace_bytes(K, H) > 4 << 20:
            continue
        nxt = {"bounds beside rollouts": other, "bounds beside merge": table}.get(how)
        out = dict(U=torch.empty_like(U_in), costs=torch.empty(K, device=dev),
                   weights=torch.empty(K, device=dev), stats=torch.empty(4, device=dev))
        print(f"K={K} H={H} {how}", flush=True)
        planner.plan_step(q0=inp.q0, qd0=inp.qd0, T_goal=inp.T_goal, grid=grid, origin=inp.origin,
                          voxel=inp.voxel, noise=noise, U_in=U_in, U_out=out["U"], dt=inp.dt,
                          lam=inp.lam, weights=inp.weights, costs_out=out["costs"],
                          weights_out=out["weights"], stats_out=out["stats"], coarse=table,
                          noalloc=how == "noalloc",
                          next_bounds=None if nxt is None else (grid, S.GRID_F32, inp.origin,
                                                                inp.voxel, nxt))
        torch.cuda.synchronize()
        results[how] = {k: v.cpu().numpy() for k, v in out.items()}
    first = results["plain"]
    _check(first["costs"], first, inp.noise, inp.U_bar, inp.lam)
    for how, out in results.items():
        for k in first:
            np.testing.assert_array_equal(out[k].view(np.uint32), first[k].view(np.uint32),
                                          err_msg=f"{how}: {k}")
    planner.close()


def test_served_with_small_controllers():
    """A folded request served with unfolded ones gives what a plan step of its own gives."""
    import torch

    from paper_2512_22575_amd import smpc as S
    dev = torch.device("cuda:0")
    sizes = [(256, 16), (6401, 64), (1024, 32)]
    inps = [W.make_inputs(40 + i, K=K, H=H, dt=0.02, n=32, voxel=0.05, n_boxes=4, n_spheres=4,
                          robot_seed=40) for i, (K, H) in enumerate(sizes)]
    planner = S.Planner(inps[0].robot, device=0)
    srv = S.Server(planner, max_batch=8)
    sigma, ids, outs, refs = np.full(7, 0.5, np.float32), [], [], []
    for inp, (K, H) in zip(inps, sizes):
        g = torch.from_numpy(inp.grid).to(dev)
        U, costs = torch.empty((H, 7), device=dev), torch.empty(K, device=dev)
        # One batch of small controllers first, then one with the folded one among them.
        ids.append(srv.add_controller(g, inp.origin, inp.voxel, K, H, inp.dt, 1.0, inp.weights,
                                      sigma, U_star_out=U, costs_out=costs))
        outs.append((U, costs))
        ref_U, ref_c = torch.empty_like(U), torch.empty_like(costs)
        planner.plan_step(q0=inp.q0, qd0=inp.qd0, T_goal=inp.T_goal, grid=g, origin=inp.origin,
                          voxel=inp.voxel, noise=None, K=K, H=H, seed=5, sigma=sigma,
                          U_in=torch.zeros((H, 7), device=dev), U_out=ref_U, dt=inp.dt, lam=1.0,
                          weights=inp.weights, costs_out=ref_c)
        torch.cuda.synchronize()
        refs.append((ref_U, ref_c))
    for group in ([0, 2], [0, 1, 2]):
        for i in group:
            srv.submit(i, ids[i], inps[i].q0, inps[i].qd0, inps[i].T_goal, 5)
        left = len(group)
        print("serving", group, flush=True)
        while left:
            srv.pump()
            for c in srv.poll():
                assert c.status == S.SMPC_OK
                left -= 1
        if group == [0, 2]:
            continue
        assert torch.equal(outs[1][0], refs[1][0]) and torch.equal(outs[1][1], refs[1][1])
    srv.close()
    planner.close()
