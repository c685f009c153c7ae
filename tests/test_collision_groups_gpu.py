"""Self-collision groups and per-link bounds at the robots where their split changes: pairs
within a link, between neighbours and only far ones (the smaller kernel), single pairs,
links with fewer than four spheres or none, with and without coarse bounds."""
import dataclasses

import numpy as np
import pytest

from oracle import smpc_oracle as O
from synth import robot as R
from synth import workload as W
from tests.gpu_helpers import COST_ATOL, COST_RTOL

pytestmark = pytest.mark.gpu


def _robot(kind):
    full = R.make_robot(5, min_link_gap=0)          # every pair, also within a link
    if kind == "every pair":
        return full
    if kind == "neighbours":
        return R.make_robot(5, min_link_gap=1)
    if kind == "far":
        return R.make_robot(5)
    if kind == "one pair":
        far = R.make_robot(5)
        return dataclasses.replace(far, pairs=far.pairs[[17]])
    if kind == "some pairs":
        keep = np.random.default_rng(3).uniform(size=len(full.pairs)) < 0.2
        return dataclasses.replace(full, pairs=full.pairs[keep])
    # thinned: 0 to 4 spheres per link, the pairs among those that are left
    far = R.make_robot(5)
    left = [s for s in range(28) if (s % 4) < (4, 1, 0, 3, 2, 4, 1)[s // 4]]
    new = {s: i for i, s in enumerate(left)}
    pairs = [(new[a], new[b]) for a, b in far.pairs if a in new and b in new]
    return dataclasses.replace(far, sphere_link=far.sphere_link[left],
                               sphere_center=far.sphere_center[left],
                               sphere_radius=far.sphere_radius[left],
                               pairs=np.asarray(pairs, np.int32))


@pytest.mark.parametrize("bounds", [False, True])
@pytest.mark.parametrize("kind", ["every pair", "neighbours", "far", "one pair", "some pairs",
                                  "thinned"])
def test_costs_of_robots(kind, bounds):
    import torch

    from paper_2512_22575_amd import smpc as S
    rob = _robot(kind)
    inp = W.make_inputs(91, K=70, H=13, dt=0.05, n=32, voxel=0.05, n_boxes=6, n_spheres=4)
    dev = torch.device("cuda:0")
    grid = torch.from_numpy(inp.grid).to(dev)
    noise = torch.from_numpy(inp.noise).to(dev)
    U = torch.from_numpy(inp.U_bar).to(dev)
    costs = torch.full((70,), float("nan"), device=dev)
    out = torch.empty_like(U)
    planner = S.Planner(rob, device=0)
    stream = torch.cuda.current_stream(dev).cuda_stream
    coarse = None
    if bounds:
        coarse = torch.empty(S.smpc_grid_coarse_cells(32, 32, 32), device=dev)
        assert S.smpc_grid_coarse_min(grid, S.GRID_F32, coarse.data_ptr(), stream) == S.SMPC_OK
    print(f"robot: {kind}, bounds {bounds}", flush=True)
    planner.plan_step(q0=inp.q0, qd0=inp.qd0, T_goal=inp.T_goal, grid=grid, origin=inp.origin,
                      voxel=inp.voxel, noise=noise, U_in=U, U_out=out, dt=inp.dt, lam=inp.lam,
                      weights=inp.weights, costs_out=costs, coarse=coarse)
    torch.cuda.synchronize()
    ref = O.plan_step(rob.rounded_f32(), inp.q0, inp.qd0, inp.T_goal, inp.grid, inp.origin,
                      inp.voxel, inp.noise, inp.U_bar, inp.dt, inp.lam, inp.weights)
    err = np.abs(costs.cpu().numpy() - ref["S"])
    assert np.all(err <= COST_RTOL * np.abs(ref["S"]) + COST_ATOL), float(err.max())
    planner.close()
