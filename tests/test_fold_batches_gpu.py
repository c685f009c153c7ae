"""Serving batches around a controller whose partials are folded: the batch before such a
controller exists, batches of unfolded requests after it (the batch graph then has a fold node
without blocks) and the folded request itself, alone and beside another, all give what a plan
step of their own gives, bit for bit."""
import numpy as np
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


def test_every_batch_equals_its_plan_steps():
    import torch

    from paper_2512_22575_amd import smpc as S
    dev = torch.device("cuda:0")
    # 64 horizon steps: 4 rollouts per partial, folded from 1537 partials on.
    sizes = [(256, 16), (6401, 64), (1024, 32), (300, 20), (6145, 64), (64, 64)]
    folded = {1, 4}
    inps = [W.make_inputs(60 + i, K=K, H=H, dt=0.02, n=32, voxel=0.05, n_boxes=4, n_spheres=4,
                          robot_seed=60) for i, (K, H) in enumerate(sizes)]
    planner = S.Planner(inps[0].robot, device=0)
    srv = S.Server(planner, max_batch=8)
    sigma = np.full(7, 0.5, np.float32)
    keep, ids, outs, refs = [], {}, {}, {}

    def add(i):
        inp, (K, H) = inps[i], sizes[i]
        g = torch.from_numpy(inp.grid).to(dev)
        keep.append(g)
        outs[i] = torch.empty((H, 7), device=dev), torch.empty(K, device=dev)
        ids[i] = srv.add_controller(g, inp.origin, inp.voxel, K, H, inp.dt, 1.0, inp.weights, sigma,
                                    U_star_out=outs[i][0], costs_out=outs[i][1])
        refs[i] = torch.empty((H, 7), device=dev), torch.empty(K, device=dev)
        planner.plan_step(q0=inp.q0, qd0=inp.qd0, T_goal=inp.T_goal, grid=g, origin=inp.origin,
                          voxel=inp.voxel, noise=None, K=K, H=H, seed=9 + i, sigma=sigma,
                          U_in=torch.zeros((H, 7), device=dev), U_out=refs[i][0], dt=inp.dt,
                          lam=1.0, weights=inp.weights, costs_out=refs[i][1])
        torch.cuda.synchronize()

    def serve(group):
        print("serving", group, flush=True)
        for i in group:
            srv.submit(i, ids[i], inps[i].q0, inps[i].qd0, inps[i].T_goal, 9 + i)
        left = len(group)
        while left:
            srv.pump()
            for c in srv.poll():
                assert c.status == S.SMPC_OK
                left -= 1
        for i in group:
            assert torch.equal(outs[i][0], refs[i][0]), f"U* of {i} (folded: {i in folded})"
            assert torch.equal(outs[i][1], refs[i][1]), f"costs of {i} (folded: {i in folded})"

    add(0)
    serve([0])
    for i in range(1, len(sizes)):
        add(i)
    for group in ([2], [1], [4, 3], [5]):
        serve(group)
    srv.close()
    planner.close()
