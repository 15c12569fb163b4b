"""Plans around the sizes up to which the places of patches and groups travel with the filling launch (158, 113 and 52
groups of 4, 8 and 16 patches) and with one launch ahead of it (66 of 16): every head's work-list against the oracle's
mask, for the largest plan that fits and the smallest that does not."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves,side,tables", [(4, 13, 38), (4, 13, 39), (8, 13, 54), (8, 13, 55), (16, 16, 51), (16, 16, 52),
                                               (16, 1, 1), (4, 1, 153), (4, 1, 154), (4, 13, 40), (4, 1, 158), (4, 1, 159),
                                               (8, 13, 56), (8, 13, 57), (16, 16, 53), (16, 16, 66), (16, 16, 67)])
def test_places(waves, side, tables):
    import oracle
    import paper_2411_17178_amd as lv
    scales = (1, 3, 7, side)
    K = len(scales)
    # distinct tables (equal ones would share a work-list): the number of the table in the query scale's row
    rad = [[[-1] * K for _ in range(K)] for _ in range(tables)]
    for h in range(tables):
        rad[h][3] = [-1 + h % 2, h // 2 % 3, h // 6 % 6, h // 36]
    print(f"  waves={waves} side={side} tables={tables}", flush=True)
    plan = lv.litevar_mask_build(scales, 1, rad, 0, (3, 4), waves_per_group=waves)
    assert plan.n_head_groups == tables
    lv.litevar_plan_check(plan)
    total = 0
    for h in range(tables):
        mask, _ = lv.litevar_mask_export_dense(plan, head=h)
        mask = mask.cpu().numpy()
        if h in (0, 1, tables // 2, tables - 1):
            assert (mask == oracle.mask_dense(scales, rad[h], 0)[-side * side:]).all()
        assert int(mask.sum()) == int(plan.retained_pairs_of_group[plan.head_group[h]])
        total += int(mask.sum())
    header = plan.blob[:256].cpu().numpy().view(np.int64)
    assert total == int(plan.retained_pairs) == int(header[6]) and int(header[3]) == plan.n_steps


@pytest.mark.parametrize("tables", [3, 70])                    # places with the filling launch, and in two launches ahead of it
def test_builds_replay(tables):
    """A captured build and call: every replay lays the plan out anew over what the eager work between left in its buffer."""
    import paper_2411_17178_amd as lv
    scales, K = (2, 5, 16), 3
    rad = [[[h % 3, h // 3 % 5, h // 15]] * K for h in range(tables)]
    n = lv.litevar_mask_plan_bytes(scales, 1, rad, 0, (2, 3), waves_per_group=16)
    blob = torch.zeros(n, dtype=torch.uint8, device="cuda")
    q, k, v = (torch.randn((1, tables, m, 64), device="cuda", dtype=torch.bfloat16) for m in (256, 285, 285))
    out = torch.zeros_like(q)

    def work(stream=None):
        plan = lv.litevar_mask_build(scales, 1, rad, 0, (2, 3), waves_per_group=16, blob=blob, stream=stream)
        lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125, out=out, stream=stream)
        return plan
    plan = work()
    lv.litevar_plan_check(plan)
    eager, laid_out = out.clone(), blob.clone()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        plan = work(side)
    for rep in range(3):
        out.fill_(float(rep))
        blob.fill_(0xff)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        lv.litevar_plan_check(plan)
        assert torch.equal(out, eager)
        used = torch.zeros(n, dtype=torch.bool, device="cuda")
        for i in range(4, 11):                                 # the sections that a plan fills whole, but for their padding
            used[int(plan.off[i]):int(plan.off[i + 1]) // 256 * 256 - 255] = True
        assert int(used.sum()) > n // 2 and torch.equal(blob[used], laid_out[used])
