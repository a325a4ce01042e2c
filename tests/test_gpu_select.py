"""Top-k selection against a stable sort of the exported scores (needs an MI355X)."""
import numpy as np
import pytest
import torch

from synth import config as C

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2504_16083_amd import mmi
    c = mmi.Ctx(0)
    yield c
    c.close()


# one score, a wave, the register variants' limits (8192 and 32768 scores) and the pass-per-launch
# variant past them; n from one element to all but one
@pytest.mark.parametrize("S", [1, 65, 8191, 8192, 8193, 32768, 32769, 70001])
def test_topk_edges(ctx, S):
    from paper_2504_16083_amd import mmi
    print(f"[gpu] topk S={S}", flush=True)
    g = torch.Generator().manual_seed(S)
    q = torch.randn(S, 4, 128, generator=g).to(torch.bfloat16).cuda()
    # keys of period 7 for the second KV head: long runs of equal scores
    k = torch.randn(S, 2, 128, generator=g)
    k[:, 1] = k[torch.arange(S) % 7, 1]
    k = k.to(torch.bfloat16).cuda()
    sizes = [(1, 1), (max(1, S - 1), min(S, 64)), (max(1, S // 3), max(1, S // 2)), (1000, S + 5)]
    heads = [C.global_head(C.vslash(a, b)) for a, b in sizes]
    plan = mmi.Plan(ctx, mmi.Problem(S, 4, 2, None), heads, q, k)
    for h, (nv, ns) in enumerate(sizes):
        for score, sel, n in (("v", "vsel", nv), ("u", "ssel", ns)):
            x, got = plan.export(h, score), plan.export(h, sel)
            want = np.sort(np.argsort(-x, kind="stable")[:min(n, S)])
            assert np.array_equal(got, want), (S, h, sel)
    plan.destroy()
