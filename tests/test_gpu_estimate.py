"""Estimation passes at the edges of their splits against float64 (needs an MI355X)."""
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


# key chunks of the LSE pass and tile runs of the score pass: one partial tile, whole chunks, one key past
# them, more chunks than the merge has waves, two batches of row sets per KV head
@pytest.mark.parametrize("S,Hq,Hkv", [(1, 1, 1), (64, 1, 1), (127, 2, 1), (128, 2, 1), (129, 5, 1), (2049, 2, 2),
                                      (4097, 9, 1), (20011, 3, 1)])
def test_estimate_edges(ctx, S, Hq, Hkv):
    from paper_2504_16083_amd import mmi
    print(f"[gpu] estimate S={S} heads {Hq}/{Hkv}", flush=True)
    g = torch.Generator().manual_seed(S)
    q = torch.randn(S, Hq, 128, generator=g).to(torch.bfloat16)
    k = torch.randn(S, Hkv, 128, generator=g).to(torch.bfloat16)
    heads = [C.global_head(C.vslash(1, 1))] * Hq
    plan = mmi.Plan(ctx, mmi.Problem(S, Hq, Hkv, None), heads, q.cuda(), k.cuda())
    n = min(64, S)
    rows = np.arange(S - n, S)
    for h in range(Hq):
        a = (q[S - n:, h].double() @ k[:, h // (Hq // Hkv)].double().t()).numpy() / np.sqrt(128.0)
        a[np.arange(S)[None] > rows[:, None]] = -np.inf
        m = a.max(1)
        lse = m + np.log(np.exp(a - m[:, None]).sum(1))
        p = np.exp(a - lse[:, None])
        u = np.zeros(S)
        for r, x in enumerate(rows):
            u[:x + 1] += p[r, :x + 1][::-1]
        # fp32 accumulation of 128 products: sum |q k| ~ 82, x 128^-0.5 x 128 x 2^-24 = 5.5e-5 on a logit, so
        # 1e-4 absolute on the LSE and twice that relative on sums of exponentials
        assert np.abs(plan.export(h, "est_lse") - lse).max() <= 1e-4
        for what, want in (("v", p.sum(0)), ("u", u)):
            assert np.abs(plan.export(h, what) - want).max() <= 2e-4 * want.max(), (h, what)
            assert np.abs(plan.export(h, what) / want - 1).max() <= 2e-4, (h, what)
    plan.destroy()
