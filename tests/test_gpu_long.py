"""Paths that only long sequences reach (needs an MI355X): items that start side by side, unions by four waves."""
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


def _layer(S, Hq, Hkv, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn(S, h, 128, generator=g, device="cuda").to(torch.bfloat16) for h in (Hq, Hkv, Hkv)]


def test_items_side_by_side(ctx):
    """Two dense heads of 256K tokens and a block: the items of every run wait for the run before. Bitwise the rows of
    the launch without waiting (a captured one), and the sampled rows against fp32 attention."""
    from paper_2504_16083_amd import mmi
    print("[gpu] long, side by side", flush=True)
    S = (1 << 18) + 33
    q, k, v = _layer(S, 2, 1, 1)
    plan = mmi.Plan(ctx, mmi.Problem(S, 2, 1, None), [C.global_head(C.dense())] * 2, q, k)
    o, e = torch.full_like(q, 7.0), torch.full_like(q, 7.0)
    for _ in range(2):
        o.fill_(7.0)
        plan.execute(q, k, v, o)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.execute(q, k, v, e)
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(o, e)
    plan.destroy()
    rows = torch.tensor([0, 63, 64, 255, 256, 4095, 100001, S // 2, S - 257, S - 256, S - 34, S - 33, S - 1], device="cuda")
    a = q[rows].float().transpose(0, 1) @ k[:, 0].float().t() / 128 ** 0.5
    a.masked_fill_(torch.arange(S, device="cuda")[None] > rows[:, None], float("-inf"))
    want = (a.softmax(-1) @ v[:, 0].float()).transpose(0, 1)
    # the output bound of the parity tests: 2e-2 plus half a bf16 spacing (|O| < 8 here: 2^-6)
    assert (o[rows].float() - want).abs().max() <= 2e-2 + 2.0 ** -6


@pytest.mark.parametrize("nblk", [10240, 10241])
def test_unions_of_long_bitmap_rows(ctx, nblk):
    """The longest bitmap row that one wave holds, and one block more: the plan's tables are consistent."""
    from paper_2504_16083_amd import mmi
    print(f"[gpu] long, {nblk} key blocks", flush=True)
    S = nblk * 64
    q, k, _ = _layer(S, 3, 1, 2)
    heads = [C.global_head(C.ashape(128, 500)), C.global_head(C.grid(250, 260)), C.global_head(C.vslash(60, 20))]
    plan = mmi.Plan(ctx, mmi.Problem(S, 3, 1, None), heads, q, k)
    assert plan.stats(0).n_kblocks == nblk
    plan.check()
    plan.destroy()
