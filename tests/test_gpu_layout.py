"""Grid orders and explicit row permutations against numpy (needs an MI355X)."""
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


# strides that divide the length, leave remainders below and above the phase, one, and half the length
@pytest.mark.parametrize("S", [64, 127, 1000, 2049])
def test_grid_order(ctx, S):
    from paper_2504_16083_amd import mmi
    print(f"[gpu] grid order S={S}", flush=True)
    strides = [s for s in (1, 2, 3, 7, 8, 31, 32, 50, 63, 64, 100, 250, 333, 500, 1000, 1024) if 2 * s <= S]
    g = torch.Generator().manual_seed(S)
    q = torch.randn(S, len(strides) * 2, 128, generator=g).to(torch.bfloat16).cuda()
    k = torch.randn(S, 2, 128, generator=g).to(torch.bfloat16).cuda()
    heads = [C.global_head(C.grid(s, s)) for s in strides] * 2
    plan = mmi.Plan(ctx, mmi.Problem(S, len(heads), 2, None), heads, q, k)
    for h in range(len(heads)):
        s, p = plan.export(h, "params")[:2]
        assert s == strides[h % len(strides)]
        c = np.arange(S)
        want = c[np.lexsort((c // s, (c - p - 1) % s))]
        got = plan.export(h, "qperm")
        assert np.array_equal(got[:S], want) and (got[S:] == -1).all(), (h, s, p)
    plan.destroy()


# one vector per row, powers of two up to the variant's limit and past it, other sizes; row counts around a
# workgroup's share; rows inside a wider buffer
@pytest.mark.parametrize("row,n", [(16, 1), (16, 1023), (256, 63), (256, 64), (256, 65), (256, 4097), (4096, 5),
                                   (8192, 3), (48, 700), (272, 129)])
def test_permute_rows(row, n):
    from paper_2504_16083_amd import mmi
    print(f"[gpu] permute row={row} n={n}", flush=True)
    rng = np.random.default_rng(n)
    src = torch.from_numpy(rng.integers(0, 256, (n + 7, row + 64), dtype=np.uint8)).cuda()
    perm = rng.permutation(n + 7)[:n].astype(np.int32)
    perm[rng.random(n) < 0.2] = -1
    pt = torch.from_numpy(perm).cuda()
    a = src[:, 16:16 + row]
    dst = torch.full((n + 2, row + 32), 9, dtype=torch.uint8, device="cuda")
    mmi.mmi_permute_rows(a, dst[:, :row], pt)
    want = np.full((n + 2, row + 32), 9, np.uint8)
    h = a.cpu().numpy()
    want[:n, :row] = np.where(perm[:, None] >= 0, h[np.maximum(perm, 0)], 0)
    assert np.array_equal(dst.cpu().numpy(), want)
    back = torch.full((n + 7, row + 64), 5, dtype=torch.uint8, device="cuda")
    mmi.mmi_unpermute_rows(dst[:, :row], back[:, 16:16 + row], pt)
    want = np.full((n + 7, row + 64), 5, np.uint8)
    want[perm[perm >= 0], 16:16 + row] = h[perm[perm >= 0]]
    assert np.array_equal(back.cpu().numpy(), want)
