"""Output differences and per-head block statistics against numpy (needs an MI355X)."""
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


# a row, a workgroup's rows and one past them, past an unrolled stretch; a head stride of its own
@pytest.mark.parametrize("S,H,n_class", [(1, 1, 1), (32, 2, 2), (33, 3, 8), (129, 2, 3), (5000, 3, 2)])
def test_sqerr(S, H, n_class):
    from paper_2504_16083_amd import mmi
    print(f"[gpu] sqerr S={S}", flush=True)
    g = torch.Generator().manual_seed(S)
    a, b = (torch.randn(S, H + 1, 128, generator=g).to(torch.bfloat16) for _ in range(2))
    cls = torch.randint(0, n_class + 1, (S,), generator=g).to(torch.uint8)   # class n_class: skipped rows
    a[cls == n_class] = float("inf")
    prob = mmi.Problem(S, H, H, None, strides={"o": ((H + 1) * 128, 128)})
    out = torch.full((H * n_class,), -1.0, device="cuda", dtype=torch.float64)
    mmi.mmi_output_sqerr(prob, a.cuda(), b.cuda(), cls.cuda(), n_class, out)
    d = (a.float() - b.float()).double().square().sum(2).numpy()
    want = np.array([[d[cls.numpy() == c, h].sum() for c in range(n_class)] for h in range(H)])
    # fp64 sums of n positive terms in another order: n 2^-53 relative
    assert np.abs(out.cpu().numpy().reshape(H, -1) - want).max() <= S * 128 * 2.0 ** -53 * max(want.max(), 1.0)


# the search sums 64 runs of rows per head: empty runs, one row a run, runs of 2 with a short last one, more rows a run
# than a workgroup reads at once, and past an unrolled stretch
@pytest.mark.parametrize("S", [5, 64, 127, 2049, 8300])
def test_search_errors(ctx, S):
    """The candidates' errors that the search reports, against fp64 sums over the outputs of the same plans."""
    from paper_2504_16083_amd import mmi
    print(f"[gpu] search errors S={S}", flush=True)
    g = torch.Generator().manual_seed(S)
    q, k, v = (torch.randn(S, h, 128, generator=g).to(torch.bfloat16).cuda() for h in (2, 1, 1))
    mod = (np.arange(S) * 5 // S % 2).astype(np.uint8)       # five stretches, two modalities
    prob = mmi.Problem(S, 2, 1, mod)
    cands = [C.ashape(2, 3), C.ashape(40, 200)]
    _, r = mmi.mmi_search(ctx, prob, q, k, v, cands, [C.none()], C.ashape(16, 64))

    def out(head):
        o = torch.empty_like(q)
        mmi.mmi_attention(ctx, prob, [head] * 2, q, k, v, o)
        return o.float().cpu()

    def check(got, d, rows):
        want = d[rows].sum()
        # fp64 sums of n positive terms in another order: n 2^-53 relative
        assert abs(got - want) <= S * 128 * 2.0 ** -53 * want, (got, want)

    inner, full = out(C.boundary2d_head({0: C.dense(), 1: C.dense()}, {})), out(C.global_head(C.dense()))
    for c, op in enumerate(cands):
        d1 = (out(C.boundary2d_head({0: op, 1: op}, {})) - inner).double().square().sum(2).numpy()
        d3 = (out(C.global_head(op)) - full).double().square().sum(2).numpy()
        for h in range(2):
            for i in range(2):
                check(r["step1_err"][h, c, i], d1[:, h], mod == i)
            check(r["step3g_err"][h, c], d3[:, h], slice(None))


def test_block_statistics(ctx):
    from paper_2504_16083_amd import mmi
    S = 2049 + 64 * 70                      # more than one run of query blocks per workgroup, a ragged tail
    rng = np.random.default_rng(0)
    mod = np.repeat(rng.integers(0, 3, S // 37 + 1), 37)[:S].astype(np.uint8)
    g = torch.Generator().manual_seed(1)
    q, k = (torch.randn(S, h, 128, generator=g).to(torch.bfloat16).cuda() for h in (4, 2))
    intra = {0: C.ashape(64, 128), 1: C.grid(30, 40), 2: C.vslash(20, 20)}
    heads = [C.global_head(C.grid(50, 60)), C.qboundary_head(intra),
             C.boundary2d_head(intra, {(0, 1): C.vert(30), (2, 0): C.dense()}), C.global_head(C.ashape(64, 256))]
    plan = mmi.Plan(ctx, mmi.Problem(S, 4, 2, mod), heads, q, k)
    for h in (2, 0, 1, 3):
        st = plan.stats(h)
        ptr, col = plan.export(h, "row_ptr"), plan.export(h, "col_idx")

        def mods(perm):
            x = perm.reshape(-1, 64)
            return [int(mod[r[r >= 0][0]]) for r in x]
        mq, mk = mods(plan.export(h, "qperm")), mods(plan.export(h, "kperm"))
        want = np.zeros((8, 8), np.int64)
        for i in range(len(mq)):
            for j in col[ptr[i]:ptr[i + 1]]:
                want[mq[i], mk[j]] += 1
        assert np.array_equal(np.array([list(r) for r in st.blocks_by_modality]), want), h
        for m in range(3 if h in (1, 2) else 1):
            if (h == 0) or (h in (1, 2) and m == 1):
                p = plan.export(h, "params", m)
                assert (st.sigma[m], st.phase[m]) == (p[0], p[1]), (h, m)
    plan.destroy()


def test_column_list_takes_no_device_memory(ctx):
    """Asking for the size of a column list, or for the list, leaves the plan's device memory as it was."""
    import ctypes as ct
    from paper_2504_16083_amd import mmi
    print("[gpu] column list", flush=True)
    S = 4097
    g = torch.Generator().manual_seed(2)
    q, k = (torch.randn(S, h, 128, generator=g).to(torch.bfloat16).cuda() for h in (4, 2))
    plan = mmi.Plan(ctx, mmi.Problem(S, 4, 2, None), [C.global_head(C.vslash(50, 50))] * 4, q, k)
    before = plan.timing()["device_bytes"]
    need = ct.c_size_t()
    assert mmi.lib().mmi_plan_export(plan.h, 1, 3, 0, None, 0, ct.byref(need)) == 0
    assert need.value == 4 * plan.stats(1).nnz_blocks
    assert plan.timing()["device_bytes"] == before
    small = np.full(3, -7, np.int32)       # too small: refused, nothing written
    assert mmi.lib().mmi_plan_export(plan.h, 1, 3, 0, small.ctypes.data_as(ct.c_void_p), 12, ct.byref(need)) == -1
    assert (small == -7).all()
    ptr, col = plan.export(1, "row_ptr"), plan.export(1, "col_idx")
    assert len(col) == ptr[-1] and all((np.diff(col[a:b]) > 0).all() for a, b in zip(ptr, ptr[1:]))
    assert plan.timing()["device_bytes"] == before
    plan.destroy()
