"""The attention launch's item queue: streams, capture, few and many items (needs an MI355X)."""
import pytest
import torch

from synth import config as C

pytestmark = pytest.mark.gpu


def _layer(S, Hq, Hkv, seed):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(S, h, 128, generator=g).to(torch.bfloat16).cuda() for h in (Hq, Hkv, Hkv)]


@pytest.fixture(scope="module")
def ctx():
    from paper_2504_16083_amd import mmi
    c = mmi.Ctx(0)
    yield c
    c.close()


def test_streams_share_a_plan(ctx):
    """One plan on more streams than it has queues, launches in flight together: every output bitwise the first."""
    from paper_2504_16083_amd import mmi
    print("[gpu] queue streams", flush=True)
    S = 5000
    q, k, v = _layer(S, 8, 2, 1)
    heads = [C.global_head(C.dense()), C.global_head(C.grid(40, 60)), C.global_head(C.ashape(64, 500)),
             C.global_head(C.vslash(100, 50))] * 2
    plan = mmi.Plan(ctx, mmi.Problem(S, 8, 2, None), heads, q, k)
    want = torch.empty_like(q)
    plan.execute(q, k, v, want)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(11)]
    outs = [torch.full_like(q, 7.0) for _ in range(33)]
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        plan.execute(q, k, v, o, None, streams[i % 11])
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        assert torch.equal(o, want), i
    plan.destroy()


@pytest.mark.parametrize("split", [True, False])
def test_streams_with_their_own_inputs(ctx, split):
    """Launches of one plan in flight on several streams, each on inputs of its own: every output bitwise that of the
    same call made alone. With split row groups they share the plan's partials."""
    from paper_2504_16083_amd import mmi
    print(f"[gpu] queue streams, own inputs, split={split}", flush=True)
    S, n = (5000, 6) if split else (3000, 6)
    mix = [C.global_head(C.dense()), C.global_head(C.ashape(64, 500)), C.global_head(C.ashape(64, 200)),
           C.global_head(C.ashape(64, 200))]
    heads = mix * 2 if split else [C.global_head(C.dense())] * 8
    ins = [_layer(S, 8, 2, 20 + i) for i in range(n)]
    plan = mmi.Plan(ctx, mmi.Problem(S, 8, 2, None), heads, *ins[0][:2])
    assert (sum(plan.stats(h).split_rows for h in range(8)) > 0) == split
    want = [(torch.empty_like(ins[0][0]), torch.empty(8, S, device="cuda")) for _ in ins]
    for x, (o, lse) in zip(ins, want):
        plan.execute(*x, o, lse)
        torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(n)]
    got = [(torch.full_like(ins[0][0], 7.0), torch.full((8, S), 7.0, device="cuda")) for _ in range(5 * n)]
    torch.cuda.synchronize()
    for i, (o, lse) in enumerate(got):
        plan.execute(*ins[i % n], o, lse, streams[(i + i // n) % n])
    torch.cuda.synchronize()
    for i, (o, lse) in enumerate(got):
        assert torch.equal(o, want[i % n][0]) and torch.equal(lse, want[i % n][1]), i
    plan.destroy()


@pytest.mark.parametrize("S", [300, 5000])
def test_created_on_one_stream_executed_on_others(ctx, S):
    """Nothing but the library orders the executes behind the creation's last launches (work list, item map, cleared
    counters); the buffers come from earlier plans, so what they hold before is another plan's. Statistics and exports
    likewise."""
    from paper_2504_16083_amd import mmi
    print(f"[gpu] queue creation S={S}", flush=True)
    heads = [C.global_head(C.dense()), C.global_head(C.grid(20, 30)), C.global_head(C.ashape(64, 500)),
             C.global_head(C.vslash(100, 50))] * 2
    q, k, v = _layer(S, 8, 2, 5)
    prob = mmi.Problem(S, 8, 2, None)
    want = torch.empty_like(q)
    mmi.mmi_attention(ctx, prob, heads, q, k, v, want)
    streams = [torch.cuda.Stream() for _ in range(4)]
    for i in range(6):
        other = mmi.Plan(ctx, mmi.Problem(S - i, 8, 2, None), heads[::-1], q, k)    # leaves its tables in the buffers
        other.destroy()
        outs = [torch.full_like(q, 7.0) for _ in streams]
        torch.cuda.synchronize()
        plan = mmi.Plan(ctx, prob, heads, q, k, streams[i % 4])
        for st, o in zip(streams, outs):
            plan.execute(q, k, v, o, None, st)
        nnz = [plan.stats(h).nnz_blocks for h in range(8)]
        assert nnz == [len(plan.export(h, "col_idx")) for h in range(8)]
        torch.cuda.synchronize()
        for j, o in enumerate(outs):
            assert torch.equal(o, want), (i, j)
        plan.destroy()


def test_destroyed_while_streams_still_execute(ctx):
    """Destroying a plan waits for its launches on every stream; the next plan takes over its buffers at once."""
    from paper_2504_16083_amd import mmi
    print("[gpu] queue destroy", flush=True)
    S = 3000
    q, k, v = _layer(S, 8, 2, 6)
    prob, dense = mmi.Problem(S, 8, 2, None), [C.global_head(C.dense())] * 8
    want, want2 = torch.empty_like(q), torch.empty_like(q)
    mmi.mmi_attention(ctx, prob, dense, q, k, v, want)
    mmi.mmi_attention(ctx, prob, [C.global_head(C.ashape(64, 300))] * 8, q, k, v, want2)
    streams = [torch.cuda.Stream() for _ in range(6)]
    for r in range(3):
        outs, o2, last = [torch.full_like(q, 7.0) for _ in range(24)], torch.full_like(q, 7.0), torch.empty_like(q)
        torch.cuda.synchronize()
        plan = mmi.Plan(ctx, prob, dense, q, k)
        for i, o in enumerate(outs):
            plan.execute(q, k, v, o, None, streams[i % 6])
        plan.execute(q, k, v, last, None, streams[r])
        plan.destroy()
        nxt = mmi.Plan(ctx, prob, [C.global_head(C.ashape(64, 300))] * 8, q, k)
        nxt.execute(q, k, v, o2)
        torch.cuda.synchronize()
        for i, o in enumerate(outs):
            assert torch.equal(o, want), (r, i)
        assert torch.equal(o2, want2), r
        nxt.destroy()


def test_short_lived_streams(ctx):
    """More streams than counter sets, each destroyed right after its launch (its handle may come back for the next
    stream): every output bitwise that of the same call made alone."""
    import ctypes
    from paper_2504_16083_amd import mmi
    print("[gpu] queue short-lived streams", flush=True)
    hip = ctypes.CDLL("libamdhip64.so")
    S, n = 3000, 5
    ins = [_layer(S, 8, 2, 40 + i) for i in range(n)]
    plan = mmi.Plan(ctx, mmi.Problem(S, 8, 2, None), [C.global_head(C.dense())] * 8, *ins[0][:2])
    want = [torch.empty_like(ins[0][0]) for _ in ins]
    for x, o in zip(ins, want):
        plan.execute(*x, o)
    got = [torch.full_like(want[0], 7.0) for _ in range(24)]
    torch.cuda.synchronize()
    for i, o in enumerate(got):
        st = ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(st)) == 0
        plan.execute(*ins[i % n], o, None, st.value)
        assert hip.hipStreamDestroy(st) == 0
    torch.cuda.synchronize()
    for i, o in enumerate(got):
        assert torch.equal(o, want[i % n]), i
    plan.execute(*ins[0], got[0])       # the default stream, after the last of them
    plan.destroy()


def test_graph_replay(ctx):
    """A captured execute replayed between eager ones on new inputs."""
    from paper_2504_16083_amd import mmi
    print("[gpu] queue capture", flush=True)
    S = 3000
    q, k, v = _layer(S, 4, 2, 2)
    plan = mmi.Plan(ctx, mmi.Problem(S, 4, 2, None), [C.global_head(C.ashape(64, 300))] * 4, q, k)
    o, e = torch.zeros_like(q), torch.zeros_like(q)
    plan.execute(q, k, v, e)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.execute(q, k, v, o)
    for i in range(3):
        v.copy_(_layer(S, 4, 2, 10 + i)[2])
        plan.execute(q, k, v, e)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, e), i
    plan.destroy()


def test_stage_times_after_a_captured_execute(ctx):
    """The stage times stay readable once an execute was captured, before and after its replay."""
    from paper_2504_16083_amd import mmi
    print("[gpu] queue capture, stage times", flush=True)
    q, k, v = _layer(3000, 4, 2, 7)
    plan = mmi.Plan(ctx, mmi.Problem(3000, 4, 2, None), [C.global_head(C.ashape(64, 300))] * 4, q, k)
    o = torch.empty_like(q)
    plan.execute(q, k, v, o)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        plan.execute(q, k, v, o)
    assert plan.timing()["attn_ms"] > 0
    g.replay()
    torch.cuda.synchronize()
    assert plan.timing()["attn_ms"] > 0
    plan.execute(q, k, v, o)
    t = plan.timing()
    assert t["attn_ms"] > 0 and t["combine_ms"] >= 0
    plan.destroy()


@pytest.mark.parametrize("S,Hq", [(1, 1), (64, 1), (257, 1), (300, 9), (2048, 40)])
def test_item_counts(ctx, S, Hq):
    """From one item to more than the CUs: rows all written, the plan's tables consistent."""
    from paper_2504_16083_amd import mmi
    print(f"[gpu] queue items S={S} Hq={Hq}", flush=True)
    q, k, v = _layer(S, Hq, 1, 3)
    plan = mmi.Plan(ctx, mmi.Problem(S, Hq, 1, None), [C.global_head(C.dense())] * Hq, q, k)
    plan.check()
    o = torch.full_like(q, float("nan"))
    for _ in range(2):
        plan.execute(q, k, v, o)
    torch.cuda.synchronize()
    plan.destroy()
    a = torch.einsum("qhd,kd->hqk", q.float().cpu(), k[:, 0].float().cpu()) / 128 ** 0.5
    a.masked_fill_(torch.ones(S, S).triu_(1).bool(), float("-inf"))
    want = torch.einsum("hqk,kd->qhd", a.softmax(-1), v[:, 0].float().cpu())
    # the output bound of the parity tests: 2e-2 plus half a bf16 spacing (|O| < 8 here: 2^-6)
    assert (o.float().cpu() - want).abs().max() <= 2e-2 + 2.0 ** -6
