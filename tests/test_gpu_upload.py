"""Table upload of the entry points that build their tables per call: staging
slots used again while earlier uploads wait on the GPU, tables of one, several
and many copy units, runs of one segment longer than a fill stripe, calls on
two streams, and calls recorded into a HIP graph, whose replays come after
other calls with other tables. The same kernels run on the same inputs either
way, so every output equals the same call made alone, bit for bit (and one of
them the oracle's)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_02945_amd as msao
from paper_2604_02945_amd import binding as B
from test_gpu_parity import _rand_seg, to_device
from workloads import AUDIO, IMAGE, TEXT, VIDEO, default_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


def table(i):
    """Table i: one segment up to many, sizes different in every one."""
    rng = np.random.default_rng(50 + i)
    if i % 4 == 0:
        return [_rand_seg(rng, 0, IMAGE, 1, 60 + i, 64, "bf16", 0.5, "relu_bg")], 1
    if i % 4 == 1:  # one wavefront per 512 rows of 16 bytes; kept rows and frames of one segment over a fill stripe
        return [_rand_seg(rng, 0, AUDIO, 1, 70_000 + i, 8, "bf16", 0.6, "relu_bg"),
                _rand_seg(rng, 0, VIDEO, 9000, 2, 8, "bf16", 0.5, "relu_bg")], 1
    R = 40 if i % 4 == 2 else 3
    segs = []
    for r in range(R):
        segs.append(_rand_seg(rng, r, IMAGE, 1, 10 + (7 * r + i) % 50, 64, "bf16", -1.0, "relu_bg"))
        segs.append(_rand_seg(rng, r, VIDEO, 3 + i % 3, 5, 64, "f32", 0.4, "relu_bg"))
        segs.append(_rand_seg(rng, r, TEXT, 1, 1 + (r + i) % 4, 128, "bf16", 1.0, "relu_bg"))
    return segs, R


def snapshot(o, R, n, segs):
    r = {k: v.cpu().numpy().copy() for k, v in o.results(R, n).items()}
    for i, rows in enumerate(msao.compacted_rows(segs, o, r["kept_count"])):
        r[f"rows{i}"] = rows.contiguous().view(torch.uint8).cpu().numpy()
    return r


@pytest.mark.parametrize("entry", ["msao_run", "stages"])
def test_uploads_waiting_on_the_gpu(entry, dev):
    print(f"[upload] {entry}", flush=True)
    ctx = msao.Context(0)
    p = default_params()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    cases, want = [], []
    for i in range(12):
        segs, R = table(i)
        ds = to_device(segs, dev)
        o, alone = msao.Outputs(ds, R), msao.Outputs(ds, R)

        def calls(out):
            if entry == "msao_run":
                return [B.prepare("msao_run", ds, R, out, p, ctx=ctx)]
            return [B.prepare("msao_mas_score", ds, R, out, p, ctx=ctx),
                    B.prepare("msao_select_tokens", ds, R, out, p, ctx=ctx, mas=out.req["mas"]),
                    B.prepare("msao_compact", ds, R, out, ctx=ctx)]
        for c in calls(alone):
            c()
            torch.cuda.synchronize()
        want.append(snapshot(alone, R, len(ds), ds))
        cases.append((ds, R, o, calls(o), segs))
    torch.cuda.synchronize()
    # work in front of the uploads, so that they wait while the host goes on
    a = torch.randn(4096, 4096, device=dev)
    for s in streams:
        with torch.cuda.stream(s):
            for _ in range(20):
                a @ a
    for i, (ds, R, o, cs, _) in enumerate(cases):
        for c in cs:
            c(streams[i % 2])
    torch.cuda.synchronize()
    for i, (ds, R, o, cs, _) in enumerate(cases):
        got = snapshot(o, R, len(ds), ds)
        for k, v in want[i].items():
            assert np.array_equal(got[k].view(np.uint8), v.view(np.uint8)), f"call {i}: {k}"
    ds, R, o, _, segs = cases[3]
    ref = oracle.run(segs, R, p)
    assert np.array_equal(want[3]["kept_idx"], ref["kept_idx"]) and np.array_equal(want[3]["kept_count"], ref["k"])
    ctx.close()


@pytest.mark.parametrize("which", [0, 3])
def test_call_recorded_into_a_graph(which, dev):
    """Tables in the scoring launch's arguments (table 0), and in pieces."""
    print("[upload] graph", flush=True)
    ctx = msao.Context(0)
    segs, R = table(which)
    ds = to_device(segs, dev)
    o = msao.Outputs(ds, R, workspace=False)
    call = B.prepare("msao_run_noalloc", ds, R, o, default_params(), ctx=ctx)
    s = torch.cuda.Stream()
    call(s)
    torch.cuda.synchronize()
    want = snapshot(o, R, len(ds), ds)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(torch.cuda.current_stream())
    for rep in range(3):
        for group in (o.tok, o.frm, o.req, o.sel):
            for t in group.values():
                t.fill_(0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = snapshot(o, R, len(ds), ds)
        for k, v in want.items():
            assert np.array_equal(got[k].view(np.uint8), v.view(np.uint8)), f"replay {rep}: {k}"
    # later calls of the context go on as before
    for _ in range(6):
        call()
    torch.cuda.synchronize()
    got = snapshot(o, R, len(ds), ds)
    assert all(np.array_equal(got[k].view(np.uint8), v.view(np.uint8)) for k, v in want.items())
    ctx.close()


def prepared(i, entry, dev, ctx, p):
    """Table i (i % 4 of 2 or 3: more than 3 KiB of tables) with its calls, outputs and the outputs of the calls made alone."""
    segs, R = table(i)
    ds = to_device(segs, dev)
    o, alone = msao.Outputs(ds, R), msao.Outputs(ds, R)

    def calls(out):
        if entry == "stages":
            return [B.prepare("msao_mas_score", ds, R, out, p, ctx=ctx),
                    B.prepare("msao_select_tokens", ds, R, out, p, ctx=ctx, mas=out.req["mas"]),
                    B.prepare("msao_compact", ds, R, out, ctx=ctx)]
        return [B.prepare("msao_run", ds, R, out, p, ctx=ctx)]
    for c in calls(alone):
        c()
    torch.cuda.synchronize()
    return ds, R, o, calls(o), snapshot(alone, R, len(ds), ds)


def cleared(*outs):
    for o in outs:
        for group in (o.tok, o.frm, o.req, o.sel):
            for t in group.values():
                t.fill_(0)
        o.out.zero_()
        if o.workspace is not None:
            o.workspace.fill_(0)
    torch.cuda.synchronize()


@pytest.mark.parametrize("entry", ["msao_run", "stages"])
def test_many_calls_in_one_graph(entry, dev):
    """More calls with large tables in one graph than the context has staging
    slots (four), each with tables of its own, and replays after eager calls
    that use every slot."""
    print(f"[upload] many calls in a graph, {entry}", flush=True)
    ctx, p = msao.Context(0), default_params()
    inside = [prepared(i, entry, dev, ctx, p) for i in (2, 3, 6, 7, 10, 11, 14)]
    between = [prepared(i, "msao_run", dev, ctx, p) for i in (15, 18, 19, 22, 23)]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _, _, _, cs, _ in inside:
            for c in cs:
                c(torch.cuda.current_stream())
    for rep in range(3):
        cleared(*[x[2] for x in inside + between])
        for _, _, _, cs, _ in between:
            cs[0]()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for i, (ds, R, o, _, want) in enumerate(inside + between):
            got = snapshot(o, R, len(ds), ds)
            for k, v in want.items():
                assert np.array_equal(got[k].view(np.uint8), v.view(np.uint8)), f"replay {rep}, call {i}: {k}"
    ctx.close()


def test_noalloc_call_in_a_graph_after_other_calls(dev):
    """A recorded msao_run_noalloc is replayed after more calls with other
    large tables than there are staging slots."""
    print("[upload] noalloc in a graph", flush=True)
    ctx, p = msao.Context(0), default_params()
    segs, R = table(3)
    ds = to_device(segs, dev)
    o = msao.Outputs(ds, R, workspace=False)
    call = B.prepare("msao_run_noalloc", ds, R, o, p, ctx=ctx)
    call()
    torch.cuda.synchronize()
    want = snapshot(o, R, len(ds), ds)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(torch.cuda.current_stream())
    others = [prepared(i, "msao_run", dev, ctx, p) for i in (6, 7, 10, 11, 14, 15, 18, 19)]
    for rep in range(3):
        cleared(o)
        for _, _, _, cs, _ in others:
            cs[0]()
        g.replay()
        torch.cuda.synchronize()
        got = snapshot(o, R, len(ds), ds)
        for k, v in want.items():
            assert np.array_equal(got[k].view(np.uint8), v.view(np.uint8)), f"replay {rep}: {k}"
    ctx.close()


@pytest.mark.parametrize("kind", ["rows", "clips", "clips and many rows"])
@pytest.mark.parametrize("n", [1, 2, 6, 8, 9, 10, 11, 12, 13, 16])
def test_tables_with_the_scoring_launch(n, kind, dev):
    """Calls on both sides of the table size that travels with the scoring
    launch (about ten segments), against the same run from a plan's tables."""
    print(f"[upload] {n} segments, {kind}", flush=True)
    rng = np.random.default_rng(n)
    segs = []
    for i in range(n):
        if kind != "rows" and i % 2 == 0:
            segs.append(_rand_seg(rng, i % 3, VIDEO, 2 + i, 3 + i % 4, 64 * (1 + i % 3), "bf16" if i % 4 else "f32", 0.4))
        else:
            rows = 5000 if kind == "clips and many rows" and i == 1 else 20 + 9 * i
            segs.append(_rand_seg(rng, i % 3, IMAGE, 1, rows, 1024 if rows == 5000 else 72, "bf16", 1.0 if i % 5 == 3 else -1.0, "relu_bg"))
    ds, p, R = to_device(segs, dev), default_params(), 3
    ctx = msao.Context(0)
    o, q = msao.Outputs(ds, R), msao.Outputs(ds, R)
    plan = msao.Plan(ds, R, q, p, ctx=ctx)
    for out in (o, q):
        out.workspace.fill_(0xA5) if out is o else None
        out.out.zero_()
    plan()
    call = B.prepare("msao_run", ds, R, o, p, ctx=ctx)
    for _ in range(2):
        call()
    torch.cuda.synchronize()
    want, got = snapshot(q, R, n, ds), snapshot(o, R, n, ds)
    for k, v in want.items():
        assert np.array_equal(got[k].view(np.uint8), v.view(np.uint8)), k
    plan.close()
    ctx.close()
