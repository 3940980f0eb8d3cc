"""k_pair on the rows it took over from the chain pass: bf16 rows that do not
fill their last unit of 512 bytes or are over 2 KiB, fp32 rows, up to 4 KiB
each; every unit count, odd position counts, ranges of two frames and more,
padded strides, specials; and the other segments of a batch in the same launch
(up to 1,024 work items) or in one of their own. The bar of the parity tests
against the oracle (integers bit-exact, sums within 2e-3 for bf16 and 1e-5 for
fp32), and the chain pass (MSAO_PAIR=0) gives the same integers."""
import re

import numpy as np
import pytest
import torch

import paper_2604_02945_amd as msao
from paper_2604_02945_amd import binding as B
from test_gpu_parity import _rand_seg, dev, host, log, run_and_compare, to_device  # noqa: F401
from workloads import AUDIO, IMAGE, TEXT, VIDEO, default_params

pytestmark = pytest.mark.gpu


def clips(seed, shapes, dtype, kind="normal"):
    rng = np.random.default_rng(seed)
    return [_rand_seg(rng, i % 2, VIDEO, T, P, C, dtype, 0.3, kind) for i, (T, P, C) in enumerate(shapes)]


@pytest.mark.parametrize("C", [8, 248, 264, 504, 520, 1016, 1032, 1152, 1280, 1288, 1536, 1544, 1792, 1800, 2040, 2048, 2056])
def test_bf16_widths(C, dev):
    log(f"[pair wide] bf16 C={C}")
    run_and_compare(clips(C, [(2, 8, C), (3, 7, C), (5, 9, C), (9, 2, C), (17, 3, C)], "bf16"), 2, default_params(), dev)


@pytest.mark.parametrize("C", [4, 124, 128, 132, 256, 260, 384, 500, 640, 768, 772, 896, 900, 1020, 1024, 1028])
def test_f32_widths(C, dev):
    log(f"[pair wide] f32 C={C}")
    run_and_compare(clips(C, [(2, 8, C), (3, 7, C), (5, 9, C), (9, 2, C), (17, 3, C)], "f32"), 2, default_params(), dev)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kind", ["special", "same", "zero", "static_video"])
def test_kinds(kind, dtype, dev):
    log(f"[pair wide] {kind} {dtype}")
    segs = clips(3, [(35, 5, 1000), (4, 3, 1024), (66, 4, 72)], dtype, kind)
    run_and_compare(segs, 2, default_params(), dev)
    run_and_compare(segs, 2, default_params(), dev, pad=24)


@pytest.mark.parametrize("rows", [40, 4096, 4100, 9000])
def test_rest_in_the_launch(rows, dev):
    """Images of 2 KiB rows, four to a work item: 10, 1,024, 1,025 and 2,250
    items, beside an audio track and texts of none to a few."""
    rng = np.random.default_rng(rows)
    segs = [_rand_seg(rng, 0, VIDEO, 6, 5, 1160, "bf16", 0.3), _rand_seg(rng, 0, IMAGE, 1, rows, 1024, "bf16", 0.25, "relu_bg"),
            _rand_seg(rng, 1, VIDEO, 3, 4, 512, "bf16", 0.5)]
    if rows == 40:
        segs += [_rand_seg(rng, 1, AUDIO, 1, 30, 1280, "f32", -1.0), _rand_seg(rng, 1, TEXT, 1, 9, 4096, "bf16", 1.0)]
    log(f"[pair wide] rest {rows}")
    run_and_compare(segs, 2, default_params(), dev)
    run_and_compare(segs, 2, default_params(), dev, compact=False)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_chain_pass_gives_the_same_integers(dtype, dev, monkeypatch):
    segs = clips(9, [(32, 10, 1000), (17, 7, 72), (40, 2, 1024)], dtype, "static_video")
    outs = []
    for flag in ("0", "1"):
        monkeypatch.setenv("MSAO_PAIR", flag)
        ctx = B.Context(0)
        got, _, _ = run_and_compare(segs, 2, default_params(), dev, ctx=ctx)
        outs.append({k: host(v).copy() for k, v in got.items()})
        ctx.close()
    for k in ("z", "d", "kept_idx", "keep", "kept_count", "agg", "dframe"):
        assert np.array_equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("dtype,C", [("f32", 64), ("bf16", 72), ("bf16", 1032)])
@pytest.mark.parametrize("entry", ["msao_run", "msao_mas_score", "Plan"])
def test_workspace_with_room_for_the_chain_pass_only(entry, dtype, C, dev, monkeypatch):
    """k_pair's short ranges are more work items than the chain pass has (300
    against 150 here): a workspace that holds only the latter is still enough."""
    log(f"[pair wide] workspace {entry} {dtype} {C}")
    segs, p = clips(4, [(200, 6, C)], dtype), default_params()
    ds = to_device(segs, dev)
    ctxs = []
    for flag in ("0", "1"):
        monkeypatch.setenv("MSAO_PAIR", flag)
        ctxs.append(B.Context(0))
    chain, pair = ctxs

    def call(o, ctx):
        if entry == "Plan":
            plan = msao.Plan(ds, 1, o, p, ctx=ctx)
            plan()
            torch.cuda.synchronize()
            plan.close()
        else:
            B.prepare(entry, ds, 1, o, p, ctx=ctx)()
            torch.cuda.synchronize()
    o, want = msao.Outputs(ds, 1), msao.Outputs(ds, 1)
    o.ws_bytes = 256
    with pytest.raises(Exception, match="needed") as e:
        call(o, chain)
    o.ws_bytes = int(re.search(r"(\d+) needed", str(e.value)).group(1))
    call(o, pair)
    call(want, pair)
    names = ["z", "d", "agg", "dframe"] + ([] if entry == "msao_mas_score" else ["keep", "kept_idx", "kept_count"])
    got, ref = o.results(1, 1), want.results(1, 1)
    for k in names:
        a, b = host(got[k]), host(ref[k])
        if k == "kept_idx":
            a, b = a[:host(ref["kept_count"])[0]], b[:host(ref["kept_count"])[0]]
        assert np.array_equal(a, b), k
    for c in ctxs:
        c.close()


@pytest.mark.parametrize("dtype,C,T,P", [("f32", 8, 2, 2046), ("f32", 8, 2, 2050), ("f32", 8, 15, 4096), ("f32", 8, 16, 4096),
                                         ("f32", 8, 33, 2100), ("bf16", 1032, 2, 2050), ("bf16", 1032, 4, 2050),
                                         ("bf16", 1544, 4, 2050), ("bf16", 1032, 9, 2050)])
def test_clips_of_more_positions_than_simds_take_pairs_of(dtype, C, T, P, dev):
    """Both sides of the rule that leaves wide rows to the chain pass when there
    are more than 1,024 pairs of positions; beside them, a clip of narrow rows."""
    log(f"[pair wide] {T} x {P} x {C} {dtype}")
    run_and_compare(clips(T + P, [(T, P, C)], dtype) + clips(1, [(5, 9, 256)], "bf16"), 2, default_params(), dev)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows", [4096, 4100, 52000])
@pytest.mark.parametrize("narrow", [False, True])
def test_small_clips_beside_many_rows(narrow, rows, dtype, dev):
    """Small wide clips beside 1,024, 1,025 and 13,000 work items of rows (107 MB),
    alone and with a clip of narrow rows: in k_pair's launch or left to k_score's."""
    rng = np.random.default_rng(rows)
    C = 1160 if dtype == "bf16" else 72
    segs = clips(rows, [(6, 5, C), (9, 4, C)], dtype) + [_rand_seg(rng, 0, AUDIO, 1, rows, 1024, "bf16", 0.25, "relu_bg")]
    if narrow:
        segs += clips(2, [(5, 9, 256)], "bf16")
    log(f"[pair wide] {dtype} beside {rows} rows, narrow {narrow}")
    run_and_compare(segs, 2, default_params(), dev)
