"""GPU parity of the draft-confidence kernel (Sec. 4.2, Eq. 9-10) against the
oracle, through the C ABI (msao_draft_entropy).

Tolerance on the entropy, derived from the kernel's arithmetic: each lane sums
at most ceil(V / 2048) * 8 terms of exp(x - m) in float32 and the block merges
256 partial sums, so s and t carry a relative rounding error of at most
gamma ~ (V / 256 + 8) * 2^-24 (3.6e-5 at V = 151,936), and v_exp_f32 adds
about 2^-22 per term. H = ln s - t / s with |t / s| <= ln V then errs by at
most gamma * (1 + 2 ln V) + 2^-21 (1 + ln V), under 1e-3 nats for V <= 2^18.
The arg max is exact (both sides compare the same float values, first index
among equal maxima). The speculation flag is checked against the kernel's own
normalised entropy, and against the oracle's wherever the oracle's value lies
more than the tolerance away from the threshold.
"""
import math
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2604_02945_amd as msao
from paper_2604_02945_amd import binding as B
from workloads import DRAFT_ROWS, DRAFT_VOCAB, draft_logits, f32_to_bf16_bits

pytestmark = pytest.mark.gpu

H_TOL = 1e-3  # nats


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


def log(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def to_dev(x, dtype, dev):
    if dtype == "f32":
        return torch.from_numpy(np.ascontiguousarray(x)).to(dev)
    return torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).to(dev).view(torch.bfloat16)


def check(x, dtype, vocab, dev, theta=0.3, rows_to_check=None):
    """Run the kernel on host array x ([rows, stride]) and compare with the oracle."""
    t = to_dev(x, dtype, dev)
    out = msao.msao_draft_entropy(t, theta, vocab=vocab)
    torch.cuda.synchronize()
    H = out["entropy"].cpu().numpy().astype(np.float64)
    Hn = out["entropy_norm"].cpu().numpy().astype(np.float64)
    am = out["draft_token"].cpu().numpy()
    sp = out["speculate"].cpu().numpy()
    rows = np.arange(x.shape[0]) if rows_to_check is None else np.asarray(rows_to_check)
    Hr, amr = oracle.entropy_rows(x[rows], dtype, vocab)
    lnV = math.log(vocab)
    nan_r = np.isnan(Hr)
    assert np.array_equal(np.isnan(H[rows]), nan_r), "NaN rows"
    ok = ~nan_r
    err = np.abs(H[rows][ok] - Hr[ok])
    assert err.size == 0 or err.max() <= H_TOL, f"entropy error {err.max()}"
    assert np.all(np.abs(Hn[rows][ok] - Hr[ok] / lnV) <= H_TOL / lnV + 1e-7), "normalised entropy"
    assert np.array_equal(am[rows], amr), "draft token"
    assert np.array_equal(sp, (Hn <= np.float32(theta)).astype(np.uint8)), "speculate vs own entropy"
    far = ok & (np.abs(Hr / lnV - theta) > H_TOL / lnV + 1e-6)
    assert np.array_equal(sp[rows][far], (Hr[far] / lnV <= theta).astype(np.uint8)), "speculate vs oracle"
    return H, Hn, am, sp, (err.max() if err.size else 0.0)


@pytest.mark.parametrize("rows,vocab,stride,dtype", [
    (3, 2, 8, "bf16"), (7, 8, 8, "bf16"), (5, 1000, 1008, "bf16"), (5, 1001, 1008, "bf16"),
    (4, 1007, 1008, "f32"), (9, 2051, 2052, "f32"), (300, 4096, 4096, "f32"), (33, 65536, 65536, "bf16"),
    (2, DRAFT_VOCAB + 5, DRAFT_VOCAB + 8, "bf16"), (64, DRAFT_VOCAB, DRAFT_VOCAB, "bf16"),
    (16, DRAFT_VOCAB, DRAFT_VOCAB, "f32"),
])
def test_entropy_matches_oracle(rows, vocab, stride, dtype, dev):
    log(f"[entropy] rows={rows} vocab={vocab} stride={stride} {dtype}")
    x = draft_logits(rows, vocab, seed=rows + vocab, dtype=dtype, row_stride=stride)
    *_, err = check(x, dtype, vocab, dev)
    log(f"[entropy] max |dH| = {err:.2e}")


def test_entropy_special_rows(dev):
    V = 4096
    rng = np.random.default_rng(3)
    x = rng.standard_normal((10, V)).astype(np.float32)
    x[0] = 1.5                                   # equal logits: H = ln V, first index
    x[1, ::3] = -np.inf                          # a third of the vocabulary masked
    x[2, :] = -np.inf
    x[2, 77] = 0.0                               # one finite logit: H = 0
    x[3, 5] = np.nan                             # NaN -> NaN
    x[4, 9] = np.inf                             # +inf -> NaN
    x[5, :] = -np.inf                            # nothing finite -> NaN
    x[6, [10, 300, 4000]] = 50.0                 # three equal maxima: the first
    x[7, 2222] = 300.0                           # one dominant logit
    x[8] *= 40.0                                 # very peaked softmax
    x[9, -1] = 60.0                              # maximum in the last chunk
    for dtype in ("f32", "bf16"):
        xx = x if dtype == "f32" else f32_to_bf16_bits(x)
        H, Hn, am, sp, _ = check(xx, dtype, V, dev)
        assert H[0] == pytest.approx(math.log(V), abs=H_TOL) and am[0] == 0
        assert abs(H[2]) <= H_TOL and am[2] == 77
        assert am[6] == 10 and am[7] == 2222 and am[9] == V - 1
        assert np.isnan(H[3]) and np.isnan(H[4]) and np.isnan(H[5])


def test_entropy_outputs_are_optional_and_zero_rows(dev):
    x = draft_logits(4, 1024, seed=5, dtype="bf16")
    t = to_dev(x, "bf16", dev)
    tok = torch.full((4,), -7, dtype=torch.int32, device=dev)
    msao.msao_draft_entropy(t, 0.5, outputs={"draft_token": tok})
    torch.cuda.synchronize()
    assert np.array_equal(tok.cpu().numpy(), oracle.entropy_rows(x, "bf16")[1])
    empty = torch.empty((0, 1024), dtype=torch.bfloat16, device=dev)
    o = msao.msao_draft_entropy(empty, 0.5)
    torch.cuda.synchronize()
    assert o["entropy"].numel() == 0


def test_entropy_rejects_bad_arguments(dev):
    ctx = B.Context(0)
    L = B.lib()
    x = torch.zeros((4, 1024), dtype=torch.bfloat16, device=dev)
    H = torch.empty(4, device=dev)
    out = B.MsaoEntropyOut(B._ptr(H), None, None, None)
    args = lambda ptr=x.data_ptr(), rows=4, V=1024, stride=1024, dt=B.BF16, th=0.5: L.msao_draft_entropy(
        ctx.handle, B.ctypes.c_void_p(ptr), rows, V, stride, dt, th, B._addr(out), None)
    assert args() == 0
    torch.cuda.synchronize()
    assert args(V=1) == 1 and args(V=2000) == 1 and args(rows=-1) == 1 and args(dt=7) == 1
    assert args(th=float("nan")) == 1
    assert args(ptr=x.data_ptr() + 2) == 2 and args(stride=1025, V=1000) == 2
    ctx.close()


def test_entropy_full_size_sampled(dev):
    """The benchmark's shape (1,280 rows x 151,936 bf16, 389 MB) in one launch;
    every 20th row against the oracle, the rest by range checks."""
    log("[entropy] full size 1280 x 151936 bf16")
    x = draft_logits(DRAFT_ROWS, DRAFT_VOCAB, seed=0, dtype="bf16")
    H, Hn, am, sp, err = check(x, "bf16", DRAFT_VOCAB, dev, theta=0.5, rows_to_check=np.arange(0, DRAFT_ROWS, 20))
    assert np.all((Hn >= -1e-6) & (Hn <= 1 + 1e-6)) and np.all((am >= 0) & (am < DRAFT_VOCAB))
    log(f"[entropy] full size: max |dH| on sampled rows {err:.2e}; speculating {int(sp.sum())} of {DRAFT_ROWS}")


def test_entropy_feeds_algorithm_1(dev):
    """The kernel's normalised entropies drive the host scheduler exactly as
    the oracle's Algorithm 1 would on the same values."""
    x = draft_logits(400, 8192, seed=9, dtype="bf16")
    out = msao.msao_draft_entropy(to_dev(x, "bf16", dev), 0.5)
    torch.cuda.synchronize()
    hn = out["entropy_norm"].cpu().numpy()
    s = msao.Scheduler(hn[:200])
    theta0, nd = s.state.theta, s.state.n_draft
    dec, th = s.run(hn[200:])
    p = s.params
    odec, oth, _ = oracle.sched_run(hn[200:].astype(np.float64), theta0, nd, p.delta, p.theta_min, p.alpha)
    assert np.array_equal(dec, odec) and np.array_equal(th, oth)


def same_bits(got, want):
    for k in ("entropy", "entropy_norm", "draft_token", "speculate"):
        a, b = got[k].cpu().numpy(), want[k].cpu().numpy()
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), (k, a, b)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,batches,extra", [
    (1, 1, 1), (1, 12, -1), (2, 12, 0), (1, 16, -1), (1, 16, 0), (1, 16, 1), (2, 31, -3), (1, 64, 5), (3, 64, 64), (1, 130, 7), (15, 17, 3),
    (16, 16, 7), (17, 16, 1)])
def test_rows_split_over_workgroups(rows, batches, extra, dtype, dev):
    """Vocabularies around whole batches of a workgroup's loads (4,096 float32
    or 8,192 bf16 logits), from too few to be split
    to many, for one row up to past the most rows that are split."""
    vocab = batches * (4096 if dtype == "f32" else 8192) + extra
    log(f"[entropy split] {rows} x {vocab} {dtype}")
    stride = -(-vocab // 8) * 8
    x = draft_logits(min(rows, 20), stride, seed=rows + batches, dtype=dtype)
    x = np.tile(x, (-(-rows // len(x)), 1))[:rows]
    check(x, dtype, vocab, dev, rows_to_check=np.unique([0, rows // 2, rows - 1, min(rows - 1, 19)]))


def test_split_rows_special_values(dev):
    """A row of -inf, one finite logit in every part of a row in turn, equal
    maxima in several parts (the first counts) and NaN in the last part."""
    V = 20 * 4096 + 3  # 4 parts for each of 16 rows
    log("[entropy split] special")
    x = np.full((16, V + 1), -np.inf, np.float32)
    for r in range(1, 8):
        x[r, min(V - 1, (r - 1) * 16384 + 17)] = 2.0
    x[8, [5000, 45000, V - 1]] = 1.0
    x[9:] = 0.0
    x[10, V - 1] = np.nan
    x[11, [4096, 30000, 70000]] = 3.0
    t = torch.from_numpy(x).to(dev)
    out = msao.msao_draft_entropy(t, 0.3, vocab=V)
    torch.cuda.synchronize()
    tok, H = out["draft_token"].cpu().numpy(), out["entropy"].cpu().numpy()
    # each row alone beside 256 others takes the path of one workgroup per row
    whole = msao.msao_draft_entropy(t.repeat(17, 1), 0.3, vocab=V)
    torch.cuda.synchronize()
    assert np.array_equal(tok, whole["draft_token"].cpu().numpy()[:16])
    np.testing.assert_allclose(H, whole["entropy"].cpu().numpy()[:16], rtol=0, atol=H_TOL)
    assert tok[8] == 5000 and tok[11] == 4096 and np.isnan(H[10])


def test_split_rows_in_flight_and_in_a_graph(dev):
    """More split calls in flight than a context has slots, on two streams; then
    one recorded into a graph; every result is the same call's made alone, bit
    for bit."""
    log("[entropy split] in flight")
    ctx = B.Context(0)
    xs = [torch.from_numpy(draft_logits(1 + i % 3, 151936, seed=i, dtype="f32")).to(dev) for i in range(12)]

    def buffers(rows):
        return {"entropy": torch.zeros(rows, device=dev), "entropy_norm": torch.zeros(rows, device=dev),
                "draft_token": torch.zeros(rows, dtype=torch.int32, device=dev),
                "speculate": torch.zeros(rows, dtype=torch.uint8, device=dev)}
    want, got = [], [buffers(len(x)) for x in xs]
    for x in xs:
        want.append(msao.msao_draft_entropy(x, 0.3, ctx=ctx))
        torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    a = torch.randn(4096, 4096, device=dev)
    torch.cuda.synchronize()
    for s in streams:
        with torch.cuda.stream(s):
            for _ in range(10):
                a @ a
    for i, x in enumerate(xs):
        msao.msao_draft_entropy(x, 0.3, ctx=ctx, stream=streams[i % 2], outputs=got[i])
    torch.cuda.synchronize()

    for g, w in zip(got, want):
        same_bits(g, w)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        msao.msao_draft_entropy(xs[0], 0.3, ctx=ctx, outputs=got[0])
    for _ in range(3):
        got[0]["entropy"].zero_()
        graph.replay()
        msao.msao_draft_entropy(xs[1], 0.3, ctx=ctx, outputs=got[1])
        torch.cuda.synchronize()
        same_bits(got[0], want[0])
        same_bits(got[1], want[1])
    ctx.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,batches,extra", [(1, 16, 0), (1, 16, 1), (1, 64, 5), (2, 31, -3), (3, 40, 64), (7, 17, 3), (16, 16, 7),
                                                (16, 38, -1), (17, 16, 1), (1, 11, 0)])
def test_results_do_not_depend_on_slots(rows, batches, extra, dtype, dev):
    """The same rows split over workgroups and, recorded into a graph, by one
    workgroup each: every output has the same bits, NaN and infinities included."""
    vocab = batches * (4096 if dtype == "f32" else 8192) + extra
    log(f"[entropy slots] {rows} x {vocab} {dtype}")
    ctx = B.Context(0)
    x = draft_logits(rows, -(-vocab // 8) * 8, seed=rows + batches, dtype=dtype)
    t = to_dev(x, dtype, dev)
    if rows >= 3:
        t[1, vocab // 3:] = -float("inf")
        t[2, vocab - 2] = float("nan")
    theta = float(msao.msao_draft_entropy(t, 0.3, vocab=vocab, ctx=ctx)["entropy_norm"][0])
    want = msao.msao_draft_entropy(t, theta, vocab=vocab, ctx=ctx)
    got = {k: torch.zeros_like(v) for k, v in want.items()}
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        msao.msao_draft_entropy(t, theta, vocab=vocab, ctx=ctx, outputs=got)
    for _ in range(3):
        for v in got.values():
            v.zero_()
        graph.replay()
        torch.cuda.synchronize()
        same_bits(got, want)
    assert int(want["speculate"][0]) == 1  # theta is row 0's own value
    ctx.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,vocab", [(6, 151936), (40, 151936), (6, 5003)])
def test_rows_masked_with_the_lowest_value(rows, vocab, dtype, dev):
    """Tokens that a decoder rules out carry the type's lowest value: the tail of
    the vocabulary, its head, and all but a few tokens, one of them the last."""
    log(f"[entropy masks] {rows} x {vocab} {dtype}")
    stride = -(-vocab // 8) * 8
    x = draft_logits(rows, stride, seed=rows, dtype="f32")
    low = float(torch.finfo(torch.float32 if dtype == "f32" else torch.bfloat16).min)
    x[0, 2 * vocab // 3:] = low
    x[1, :2 * vocab // 3] = low
    for r, kept in ((2, [vocab // 2]), (3, [7, vocab // 5, vocab - 1]), (4, range(vocab // 3, vocab // 3 + 300))):
        v = x[r, list(kept)].copy()
        x[r] = low
        x[r, list(kept)] = v
    x[5] = low
    x = x if dtype == "f32" else (torch.from_numpy(x).to(torch.bfloat16).view(torch.int16).numpy())
    H = check(x, dtype, vocab, dev, rows_to_check=np.arange(6))[0]
    assert np.all(np.isfinite(H))
