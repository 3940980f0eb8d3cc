"""Selection over its sizes: the keys of up to 16,384 tokens (24,576 of one
term) sit in the registers of a block (4, 8, 16 or 24 a thread), and while there are fewer than 256
selections each round of four a thread is written by a block of its own; larger
selections take the
two passes over chunks of 4,096, or, in the smallest workspace that is
accepted, blocks that re-read all keys. Every size at the edges of those
ranges, every kind of key (activity, temporal, both; tied in long runs, one
value, spread out), token offsets that are no multiple of four, fixed and
MAS-guided counts, whole-segment and per-frame scope, against a sort of the
exact keys (key, then index)."""
import re

import numpy as np
import pytest
import torch

import paper_2604_02945_amd as msao
from paper_2604_02945_amd import binding as B

pytestmark = pytest.mark.gpu

IMAGE, VIDEO = B.IMAGE, B.VIDEO
SIZES = [1, 2, 3, 4, 5, 7, 63, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 8191, 8192, 8193,
         16383, 16384, 16385, 20480, 20481, 24575, 24576, 24577, 40000, 65537]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


def values(rng, n, C, how):
    """z or d of n tokens, in [0, C]."""
    if how == "spread":
        return rng.integers(0, C + 1, n)
    if how == "tied":  # runs of the largest value, the others in few values
        v = rng.integers(C // 2, C // 2 + 4, n)
        v[n // 5: n // 2] = C
        return v
    if how == "one":
        return np.full(n, C)
    return np.clip(rng.normal(C / 2, C / 40, n), 0, C).astype(np.int64)  # crowded


def q24(x):
    return int(np.rint(np.float64(np.float32(x)) * 2 ** 24))


def expected(segs, z, d, lam_s, lam_t, mas, per_frame):
    keep, idx, count, off = [], [], [], 0
    for (m, T, P, C, ratio) in segs:
        N = T * P
        zz, dd = z[off:off + N].astype(object), d[off:off + N].astype(object)
        key = q24(lam_s[m]) * zz
        if m == VIDEO and T > 1:
            key = key + q24(lam_t[m]) * (C - dd)
        kappa = float(np.float32(ratio)) if ratio >= 0 else 1.0 - float(np.float32(mas[m]))
        f = np.zeros(N, np.uint8)
        frames = T if per_frame and T > 1 else 1
        n = N // frames
        k = min(n, int(np.ceil(kappa * n)))
        for t in range(frames):
            part = np.array(key[t * n:(t + 1) * n], dtype=np.uint64)
            f[t * n + np.argsort(part, kind="stable")[:k]] = 1
        keep.append(f)
        i = np.full(N, -1, np.int32)
        at = np.flatnonzero(f)
        i[:len(at)] = at
        idx.append(i)
        count.append(len(at))
        off += N
    return np.concatenate(keep), np.concatenate(idx), np.array(count, np.int32)


def check(segs, how, dev, lam_s=(0, .6, .6, .6), lam_t=(0, 0, .4, 0), per_frame=False, smallest=False, seed=0):
    rng = np.random.default_rng(seed)
    z = np.concatenate([values(rng, T * P, C, how) for (_, T, P, C, _) in segs]).astype(np.int32)
    d = np.concatenate([values(rng, T * P, C, how) for (_, T, P, C, _) in segs]).astype(np.int32)
    mas = np.array([0.1, 0.37, 0.55, 0.9], np.float32)
    table = [msao.DeviceSegment(torch.empty(T * P, C, dtype=torch.bfloat16, device=dev), 0, m, ratio, T)
             for (m, T, P, C, ratio) in segs]
    p = dict(msao.default_params(), lambda_s=list(lam_s), lambda_t=list(lam_t), flags=B.FLAG_SELECT_PER_FRAME if per_frame else 0)
    o = msao.Outputs(table, 1, compact=False)
    zt, dt = torch.from_numpy(z).to(dev), torch.from_numpy(d).to(dev)
    mt = torch.from_numpy(mas).to(dev)
    if smallest:
        full = o.ws_bytes
        o.ws_bytes = 1
        with pytest.raises(msao.MsaoError) as e:
            msao.msao_select_tokens(table, 1, zt, dt, mt, params=p, outputs=o)
        o.ws_bytes = int(re.search(r"(\d+) needed", str(e.value)).group(1))
        assert o.ws_bytes < full
    for t in (o.sel["keep"], o.sel["kept_idx"], o.sel["kept_count"]):
        t.fill_(77)
    msao.msao_select_tokens(table, 1, zt, dt, mt, params=p, outputs=o)
    torch.cuda.synchronize()
    keep, idx, count = expected(segs, z, d, lam_s, lam_t, mas, per_frame)
    r = o.results(1, len(segs))
    assert np.array_equal(r["kept_count"].cpu().numpy(), count)
    assert np.array_equal(r["keep"].cpu().numpy(), keep)
    assert np.array_equal(r["kept_idx"].cpu().numpy(), idx)


@pytest.mark.parametrize("how", ["spread", "tied", "one", "crowded"])
@pytest.mark.parametrize("n", SIZES)
def test_sizes(n, how, dev):
    print(f"[selection] {n} {how}", flush=True)
    C = 64 if n > 20000 else 512
    check([(IMAGE, 1, n, C, 0.4)], how, dev, seed=n)
    # three segments, the second and third at odd token offsets; the third's count from MAS
    check([(IMAGE, 1, 3, C, 0.5), (VIDEO, max(1, n // 7), min(n, 7), C, 0.3), (IMAGE, 1, n, C, -1.0)], how, dev, seed=n + 1)


@pytest.mark.parametrize("lam", [(0.6, 0.4), (0.0, 1.0), (1.0, 0.0), (0.0, 0.0)])
@pytest.mark.parametrize("T,P", [(2, 513), (3, 3000), (5, 4097), (2, 20000)])
def test_keys_and_scopes(T, P, lam, dev):
    print(f"[selection] {T} x {P} weights {lam}", flush=True)
    for per_frame in (False, True):
        for ratio in (0.25, -1.0, 0.0, 1.0):
            check([(IMAGE, 1, 1, 40, 1.0), (VIDEO, T, P, 40, ratio)], "spread", dev, lam_s=(0, .6, lam[0], .6),
                  lam_t=(0, 0, lam[1], 0), per_frame=per_frame, seed=T * P)


@pytest.mark.parametrize("how", ["spread", "tied", "one", "crowded"])
def test_wide_keys_of_large_selections(how, dev):
    """4,096 channels: 13-bit and, with the temporal term, 37-bit keys, so the first digit leaves candidates."""
    print(f"[selection] wide {how}", flush=True)
    check([(IMAGE, 1, 5, 4096, 0.5), (IMAGE, 1, 18001, 4096, 0.3)], how, dev, seed=1)
    check([(IMAGE, 1, 5, 4096, 0.5), (VIDEO, 9, 2003, 4096, 0.7)], how, dev, seed=2)


@pytest.mark.parametrize("n", [16385, 24577, 40000])
@pytest.mark.parametrize("how", ["spread", "tied"])
def test_smallest_workspace(n, how, dev):
    print(f"[selection] smallest workspace {n} {how}", flush=True)
    check([(IMAGE, 1, 3, 512, 0.5), (IMAGE, 1, n, 512, 0.4)], how, dev, smallest=True, seed=n)
    check([(VIDEO, 5, n // 5, 512, -1.0)], how, dev, smallest=True, seed=n + 1)


@pytest.mark.parametrize("largest", [4095, 4096, 16384])
@pytest.mark.parametrize("count", [31, 43, 64, 255, 256, 257])
def test_one_block_or_one_per_round(count, largest, dev):
    """On both sides of the 256 selections up to which a selection is written
    by a block per round (1,024 tokens), and of the 128 blocks (rounds of 4,096,
    beside a selection of 4,096 and more)."""
    print(f"[selection] {count} selections up to {largest}", flush=True)
    n = [1 + (37 * i) % 1100 for i in range(count - 5)] + [1024, 1025, 2049, 3000, largest]
    segs = [(VIDEO, 3, -(-x // 3), 40, -1.0) if i % 7 == 2 else (IMAGE, 1, x, 40, 0.0 if i % 11 == 3 else 0.37)
            for i, x in enumerate(n)]
    check(segs, "crowded", dev, seed=count)
    check(segs[-3:-1], "tied", dev, seed=count + 1)
