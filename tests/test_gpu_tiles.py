"""Pass 1 by tiles (k_pass1) on adversarial data, at sizes just above those that go by rows: five, two and one
element groups, two and four workers per wavefront, one and two row groups.  Four buckets hold the four kinds of
chunk: element-wise mixed, all eligible and all routed, short FP32 runs, and eligible with a ragged end.

  wide      |g| over 2^-60 .. 2^60 and subnormals, so that tiles leave the proof of an exact sum and every rounding
            error is carried: |g| sums, thresholds and scales bit for bit
  midpoint  sums just above a rounding midpoint: uncertified partials, each worker summed again
  faults    a NaN, an infinity at a routed position, an FP32 sum that overflows, each in a bucket of its own
"""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

import oracle as nfo
import paper_2606_25759_amd as nf
from tests.nfgpu import POOL, Bucket, check_route
from tests.test_gpu_exact_sums import midpoint_rows
from tests.test_gpu_ternary import check_ternary_bucket, ternary_route

pytestmark = pytest.mark.gpu

WORKERS = [3, 8, 16, 20, 70]
TERNARY = nf.policy(format=nf.NF_FORMAT_TERNARY, tau=0.5)


def sizes(W):
    """(elements, bucket elements) just above the sizes that go by rows."""
    n = ((160 << 20) if W <= 16 else (1 << 30)) // (4 * W) + 4099
    bn = n // 4 // 64 * 64 + 64
    for fmt in (nf.NF_FORMAT_BINARY, nf.NF_FORMAT_TERNARY):
        path = nf.nf_pass1_path(W, n, bn, fmt)
        assert not path & nf.NF_PASS1_ROWS and bool(path & nf.NF_PASS1_PLANES) == (fmt == 1 and W > 16)
    assert -(-n // bn) == 4
    return n, bn


def mask_of(n, bn):
    rng = np.random.default_rng(n)
    el = np.ones(n, bool)
    el[:bn] = rng.random(bn) < 0.8
    el[bn + bn // 2: 2 * bn] = False
    for a in range(2 * bn, 3 * bn, 40_000):
        el[a: a + 700] = False
    return el, np.packbits(np.pad(el, (0, -n % 64)), bitorder="little").view(np.uint64).copy()


def rows(W, n, base):
    """W rows of a stride that is a multiple of 4, as shifted copies of base (n + 67 W elements) with alternating
    signs."""
    g = np.zeros((W, -(-n // 4) * 4), np.float32)
    for w in range(W):
        np.multiply(base[67 * w: 67 * w + n], np.float32(1 - 2 * (w % 2)), out=g[w, :n])
    return g


def check(jobs):
    """Oracle checks in a pool of host threads (its calls release the interpreter lock)."""
    with ThreadPoolExecutor(POOL) as ex:
        for f in [ex.submit(*j) for j in jobs]:
            f.result()


def route(g, mask, n, pol, bn):
    res = Bucket(g, mask, n, bn).route(pol)
    torch.cuda.empty_cache()
    return res


@pytest.mark.parametrize("W", WORKERS)
def test_wide_range(W):
    n, bn = sizes(W)
    rng = np.random.default_rng(W)
    base = rng.standard_normal(n + 67 * W, dtype=np.float32) * np.exp2(rng.integers(-60, 61, n + 67 * W)).astype(np.float32)
    base[::97] = np.float32(3e-45)
    g, (_, mask) = rows(W, n, base), mask_of(n, bn)
    veto = nf.policy(veto=1, fp32_op=nf.NF_FP32_MEAN)
    tern, vetoed = ternary_route(g, mask, n, TERNARY, bn), route(g, mask, n, veto, bn)
    check([(check_ternary_bucket, tern, g, mask, n, TERNARY, b, bn, f"W={W} bucket {b}") for b in range(4)] +
          [(check_route, vetoed, g[:, :n], mask, n, veto, bn, True, f"W={W} vetoed", [b]) for b in range(4)])


@pytest.mark.parametrize("W", WORKERS)
def test_midpoint_sums(W):
    n, bn = sizes(W)
    g = np.zeros((W, -(-n // 4) * 4), np.float32)
    g[:, :n] = midpoint_rows(W, n, W, True, bn)
    mask = np.full((n + 63) // 64, ~np.uint64(0))
    mask[-1] >>= np.uint64(-n % 64)
    pol = nf.policy(format=nf.NF_FORMAT_TERNARY, tau=0.5, force_lowbit=1)
    res = ternary_route(g, mask, n, pol, bn)
    check([(check_ternary_bucket, res, g, mask, n, pol, b, bn, f"W={W} bucket {b}") for b in range(4)])
    for w in range(W):
        assert res["stats"][w % 4]["sum_abs_elig"][w] == 1.0 + 2.0 ** -52
    assert [int(d["resummed"]) for d in res["dec"]] == [len(range(b, W, 4)) for b in range(4)]


@pytest.mark.parametrize("W", WORKERS)
def test_faults(W):
    n, bn = sizes(W)
    base = np.random.default_rng(W).standard_normal(n + 67 * W, dtype=np.float32) * np.float32(1e-3)
    g, (el, mask) = rows(W, n, base), mask_of(n, bn)
    routed = np.flatnonzero(~el)
    g[W // 2, np.flatnonzero(el[:bn])[1000]] = np.nan
    g[W - 1, 2 * bn - 5] = np.inf
    over = routed[np.searchsorted(routed, 2 * bn + 100)]
    g[:, over] = np.float32(3e38)
    pols = (nf.policy(), nf.policy(force_lowbit=1, fp32_op=nf.NF_FP32_MEAN), nf.policy(veto=1, fp32_op=nf.NF_FP32_MEAN))
    res = [route(g, mask, n, p, bn) for p in pols]
    check([(check_route, r, g[:, :n], mask, n, p, bn, True, f"W={W} policy {k}", [b])
           for k, (r, p) in enumerate(zip(res, pols)) for b in range(4)])
    assert [int(d["route"]) for d in res[0]["dec"]] == [nfo.ROUTE_F, nfo.ROUTE_F, nfo.ROUTE_L, nfo.ROUTE_L]
    assert np.isinf(res[0]["out"][over])
