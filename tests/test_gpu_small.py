"""Pass 1 by rows and the fused decision and read side of small problems, at
the edges of their rules: one word to whole batches of eight words, ragged
ends, fewer and more workers than wavefronts, one chunk to the last small
size and the first above it, the most partials a read-side block reduces, row
groups above 64 workers, and every route.  Bits, counts, routes and FP32 sums
bit for bit against the oracle; the FP64 sums and the scale within the bars of
nfgpu (another order of exact FP64 sums; |g| sums exact without sign words)."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle as nfo
import paper_2606_25759_amd as nf
import synth
from tests.nfgpu import Bucket, check_route
from tests.test_gpu_ternary import check_ternary_bucket, ternary_route

pytestmark = pytest.mark.gpu

MB160, GB1 = 160 << 20, 1 << 30


def tile(W):
    """Elements of a pass-1 tile (the unit of the small-problem rule)."""
    rows = W if W <= 32 else -(-W // 2) if W <= 64 else -(-W // -(-W // 64))
    return (16 // min(rows, 16)) * {1: 512, 2: 256, 3: 256, 4: 256}[-(-rows // 16)]


def case(W, n, seed, elig=0.85):
    lay = synth.small(W, n, seed, elig_frac=elig, nruns=13)
    return synth.generate_host(lay), nfo.mask_from_segments(*synth.mask_segments(lay), n)


EDGES = [(W, n) for W in (1, 3, 9, 16, 17, 64, 65, 255) for n in (1, 64, 511, 513, 4095, 20_001)]
# the last small size and the first above it; 256 chunks of 64 workers are too many partials for the fused decision
EDGES += [(W, 1024 * tile(W) + d) for W in (2, 16, 33, 64, 130) for d in (0, 1)]
# the largest by rows up to 16 workers, the smallest by tiles, a middling one by rows
EDGES += [(12, MB160 // 48), (8, MB160 // 32 + 1), (40, 1_500_000)]
# the largest by rows above 16 workers and the smallest by tiles; 17 to 64 workers by rows again above 4,096 chunks
LIMITS = [(24, GB1 // 96, True), (24, GB1 // 96 + 1, False), (70, GB1 // 280, True), (70, GB1 // 280 + 1, False),
          (17, 4096 * 8192 + 1, True)]


@pytest.mark.parametrize("W,n", EDGES)
def test_low_bit_and_vetoed(W, n):
    g, mask = case(W, n, 5 * W + n)
    k = Bucket(g, mask, n)
    for pol in (nf.policy(), nf.policy(veto=1, fp32_op=nf.NF_FP32_MEAN)):
        check_route(k.route(pol), g, mask, n, pol, what=f"W={W} n={n} veto={pol.veto}")


@pytest.mark.parametrize("W,n,by_rows", LIMITS)
def test_limits_above_16_workers(W, n, by_rows):
    assert bool(nf.nf_pass1_path(W, n, n) & nf.NF_PASS1_ROWS) == by_rows
    g, mask = case(W, n, W + n)
    k = Bucket(g, mask, n)
    pols = (nf.policy(), nf.policy(veto=1, fp32_op=nf.NF_FP32_MEAN))
    res = [k.route(pol) for pol in pols]
    with ThreadPoolExecutor(2) as ex:  # the oracle's calls release the interpreter lock
        list(ex.map(lambda i: check_route(res[i], g, mask, n, pols[i], what=f"W={W} n={n} veto={i}"), range(2)))


@pytest.mark.parametrize("W,n", [(W, n) for W in (1, 3, 9, 16, 17, 64, 65) for n in (1, 64, 513, 20_001)] +
                         [(W, 1024 * tile(W) + d) for W in (16, 33) for d in (0, 1)])
def test_ternary(W, n):
    g, mask = case(W, n, 7 * W + n)
    pol = nf.policy(format=nf.NF_FORMAT_TERNARY, tau=0.5, decode_mode=W % 2)
    res = ternary_route(g, mask, n, pol)
    check_ternary_bucket(res, g, mask, n, pol, 0, max(n, 1), f"W={W} n={n}")


@pytest.mark.parametrize("W", [2, 8, 24, 64])
@pytest.mark.parametrize("n", [700, 50_003])
@pytest.mark.parametrize("fault", ["nan", "inf", "dead", "spike", "overflow"])
def test_fallback(W, n, fault):
    """What the data sends to the FP32 fallback, both formats."""
    g, mask = case(W, n, W + n, elig=0.9)
    if fault == "nan":
        g[W // 2, n // 3] = np.nan
    elif fault == "inf":
        g[0, n - 1] = -np.inf
    elif fault == "dead":
        g[W - 1] = 0.0
    elif fault == "spike":
        g[W - 1] *= 30
    else:  # every worker finite, their FP32 sum not
        g[:, n // 2] = np.float32(3e38)
    for fmt in (nf.NF_FORMAT_BINARY, nf.NF_FORMAT_TERNARY):
        pol = nf.policy(format=fmt)
        if fmt == nf.NF_FORMAT_BINARY:
            check_route(Bucket(g, mask, n).route(pol), g, mask, n, pol, what=f"{fault} W={W} n={n}")
        else:
            check_ternary_bucket(ternary_route(g, mask, n, pol), g, mask, n, pol, 0, n, f"{fault} W={W} n={n} ternary")


@pytest.mark.parametrize("W", [4, 20, 80])
@pytest.mark.parametrize("n,bucket_n", [(9_000, 64), (100_001, 6_400), (300_000, 131_072)])
def test_many_small_buckets(W, n, bucket_n):
    """One of them without an eligible element, one with a NaN."""
    g, mask = case(W, n, W + bucket_n)
    mask[bucket_n // 64: 2 * bucket_n // 64] = 0
    g[1, 2 * bucket_n + 5] = np.nan
    pol = nf.policy()
    check_route(Bucket(g, mask, n, bucket_n).route(pol), g, mask, n, pol, bucket_n, what=f"W={W}")
    pol = nf.policy(format=nf.NF_FORMAT_TERNARY)
    res = ternary_route(g, mask, n, pol, bucket_n)
    for b in range(-(-n // bucket_n)):
        check_ternary_bucket(res, g, mask, n, pol, b, bucket_n, f"W={W} bucket {b}")
