"""G-Ternary in one read, above the small problems: pass 1 packs by a window
that a sample puts around each worker's threshold, the count settles what the
window left open, and a worker whose threshold missed its window is packed
anew, as is a bucket whose foretold fallback does not come.  Every output bit for bit against the oracle, by rows and by tiles, on
data that makes the window good, poor, useless or wrong."""
import numpy as np
import pytest

import oracle as nfo
import paper_2606_25759_amd as nf
import synth
from tests.test_gpu_ternary import check_ternary_bucket, ternary_route

pytestmark = pytest.mark.gpu

GIB = 1 << 30  # by tiles above, with more than 16 workers
BYTES = 640 << 20  # planes in one read above, and from eight workers
# sizes just above it: eight workers by tiles, 24 by rows
SIZES = [(8, BYTES // 32 + 77), (24, BYTES // 96 + 77)]


def data(W, n, seed):
    lay = synth.small(W, n, seed, elig_frac=0.85, nruns=17)
    return synth.generate_host(lay), nfo.mask_from_segments(*synth.mask_segments(lay), n)


@pytest.mark.parametrize("W,n", SIZES)
@pytest.mark.parametrize("kind", ["normal", "tau0", "all_gated", "outliers", "sparse", "constant", "forced",
                                  "overflow", "spike", "false_spike"])
def test_windows(kind, W, n):
    g, mask = data(W, n, n)
    pol = nf.policy(format=nf.NF_FORMAT_TERNARY, tau={"tau0": 0.0, "all_gated": 1e30, "constant": 1.0}.get(kind, 0.5),
                    force_lowbit=int(kind == "forced"))
    rng = np.random.default_rng(1)
    if kind == "outliers":
        # a few huge elements between the sampled words move the mean
        for w in range(3):
            g[w, rng.choice(n, 40, replace=False)] = 3.0
    elif kind == "sparse":
        g[:, :n] *= rng.random((W, n), dtype=np.float32) < 1e-4
        g[0, :n] = 0
        g[0, n // 2: n // 2 + 5] = 1e-3
    elif kind == "constant":
        # |g| = theta = the mean everywhere: neither below the gate nor far from it
        g[:, :n] = np.where(rng.random((W, n)) < 0.5, np.float32(-2.0 ** -9), np.float32(2.0 ** -9))
    elif kind == "forced":
        g[1, ::1001] = np.nan
        g[2, 5::100_003] = np.inf
    elif kind == "overflow":
        # found while pass 1 reads, which then stores no more planes
        g[W // 3, rng.choice(n, 40, replace=False)] = np.inf
    elif kind == "spike":
        g[W // 2] *= 10
    elif kind == "false_spike":
        # a spike of the eligible elements, foretold by the sample, drowns in the routed ones: no planes from pass 1,
        # yet the low-bit route
        el = np.unpackbits(mask.view(np.uint8), bitorder="little")[:n].astype(bool)
        g[W // 2, :n][el] *= 10
        g[:, :n][:, ~el] *= 1e4
    res = ternary_route(g, mask, n, pol)
    route = check_ternary_bucket(res, g, mask, n, pol, 0, n, f"{kind} W={W}")
    if kind in ("overflow", "spike"):
        assert route == nfo.ROUTE_F
    else:
        assert kind in ("sparse", "outliers") or route == nfo.ROUTE_L


@pytest.mark.parametrize("W,n,bucket_n", [(17, 9_900_001, 3_000_000), (70, 2_400_001, 131_072), (66, 4_200_000, 2_000_000)])
def test_windows_many_workers(W, n, bucket_n):
    """Row groups, several buckets, one of them falling back, one all FP32."""
    g, mask = data(W, n, W)
    if bucket_n < n:
        mask[:bucket_n // 64] = 0
        g[W - 1, n - 1] = np.inf
    pol = nf.policy(format=nf.NF_FORMAT_TERNARY, decode_mode=1)
    res = ternary_route(g, mask, n, pol, bucket_n)
    for b in range(-(-n // bucket_n)):
        check_ternary_bucket(res, g, mask, n, pol, b, bucket_n, f"W={W} bucket {b}")


@pytest.mark.parametrize("W,n", [(8, BYTES // 32 + 77), (16, BYTES // 64 + 77), (24, BYTES // 96 + 77),
                                 (20, GIB // 80 + 4099), (70, GIB // 280 + 4099)])
@pytest.mark.parametrize("kind", ["spike", "dead", "sampled_inf", "false_spike"])
def test_foretold_fallback(kind, W, n):
    """A fallback that the sample foretells packs no planes: bits stay as they were; one that does not come packs
    them all after all.  By tiles with one (two element groups, one), two and four workers a wavefront, and by rows."""
    g, mask = data(W, n, n)
    mask[5000:9000] = 0  # chunks without an eligible element
    pol = nf.policy(format=nf.NF_FORMAT_TERNARY)
    el = np.unpackbits(mask.view(np.uint8), bitorder="little")[:n].astype(bool)
    if kind == "spike":
        g[W // 2] *= 10
    elif kind == "dead":
        g[W - 1] = 0
    elif kind == "sampled_inf":
        g[W // 3, :n:97] = -np.inf
    else:
        g[W // 2, :n][el] *= 10
        g[:, :n][:, ~el] *= 1e4
    res = ternary_route(g, mask, n, pol)
    route = check_ternary_bucket(res, g, mask, n, pol, 0, n, f"{kind} W={W}")
    if kind == "false_spike":
        assert route == nfo.ROUTE_L
    else:
        assert route == nfo.ROUTE_F
        assert (res["bits"] == ~np.uint64(0)).all()


@pytest.mark.parametrize("W,n", [(8, BYTES // 32 + 77), (20, GIB // 80 + 4099), (70, GIB // 280 + 4099)])
def test_fallback_met_while_reading(W, n):
    """One infinity, which the sample misses: some chunks have packed planes when pass 1 meets it, later ones do not."""
    g, mask = data(W, n, n)
    g[W // 3, n // 4] = np.inf
    pol = nf.policy(format=nf.NF_FORMAT_TERNARY)
    res = ternary_route(g, mask, n, pol)
    assert check_ternary_bucket(res, g, mask, n, pol, 0, n, f"W={W}") == nfo.ROUTE_F
