"""9 to 15 workers: pass 1 and the G-Ternary pack give a worker to a wavefront
of their 16, and the wavefronts without one leave the others' sign words,
planes and partial statistics alone.  Sizes above those that pass 1 takes by
rows; everything against the oracle."""
import pytest

import oracle as nfo
import paper_2606_25759_amd as nf
import synth
from tests.nfgpu import Bucket, check_route
from tests.test_gpu_ternary import check_ternary_bucket, ternary_route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [9, 12, 15])
def test_idle_wavefronts(W):
    n = (160 << 20) // (4 * W) + 70_000
    lay = synth.small(W, n, W, elig_frac=0.85, nruns=13)
    g, mask = synth.generate_host(lay), nfo.mask_from_segments(*synth.mask_segments(lay), n)
    pol = nf.policy()
    check_route(Bucket(g, mask, n).route(pol), g, mask, n, pol, what=f"W={W}")
    pol = nf.policy(format=nf.NF_FORMAT_TERNARY)
    check_ternary_bucket(ternary_route(g, mask, n, pol), g, mask, n, pol, 0, n, f"W={W} ternary")
