"""Pass 1's block protocol on the CPU: k_pass1's own source, compiled for the host with a fibre per thread
(tests/block_cpu), run block by block while another block turns the bucket's fallback flag between this block's
wavefronts.  Every block barrier has to be met by all wavefronts of the block, and the chunk's statistics have to be
those of its data whatever the wavefronts saw."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2606_25759_amd", "csrc")
CPU = os.path.join(HERE, "block_cpu")
CLANG = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")


def host_source(name):
    """A kernel source for the host: dynamic LDS is an ordinary array, the lane writes in assembly are C++."""
    text = open(os.path.join(CSRC, name)).read().replace("extern __shared__", "extern")
    text = text.split("// --------------------------------------------------------------- launchers")[0]
    text = re.sub(r"__attribute__\(\(amdgpu_waves_per_eu\(.*?\)\)\)", "", text)
    if "void lanes_from_ballots(" in text:
        head, rest = text.split("  uint32_t l[8], h[8];", 1)
        rest = rest[re.search(r"\n}\n", rest).end():]
        text = head + ("  const int k = cpu::lane() < NW ? cpu::lane() : 0;\n"
                       "  lo = (uint32_t)bb[k];\n  hi = (uint32_t)(bb[k] >> 32);\n}\n") + rest
    return text


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++ of the ROCm toolchain")
    d = tmp_path_factory.mktemp("pass1")
    for name in ("nf_device.h", "nf_decide.h"):
        (d / name).write_text(host_source(name))
    (d / "kernels.h").write_text(host_source("nf_pass1.hip") + "\n}  // namespace nf\n")
    so = str(d / "pass1.so")
    subprocess.check_call([CLANG, "-x", "c++", "-O1", "-std=c++17", "-fPIC", "-shared", "-w", "-ffp-contract=off",
                           f'-DPASS1_KERNELS="{d}/kernels.h"', "-I", str(d), "-I", CPU, "-I", CSRC, "-I",
                           os.path.join(ROOT, "include"), os.path.join(CPU, "pass1.cpp"), "-o", so])
    return ctypes.CDLL(so)


def ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)


PARTIAL = np.dtype([("sabs", "f8"), ("ssq", "f8"), ("nonfinite", "u8"), ("sabs_c", "f8"), ("sabs_b", "f8")])


# tiles of 1,024 elements at 8 workers (two element groups), 2,048 at 4, 512 at 9 and 16 (one group), 256 at 70 (two
# row groups, four workers a wavefront): chunks that are all eligible, mixed, all FP32, and a ragged last one
@pytest.mark.parametrize("turn", [0, 1, 7, 8, 15, 16])
@pytest.mark.parametrize("W", [4, 8, 9, 16, 70])
def test_flag_turns_between_wavefronts(lib, W, turn):
    found = run_planes(lib, W, turn, None)
    assert not found


@pytest.mark.parametrize("W,bad", [(8, 3), (16, 15), (70, 2), (70, 69)])
def test_nonfinite_value_sets_the_flag(lib, W, bad):
    """Chunks that start later then pack no planes."""
    assert run_planes(lib, W, 16, bad)


def run_planes(lib, W, turn, bad):
    """Pass 1 over a bucket, everything checked; worker `bad` has an infinity.  Returns whether the flag was set."""
    tile = (16 // W) * 512 if W <= 16 else 256
    G, n = 2, 7 * tile + 333 % tile
    rng = np.random.default_rng(W)
    g = rng.standard_normal((W, n)).astype(np.float32)
    words = (n + 63) // 64
    el = np.ones(words * 64, bool)
    el[2 * tile + 70:2 * tile + 700] = False  # second chunk: mixed
    el[4 * tile:6 * tile] = False  # third: FP32
    el[n:] = False
    if bad is not None:
        g[bad, tile + 5] = np.inf
    mask = np.packbits(el, bitorder="little").view(np.uint64).copy()
    chunks = -(-n // (G * tile))
    bits = np.full((2 * W, words), 0x5555, np.uint64)
    out = np.zeros(n, np.float32)
    part = np.zeros((chunks, W), PARTIAL)
    part_ne = np.zeros(chunks, np.uint64)
    stats = np.zeros((W, 24), np.uint8)
    win = stats.view(np.float32)
    win[:, 0], win[:, 1], win[:, 2] = 0.4, 0.4, 1.0  # the thresholds, nothing left open, nothing foretold
    msg = ctypes.create_string_buffer(200)
    rc = lib.pass1_planes(ptr(g), ptr(mask), W, ctypes.c_int64(n), G, turn, ptr(bits), ptr(out), ptr(part),
                          ptr(part_ne), ptr(stats), msg)
    assert rc == 0, msg.value.decode()
    el = el[:n]
    for c in range(chunks):
        s = slice(c * G * tile, min((c + 1) * G * tile, n))
        assert part_ne[c] == el[s].sum()
        x = g[:, s].astype(np.float64)
        np.testing.assert_allclose(part["sabs"][c] + part["sabs_c"][c] if bad is None else part["sabs"][c],
                                   np.abs(x[:, el[s]]).sum(1), rtol=1e-14)
        np.testing.assert_allclose(part["ssq"][c], (x * x).sum(1), rtol=1e-13)  # 4,096 terms in another order
        assert np.array_equal(part["nonfinite"][c], (~np.isfinite(x)).sum(1))
    want = g[0].copy()
    for w in range(1, W):
        want = want + g[w]
    assert np.array_equal(out[~el], want[~el])
    if turn == 16:  # nobody saw the flag: both planes whole
        keep = (np.abs(g) >= np.float32(0.4)) & el
        planes = np.concatenate([keep & (g > 0), keep & (g < 0)])
        planes = np.pad(planes, ((0, 0), (0, words * 64 - n)))
        assert np.array_equal(np.packbits(planes, axis=1, bitorder="little").view(np.uint64), bits)
    if turn == 0:  # the whole block did
        assert (bits == 0x5555).all()
    return win[0, 3] != 0
