"""The work that users of the bucket reducer have it do, as cases that can be measured.

Each case is one pass through the library's public entry points on W workers' FP32 gradient rows: a training
step's reduction of every bucket (`what` = "route": one bucket, a flat buffer of equal buckets with or without a
workspace, or DDP's buckets through a bucket table), the chain with the compacted payload and per-slice scales
("sliced"), or hierarchical counting of packed signs ("hier").

Layouts (parameter runs in the order their gradients become ready, each low-bit eligible or FP32):
  runs    sixteen alternating runs, about 90% eligible
  conv    a convolutional backbone: eligible runs of 16K to 196K elements, FP32 runs of 64 to 2,048 between them
  blocks  a Transformer of `layers` blocks of width d with a vocabulary and a context: matrices eligible;
          embeddings, norms, biases and the head FP32

Conditions (`when`): "ordinary" gradients; a "vetoed" step (cooldown: the policy fixes the FP32 route); a worker
whose gradients "spike"; a "dead" worker (all zeros); an "overflow" (infinities in one worker).  The last three
make the buckets fall back to FP32 by what is found in the data.
"""
import math
import random

import numpy as np
import torch

import paper_2606_25759_amd as nf

DEV = "cuda"
BUCKET_N = 6_553_600  # 25 MiB of FP32, DDP's bucket


def _route(name, api, W, layout, format="binary", when="ordinary", decode="soft", mean=False, **size):
    return dict(name=name, what="route", api=api, W=W, layout=layout, format=format, when=when, decode=decode,
                mean=mean, **size)


def listed():
    return [
        # one small ragged bucket: a small model, or the last bucket of one; all latency
        _route("bucket_w8_70k", "bucket", 8, "runs", n=70_001),
        # a 4 MiB bucket of four workers from a loop that must not allocate; caches hold it
        _route("noalloc_w4_1m", "noalloc", 4, "runs", n=1_048_576),
        # one DDP bucket of eight workers in G-Ternary
        _route("ternary_w8_bucket", "bucket", 8, "conv", format="ternary", n=BUCKET_N),
        # ResNet-50's size: four buckets, many short FP32 runs
        _route("conv_w8_26m", "buckets", 8, "conv", n=25_600_000),
        # ViT-B/16's size cut at parameter boundaries, as DDP cuts it
        _route("ddp_w16_vit", "table", 16, "blocks", d=768, layers=12, vocab=1_970, context=197),
        # the same model in G-Ternary with equal buckets
        _route("ternary_w16_vit", "buckets", 16, "blocks", format="ternary", d=768, layers=12, vocab=1_970,
               context=197),
        # half of a 1.3B-parameter decoder (12 of 24 blocks and the embeddings): the largest
        _route("gpt_w16_714m", "buckets", 16, "blocks", d=2048, layers=12, vocab=50_257, context=2_048),
        # high fan-in, one large bucket that falls back to FP32 after it has been read
        _route("fallback_w64_25m", "bucket", 64, "runs", when="overflow", n=25_000_003),
        # a cooldown step: FP32 mean of everything, with health statistics
        _route("vetoed_w16_26m", "buckets", 16, "conv", when="vetoed", mean=True, n=25_557_032),
        # the largest fan-in that uint8 counts hold: one decoder block of width 1024
        _route("block_w255", "buckets", 255, "blocks", decode="majority", d=1024, layers=1, vocab=0, context=0),
        # compacted payload and a scale per parameter: four decoder blocks of width 2048
        dict(name="sliced_w16_201m", what="sliced", W=16, layout="blocks", d=2048, layers=4, vocab=0, context=0,
             decode="soft"),
        # 8 nodes x 8 GPUs: node-local counts of one DDP bucket, then their exchange and decode
        dict(name="hier_w64_bucket", what="hier", W=64, P=8, layout="conv", n=BUCKET_N, decode="soft"),
    ]


MOST = 12e9  # bytes of gradients of a drawn case at most


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    what = rng.choice(["route"] * 8 + ["sliced", "hier"])
    W = rng.choice([rng.randint(1, 8), rng.choice([4, 8, 16, 32, 64]), rng.randint(2, 64),
                    int(_log(rng, 16, 255.9))])
    decode = rng.choice(["soft", "soft", "majority"])
    if what == "hier":
        P = rng.choice([2, 4, 8])
        W = P * rng.randint(2, 96 // P)
        n = int(_log(rng, 60_000, 30_000_000))
        return dict(what="hier", W=W, P=P, layout="conv", n=n, decode=decode)
    n = int(_log(rng, 60_000, MOST / 4 / W))
    if what == "sliced" or rng.random() < 0.35:
        d = 64 * int(_log(rng, 1, 32.9)) + rng.choice([0, 0, 16, 40])
        per = 12 * d * d + 13 * d
        layers = max(1, min(48, n // per))
        while layers * per * 4 * W > MOST:
            d = max(64, d // 2)
            per = 12 * d * d + 13 * d
            layers = max(1, min(layers, int(MOST / 4 / W) // per))
        size = dict(layout="blocks", d=d, layers=layers, vocab=rng.choice([0, rng.randint(100, 3_000)]),
                    context=rng.randint(16, 512))
    else:
        size = dict(layout=rng.choice(["runs", "conv"]), n=n)
    if what == "sliced":
        return dict(what="sliced", W=W, decode=decode, **size)
    when = rng.choice(["ordinary"] * 7 + ["vetoed", "spike", "dead", "overflow"])
    if W < 3 and when == "spike":
        when = "dead"
    api = rng.choice(["bucket", "buckets", "noalloc", "table"])
    if api == "noalloc":
        api = "noalloc" if nf.nf_workspace_bytes_buckets(W, _total(size), BUCKET_N) <= nf.NF_STATIC_SCRATCH_BYTES \
            else "buckets"
    return dict(what="route", api=api, W=W, format=rng.choice(["binary", "binary", "ternary"]), when=when,
                decode=decode, mean=rng.random() < 0.3, **size)


# ------------------------------------------------------------------- layouts

def _tensors(case):
    """(lengths, eligible) of the layout's runs in bucket order."""
    if case["layout"] == "blocks":
        d = case["d"]
        t = [(case["vocab"] * d, 0), (case["context"] * d, 0)]
        for _ in range(case["layers"]):
            t += [(d, 0), (d, 0), (3 * d * d, 1), (3 * d, 0), (d * d, 1), (d, 0),
                  (d, 0), (d, 0), (4 * d * d, 1), (4 * d, 0), (4 * d * d, 1), (d, 0)]
        t = [x for x in reversed(t) if x[0]]
        return np.array([x[0] for x in t], np.int64), np.array([x[1] for x in t], np.uint8)
    n = case["n"]
    rng = random.Random(n)
    lengths, eligible = [], []
    if case["layout"] == "runs":
        cuts = sorted(rng.sample(range(1, 997), 7))
        for k, (a, b) in enumerate(zip([0] + cuts, cuts + [997])):
            run = (n * b // 997) - (n * a // 997)
            f = run * rng.randint(50, 150) // 1000
            lengths += [run - f, f]
            eligible += [1, 0]
    else:
        left = n
        while left > 0:
            for length, e in ((rng.randint(16_384, 196_608), 1), (rng.randint(64, 2_048), 0)):
                length = min(length, left)
                if length:
                    lengths.append(length)
                    eligible.append(e)
                left -= length
    keep = [k for k in range(len(lengths)) if lengths[k]]
    return np.array([lengths[k] for k in keep], np.int64), np.array([eligible[k] for k in keep], np.uint8)


def _total(case):
    return int(_tensors(case)[0].sum())


def _offsets(lengths):
    """DDP's cut: a bucket closes with the tensor that fills it (the first one sooner); starts move down to
    multiples of 64."""
    ends, size, cap, at = [], 0, 1 << 20, 0
    for length in lengths.tolist():
        at += length
        size += 4 * length
        if size >= cap:
            ends.append(at)
            size, cap = 0, 25 << 20
    starts = sorted({0} | {e // 64 * 64 for e in ends if e // 64 * 64 < at})
    return np.array(starts + [at], np.int64)


def _gradients(case, lengths, seed):
    """[W, stride] rows: per-run scales spread over three decades, Student-t(3) for the Transformers (heavy
    tails), normal else, and the case's condition."""
    W, n = case["W"], int(lengths.sum())
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed * 1_000_003 + W)
    sigma = np.exp(np.random.default_rng(seed).uniform(math.log(1e-6), math.log(1e-3), len(lengths)))
    sigma = torch.repeat_interleave(torch.from_numpy(sigma.astype(np.float32)).to(DEV),
                                    torch.from_numpy(lengths).to(DEV))
    g = torch.zeros(W, -(-n // 64) * 64, dtype=torch.float32, device=DEV)
    for w in range(W):
        row = g[w, :n]
        row.normal_(generator=gen)
        if case["layout"] == "blocks" and n < 150_000_000:
            t = torch.empty(n, dtype=torch.float32, device=DEV)
            chi = t.normal_(generator=gen).square()
            for _ in range(2):
                chi += t.normal_(generator=gen).square_()
            row /= chi.div_(3).sqrt_().clamp_(min=1e-3)
        row *= sigma
    when = case.get("when")
    if when == "spike":
        g[W // 2] *= 10
    elif when == "dead":
        g[W - 1] = 0
    elif when == "overflow":
        at = torch.randint(n, (100,), generator=gen, device=DEV)
        g[W // 3, at] = math.inf
    return g


def _words(n):
    return (n + 63) // 64


# ------------------------------------------------------------------ the pass

class State:
    pass


def prepare(case, seed):
    s = State()
    s.case, s.W = case, case["W"]
    lengths, eligible = _tensors(case)
    s.n = n = int(lengths.sum())
    W, nw = s.W, _words(n)
    starts = np.cumsum(lengths) - lengths
    s.mode = nf.NF_DECODE_MAJORITY if case["decode"] == "majority" else nf.NF_DECODE_SOFT
    s.out = torch.zeros(n, dtype=torch.float32, device=DEV)
    if case["what"] == "hier":
        mask = nf.nf_mask_from_segments(starts, lengths, eligible, n)
        s.mask = torch.from_numpy(mask.view(np.int64)).to(DEV)
        gen = torch.Generator(device=DEV)
        gen.manual_seed(seed)
        s.bits = torch.randint(-2**63, 2**63 - 1, (W, nw), dtype=torch.int64, device=DEV, generator=gen)
        s.bits &= s.mask
        s.partial = torch.empty(W // case["P"], -(-n // 16) * 16, dtype=torch.uint8, device=DEV)
        s.counts = torch.empty(n, dtype=torch.uint8, device=DEV)
        s.scale = torch.rand(1, device=DEV, generator=gen) * 1e-3
        s.result = {"partial": s.partial[:, :n], "counts": s.counts, "out": s.out}
        return s
    s.grads = _gradients(case, lengths, seed)
    if case["what"] == "sliced":
        e = eligible.astype(bool)
        s.lay = nf.SlicedLayout(starts[e], lengths[e], n, device=DEV)
        s.bits = torch.empty(W, nw, dtype=torch.int64, device=DEV)
        s.cbits = torch.empty(W, _words(s.lay.n_eligible), dtype=torch.int64, device=DEV)
        s.stats = torch.empty(W * nf.STATS_BYTES, dtype=torch.uint8, device=DEV)
        s.ws = nf.empty_workspace(nf.nf_workspace_bytes(W, n), DEV)
        s.sums = torch.empty(s.lay.S, W, dtype=torch.float64, device=DEV)
        s.scales = torch.empty(s.lay.S, dtype=torch.float32, device=DEV)
        s.counts = torch.empty(s.lay.n_eligible, dtype=torch.uint8, device=DEV)
        s.result = {"bits": s.bits, "cbits": s.cbits, "sums": s.sums, "scales": s.scales, "counts": s.counts,
                    "out": s.out, **_stats_views(s.stats, 1, W)}
        return s
    mask = nf.nf_mask_from_segments(starts, lengths, eligible, n)
    s.mask = torch.from_numpy(mask.view(np.int64)).to(DEV)
    ternary = case["format"] == "ternary"
    s.pol = nf.policy(veto=int(case["when"] == "vetoed"), decode_mode=s.mode,
                      fp32_op=nf.NF_FP32_MEAN if case["mean"] else nf.NF_FP32_SUM,
                      format=nf.NF_FORMAT_TERNARY if ternary else nf.NF_FORMAT_BINARY)
    s.offsets = _buckets(case, lengths)
    nb = len(s.offsets) - 1
    s.bits = torch.zeros((2 if ternary else 1) * W, nw, dtype=torch.int64, device=DEV)
    s.counts = torch.zeros((2 if ternary else 1) * n, dtype=torch.uint8, device=DEV)
    s.stats = torch.empty(nb * W * nf.STATS_BYTES, dtype=torch.uint8, device=DEV)
    s.dec = torch.empty(nb * nf.DECISION_BYTES, dtype=torch.uint8, device=DEV)
    if case["api"] == "bucket":
        s.ws = nf.empty_workspace(nf.nf_workspace_bytes(W, n), DEV)
    elif case["api"] == "buckets":
        s.ws = nf.empty_workspace(nf.nf_workspace_bytes_buckets(W, n, BUCKET_N), DEV)
    elif case["api"] == "table":
        s.ws = nf.empty_workspace(nf.nf_workspace_bytes_table(W, s.offsets), DEV)
        s.table = torch.empty(nf.nf_bucket_table_bytes(W, s.offsets), dtype=torch.uint8, device=DEV)
        nf.nf_bucket_table_init(W, s.offsets, s.table)
    d32 = s.dec.view(torch.int32).view(nb, 10)
    s.result = {"out": s.out, "route": d32[:, 0], "reasons": d32[:, 1], "scale": s.dec.view(torch.float32).view(nb, 10)[:, 2],
                "n_eligible": s.dec.view(torch.int64).view(nb, 5)[:, 2],
                "bytes": s.dec.view(torch.float64).view(nb, 5)[:, 3:], **_stats_views(s.stats, nb, W)}
    # what the route writes: payload and counts of the low-bit route (a bucket without an eligible element keeps
    # its counts), the sign words of a binary fallback
    if case["when"] == "ordinary":
        s.result.update(bits=s.bits, counts=s.counts)
    elif case["when"] != "vetoed" and not ternary:
        s.result.update(bits=s.bits)
    return s


def _buckets(case, lengths):
    n = int(lengths.sum())
    if case["api"] == "bucket":
        return np.array([0, n], np.int64)
    if case["api"] == "table":
        return _offsets(lengths)
    return np.array(list(range(0, n, BUCKET_N)) + [n], np.int64)


def _stats_views(stats, nb, W):
    return {"nonfinite": stats.view(torch.int64).view(nb, W, 3)[:, :, 0],
            "sum_abs": stats.view(torch.float64).view(nb, W, 3)[:, :, 1],
            "sum_sq": stats.view(torch.float64).view(nb, W, 3)[:, :, 2]}


def run(s):
    case = s.case
    if case["what"] == "hier":
        nf.nf_partial_counts(s.bits, s.W, case["P"], s.n, s.partial)
        nf.nf_partial_count_reduce(s.partial, s.W, s.n, s.mask, s.scale, s.mode, s.counts, s.out)
    elif case["what"] == "sliced":
        nf.nf_pack_signs(s.grads, s.n, s.lay.d_mask, s.bits, s.stats, s.ws)
        nf.nf_compact_signs(s.bits, s.W, s.n, s.lay, s.cbits)
        nf.nf_slice_scales_from_pass1(s.grads, s.n, s.lay, s.sums, s.scales, s.ws)
        nf.nf_compact_signcount_reduce(s.cbits, s.W, s.lay, s.scales, s.mode, s.counts, s.out)
        nf.nf_fp32_reduce(s.grads, s.n, s.lay.d_mask, nf.NF_SEL_ROUTED, nf.NF_FP32_SUM, s.out)
    elif case["api"] == "bucket":
        nf.nf_route_bucket(s.grads, s.n, s.mask, s.pol, s.bits, s.counts, s.out, s.stats, s.dec, s.ws)
    elif case["api"] == "buckets":
        nf.nf_route_buckets(s.grads, s.n, BUCKET_N, s.mask, s.pol, s.bits, s.counts, s.out, s.stats, s.dec, s.ws)
    elif case["api"] == "noalloc":
        nf.nf_route_buckets_noalloc(s.grads, s.n, BUCKET_N, s.mask, s.pol, s.bits, s.counts, s.out, s.stats, s.dec)
    else:
        nf.nf_route_bucket_table(s.grads, s.offsets, s.table, s.mask, s.pol, s.bits, s.counts, s.out, s.stats, s.dec,
                                 s.ws)
    return s.result


def work(case):
    W, (lengths, eligible) = case["W"], _tensors(case)
    n, ne, nw = int(lengths.sum()), int(lengths[eligible.astype(bool)].sum()), _words(int(lengths.sum()))
    if case["what"] == "hier":
        # sign words and mask in; partial counts, counts and decoded values out
        return {"bytes": 8 * W * nw + 8 * nw + (W // case["P"]) * n + n + 4 * ne, "flops": W * n}
    # gradients and mask in; a comparison, |g| and g*g with their sums, per element and worker
    read, flops = 4 * W * n + 8 * nw, 5 * W * n
    if case["what"] == "sliced":
        return {"bytes": read + 8 * W * nw + 8 * W * _words(ne) + ne + 4 * n, "flops": flops}
    if case["when"] == "vetoed":
        return {"bytes": read + 4 * n, "flops": flops}
    planes = 2 if case["format"] == "ternary" else 1
    if case["when"] != "ordinary":
        return {"bytes": read + (8 * W * nw if planes == 1 else 0) + 4 * n, "flops": flops}
    return {"bytes": read + planes * 8 * W * nw + planes * n + 4 * n, "flops": flops}


def tolerance(case):
    # Whole numbers (signs, counts, routes) are the same.  Against 64 bits, FP32 sums over the workers, decoded
    # values and scales are 1e-7 off in the 2-norm (2e-7 at 64 workers, 3e-7 at 255); a sum that cancels, by more.
    return {"rel": 6e-7 if case["W"] <= 64 else 1e-6, "max": 1e-5}


# ----------------------------------------------------------- 64-bit reference

def _unpacked(words, n):
    """bool [n] of little-endian 64-bit words."""
    b = words.view(torch.uint8).unsqueeze(1) >> torch.arange(8, dtype=torch.uint8, device=DEV)
    return (b & 1).bool().reshape(-1)[:n]


def _packed(x):
    x = torch.nn.functional.pad(x.to(torch.uint8), (0, -len(x) % 64)).view(-1, 8)
    word = x[:, 0].clone()
    for k in range(1, 8):
        word |= x[:, k] << k
    return word.view(torch.int64)


def _decoded(vote, W, scale, mode):
    """Decoded values of vote margins in [-W, W]."""
    return scale * (torch.sign(vote) if mode == nf.NF_DECODE_MAJORITY else vote / W)


def exact(case, seed):
    if 4 * case["W"] * _total(case) > 50e9:
        return None
    s = prepare(case, seed)
    W, n = s.W, s.n
    lengths, eligible = _tensors(case)
    starts = np.cumsum(lengths) - lengths
    mask = torch.repeat_interleave(torch.from_numpy(eligible).to(DEV), torch.from_numpy(lengths).to(DEV)).bool()
    if case["what"] == "hier":
        P = case["P"]
        partial = torch.stack([sum(_unpacked(s.bits[w], n).to(torch.uint8) for w in range(g, g + P))
                               for g in range(0, W, P)])
        counts = partial.sum(0)
        out = _decoded(2.0 * counts - W, W, s.scale.double(), s.mode)
        return {"partial": partial, "counts": counts.to(torch.uint8), "out": torch.where(mask, out, 0.0)}
    sums = torch.zeros(n, dtype=torch.float64, device=DEV)
    counts = torch.zeros(n, dtype=torch.uint8, device=DEV)
    bits = []
    if case["what"] == "sliced":
        edges = torch.from_numpy(np.append(starts, n))
        e = eligible.astype(bool)
        stat = {"nonfinite": [], "sum_abs": [], "sum_sq": []}
        slices = []
        for w in range(W):
            x = s.grads[w, :n].double()
            sums += x
            up = (x > 0) & mask
            counts += up
            bits.append(up)
            a = x.abs()
            per = torch.stack([a[i:j].sum() for i, j in zip(edges[:-1].tolist(), edges[1:].tolist())])[torch.from_numpy(e).to(DEV)]
            slices.append(per)
            stat["nonfinite"].append((~torch.isfinite(x)).sum())
            stat["sum_abs"].append(per.sum())
            stat["sum_sq"].append(x.square().sum())
        slices = torch.stack(slices, 1)
        length = torch.from_numpy(lengths[e]).to(DEV)
        scales = (slices / length[:, None]).mean(1)
        out = _decoded(2.0 * counts[mask] - W, W, torch.repeat_interleave(scales, length), s.mode)
        sums[mask] = out
        return {"bits": torch.stack([_packed(b) for b in bits]), "cbits": torch.stack([_packed(b[mask]) for b in bits]),
                "sums": slices, "scales": scales, "counts": counts[mask], "out": sums,
                **{k: torch.stack(v).view(1, W) for k, v in stat.items()}}
    spans = list(zip(s.offsets[:-1].tolist(), s.offsets[1:].tolist()))
    ne = torch.stack([mask[a:b].sum() for a, b in spans])
    stat = {"nonfinite": [], "sum_abs": [], "sum_sq": []}
    down = torch.zeros(n, dtype=torch.uint8, device=DEV)
    ternary = case["format"] == "ternary"
    low = []  # negative planes
    for w in range(W):
        x = s.grads[w, :n].double()
        sums += x
        a = torch.where(mask, x.abs(), 0.0)
        stat["nonfinite"].append(torch.stack([(~torch.isfinite(x[i:j])).sum() for i, j in spans]))
        stat["sum_abs"].append(torch.stack([a[i:j].sum() for i, j in spans]))
        stat["sum_sq"].append(torch.stack([x[i:j].square().sum() for i, j in spans]))
        if ternary:  # the gate, at the FP32 threshold that its definition rounds to
            theta = 0.5 * (stat["sum_abs"][-1] / ne).float()
            keep = mask & (s.grads[w, :n].abs() >= torch.repeat_interleave(theta, torch.tensor([j - i for i, j in spans], device=DEV)))
            up, dn = keep & (x > 0), keep & (x < 0)
            down += dn
            low.append(_packed(dn))
        else:
            up = mask & (x > 0)
        counts += up
        bits.append(_packed(up))
    stat = {k: torch.stack(v, 1) for k, v in stat.items()}
    scale = torch.where(ne > 0, (stat["sum_abs"] / ne[:, None]).mean(1), 0.0)
    if case["mean"]:
        sums /= W
    if case["when"] == "ordinary":
        vote = counts.double() - down if ternary else 2.0 * counts - W
        per = torch.repeat_interleave(scale, torch.tensor([j - i for i, j in spans], device=DEV))
        sums = torch.where(mask, _decoded(vote, W, per, s.mode), sums)
    want = {"out": sums, "scale": scale, "n_eligible": ne, "route": None, "reasons": None, "bytes": None, **stat}
    if "bits" in s.result:
        want["bits"] = torch.stack(bits + low)
    if "counts" in s.result:
        vote = [counts, down] if ternary else [counts]
        want["counts"] = torch.cat(vote)
    return want
