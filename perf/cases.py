"""Timing cases of the sharded AdamW commit and the state digests.

Each case is one call, or one short sequence of calls, that a training rank
makes through the package's public entry points on its own shard:

* ``commit``        the commit after an optimizer step (binary32 state, bf16 copy)
* ``commit_zero``   the commit that also zeroes the gradient
* ``commit_static`` the commit that takes no workspace (capture, no allocation)
* ``boundary``      the committed boundary of in-memory recovery: the commit that
                    zeroes the gradient, the gradient guard, the state digest
* ``digest``        the state digest alone (cross-rank state check)
* ``copy_digest``   the digest of the bf16 working copy
* ``guard``         the gradient guard alone
* ``bf16_commit``   the commit on state held in BF16
* ``bf16_digest``   the state digest of BF16 state
* ``bf16_boundary`` the BF16 commit followed by the BF16 state digest

A shard is laid out in one of three ways:

* ``flat``    one segment, the whole shard
* ``layers``  one segment per tensor of a decoder, each padded to 128 elements
* ``slice``   rank ``rank`` of ``world`` equal parts of the decoder's tensors laid
              end to end without padding: segments start at any element and the
              first and last one are cut

The arrays are separate torch allocations, as a program that keeps its own
optimizer state has them.
"""
from __future__ import annotations

import math

import torch

import paper_2609_18178_amd as pk

PAD = 128  # elements a tensor is padded to in the ``layers`` layout

# bytes per element that one pass has to move: each input read once, each output written once
BYTES = {
    "commit": 30, "commit_zero": 34, "commit_static": 30, "boundary": 34 + 4 + 12, "digest": 12, "copy_digest": 2,
    "guard": 4, "bf16_commit": 14, "bf16_digest": 6, "bf16_boundary": 14 + 6,
}
# arithmetic per element: the update is 14 binary32 operations, a digest word 9 operations on 64 bits
UPDATE, WORD = 14, 9
FLOPS = {
    "commit": UPDATE + 3 * WORD, "commit_zero": UPDATE + 3 * WORD, "commit_static": UPDATE + 3 * WORD,
    "boundary": UPDATE + 6 * WORD + 1, "digest": 3 * WORD, "copy_digest": WORD, "guard": 1,
    "bf16_commit": UPDATE + 3 * WORD, "bf16_digest": 3 * WORD, "bf16_boundary": UPDATE + 6 * WORD,
}
OPS = tuple(BYTES)

HYPERS = (
    dict(lr=3e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1),    # matrices, and flat shards
    dict(lr=1.5e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1),  # embedding
    dict(lr=1.5e-4, beta1=0.9, beta2=0.99, eps=1e-8, weight_decay=0.1),  # output head
    dict(lr=3e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.0),    # norms
)


def listed():
    return [
        # the smallest real shard: a few workgroups and a ragged tail, all latency
        dict(name="commit_100k_odd", op="commit", layout="flat", numel=100_003, offset=15 * 100_003, step=5),
        # a small shard at its first step (moments zero): fits the on-chip cache, launches count
        dict(name="commit_1m_first", op="commit", layout="flat", numel=1 << 20, offset=0, step=1),
        # a 1.2B decoder over 16 ranks
        dict(name="commit_76m", op="commit", layout="flat", numel=76_000_000, offset=15 * 76_000_000, step=100),
        # a 7B decoder over 16 ranks: the headline shard
        dict(name="commit_453m", op="commit", layout="flat", numel=453_001_472, offset=15 * 453_001_472, step=5),
        # a whole 32-layer decoder on one rank, a segment per tensor, four sets of hyperparameters
        dict(name="commit_layers_143m", op="commit", layout="layers", layers=32, hidden=512, intermediate=1792, kv=128,
             vocab=32768, step=5),
        # one rank's part of a flat vector without padding, gradients zeroed in the same pass
        dict(name="zero_slice_20m", op="commit_zero", layout="slice", layers=24, hidden=1000, intermediate=2750, kv=250,
             vocab=32003, rank=7, world=16, step=40),
        # a two-layer decoder with the entry point that allocates nothing
        dict(name="static_layers_1m", op="commit_static", layout="layers", layers=2, hidden=200, intermediate=520, kv=40,
             vocab=1003, step=9),
        # the committed boundary of one rank in the recovery protocol's own rehearsal
        dict(name="boundary_1m_odd", op="boundary", layout="flat", numel=1_000_003, offset=3 * 1_000_003, step=3),
        # cross-rank state check of the headline shard
        dict(name="digest_453m", op="digest", layout="flat", numel=453_001_472, offset=7 * 453_001_472, step=5),
        # check of the working copy of the 1.2B decoder's shard
        dict(name="copy_digest_76m", op="copy_digest", layout="flat", numel=76_000_000, offset=3 * 76_000_000, step=5),
        # the headline shard with weights and moments in BF16
        dict(name="bf16_commit_453m", op="bf16_commit", layout="flat", numel=453_001_472, offset=15 * 453_001_472, step=5),
        # commit and state check of one rank's unpadded part in BF16
        dict(name="bf16_boundary_slice_20m", op="bf16_boundary", layout="slice", layers=24, hidden=1000, intermediate=2750,
             kv=250, vocab=32003, rank=9, world=16, step=40),
    ]


COST = 30 * 453_001_472  # bytes of the largest listed case


def draw(rng):
    while True:
        op = rng.choice(OPS)
        layout = rng.choice(("flat", "layers", "slice"))
        case = dict(op=op, layout=layout, step=rng.choice((1, 2, 5, 18, 100, 1000)))
        most = COST // BYTES[op] if op not in ("digest", "copy_digest", "guard", "bf16_digest") else 453_001_472
        size = int(math.exp(rng.uniform(math.log(20_000), math.log(min(most, 453_001_472)))))
        if layout == "flat":
            # whole vectors, and sizes with any remainder
            numel = size if rng.random() < 0.6 else max(4096, size // 4096 * 4096)
            case.update(numel=numel, offset=rng.randrange(16) * numel)
            return case
        world = rng.choice((2, 3, 4, 8, 16)) if layout == "slice" else 1
        layers = rng.randint(1, 32)
        # a hidden size that brings the shard near `size`: about 12 hidden^2 a layer and 16 hidden^2 in the embeddings
        hidden = max(16, min(4096, int(math.sqrt(size * world / (12 * layers + 16)))))
        if rng.random() < 0.6:
            hidden = max(16, hidden // 8 * 8)
        case.update(layers=layers, hidden=hidden, intermediate=hidden * rng.randint(22, 36) // 10,
                    kv=max(1, hidden // rng.choice((1, 2, 4, 5, 8))), vocab=min(65536, max(500, 8 * hidden + rng.randint(-9, 9))))
        if layout == "slice":
            case.update(rank=rng.randrange(world), world=world)
        numel = _shape(case)[0]
        # (the entry point without a workspace takes at most 512 segments: 32 layers have 291)
        if 4096 <= numel <= 453_001_472 and numel * BYTES[op] <= COST:
            return case


def _tensors(case):
    """(numel, hyperparameter index) of a decoder's tensors in order."""
    h, inter, kv, vocab = case["hidden"], case["intermediate"], case["kv"], case["vocab"]
    out = [(vocab * h, 1)]
    for _ in range(case["layers"]):
        out += [(h * h, 0), (kv * h, 0), (kv * h, 0), (h * h, 0), (inter * h, 0), (inter * h, 0), (h * inter, 0), (h, 3),
                (h, 3)]
    return out + [(h, 3), (vocab * h, 2)]


def _shape(case):
    """(elements of the shard, flat index of its first, segment table or None)."""
    if case["layout"] == "flat":
        return case["numel"], case["offset"], None
    segs, off = [], 0
    if case["layout"] == "layers":
        for n, hi in _tensors(case):
            segs.append((off, n, hi))
            off += (n + PAD - 1) // PAD * PAD
        return off, 0, segs
    tensors = _tensors(case)
    total = sum(n for n, _ in tensors)
    part = -(-total // case["world"])
    first = case["rank"] * part
    last = min(total, first + part)
    for n, hi in tensors:
        lo, hi_end = max(off, first), min(off + n, last)
        if lo < hi_end:
            segs.append((lo - first, hi_end - lo, hi))
        off += n
    return last - first, first, segs


def _is_bf16(case):
    return case["op"].startswith("bf16_")


def _arrays(case, seed):
    """Weights, gradient and moments as a training run has them; zero moments at the first step."""
    n, offset, segs = _shape(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(sigma):
        return torch.empty(n, dtype=torch.float32, device="cuda").normal_(0.0, sigma, generator=gen)

    p, g = normal(0.02), normal(1e-3)
    if case["step"] == 1:
        m, v = torch.zeros_like(p), torch.zeros_like(p)
    else:
        m, v = normal(1e-4), normal(1e-7).abs_()
    if _is_bf16(case):
        p, g, m, v = (x.to(torch.bfloat16) for x in (p, g, m, v))
    return p, g, m, v, offset, segs


def prepare(case, seed):
    p, g, m, v, offset, segs = _arrays(case, seed)
    hypers = None if segs is None else [pk.Hyper(**h) for h in HYPERS]
    if _is_bf16(case):
        shard = pk.ShardBf16(p, g, m, v, offset, segments=segs, hypers=hypers)
    else:
        shard = pk.Shard(p, g, m, v, p.to(torch.bfloat16), offset, segments=segs, hypers=hypers)
    return {"op": case["op"], "shard": shard, "hyper": pk.Hyper(**HYPERS[0]) if segs is None else None, "step": case["step"]}


def run(state):
    op, shard, hyper, step = state["op"], state["shard"], state["hyper"], state["step"]
    if op == "digest":
        return {"digest": pk.shard_digest(shard)}
    if op == "copy_digest":
        return {"digest": pk.bf16_digest(shard)}
    if op == "guard":
        return {"count": pk.grad_guard(shard)}
    if op == "bf16_digest":
        return {"digest": pk.shard_digest_bf16(shard)}
    state["step"] = step + 1  # each commit is the next optimizer step
    if op.startswith("bf16_"):
        out = {"digest": pk.adamw_commit_bf16(shard, step, hyper)}
        if op == "bf16_boundary":
            out["check"] = pk.shard_digest_bf16(shard)
    elif op == "commit_static":
        out = {"digest": pk.adamw_commit_static(shard, step, hyper)}
    else:
        out = {"digest": pk.adamw_commit(shard, step, hyper, zero_grad=op in ("commit_zero", "boundary"))}
        if op == "boundary":
            out["count"] = pk.grad_guard(shard)
            out["check"] = pk.shard_digest(shard)
        if op in ("commit_zero", "boundary"):
            out["grad"] = shard.grad
    out.update(param=shard.param, exp_avg=shard.exp_avg, exp_avg_sq=shard.exp_avg_sq)
    if not op.startswith("bf16_"):
        out["copy"] = shard.param_bf16
    return out


def work(case):
    segs = _shape(case)[2]
    n = _shape(case)[0] if segs is None else sum(length for _, length, _ in segs)
    return {"bytes": BYTES[case["op"]] * n, "flops": FLOPS[case["op"]] * n}


def tolerance(case):
    # one IEEE rounding per operation in a fixed order, and a digest of the resulting bits: ranks compare state bit for bit
    return "exact"


# --------------------------------------------------------------------------
# the same in plain torch and 64 bits
# --------------------------------------------------------------------------
CHUNK = 1 << 24


def _shift(z, s):
    return (z >> s) & ((1 << (64 - s)) - 1)


def _i64(x):
    return x - (1 << 64) if x >> 63 else x


def _hash_sum(words, first, tag):
    """Wrapping sum of splitmix64(word ^ (index | tag << 56)) over int64 words."""
    index = torch.arange(first, first + words.numel(), dtype=torch.int64, device=words.device)
    z = (words ^ (index | (tag << 56))) + _i64(0x9E3779B97F4A7C15)
    z = (z ^ _shift(z, 30)) * _i64(0xBF58476D1CE4E5B9)
    z = (z ^ _shift(z, 27)) * _i64(0x94D049BB133111EB)
    return (z ^ _shift(z, 31)).sum()


def _words(t):
    if t.dtype == torch.float32:
        return t.view(torch.int32).to(torch.int64) & 0xFFFFFFFF
    return t.view(torch.int16).to(torch.int64) & 0xFFFF


def _slots(per, segs):
    """Result slots as a call gives them: one, or one per segment and their sum."""
    return torch.stack(per) if segs is None else torch.stack(per + [torch.stack(per).sum()])


def exact(case, seed):
    p, g, m, v, offset, segs = _arrays(case, seed)
    op, table = case["op"], segs if segs is not None else [(0, p.numel(), 0)]
    if op == "guard":
        return {"count": _slots([(_words(g[o:o + n]) != 0).sum() for o, n, _ in table], segs)}
    if op in ("digest", "bf16_digest", "copy_digest"):
        arrays = [(p.to(torch.bfloat16), 3)] if op == "copy_digest" else [(p, 0), (m, 1), (v, 2)]
        per = []
        for o, n, _ in table:
            total = torch.zeros((), dtype=torch.int64, device=p.device)
            for lo in range(o, o + n, CHUNK):
                hi = min(lo + CHUNK, o + n)
                for x, tag in arrays:
                    total = total + _hash_sum(_words(x[lo:hi]), offset + lo, tag)
            per.append(total)
        return {"digest": _slots(per, segs)}
    out = [x.double() for x in (p, m, v)]  # elements between segments stay as they are
    f32 = lambda x: float(torch.tensor(x, dtype=torch.float32))  # noqa: E731
    t = case["step"]
    for o, n, hi in table:
        lr, b1, b2, eps, wd = (f32(HYPERS[hi][k]) for k in ("lr", "beta1", "beta2", "eps", "weight_decay"))
        for lo in range(o, o + n, CHUNK):
            at = slice(lo, min(lo + CHUNK, o + n))
            pp, gg, mm, vv = out[0][at], g[at].double(), out[1][at], out[2][at]
            mm = b1 * mm + (1 - b1) * gg
            vv = b2 * vv + (1 - b2) * gg * gg
            den = vv.sqrt() / math.sqrt(1 - b2 ** t) + eps
            out[0][at] = pp * (1 - lr * wd) - lr / (1 - b1 ** t) * (mm / den)
            out[1][at], out[2][at] = mm, vv
    want = {"digest": None, "param": out[0], "exp_avg": out[1], "exp_avg_sq": out[2]}
    if op in ("boundary", "bf16_boundary"):
        want["check"] = None
    if op == "boundary":
        want["count"] = torch.zeros(len(table) if segs is None else len(table) + 1, dtype=torch.int64)
    if op in ("commit_zero", "boundary"):
        grad = g.double()
        for o, n, _ in table:
            grad[o:o + n] = 0.0
        want["grad"] = grad
    if not op.startswith("bf16_"):
        # elements between segments keep the copy that prepare() made of the weights
        want["copy"] = out[0]
    return want
