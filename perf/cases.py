"""Performance cases of libsalt: the calls a serving program makes, at the sizes it makes them.

Every case goes through the Python binding of the C ABI (``paper_2608_03579_amd.salt``).
torch owns the activations: it is imported before the binding, so that libsalt
resolves to the HIP runtime torch has loaded and both see one device.  All work
goes to torch's current stream.

A case is a dict of plain values:

``kind``
    ``layer``     the centroid + residual apply of one decoder layer (its seven
                  projections, or q_proj alone) in one call.
    ``one_shot``  ``salt_apply_map``: host maps in, one table applied.
    ``swap``      a decode step that first swaps residuals of new users in.
    ``fuse``      a centroid folded into a layer's base weights.
    ``gram``      Eq. 2's terms of two adapters over every table of a model.
``hidden, kv, ffn``
    the layer's shapes (q, o: hidden x hidden; k, v: hidden x kv; gate, up:
    hidden x ffn; down: ffn x hidden).  q, k and v read one x, and so do gate and
    up, as in a decoder layer.
``batch``
    ``decode``  T users, one token each;  ``zipf``  T tokens of users drawn from a
    truncated Zipf(1.1);  ``prefill``  contiguous runs of tokens, one user each.
``residual``
    ``1``, ``2``: that rank;  ``mixed``: 1 or 2 per user;  ``lora``: rank 16 and no
    centroids (plain per-user LoRA);  ``tail``: mixed, and the rare users on
    concatenated adapters of rank r_c + 1 or r_c + 2 without a centroid.
``gamma``     per-user centroid scales from {0.6, 0.8, 1.0}.
``new_batch`` the pass starts from host maps (stage, build, apply); otherwise the
              plan is the one the batch's earlier layers used.
"""
from __future__ import annotations

import math

import numpy as np
import torch  # noqa: F401  (before the binding: one HIP runtime for both)

from paper_2608_03579_amd import salt

LLAMA_3B = dict(hidden=3072, kv=1024, ffn=8192)     # Llama-3.2-3B
LLAMA_8B = dict(hidden=4096, kv=1024, ffn=14336)    # Llama-3.1-8B
STD = 0.02                                          # adapter and base-weight scale


def listed():
    return [
        # one small fp32 projection through the one-shot call: the smallest call there is, all launches and host work
        dict(name="one_shot_f32_256_T64", kind="one_shot", dtype="f32", proj="q", hidden=256, kv=256, ffn=256, T=64,
             batch="zipf", users=16, C=4, r_c=8, residual="2", gamma=False),
        # a handful of interactive users: the layer of a decode step at its lowest latency, new maps each step
        dict(name="decode_3b_T4", kind="layer", dtype="bf16", proj="all", **LLAMA_3B, T=4, batch="decode", users=64,
             C=4, r_c=32, residual="2", gamma=False, new_batch=True),
        # q_proj alone adapted (the common LoRA target), 64 users decoding
        dict(name="decode_qproj_3b_T64", kind="layer", dtype="bf16", proj="q", **LLAMA_3B, T=64, batch="decode",
             users=64, C=4, r_c=32, residual="2", gamma=True, new_batch=True),
        # one layer of a 256-user decode step; its plan is shared with the step's other layers
        dict(name="decode_8b_T256", kind="layer", dtype="bf16", proj="all", **LLAMA_8B, T=256, batch="decode",
             users=1024, C=16, r_c=32, residual="2", gamma=False, new_batch=False),
        # the same step when 32 of its users are new: their residuals come over PCIe first
        dict(name="swap32_decode_8b_T256", kind="swap", dtype="bf16", proj="all", **LLAMA_8B, T=256, batch="decode",
             users=1024, C=16, r_c=32, residual="2", gamma=False, new_batch=True, swaps=32),
        # a skewed multi-tenant batch, ranks 1 and 2
        dict(name="zipf_3b_T512", kind="layer", dtype="bf16", proj="all", **LLAMA_3B, T=512, batch="zipf", users=2000,
             C=8, r_c=64, residual="mixed", gamma=False, new_batch=False),
        # the same users on plain rank-16 LoRAs
        dict(name="lora16_zipf_3b_T512", kind="layer", dtype="bf16", proj="all", **LLAMA_3B, T=512, batch="zipf",
             users=2000, C=0, r_c=0, residual="lora", gamma=False, new_batch=False),
        # the same users, the rare ones on concatenated rank-65/66 adapters
        dict(name="tail_zipf_3b_T512", kind="layer", dtype="bf16", proj="all", **LLAMA_3B, T=512, batch="zipf",
             users=2000, C=8, r_c=64, residual="tail", gamma=False, new_batch=False),
        # a chunk of a mixed prefill with shapes that fill no tile evenly
        dict(name="prefill_ragged_T1531", kind="layer", dtype="bf16", proj="all", hidden=2056, kv=520, ffn=5496,
             T=1531, batch="prefill", users=61, C=6, r_c=48, residual="mixed", gamma=True, new_batch=True),
        # one layer of a full prefill batch: the largest call
        dict(name="prefill_3b_T8192", kind="layer", dtype="bf16", proj="all", **LLAMA_3B, T=8192, batch="prefill",
             users=256, C=8, r_c=64, residual="1", gamma=False, new_batch=False),
        # start-up of a node that serves one domain: a centroid folded into a layer's weights
        dict(name="fuse_3b_r64", kind="fuse", dtype="bf16", proj="all", **LLAMA_3B, C=2, r_c=64),
        # the layer-wise cosine of two rank-16 adapters over a whole model
        dict(name="gram_3b_r16_28_layers", kind="gram", dtype="bf16", proj="all", **LLAMA_3B, layers=28, r1=16, r2=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shapes(rng, most=None):
    model = rng.choice(["3b", "8b", "ragged", "ragged"]) if most is None else "ragged"
    if model == "3b":
        return dict(LLAMA_3B)
    if model == "8b":
        return dict(LLAMA_8B)
    hidden = 8 * _log_int(rng, 32, (most or 4096) // 8)
    return dict(hidden=hidden, kv=max(8, hidden // rng.choice([1, 3, 4, 8]) // 8 * 8),
                ffn=max(8, int(hidden * rng.uniform(1.5, 3.5)) // 8 * 8))


def draw(rng):
    most = max(work(c)["bytes"] for c in listed() if c["name"] == "prefill_3b_T8192")
    while True:
        kind = rng.choice(["layer"] * 8 + ["one_shot", "swap", "fuse", "gram"])
        if kind == "gram":
            c = dict(kind=kind, dtype=rng.choice(["bf16"] * 5 + ["f32"]), proj="all", **_draw_shapes(rng),
                     layers=_log_int(rng, 2, 32), r1=rng.choice([1, 2, 8, 16, 17, 32, 65]),
                     r2=rng.choice([1, 2, 16, 32, 64]))
        elif kind == "fuse":
            c = dict(kind=kind, dtype=rng.choice(["bf16"] * 5 + ["f32"]), proj="all", **_draw_shapes(rng), C=2,
                     r_c=8 * rng.randint(1, 16))
        else:
            f32 = kind != "swap" and rng.random() < 0.15
            c = dict(kind=kind, dtype="f32" if f32 else "bf16",
                     proj="q" if kind == "one_shot" or rng.random() < 0.15 else "all",
                     **_draw_shapes(rng, 1024 if f32 else None))
            batch = "decode" if kind == "swap" else rng.choice(["decode", "zipf", "zipf", "prefill", "prefill"])
            T = _log_int(rng, 1, 512) if f32 or batch != "prefill" else _log_int(rng, 64, 8192)
            users = {"decode": T + rng.randint(0, 256), "zipf": _log_int(rng, 4, 2000),
                     "prefill": max(1, min(T, 256, T // rng.randint(8, 64)))}[batch]
            residual = rng.choice(["1", "2", "mixed", "mixed"] if batch != "zipf" else ["mixed", "mixed", "lora", "tail"])
            C = 0 if residual == "lora" else rng.randint(1, 16)
            c.update(T=T, batch=batch, users=users, C=C,
                     r_c=0 if C == 0 else rng.choice([8, 16, 16, 24, 32, 32, 40, 64, 64]), residual=residual,
                     gamma=rng.random() < 0.4)
            if kind != "one_shot":
                c["new_batch"] = kind == "swap" or rng.random() < 0.5
            if kind == "swap":
                c["swaps"] = rng.randint(1, max(1, min(64, T)))
        if work(c)["bytes"] <= most:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _shapes(case):
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    if case["proj"] == "q":
        return [(h, h)]
    return [(h, h), (h, kv), (h, kv), (h, h), (h, f), (h, f), (f, h)]


def _inputs_of(case):
    """Which activation each table reads: q, k, v one; o; gate, up one; down."""
    return [0] if case["proj"] == "q" else [0, 0, 0, 1, 2, 2, 3]


def _esize(case):
    return 4 if case["dtype"] == "f32" else 2


def _maps(case, seed):
    """(tok_c, tok_u, gamma or None, rank per slot) of the batch; slots are the users, in a random order."""
    rng = np.random.default_rng([2608, 3579, int(seed)])
    T, n, C, kind = case["T"], case["users"], case["C"], case["residual"]
    if case["batch"] == "decode":
        user = rng.choice(n, size=T, replace=False)
    elif case["batch"] == "zipf":
        p = np.arange(1, n + 1, dtype=np.float64) ** -1.1
        user = rng.choice(n, size=T, p=p / p.sum())
    else:
        length = rng.integers(1, 513, size=n).astype(np.float64)
        edge = np.round(np.cumsum(length) * T / length.sum()).astype(np.int64)
        user = np.searchsorted(edge, np.arange(T), side="right").clip(0, n - 1)
    rank = {"1": np.full(n, 1), "2": np.full(n, 2), "lora": np.full(n, 16)}.get(kind)
    if rank is None:
        rank = rng.integers(1, 3, size=n)
    cent = rng.integers(0, C, size=n) if C else np.full(n, -1)
    if kind == "tail":
        rare = np.arange(n) >= min(100, (n + 1) // 2)
        rank = np.where(rare, case["r_c"] + rank, rank)
        cent = np.where(rare, -1, cent)
    g = np.asarray([0.6, 0.8, 1.0], np.float32)[rng.integers(0, 3, size=n)]
    # the pool holds the users that the batch references, and up to 1024 others
    seen = np.unique(user)
    n_slots = len(seen) if kind == "tail" else min(n, max(len(seen), 1024))
    slot_of = np.full(n, -1)
    slot_of[seen] = rng.permutation(n_slots)[: len(seen)]
    slot_rank = np.zeros(n_slots, np.int32)
    slot_rank[slot_of[seen]] = rank[seen]
    return (cent[user].astype(np.int32), slot_of[user].astype(np.int32), g[user] if case["gamma"] else None, slot_rank)


class _Values:
    """The numbers of a case, drawn on the GPU from the seed: activations N(0, 1), adapters and weights N(0, 0.02^2)."""

    def __init__(self, case, seed):
        self.case = case
        self.seed = int(seed)
        self.dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16

    def _normal(self, key, shape, std=1.0):
        g = torch.Generator(device="cuda")
        g.manual_seed((self.seed * 1000003 + key * 7919 + 17) % (1 << 62))
        return (torch.randn(shape, generator=g, device="cuda") * std).to(self.dtype)

    def x(self, i, width):
        return self._normal(100 + i, (self.case["T"], width))

    def y0(self, t, width):
        return self._normal(200 + t, (self.case["T"], width))

    def centroids(self, t, shape):
        C, r = self.case["C"], self.case["r_c"]
        return self._normal(300 + t, (C, r, shape[0]), STD), self._normal(400 + t, (C, r, shape[1]), STD)

    def blobs(self, elems, generation=0):
        return self._normal(500 + generation, (elems,), STD)

    def weight(self, t, shape):
        return self._normal(600 + t, shape, STD)


def _host(a):
    """A device tensor as a numpy array of its bits."""
    a = a.cpu()
    return a.numpy() if a.dtype == torch.float32 else a.view(torch.uint16).numpy()


def _pinned(buf, a):
    """Copy a device tensor of adapter elements into page-locked memory."""
    torch.from_numpy(buf.view(np.float32 if a.dtype == torch.float32 else np.uint16))[: a.numel()].copy_(
        a if a.dtype == torch.float32 else a.view(torch.uint16))


def _load_slots(ctx, slots, ranks, blob_of, per_rank, esize, keep=None):
    """Swap the blobs of `slots` in, 32 at a time, through one page-locked buffer (or `keep`)."""
    step = len(slots) if keep is not None else 32
    for i in range(0, len(slots), step):
        part = slots[i: i + step]
        sizes = [int(ranks[s]) * per_rank * esize for s in part]
        offs = np.concatenate([[0], np.cumsum(sizes)])
        buf = keep if keep is not None else salt.HostBuffer(int(offs[-1]))
        lo, hi = blob_of(part[0])[0], blob_of(part[-1])[1]
        _pinned(buf, blob_of(None)[lo:hi])
        args = ([int(s) for s in part], [int(ranks[s]) for s in part], [buf.ptr + int(o) for o in offs[:-1]], sizes)
        if keep is not None:
            return args
        st = ctx.load_residuals_ptr(*args)
        if st != salt.OK:
            raise salt.SaltError(st, "load_residuals")
        ctx.wait_loads()


def _blob_layout(slots, slot_rank, per_rank):
    """Where each slot's blob lies in one long draw, in the order of `slots`."""
    off, at = {}, 0
    for s in slots:
        n = int(slot_rank[s]) * per_rank
        off[int(s)] = (at, at + n)
        at += n
    return off, at


def _swapped(case, tok_u, seed):
    rng = np.random.default_rng([2608, 3580, int(seed)])
    return [int(s) for s in np.sort(rng.choice(np.unique(tok_u), size=case["swaps"], replace=False))]


# ---------------------------------------------------------------------------
# the five functions
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind, shapes, v, es = case["kind"], _shapes(case), _Values(case, seed), _esize(case)
    s = dict(kind=kind, stream=torch.cuda.current_stream().cuda_stream)
    if kind == "gram":
        shapes = shapes * case["layers"]
        per_rank = sum(i + o for i, o in shapes)
        s["blobs"] = [v.blobs(case["r1"] * per_rank), v.blobs(case["r2"] * per_rank, 1)]
        s["ranks"] = case["r1"], case["r2"]
        s["ctx"] = salt.Context(case["dtype"], shapes, 0, 0, 1, 0, 1)
        return s
    if kind == "fuse":
        s["ctx"] = ctx = salt.Context(case["dtype"], shapes, case["C"], case["r_c"], 1, 0, 1)
        for t, sh in enumerate(shapes):
            ctx.pin_centroids(t, *(_host(a) for a in v.centroids(t, sh)))
        s["w"] = [v.weight(t, sh) for t, sh in enumerate(shapes)]
        return s
    tok_c, tok_u, gamma, slot_rank = _maps(case, seed)
    s["ctx"] = ctx = salt.Context(case["dtype"], shapes, case["C"], case["r_c"], len(slot_rank), int(slot_rank.max()),
                                  case["T"])
    if case["C"]:
        for t, sh in enumerate(shapes):
            ctx.pin_centroids(t, *(_host(a) for a in v.centroids(t, sh)))
    per_rank = sum(i + o for i, o in shapes)
    slots = [int(u) for u in np.unique(tok_u)]
    off, total = _blob_layout(slots, slot_rank, per_rank)
    draw_ = v.blobs(total)
    _load_slots(ctx, slots, slot_rank, lambda u: draw_ if u is None else off[u], per_rank, es)
    if kind == "swap":
        new = _swapped(case, tok_u, seed)
        noff, ntotal = _blob_layout(new, slot_rank, per_rank)
        fresh = v.blobs(ntotal, 1)
        s["host"] = salt.HostBuffer(ntotal * es)
        s["swap"] = _load_slots(ctx, new, slot_rank, lambda u: fresh if u is None else noff[u], per_rank, es, s["host"])
    ins = _inputs_of(case)
    width = {i: sh[0] for i, sh in zip(ins, shapes)}
    xs = {i: v.x(i, w) for i, w in width.items()}
    s["x"] = [xs[i] for i in ins]
    s["y"] = [v.y0(t, sh[1]) for t, sh in enumerate(shapes)]
    s["tables"] = list(range(len(shapes)))
    s["maps"] = tok_c, tok_u, gamma
    if kind != "one_shot":
        s["new_batch"] = case["new_batch"]
        s["plan"] = ctx.plan()
        s["plan"].set_maps(tok_c, tok_u, gamma, s["stream"])
        s["plan"].build(s["stream"])
    return s


def run(state):
    s, ctx, stream = state, state["ctx"], state["stream"]
    if s["kind"] == "gram":
        a, b = s["blobs"]
        return ctx.adapter_gram(a.data_ptr(), s["ranks"][0], b.data_ptr(), s["ranks"][1], stream)
    if s["kind"] == "fuse":
        for t, w in enumerate(s["w"]):
            ctx.fuse_centroid(t, 1, 0.8, w.data_ptr(), w.shape[1], stream)
        return s["w"]
    if s["kind"] == "one_shot":
        ctx.apply_map(0, *s["maps"], s["x"][0].data_ptr(), s["y"][0].data_ptr(), stream)
        return s["y"]
    if s["kind"] == "swap":
        st = ctx.load_residuals_ptr(*s["swap"])
        if st != salt.OK:
            raise salt.SaltError(st, "load_residuals")
    if s["new_batch"]:
        s["plan"].set_maps(*s["maps"], stream)
        s["plan"].build(stream)
    ctx.apply_batch(s["tables"], s["plan"], [x.data_ptr() for x in s["x"]], [y.data_ptr() for y in s["y"]], stream)
    return s["y"]


def work(case):
    shapes, es = _shapes(case), _esize(case)
    if case["kind"] == "gram":
        per_rank = sum(i + o for i, o in shapes) * case["layers"]
        r1, r2 = case["r1"], case["r2"]
        return dict(bytes=es * per_rank * (r1 + r2) + 24 * len(shapes) * case["layers"],
                    flops=2 * per_rank * (r1 * r2 + r1 * r1 + r2 * r2))
    if case["kind"] == "fuse":
        return dict(bytes=sum(es * (2 * i * o + case["r_c"] * (i + o)) for i, o in shapes),
                    flops=sum(2 * i * o * case["r_c"] for i, o in shapes))
    # the batch of seed 0 stands for those of the other seeds
    tok_c, tok_u, _, slot_rank = _maps(case, 0)
    T = case["T"]
    ranks = int(slot_rank[np.unique(tok_u)].sum()) + case["r_c"] * len(np.unique(tok_c[tok_c >= 0]))
    n_in = sum({i: sh[0] for i, sh in zip(_inputs_of(case), shapes)}.values())
    n_out = sum(o for _, o in shapes)
    per_rank = sum(i + o for i, o in shapes)
    per_tok = slot_rank[tok_u].astype(np.int64) + np.where(tok_c >= 0, case["r_c"], 0)
    b = es * (T * (n_in + 2 * n_out) + ranks * per_rank) + 12 * T
    if case["kind"] == "swap":      # the new users' blobs, from host memory into the pool
        b += 2 * es * per_rank * int(slot_rank[_swapped(case, tok_u, 0)].sum())
    return dict(bytes=b, flops=2 * int(per_tok.sum()) * per_rank)


def tolerance(case):
    # measured against exact(): 4e-8 (fp32 y) and 7e-8 (Gram terms, fp32 sums); longer sums at the ends of the ranges
    if case["kind"] == "gram" or case["dtype"] == "f32":
        return dict(rel=1e-6, max=1e-5)
    # bf16 y and weights: one rounding, 1.7e-3 against exact(), times four
    return dict(rel=7e-3, max=2e-2)


def exact(case, seed):
    kind, shapes, v = case["kind"], _shapes(case), _Values(case, seed)
    if kind == "gram":
        shapes = shapes * case["layers"]
        per_rank = sum(i + o for i, o in shapes)
        r1, r2 = case["r1"], case["r2"]
        one, two = v.blobs(r1 * per_rank), v.blobs(r2 * per_rank, 1)
        out, at = [], 0

        def factors(blob, r, i, o):
            b = blob[r * at: r * (at + i + o)].double()
            return b[: r * i].view(r, i), b[r * i:].view(r, o)

        for i, o in shapes:
            a1, b1 = factors(one, r1, i, o)
            a2, b2 = factors(two, r2, i, o)
            out.append(torch.stack([((a1 @ a2.T) * (b1 @ b2.T)).sum(), ((a1 @ a1.T) * (b1 @ b1.T)).sum(),
                                    ((a2 @ a2.T) * (b2 @ b2.T)).sum()]))
            at += i + o
        return torch.stack(out)
    if kind == "fuse":
        res = []
        for t, sh in enumerate(shapes):
            at, b = v.centroids(t, sh)
            g = float(np.float32(0.8))
            res.append(v.weight(t, sh).double() + g * (at[1].double().T.contiguous() @ b[1].double()))
        return res
    tok_c, tok_u, gamma, slot_rank = _maps(case, seed)
    per_rank = sum(i + o for i, o in shapes)
    slots = [int(u) for u in np.unique(tok_u)]
    off, total = _blob_layout(slots, slot_rank, per_rank)
    blob = v.blobs(total)
    where = {u: (blob, *off[u]) for u in slots}
    if kind == "swap":
        new = _swapped(case, tok_u, seed)
        noff, ntotal = _blob_layout(new, slot_rank, per_rank)
        fresh = v.blobs(ntotal, 1)
        where.update({u: (fresh, *noff[u]) for u in new})
    scale = torch.ones(case["T"], dtype=torch.float64, device="cuda")
    if gamma is not None:
        scale = torch.from_numpy(gamma.astype(np.float64)).cuda()
    rows_c = {c: torch.from_numpy(np.nonzero(tok_c == c)[0]).cuda() for c in np.unique(tok_c) if c >= 0}
    rows_u = {u: torch.from_numpy(np.nonzero(tok_u == u)[0]).cuda() for u in slots}
    ins, res, prefix = _inputs_of(case), [], 0
    for t, (i, o) in enumerate(shapes):
        x = v.x(ins[t], i).double()
        y = v.y0(t, o).double()
        if case["C"]:
            at, b = v.centroids(t, (i, o))
            for c, rows in rows_c.items():
                low = (x[rows] @ at[c].double().T.contiguous()) * scale[rows, None]
                y[rows] += low @ b[c].double()
        for u, rows in rows_u.items():
            r = int(slot_rank[u])
            src, lo, _ = where[u]
            f = src[lo + r * prefix: lo + r * (prefix + i + o)].double()
            y[rows] += (x[rows] @ f[: r * i].view(r, i).T.contiguous()) @ f[r * i:].view(r, o)
        res.append(y)
        prefix += i + o
    return res
