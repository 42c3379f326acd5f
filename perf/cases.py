"""Timing cases of the decode/evict path: what a program that uses this package has it do.

A case is one of five kinds of call:
  decode   gkv_attend_decode: one decode step of all layers that share a context
  cycle    s decode steps and the compression that ends them (gkv_evict), call by call or, with
           "graph", recorded once into a HIP graph and replayed
  score    the compression's scoring half: window score, global score, top-(b - w)
  gkv      the same with the redundancy term, and the eviction log
  compact  gkv_compact: the kept rows of K and V moved to the front, in place

Shapes are the workload configurations in gkv_traces and the head shapes, dtypes and window sizes
the tests cover.  Values follow the trace recipes: keys with outlier channels and a few boosted
positions ("recurring") or Student-t keys ("heavy_tail"), drawn on the GPU.
"""
import math

import torch

from paper_2512_00504_amd.binding import make_config
from paper_2512_00504_amd.state import DecodeState, k_rows_to_cache

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}
LAM, TAU = 0.7, 0.5          # redundancy weight and threshold of the "gkv" cases


def _case(name, kind, L, B, hq, hkv, d, dtype, b, w, s, rows=0, recipe="recurring", **more):
    """rows: cache rows when the call is made (decode: before the step; 0 = the middle of a cycle
    for decode, b + s for the others).  lens = "ragged": decode only, rows is the longest sequence."""
    c = dict(name=name, kind=kind, L=L, B=B, hq=hq, hkv=hkv, d=d, dtype=dtype, b=b, w=w, s=s,
             rows=rows or (b + s // 2 if kind == "decode" else b + s), recipe=recipe, lens="equal", graph=False)
    c.update(more)
    return c


def listed():
    return [
        # the tiny fp32 configuration, call by call: a correctness run or a small experiment
        _case("tiny_f32_cycle", "cycle", 1, 1, 8, 2, 64, "f32", 64, 8, 16),
        # one sequence, one layer at the 7B head shape, its cycle recorded into a graph: latency
        _case("single_cycle_graph", "cycle", 1, 1, 28, 4, 128, "bf16", 512, 16, 128, graph=True),
        # one layer of a layer-at-a-time model at batch 32, budget 2048
        _case("layer_decode_b2048", "decode", 1, 32, 28, 4, 128, "bf16", 2048, 16, 128),
        # a batch whose prompts differ: lengths from a few hundred rows to the largest capacity
        _case("ragged_decode", "decode", 4, 8, 28, 4, 128, "bf16", 3840, 16, 96, rows=3900, lens="ragged"),
        # the headline configuration's decode step, all 28 layers in one launch
        _case("decode_28layer_b512", "decode", 28, 8, 28, 4, 128, "bf16", 512, 16, 128),
        # the large-batch configuration's decode step: 10 GB of cache, heavy-tailed keys
        _case("decode_large_batch", "decode", 36, 64, 40, 8, 128, "bf16", 1024, 32, 64, recipe="heavy_tail"),
        # a medium batch of the 40q/8kv shape through a whole compression cycle
        _case("medium_cycle", "cycle", 4, 8, 40, 8, 128, "bf16", 1024, 32, 64, recipe="heavy_tail"),
        # fp32 caches at the 7B head shape: reference runs of the method
        _case("f32_cycle", "cycle", 2, 4, 28, 4, 128, "f32", 512, 16, 32),
        # bf16 with head_dim 64: the small-model head shape
        _case("d64_cycle", "cycle", 8, 8, 10, 2, 64, "bf16", 512, 32, 32),
        # scoring at budget 1024, batch 16, 28 layers
        _case("score_28layer_b1024", "score", 28, 16, 28, 4, 128, "bf16", 1024, 16, 128),
        # the full method with the redundancy term at the headline configuration
        _case("gkv_28layer_b512", "gkv", 28, 8, 28, 4, 128, "bf16", 512, 16, 128),
        # compaction at budget 2048, batch 16, 28 layers
        _case("compact_28layer_b2048", "compact", 28, 16, 28, 4, 128, "bf16", 2048, 16, 128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "cycle", "cycle", "score", "score", "gkv", "compact", "compact"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "bf16", "f32"])
    d = rng.choice([128, 128, 128, 64])
    hkv = rng.choice([1, 2, 4, 8])
    g = rng.choice([1, 2, 3, 4, 5, 7, 7, 8, 16])
    w = rng.choice([8, 16, 16, 32])
    s = rng.choice([32, 48, 64, 100, 128]) if kind != "cycle" else rng.choice([32, 64])
    b = _log_int(rng, 64, 2048)
    recipe = rng.choice(["recurring", "recurring", "heavy_tail"])
    lens, rows, graph = "equal", 0, False
    plain = dtype == "f32" or d != 128
    if kind == "decode":
        units = _log_int(rng, 4, 2000)
        rows = b + rng.randrange(s)
        lens = rng.choice(["equal", "equal", "ragged"])
        limit = 1 << (28 if plain else 30)
    elif kind == "cycle":
        units = _log_int(rng, 4, 256)
        graph = rng.random() < 0.25
        limit = 1 << (24 if plain else 27)
    elif kind == "gkv":
        units = _log_int(rng, 4, 900)
        b = min(b, 300 if plain else 1100)
        limit = 1 << (22 if plain else 28)
    else:
        units = _log_int(rng, 4, 2000)
        # a prompt longer than the budget meets its first compression with more than b + s rows
        if rng.random() < 0.3:
            rows = rng.randrange(b + s, min(3 * b + s, 3000))
        limit = 1 << (25 if plain and kind == "score" else 29)
    if graph:
        b = max(s, b // s * s)            # a recorded cycle wants step bases that are multiples of s and w
    row_bytes = 2 * d * (4 if dtype == "f32" else 2)
    units = max(hkv, min(units, limit // (row_bytes * (rows or b + s))))
    lb = max(1, units // hkv)
    L = rng.choice([x for x in (1, 1, 2, 4, 14, 28) if x <= lb])
    return {k: v for k, v in _case("", kind, L, max(1, lb // L), g * hkv, hkv, d, dtype, b, w, s, rows, recipe,
                                   lens=lens, graph=graph).items() if k != "name"}


# ---- inputs ---------------------------------------------------------------------------------
def _lens(case):
    B, n = case["B"], case["rows"]
    if case["lens"] == "equal":
        return [n] * B
    return [max(1, n * (i + 1) // B - (i * 7) % 13) for i in range(B)]


class _Inputs:
    """Draws, layer by layer, from one generator: the same values for prepare() and exact()."""

    def __init__(self, case, seed):
        self.c = case
        self.dev = torch.device("cuda")
        self.g = torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)
        L, hkv, d = case["L"], case["hkv"], case["d"]
        u = torch.randn(L, hkv, d, generator=self.g, device=self.dev)
        self.u = u / u.norm(dim=-1, keepdim=True)
        self.scale = torch.ones(L, hkv, d, device=self.dev)
        ch = torch.rand(L, hkv, d, generator=self.g, device=self.dev).topk(4, dim=-1).indices
        self.scale.scatter_(-1, ch, 10.0)
        self.boost = math.sqrt(8.0 * math.sqrt(d))

    def _n(self, *shape):
        return torch.randn(*shape, generator=self.g, device=self.dev)

    def keys(self, layer, *lead):
        """[*lead, hkv, d] keys of one layer, as float32 on the case's dtype grid."""
        shape = (*lead, self.c["hkv"], self.c["d"])
        k = self._n(*shape)
        if self.c["recipe"] == "heavy_tail":
            chi = self._n(*shape).square_()
            chi += self._n(*shape).square_()
            chi += self._n(*shape).square_()
            k /= (chi / 3.0).sqrt_()
        else:
            k *= self.scale[layer]
            hit = torch.rand(*lead, 1, 1, generator=self.g, device=self.dev) < 0.01
            k += hit * (self.boost * self.u[layer])
        return k.to(_DT[self.c["dtype"]])

    def values(self, *lead):
        return self._n(*lead, self.c["hkv"], self.c["d"]).to(_DT[self.c["dtype"]])

    def queries(self, layer, n):
        """[n, B, hq, d]; a recall burst covers a tenth of the steps."""
        c = self.c
        q = self._n(n, c["B"], c["hq"], c["d"])
        if c["recipe"] != "heavy_tail":
            hit = torch.rand(n, 1, 1, 1, generator=self.g, device=self.dev) < 0.1
            q += hit * (self.boost * self.u[layer].repeat_interleave(c["hq"] // c["hkv"], dim=0))
        return q.to(_DT[c["dtype"]])

    def cache(self, layer, rows):
        """K, V [B, hkv, rows, d] of one layer."""
        k = self.keys(layer, self.c["B"], rows).transpose(1, 2).contiguous()
        v = self.values(self.c["B"], rows).transpose(1, 2).contiguous()
        return k, v

    def history(self, rows):
        """Recorded scores: normalised, most of them small."""
        c = self.c
        return torch.rand(c["L"], c["B"], c["hkv"], rows, generator=self.g, device=self.dev).pow_(4)

    def tokens(self, n):
        """q [n, L, B, hq, d], k, v [n, L, B, hkv, d]."""
        c = self.c
        q, k, v = [], [], []
        for layer in range(c["L"]):
            q.append(self.queries(layer, n))
            k.append(self.keys(layer, n, c["B"]))
            v.append(self.values(n, c["B"]))
        return [torch.stack(x, dim=1).contiguous() for x in (q, k, v)]

    def keep(self, n_cand, n_keep):
        """Kept candidates [L, B, hkv, n_keep], ascending."""
        c = self.c
        out = []
        for _ in range(c["L"]):
            r = torch.rand(c["B"], c["hkv"], n_cand, generator=self.g, device=self.dev)
            out.append(r.topk(n_keep, dim=-1).indices.sort(dim=-1).values.int())
        return torch.stack(out)


def _rows0(case):
    """Rows of the cache that are placed before the decode calls of prepare() and run()."""
    kind = case["kind"]
    if kind == "cycle":
        return case["b"]
    if kind in ("score", "gkv"):
        return case["rows"] - case["w"]
    return case["rows"]


def _t0(case):
    """The decode step that follows those rows; a multiple of w and s where a graph asks for one."""
    if case["kind"] == "cycle":
        m = math.lcm(case["w"], case["s"])
        return -(-(case["b"] + case["s"]) // m) * m
    return case["rows"] + 1024


POOL = 4                     # cycles of new tokens that a "cycle" program goes through in turn


class _State:
    pass


def prepare(case, seed):
    c, x, S = case, _Inputs(case, seed), _State()
    L, B, b, w = c["L"], c["B"], c["b"], c["w"]
    cap = -(-max(b + c["s"], c["rows"] + (c["kind"] == "decode")) // 32) * 32
    cfg = make_config(L, B, c["hq"], c["hkv"], c["d"], b, w, c["s"], cap, c["dtype"])
    S.case, S.st = c, DecodeState(cfg)
    st, n, t0 = S.st, _rows0(c), _t0(c)
    tiled = b // 16 * 16 if n >= b // 16 * 16 else 0      # as the last compression left them
    if c["lens"] == "ragged" or c["rows"] > b + c["s"]:
        tiled = 0                                         # prompts: rows as they were placed
    for layer in range(L):
        k, v = x.cache(layer, n)
        st.K[layer, :, :, :n] = k_rows_to_cache(k, tiled)
        st.V[layer, :, :, :n] = v
    del k, v
    n_hist = b - w if tiled else 0
    if n_hist:
        st.F_hist[..., :n_hist] = x.history(n_hist)
    st.pos[..., :n] = torch.arange(t0 - n, t0, dtype=torch.int32, device=x.dev)
    since = 0 if c["kind"] in ("decode", "cycle", "score", "gkv") else w
    rec = [[r - (since or 0), t0 - since, n_hist, tiled] for r in
           (_lens(c) if c["kind"] == "decode" else [n] * B)]
    st.d_state.copy_(torch.tensor(rec, dtype=torch.int32).expand(L, B, 4))
    S.step = t0
    if c["kind"] == "decode":
        q, k, v = x.tokens(1)
        S.q, S.k, S.v = q[0], k[0], v[0]
    elif c["kind"] == "cycle":
        s = c["s"]
        q, k, v = x.tokens(s * (1 if c["graph"] else POOL))
        S.outs = torch.zeros(s, L, B, c["hq"], c["d"], dtype=_DT[c["dtype"]], device=x.dev)
        S.out = S.outs.unbind(0)
        S.q, S.k, S.v = q.unbind(0), k.unbind(0), v.unbind(0)
        S.at = 0
        st.set_state(b, t0, n_hist, tiled)
        if c["graph"]:
            S.base = torch.tensor([t0], dtype=torch.int32, device=x.dev)
            st.ctx.set_step_base(S.base)
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            S.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(S.graph, stream=side):
                for i in range(s):
                    st.ctx.attend_decode(S.q[i], S.k[i], S.v[i], st.K, st.V, st.pos, i, st.qwin, st.d_state, b + i,
                                         S.out[i], st.workspace)
                st.ctx.evict(st.qwin, st.K, st.V, st.F_hist, st.pos, st.d_state, s - 1, b + s, st.S, st.F,
                             st.keep_idx, st.workspace)
                st.ctx.advance_step_base(s)
    elif c["kind"] == "compact":
        S.step = t0 - 1
        st.keep_idx.copy_(x.keep(n - w, b - w))
        st.F.copy_(x.history(st.F.shape[-1]))
    else:                                                 # the window's decode steps
        q, k, v = x.tokens(w)
        for i in range(w):
            st.ctx.attend_decode(q[i], k[i], v[i], st.K, st.V, st.pos, t0 + i, st.qwin, st.d_state, n + i, st.out,
                                 st.workspace)
        S.step = t0 + w - 1
        st.len_host = c["rows"]
    return S


def run(S):
    c, st, t = S.case, S.st, S.step
    if c["kind"] == "decode":
        st.ctx.attend_decode(S.q, S.k, S.v, st.K, st.V, st.pos, t, st.qwin, st.d_state, c["rows"], st.out, st.workspace)
        return {"out": st.out, "pos": st.pos, "qwin": st.qwin}
    if c["kind"] == "cycle":
        if c["graph"]:
            S.graph.replay()
        else:
            for i in range(c["s"]):
                j = S.at + i
                st.out = S.out[i]
                st.attend_decode(S.q[j], S.k[j], S.v[j], t + i)
            st.evict(t + c["s"] - 1)
            S.step = t + c["s"]
            S.at = (S.at + c["s"]) % len(S.q)
        return {"out": S.outs, "S": st.S, "F": st.F, "keep": st.keep_idx, "pos": st.pos, "F_hist": st.F_hist,
                "K": st.K, "V": st.V, "d_state": st.d_state}
    if c["kind"] == "compact":
        # the s rows behind the budget are there again (the decode steps' part), and the next
        # compression comes s steps later
        st.ctx.compact(st.keep_idx, st.F, st.K, st.V, st.F_hist, st.pos, st.d_state, t, st.workspace)
        S.step = t + c["rows"] - c["b"]
        return {"K": st.K, "V": st.V, "pos": st.pos, "F_hist": st.F_hist, "d_state": st.d_state}
    st.score_window(t)
    st.global_update(t)
    if c["kind"] == "score":
        st.select_topk(t)
        return {"S": st.S, "F": st.F, "keep": st.keep_idx}
    st.redundancy_combine(t, LAM, TAU, c["w"])
    st.select_topk(t, on_combined=True)
    st.evicted_positions(t)
    return {"S": st.S, "F": st.F, "R": st.R, "F_sel": st.F_sel, "keep": st.keep_idx, "evicted": st.evicted}


# ---- what a pass cannot do without ----------------------------------------------------------
def _evict_work(c, l, e):
    g, w, b, d = c["hq"] // c["hkv"], c["w"], c["b"], c["d"]
    n_hist = b - w if l <= b + c["s"] else 0
    score = (e * d * (l + g * w) + 4 * (l - w), 2.0 * g * w * d * l)
    update = 4 * (l - w) + 4 * n_hist + 4 * (l - w)
    topk = 4 * (b - w)
    compact = 2 * (2 * e * d + 4) * b + 4 * (b - w) * 3
    return score, update, topk, compact


def work(case):
    c = case
    e, d, g = (4 if c["dtype"] == "f32" else 2), c["d"], c["hq"] // c["hkv"]
    units, lb = c["L"] * c["B"] * c["hkv"], c["L"] * c["hkv"]
    if c["kind"] == "decode":
        rows = sum(n + 1 for n in _lens(c)) * lb
        return {"bytes": e * d * (2 * rows + units * (2 * g + 2)), "flops": 4.0 * g * d * rows}
    l = c["rows"]
    score, update, topk, compact = _evict_work(c, l, e)
    if c["kind"] == "compact":
        return {"bytes": units * compact, "flops": 0}
    if c["kind"] == "cycle":
        rows = sum(range(c["b"] + 1, c["b"] + c["s"] + 1))
        return {"bytes": units * (e * d * (2 * rows + c["s"] * (2 * g + 2)) + score[0] + update + topk + compact),
                "flops": units * (4.0 * g * d * rows + score[1])}
    total = {"bytes": units * (score[0] + update + topk), "flops": units * score[1]}
    if c["kind"] == "gkv":
        # the cosine matrix is symmetric: half of it, and its diagonal is not wanted
        total["bytes"] += units * (e * d * l + 4 * l + 4 * (l - c["w"]) + 4 * (l - c["b"]))
        total["flops"] += units * 1.0 * d * l * (l - 1)
    return total


def tolerance(case):
    """About four times what the path measures against exact(): bf16 outputs 1.7e-3 (their own
    rounding), fp32 scores and outputs up to 1e-6.  An entry of the redundancy score's cosine matrix
    that lies on the threshold falls on either side, which moves one R by a factor e^TAU: seldom a
    head's largest, and then 2e-2 of the norm.  Near-equal scores at the top-(b - w) border swap."""
    if case["kind"] == "compact":
        return "exact"
    if case["kind"] == "gkv":
        return {"rel": 0.03, "max": 0.99, "differ": 0.005}
    if case["kind"] == "score" or case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4, "differ": 0.002}
    return {"rel": 8e-3, "max": 0.1, "differ": 0.002}


# ---- the same in 64 bits --------------------------------------------------------------------
def _attend64(q, K, V, n):
    """q [B, hq, d], K, V [B, hkv, rows, d] (float64), n: rows seen, per sequence [B]."""
    B, hkv, rows, d = K.shape
    z = torch.matmul(q.view(B, hkv, -1, d), K.transpose(2, 3).contiguous()) / math.sqrt(d)
    dead = torch.arange(rows, device=K.device).view(1, 1, 1, -1) >= n.view(-1, 1, 1, 1)
    p = torch.softmax(z.masked_fill(dead, float("-inf")), dim=-1)
    return torch.matmul(p, V).view(B, -1, d)


def _scores64(qw, K, l, hist, n_hist, alpha=0.8):
    """qw [w, B, hq, d], K [B, hkv, l, d]: local and global score of the l - w candidates."""
    w, c = qw.shape[0], l - qw.shape[0]
    B, hkv, _, d = K.shape
    KT = K.transpose(2, 3).contiguous()
    S = torch.zeros(B, hkv, c, dtype=torch.float64, device=K.device)
    for k in range(w):
        z = torch.matmul(qw[k].view(B, hkv, -1, d), KT[..., : c + k + 1].contiguous()) / math.sqrt(d)
        S += torch.softmax(z, dim=-1)[..., :c].amax(dim=2)
    S /= w
    F = S / S.amax(dim=-1, keepdim=True)
    if n_hist:
        F[..., :n_hist] = torch.maximum(alpha * hist[..., :n_hist], F[..., :n_hist])
    return S, F


def _redundancy64(K, F, w):
    l = K.shape[2]
    Kn = K / (K.norm(dim=-1, keepdim=True) + 1e-8)
    lam, tau = (float(torch.tensor(v, dtype=torch.float32)) for v in (LAM, TAU))
    R = torch.zeros(K.shape[:3], dtype=torch.float64, device=K.device)
    for b in range(K.shape[0]):
        C = torch.matmul(Kn[b], Kn[b].transpose(1, 2).contiguous())
        C = C.masked_fill(C < tau, 0.0)
        C.diagonal(dim1=1, dim2=2).zero_()
        R[b] = C.sum(dim=1)
    R[..., l - w:] = 0.0
    R = torch.exp(R - R.amax(dim=-1, keepdim=True))
    return R, lam * F - (1.0 - lam) * R[..., : l - w]


def exact(case, seed):
    c = case
    if c["kind"] == "compact":
        return None
    x = _Inputs(c, seed)
    L, b, w, n = c["L"], c["b"], c["w"], _rows0(c)
    caches = []
    for layer in range(L):                                # the same draws in the same order as prepare()
        k, v = x.cache(layer, n)
        caches.append((k, v))
    tiled = b // 16 * 16 if n >= b // 16 * 16 else 0
    if c["lens"] == "ragged" or c["rows"] > b + c["s"]:
        tiled = 0
    n_hist = b - w if tiled else 0
    hist = x.history(n_hist).double() if n_hist else None
    cap = -(-max(b + c["s"], c["rows"] + (c["kind"] == "decode")) // 32) * 32
    steps = {"decode": 1, "cycle": c["s"] * (1 if c["graph"] else POOL)}.get(c["kind"], w)
    q, k, v = x.tokens(steps)
    if c["kind"] == "cycle":
        steps = c["s"]
    out = []
    full = {m: [] for m in ("S", "F", "R", "F_sel")}

    def padded(t):
        return torch.nn.functional.pad(t, (0, cap - t.shape[-1]))

    for layer in range(L):
        K0, V0 = (t.double() for t in caches[layer])
        shape = (c["B"], c["hkv"], steps, c["d"])
        kn = k[:steps, layer].permute(1, 2, 0, 3).double().reshape(shape)
        vn = v[:steps, layer].permute(1, 2, 0, 3).double().reshape(shape)
        if c["kind"] == "decode":
            lens = torch.tensor(_lens(c), device=x.dev)
            at = lens.view(-1, 1, 1, 1).expand(-1, c["hkv"], 1, c["d"])
            K = torch.nn.functional.pad(K0, (0, 0, 0, 1)).scatter_(2, at, kn)
            V = torch.nn.functional.pad(V0, (0, 0, 0, 1)).scatter_(2, at, vn)
            out.append(_attend64(q[0, layer].double(), K, V, lens + 1))
            continue
        K, V = torch.cat([K0, kn], dim=2), torch.cat([V0, vn], dim=2)
        if c["kind"] == "cycle":
            one = torch.ones(c["B"], dtype=torch.int64, device=x.dev)
            out.append(torch.stack([_attend64(q[i, layer].double(), K[:, :, : n + i + 1], V[:, :, : n + i + 1],
                                              one * (n + i + 1)) for i in range(steps)]))
        S, F = _scores64(q[steps - w:steps, layer].double(), K, n + steps, hist[layer] if n_hist else None, n_hist)
        full["S"].append(padded(S))
        full["F"].append(padded(F))
        if c["kind"] == "gkv":
            R, F_sel = _redundancy64(K, F, w)
            full["R"].append(padded(R))
            full["F_sel"].append(padded(F_sel))
    got = {m: torch.stack(t) for m, t in full.items() if t}
    if out:
        got["out"] = torch.stack(out, dim=1 if c["kind"] == "cycle" else 0)
    return got
