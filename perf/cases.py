"""Performance cases of the METRO hot path: what a serving program has one rank of this library do.

Three kinds of pass, each through the package's public calls with the buffers a serving loop keeps:

  layer  one MoE layer of one rank as a decode (or prefill-chunk) step runs it: routing + token lists in one
         launch, grouped SwiGLU expert FFN, weighted combine.  The rank is the one the step waits for.
  gate   router logits, top-k, gating weights and pairs per expert on the gathered batch.
  route  the routing solve of all MoE layers of a model in one launch.

Shapes are those of workloads.py (experts, top-k, ranks, slots, hidden and intermediate sizes) and generic ragged ones.
"""
import functools
import math

import numpy as np
import torch

from paper_2512_09277_amd import api
from paper_2512_09277_amd import workloads as W

DEV = "cuda"
_BF16, _F32 = "bf16", "f32"


def _layer(routing, dtype, N, k, G, spr, T, s, H, I):
    return dict(kind="layer", routing=routing, dtype=dtype, N=N, k=k, G=G, spr=spr, T=T, s=s, H=H, I=I)


def _model_layer(w, routing, T, s=None, dtype=_BF16):
    return _layer(routing, dtype, w.N, w.k, w.G, w.spr, T, w.s if s is None else s, w.H, w.I)


def _gate(dtype, T, H, N, k, valid):
    return dict(kind="gate", dtype=dtype, T=T, H=H, N=N, k=k, valid=valid)


def _route(routing, L, N, k, G, spr, T, s):
    return dict(kind="route", routing=routing, L=L, N=N, k=k, G=G, spr=spr, T=T, s=s)


def listed():
    t = W.TINY
    return [
        # smallest layer (16 experts, 4 ranks, fp32): a test model's decode step, launches and latency only
        dict(_model_layer(t, "metro", t.T, dtype=_F32), name="layer_tiny_f32"),
        # interactive serving: 8 tokens in flight, most of a rank's slots idle, a few rows per activated expert
        dict(_model_layer(W.QWEN3_30B, "metro", 8), name="layer_30b_t8"),
        # the ordinary decode batches of the three model shapes
        dict(_model_layer(W.QWEN3_30B, "metro", 256), name="layer_30b_t256"),
        dict(_model_layer(W.QWEN3_235B, "metro", 512), name="layer_235b_t512"),
        dict(_model_layer(W.DSV3, "metro", 1024), name="layer_dsv3_t1024"),
        # a ragged, small batch of the largest shape under the baseline routing
        dict(_model_layer(W.DSV3, "token_balanced", 97), name="layer_dsv3_t97_balanced"),
        # a prefill chunk (or the largest batch of the routing sweep): hundreds of rows per expert
        dict(_model_layer(W.QWEN3_30B, "token_balanced", 4096), name="layer_30b_t4096_balanced"),
        # fp32 storage and arithmetic: numerics work and reference runs at a real shape
        dict(_model_layer(W.QWEN3_30B, "metro", 256, dtype=_F32), name="layer_30b_f32_t256"),
        # hidden and intermediate sizes that fit no tile, odd batch
        dict(_layer("metro", _BF16, 128, 8, 8, 18, 133, 0.8, 2000, 712), name="layer_ragged_t133"),
        # router gate of the largest decode batch, padded to a power of two
        dict(_gate(_BF16, 1024, 7168, 256, 8, 1000), name="gate_dsv3_t1024"),
        # router kept in fp32 (usual where its logits decide the top-k)
        dict(_gate(_F32, 256, 2048, 128, 8, 256), name="gate_30b_f32_t256"),
        # all 58 MoE layers of a model in one launch
        dict(_route("metro", 58, 256, 8, 16, 18, 1024, 1.0), name="route_58x1024"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    s = round(rng.uniform(0.6, 1.4), 2)
    routing = rng.choice(["metro", "token_balanced"])
    what = rng.random()
    if what < 0.45:                                   # a model's layer, any batch it is served at
        w, most = rng.choice([(W.QWEN3_30B, 4096), (W.QWEN3_235B, 1024), (W.DSV3, 1024)])
        return _model_layer(w, routing, _log_int(rng, 1, most), s)
    if what < 0.65:                                   # other sizes, fp32 among them
        dtype = rng.choice([_F32, _BF16])
        return _layer(routing, dtype, 128, 8, 8, 18, _log_int(rng, 1, 256), min(s, 1.0), _log_int(rng, 64, 2048),
                      _log_int(rng, 64, 768))
    if what < 0.85:
        dtype = rng.choice([_F32, _BF16])
        T = _log_int(rng, 1, 4096 if dtype == _BF16 else 512)
        H = rng.choice([2048, 4096, 7168, _log_int(rng, 100, 4096)]) if dtype == _BF16 else _log_int(rng, 100, 2048)
        N = rng.choice([64, 128, 256, rng.randint(16, 200)]) if dtype == _BF16 else rng.choice([64, 128, rng.randint(16, 128)])
        return _gate(dtype, T, H, N, 8, max(1, T - rng.randint(0, T // 4)))
    N, G, spr = rng.choice([(128, 8, 18), (256, 8, 36), (256, 16, 18)])
    return _route(routing, _log_int(rng, 1, 58), N, 8, G, spr, _log_int(rng, 16, 4096), s)


# ------------------------------------------------------------------------------------------ inputs
def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == _BF16 else torch.float32


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) % (1 << 62))
    return g


def _routing_inputs(case, seed, layer=0):
    """(slot_to_expert[S], ids[T,k]): popularity, its replica placement and a trace drawn from it."""
    base = (int(seed) * 1009 + layer * 31) % (1 << 40)
    p = W.popularity(case["N"], case["s"], base)
    return W.placement(p, case["G"], case["spr"]), W.topk_trace(p, case["T"], case["k"], base + 7)


def _weights(gen, slots, rows, K, dtype):
    """[slots, rows, K] ~ N(0, 0.02), rows laid out with the pitch the library recommends (a multiple of 8)."""
    elt = 2 if dtype == torch.bfloat16 else 4
    K8 = (K + 7) // 8 * 8
    buf = torch.zeros((slots, rows, W.padded_pitch(K8, elt)), dtype=dtype, device=DEV)
    out = buf[:, :, :K]
    for l in range(slots):                            # per slot: the fp32 staging stays small
        out[l] = 0.02 * torch.randn((rows, K), generator=gen, device=DEV)
    return out


def _prepare_layer(case, seed):
    T, k, H, I, N, G, spr = (case[n] for n in ("T", "k", "H", "I", "N", "G", "spr"))
    s2e, ids = _routing_inputs(case, seed)
    g = _generator(seed)
    dt = _torch_dtype(case)
    st = dict(case=case, rank=_waited_for(case, s2e, ids), ids=torch.from_numpy(ids).to(DEV),
              s2e=torch.from_numpy(s2e).to(DEV), x=torch.randn((T, H), generator=g, device=DEV).to(dt),
              topk_w=torch.softmax(torch.randn((T, k), generator=g, device=DEV), dim=1),
              w13=_weights(g, spr, 2 * I, H, dt), w2=_weights(g, spr, H, I, dt))
    st["routing"] = {n: t.fill_(-1) for n, t in api.route_buffers(1, T, k, N, G, DEV).items()}
    st["lists"] = {n: t.fill_(-1) for n, t in api.permute_buffers(T, k, spr, DEV).items()}
    st["ws"] = torch.empty((api.moe_grouped_ffn_workspace_bytes(T, k, spr, H, I, dt),), dtype=torch.uint8, device=DEV)
    st["y"] = torch.zeros((T * k, H), dtype=dt, device=DEV)
    st["out"] = torch.empty((T, H), dtype=dt, device=DEV)
    return st


def _prepare_gate(case, seed):
    T, H, N, k = (case[n] for n in ("T", "H", "N", "k"))
    g = _generator(seed)
    dt = _torch_dtype(case)
    K8 = (H + 7) // 8 * 8
    w = torch.zeros((N, K8), dtype=dt, device=DEV)[:, :H]
    w.copy_(torch.randn((N, H), generator=g, device=DEV) / math.sqrt(H))
    code = api.DTYPE_BF16 if dt == torch.bfloat16 else api.DTYPE_F32
    return dict(case=case, x=torch.randn((T, H), generator=g, device=DEV).to(dt), w=w,
                n_valid=torch.tensor([case["valid"]], dtype=torch.int32, device=DEV),
                ws=torch.empty((int(api.load().moe_gate_topk_workspace_bytes(T, H, N, code)),), dtype=torch.uint8,
                               device=DEV),
                out=dict(topk_ids=torch.empty((T, k), dtype=torch.int32, device=DEV),
                         topk_w=torch.empty((T, k), dtype=torch.float32, device=DEV),
                         expert_count=torch.empty((N,), dtype=torch.int32, device=DEV)))


def _prepare_route(case, seed):
    L, T, k, N, G = (case[n] for n in ("L", "T", "k", "N", "G"))
    pairs = [_routing_inputs(case, seed, layer) for layer in range(L)]
    return dict(case=case, s2e=torch.from_numpy(np.stack([a for a, _ in pairs])).to(DEV),
                ids=torch.from_numpy(np.stack([b for _, b in pairs])).to(DEV),
                routing={n: t.fill_(-1) for n, t in api.route_buffers(L, T, k, N, G, DEV).items()})


def prepare(case, seed):
    return {"layer": _prepare_layer, "gate": _prepare_gate, "route": _prepare_route}[case["kind"]](case, seed)


# ------------------------------------------------------------------------------------------ the pass
def run(state):
    c = state["case"]
    if c["kind"] == "layer":
        fn = api.metro_route_permute if c["routing"] == "metro" else api.metro_route_token_balanced_permute
        routing, lists = fn(state["ids"], state["s2e"], c["N"], c["G"], c["spr"], state["rank"], out=state["routing"],
                            lists=state["lists"])
        y = api.moe_grouped_ffn(state["x"], lists["perm_pair"], lists["group_offsets"], c["k"], state["w13"],
                                state["w2"], y_perm=state["y"], ws=state["ws"])
        out = api.moe_unpermute(y, lists["pair_row"], state["topk_w"], out=state["out"])
        return dict(out=out, lists=lists, routing=routing)
    if c["kind"] == "gate":
        return api.moe_gate_topk(state["x"], state["w"], c["k"], out=state["out"], ws=state["ws"],
                                 n_valid=state["n_valid"])
    fn = api.metro_route if c["routing"] == "metro" else api.metro_route_token_balanced
    return fn(state["ids"], state["s2e"], c["N"], c["G"], c["spr"], out=state["routing"])


# ------------------------------------------------------------------------------------------ plain definitions
def _replicas(s2e, N, G, spr):
    """Per expert: {rank: its lowest slot there}, ranks ascending."""
    reps = [dict() for _ in range(N)]
    for slot in range(G * spr):
        if s2e[slot] >= 0:
            reps[s2e[slot]].setdefault(slot // spr, slot)
    return reps


def _plain_route(case, s2e, ids):
    """Slot of every pair, activated slot per expert, activated experts per rank and their bitmaps."""
    N, G, spr = case["N"], case["G"], case["spr"]
    reps = _replicas(s2e, N, G, spr)
    flat = ids.reshape(-1)
    count = np.bincount(flat, minlength=N)
    expert_slot = np.full(N, -1, np.int32)
    if case["routing"] == "metro":
        load = [0] * G
        for e in range(N):
            if count[e]:
                g = min(reps[e], key=lambda r: (load[r], r))
                load[g] += 1
                expert_slot[e] = reps[e][g]
        pair_slot = expert_slot[flat]
    else:
        order = np.argsort(flat, kind="stable")
        first = np.concatenate([[0], np.cumsum(count)[:-1]])
        nth = np.empty_like(flat)
        nth[order] = np.arange(flat.size) - first[flat[order]]
        slots = [list(r.values()) for r in reps]
        pair_slot = np.array([slots[e][q % len(slots[e])] for e, q in zip(flat.tolist(), nth.tolist())], np.int32)
    used = np.zeros(G * spr, bool)
    used[pair_slot] = True
    used = used.reshape(G, spr)
    bitmap = (used.astype(np.uint64) << np.arange(spr, dtype=np.uint64)).sum(axis=1, dtype=np.uint64)
    return dict(pair_slot=pair_slot.reshape(ids.shape), expert_slot=expert_slot,
                rank_active=used.sum(axis=1).astype(np.int32), rank_bitmap=bitmap.view(np.int64))


def _waited_for(case, s2e, ids):
    """The rank with the most activated slots, of those the one with the most pairs."""
    r = _plain_route(case, s2e, ids)
    pairs = np.bincount(r["pair_slot"].reshape(-1) // case["spr"], minlength=case["G"])
    return int(np.lexsort((pairs, r["rank_active"]))[-1])


def _exact_layer(case, seed):
    st = _prepare_layer(case, seed)
    T, k, I, spr, rank = case["T"], case["k"], case["I"], case["spr"], st["rank"]
    s2e, ids = _routing_inputs(case, seed)
    r = _plain_route(case, s2e, ids)
    local = r["pair_slot"].reshape(-1) - rank * spr
    here = (local >= 0) & (local < spr)
    order = np.flatnonzero(here)[np.argsort(local[here], kind="stable")]
    n = order.size
    offsets = np.concatenate([[0], np.cumsum(np.bincount(local[here], minlength=spr))])
    perm = np.full(T * k, -1, np.int64)
    perm[:n] = order
    row = np.full(T * k, -1, np.int64)
    row[order] = np.arange(n)
    x, topk_w = st["x"].double(), st["topk_w"].double().reshape(-1)
    out = torch.zeros(x.shape, dtype=torch.float64, device=DEV)
    for l in range(spr):
        rows = torch.from_numpy(order[offsets[l]:offsets[l + 1]]).to(DEV)
        if rows.numel() == 0:
            continue
        h = torch.mm(x[rows // k], st["w13"][l].double().t().contiguous())
        y = torch.mm(torch.nn.functional.silu(h[:, :I]) * h[:, I:], st["w2"][l].double().t().contiguous())
        out.index_add_(0, rows // k, y * topk_w[rows, None])
    as_t = torch.from_numpy
    routing = {m: as_t(v).unsqueeze(0) for m, v in r.items()}
    routing["err_flag"] = torch.zeros(1, dtype=torch.int32)
    if case["routing"] != "metro":
        routing["expert_slot"] = None
    return dict(out=out, routing=routing,
                lists=dict(group_offsets=as_t(offsets), perm_pair=as_t(perm), pair_row=as_t(row).reshape(T, k),
                           n_pairs=torch.tensor([n])))


def _exact_gate(case, seed):
    st = _prepare_gate(case, seed)
    k, valid = case["k"], case["valid"]
    top, ids = torch.sort(torch.mm(st["x"].double(), st["w"].double().t().contiguous()), dim=1, descending=True,
                          stable=True)
    w = torch.softmax(top[:, :k], dim=1)
    ids = ids[:, :k].clone()
    w[valid:] = 0
    ids[valid:] = -1
    return dict(topk_ids=ids, topk_w=w, expert_count=torch.bincount(ids[:valid].reshape(-1), minlength=case["N"]))


def exact(case, seed):
    if case["kind"] == "layer":
        return _exact_layer(case, seed)
    if case["kind"] == "gate":
        return _exact_gate(case, seed)
    return None                                       # whole numbers only: they stay the same


# ------------------------------------------------------------------------------------------ what a pass cannot do without
@functools.lru_cache(maxsize=64)
def _share(items):
    """(activated slots, rows) of the rank a layer waits for, on one drawn instance."""
    case = dict(items)
    s2e, ids = _routing_inputs(case, 1)
    r = _plain_route(case, s2e, ids)
    rank = _waited_for(case, s2e, ids)
    return int(r["rank_active"][rank]), int((r["pair_slot"] // case["spr"] == rank).sum())


def work(case):
    T, k, N = case["T"], case["k"], case["N"]
    if case["kind"] == "route":
        L, G, S = case["L"], case["G"], case["G"] * case["spr"]
        return dict(bytes=4 * L * (2 * T * k + S + N + 3 * G + 1), flops=0)
    elt = 2 if case["dtype"] == _BF16 else 4
    H = case["H"]
    if case["kind"] == "gate":
        return dict(bytes=elt * H * (T + N) + 8 * T * k + 4 * N, flops=2 * T * H * N)
    I, G, S = case["I"], case["G"], case["G"] * case["spr"]
    active, rows = _share(tuple(sorted((n, v) for n, v in case.items() if n != "name")))
    lists = 4 * (2 * T * k + S + N + 3 * G) + 4 * (T * k + rows + case["spr"]) + 4 * rows
    tokens = min(rows, T)
    return dict(bytes=elt * (active * 3 * H * I + tokens * H + T * H) + lists, flops=6 * rows * H * I)


def tolerance(case):
    if case["kind"] == "route":
        return "exact"
    if case["kind"] == "gate":
        # fp32 logits summed in another order: the weights move by the logits' error, and two experts whose logits
        # tie to within it may change places
        return {"rel": 1e-5, "max": 1e-4, "differ": 1e-3}
    # bf16: the intermediate, y and the output are rounded to bf16 (2^-9 each); the 16-bit path of ragged sizes keeps
    # the intermediate in fp32.  fp32: sums of some hundred to some thousand products in another order.
    return {"rel": 1e-2, "max": 1e-1} if case["dtype"] == _BF16 else {"rel": 4e-6, "max": 4e-5}
