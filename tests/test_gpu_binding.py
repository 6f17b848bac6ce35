"""The native marshalling of the binding against its Python checks: over argument forms that are plain, odd and wrong,
a call gives the same outputs or raises the same exception with the same words on both ways."""
import numpy as np
import pytest

from paper_2512_09277_amd import workloads as W

pytestmark = pytest.mark.gpu

T, K, N, G, SPR, H, I = 12, 2, 16, 4, 5, 64, 32


class OnlyPython:
    """Stands in for the native module: nothing is its plain case."""

    def __getattr__(self, name):
        return lambda *a: 1


def made(dtype="f32"):
    import torch

    from paper_2512_09277_amd import api

    api.load()
    w = W.TINY
    s2e = W.placement(W.popularity(N, 1.0, 1), G, SPR)
    ids = W.topk_trace(W.popularity(N, 1.0, 1), T, K, 2)
    g = torch.Generator().manual_seed(3)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    rnd = lambda *s: torch.randn(s, generator=g).to(dt).cuda()  # noqa: E731
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()  # noqa: E731
    return dict(ids=i32(ids), s2e=i32(s2e), x=rnd(T, H), w13=rnd(SPR, 2 * I, H), w2=rnd(SPR, H, I), tw=rnd(T, K).float(),
                wg=rnd(N, H), out={n: t.zero_() for n, t in api.route_buffers(1, T, K, N, G, "cuda").items()},
                lists={n: t.zero_() for n, t in api.permute_buffers(T, K, SPR, "cuda").items()},
                y=rnd(T * K, H), comb=rnd(T, H), n_valid=i32([T - 3]),
                ws=torch.zeros((api.moe_grouped_ffn_workspace_bytes(T, K, SPR, H, I, dt),), dtype=torch.uint8, device="cuda"),
                gws=torch.zeros((1 << 20,), dtype=torch.uint8, device="cuda"),
                gate=dict(topk_ids=i32(np.zeros((T, K))), topk_w=rnd(T, K).float(), expert_count=i32(np.zeros(N))))


def calls():
    from paper_2512_09277_amd import api

    return {
        "route": lambda a: api.metro_route(a["ids"], a["s2e"], N, G, SPR, out=a["out"]),
        "balanced": lambda a: api.metro_route_token_balanced(a["ids"], a["s2e"], N, G, SPR, out=a["out"]),
        "route_permute": lambda a: api.metro_route_permute(a["ids"], a["s2e"], N, G, SPR, a.get("rank", 1), out=a["out"], lists=a["lists"]),
        "balanced_permute": lambda a: api.metro_route_token_balanced_permute(a["ids"], a["s2e"], N, G, SPR, a.get("rank", 1), out=a["out"],
                                                                             lists=a["lists"]),
        "ffn": lambda a: api.moe_grouped_ffn(a["x"], a["lists"]["perm_pair"], a["lists"]["group_offsets"], a.get("k", K), a["w13"],
                                             a["w2"], y_perm=a["y"], ws=a["ws"]),
        "unpermute": lambda a: api.moe_unpermute(a["y"], a["lists"]["pair_row"], a["tw"], out=a["comb"]),
        "gate": lambda a: api.moe_gate_topk(a["x"], a["wg"], a.get("k", K), out=a["gate"], ws=a["gws"], n_valid=a["n_valid"]),
    }


def outcome(call, args):
    import torch

    try:
        r = call(args)
        torch.cuda.synchronize()
    except Exception as e:
        return type(e).__name__, str(e)
    flat = []

    def walk(v):
        if isinstance(v, dict):
            for n in sorted(v):
                walk(v[n])
        elif isinstance(v, (tuple, list)):
            for x in v:
                walk(x)
        else:
            flat.append(v.cpu())
    walk(r)
    return flat


def padded(t):
    import torch

    buf = torch.zeros((*t.shape[:-1], t.shape[-1] + 8), dtype=t.dtype, device=t.device)
    buf[..., :t.shape[-1]] = t
    return buf[..., :t.shape[-1]]


def parameter(t):
    import torch

    return torch.nn.Parameter(t, requires_grad=False)


FORMS = {
    "plain": lambda a: None,
    "padded weights": lambda a: a.update(w13=padded(a["w13"]), w2=padded(a["w2"]), wg=padded(a["wg"])),
    "pitch not a multiple of 8": lambda a: a.update(w13=padded(a["w13"])[:, :, :H - 4], x=a["x"][:, :H - 4].contiguous(), w2=a["w2"][:, :H - 4].contiguous()),
    "weights transposed": lambda a: a.update(w13=a["w13"].transpose(1, 2).contiguous().transpose(1, 2), wg=a["wg"].t().contiguous().t()),
    "weights of another type": lambda a: a.update(w13=a["w13"].double(), wg=a["wg"].double()),
    "weights of another shape": lambda a: a.update(w2=a["w2"][:, :, :I - 8].contiguous(), wg=a["wg"][:, :H - 8].contiguous()),
    "activations strided": lambda a: a.update(x=padded(a["x"]), y=padded(a["y"])),
    "activations on the host": lambda a: a.update(x=a["x"].cpu(), y=a["y"].cpu(), ids=a["ids"].cpu()),
    "float64 activations": lambda a: a.update(x=a["x"].double(), y=a["y"].double()),
    "ids of 64 bits": lambda a: a.update(ids=a["ids"].long(), lists=dict(a["lists"], pair_row=a["lists"]["pair_row"].long())),
    "ids and placement with a layer axis": lambda a: a.update(ids=a["ids"].unsqueeze(0), s2e=a["s2e"].unsqueeze(0)),
    "two layers of ids": lambda a: a.update(ids=a["ids"].repeat(2, 1, 1)),
    "placement too short": lambda a: a.update(s2e=a["s2e"][:-1].contiguous()),
    "no buffers": lambda a: a.update(out=None),
    "a buffer missing": lambda a: a.update(out={n: t for n, t in a["out"].items() if n != "rank_active"}),
    "an offset too few": lambda a: a.update(lists=dict(a["lists"], group_offsets=a["lists"]["group_offsets"][:-1].contiguous())),
    "perm_pair too short": lambda a: a.update(lists=dict(a["lists"], perm_pair=a["lists"]["perm_pair"][:-1].contiguous())),
    "workspace too small": lambda a: a.update(ws=a["ws"][:256], gws=a["gws"][:256]),
    "workspace misaligned": lambda a: a.update(ws=a["gws"][1:], gws=a["gws"][1:]),
    "rank out of range": lambda a: a.update(rank=G),
    "k too large": lambda a: a.update(k=N + 1),
    "k a tensor": lambda a: a.update(k=__import__("torch").tensor(2)),
    "no valid count": lambda a: a.update(n_valid=None),
    "valid count of 64 bits": lambda a: a.update(n_valid=a["n_valid"].long()),
    "parameters": lambda a: a.update(w13=parameter(a["w13"]), w2=parameter(a["w2"]), wg=parameter(a["wg"])),
    "empty batch": lambda a: a.update(ids=a["ids"][:0], x=a["x"][:0], y=a["y"][:0]),
}


@pytest.mark.parametrize("form", FORMS)
def test_both_ways_agree(monkeypatch, form):
    import torch

    from paper_2512_09277_amd import api

    api.load()
    native = api._native
    for name, call in calls().items():
        print(f"binding {name}: {form}", flush=True)
        seen = []
        for way in (native, OnlyPython()):
            monkeypatch.setattr(api, "_native", way)
            a = made()
            calls()["route_permute"](a)                                  # lists the FFN and the combine can read
            torch.cuda.synchronize()
            FORMS[form](a)
            if a["out"] is None and "permute" in name:
                a["lists"] = None
            seen.append(outcome(call, a))
        fast, slow = seen
        if isinstance(slow, tuple):
            assert fast == slow, name
        else:
            assert not isinstance(fast, tuple), (name, fast)
            assert len(fast) == len(slow) and all(p.dtype == q.dtype and p.shape == q.shape for p, q in zip(fast, slow)), name
            if a["out"] is not None:                                     # given buffers: their unwritten parts are alike too
                assert all(torch.equal(p, q) for p, q in zip(fast, slow)), name


def test_the_plain_case_is_native(monkeypatch):
    """Every plain call is taken by the native way, and on the caller's current stream."""
    import torch

    from paper_2512_09277_amd import api

    api.load()
    a = made("bf16")
    monkeypatch.setattr(api, "_dev", None)                               # the Python checks would fail here
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for call in calls().values():
            call(a)
    torch.cuda.synchronize()
    assert int(a["out"]["err_flag"].item()) == 0


@pytest.mark.parametrize("native", [True, False])
def test_lazily_cloned_buffers(monkeypatch, native):
    """A written buffer that is a lazy (copy-on-write) clone gets memory of its own: the tensor that it was cloned from stays."""
    import torch

    from paper_2512_09277_amd import api

    api.load()
    if not native:
        monkeypatch.setattr(api, "_native", OnlyPython())
    for name, call in calls().items():
        plain, a = made(), made()
        for args in (plain, a):
            calls()["route_permute"](args)                               # lists the FFN and the combine can read
        torch.cuda.synchronize()
        sources = []

        def lazy(t):
            sources.append((t, t.clone()))
            return torch._lazy_clone(t)

        for group in ("out", "lists", "gate"):
            if not (group == "lists" and "permute" not in name):         # those are inputs of the FFN and the combine
                a[group] = {n: lazy(t) for n, t in a[group].items()}
        for n in ("ws", "gws", "comb") + (("y",) if name == "ffn" else ()):
            a[n] = lazy(a[n])
        got, want = outcome(call, a), outcome(call, plain)
        assert not isinstance(got, tuple), (name, got)
        assert all(torch.equal(p, q) for p, q in zip(got, want)), name
        for source, before in sources:
            assert torch.equal(source, before), name
