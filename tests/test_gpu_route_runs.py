"""Routing calls that number pairs (token lists, token-balanced routing) at the sizes where a layer's pairs are cut into
runs of several workgroups: one pair short of, at and past a run, runs whose length is no multiple of four ids or of a
chunk, more layers than leave a workgroup each, and batches whose runs outgrow the registers.  Whole numbers: bit for bit."""
import numpy as np
import pytest

from paper_2512_09277_amd import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


@pytest.mark.parametrize("N,k,G,spr,T", [(16, 1, 4, 5, 1), (16, 1, 4, 5, 63), (16, 1, 4, 5, 2047), (16, 1, 4, 5, 2048), (16, 1, 4, 5, 2049),
                                         (128, 8, 8, 18, 257), (128, 8, 8, 18, 4096), (256, 3, 16, 18, 5461), (512, 5, 64, 32, 3001),
                                         (64, 7, 33, 3, 20011), (256, 8, 8, 36, 70000)])
@pytest.mark.parametrize("routing", ["metro", "token_balanced"])
def test_runs_of_one_layer(oracle, routing, N, k, G, spr, T):
    from paper_2512_09277_amd import api

    api.load()
    print(f"runs {routing} N={N} k={k} G={G} spr={spr} T={T}", flush=True)
    p = W.popularity(N, 1.0, T)
    s2e = W.placement(p, G, spr) if G * spr - N <= N * (G - 1) else None
    ids = W.topk_trace(p, T, k, T + 1)
    if T > 1:
        ids[np.random.default_rng(T).random(ids.shape) < 0.05] = -1
    ref = (oracle.route_metro if routing == "metro" else oracle.route_token_balanced)(ids, s2e, N, G, spr)
    fused = api.metro_route_permute if routing == "metro" else api.metro_route_token_balanced_permute
    plain = api.metro_route if routing == "metro" else api.metro_route_token_balanced
    alone = plain(dev(ids), dev(s2e), N, G, spr)
    for rank in sorted({0, G // 2, G - 1}):
        out, lists = fused(dev(ids), dev(s2e), N, G, spr, rank)
        want = oracle.permute(ref["pair_slot"], rank, spr)
        for got in (out, alone):
            assert int(got["err_flag"].item()) == 0
            for name in ("pair_slot", "rank_active") + (("expert_slot",) if routing == "metro" else ()):
                assert np.array_equal(got[name][0].cpu().numpy(), ref[name]), name
            assert np.array_equal(got["rank_bitmap"][0].cpu().numpy().view(np.uint64), ref["rank_bitmap"])
        n = want["n_pairs"]
        assert int(lists["n_pairs"].item()) == n
        assert np.array_equal(lists["group_offsets"].cpu().numpy(), want["group_offsets"])
        assert np.array_equal(lists["perm_pair"].cpu().numpy()[:n], want["perm_pair"])
        assert np.array_equal(lists["pair_row"].cpu().numpy(), want["pair_row"])


# experts with a choice on both sides of a batch of 8 and of the 64 prepared at a time, up to all 512; ranks in groups of 8, of 16 and
# more; ids out of range and experts without a replica beside them
@pytest.mark.parametrize("N,G,spr,choices", [(70, 3, 32, 0), (70, 8, 18, 7), (70, 8, 18, 8), (70, 9, 18, 9), (200, 16, 32, 63), (200, 17, 32, 64),
                                             (200, 8, 36, 65), (300, 32, 20, 129), (512, 16, 64, 512), (512, 64, 32, 300)])
def test_chain_lengths(oracle, N, G, spr, choices):
    from paper_2512_09277_amd import api

    api.load()
    print(f"chain N={N} G={G} spr={spr} choices={choices}", flush=True)
    rng = np.random.default_rng(N * G + choices)
    slots = [[] for _ in range(G)]
    for e in rng.permutation(N):
        if e != 5:                                        # expert 5 has no replica
            slots[min(range(G), key=lambda g: len(slots[g]))].append(e)
    for e in rng.permutation(N)[:choices]:
        for g in rng.permutation(G)[:int(rng.integers(2, 4))]:
            if e != 5 and e not in slots[g] and len(slots[g]) < spr:
                slots[g].append(e)
    s2e = np.concatenate([(s + [-1] * spr)[:spr] for s in slots]).astype(np.int32)
    for T in (3, 600):
        ids = np.stack([rng.permutation(N)[:4] for _ in range(T)]).astype(np.int32)
        ids[0, 0] = -1
        for bad in (None, N, -2, 2**31 - 1):
            if bad is not None:
                ids[T - 1, 3] = bad
            served = np.where((ids < 0) | (ids >= N) | (ids == 5), -1, ids)              # the others get no slot
            ref = oracle.route_metro(served, s2e, N, G, spr)
            flag = (api.FLAG_BAD_ID if bad is not None else 0) | (api.FLAG_NO_REPLICA if (ids == 5).any() else 0)
            for got in (api.metro_route(dev(ids), dev(s2e), N, G, spr), api.metro_route_permute(dev(ids), dev(s2e), N, G, spr, 1)[0]):
                assert int(got["err_flag"].item()) == flag
                for name in ("pair_slot", "expert_slot", "rank_active"):
                    assert np.array_equal(got[name][0].cpu().numpy(), ref[name]), (name, T, bad)


# With lists the chain has two forms; which one takes a call hangs on its spare slots (S - N) and pairs, on both sides of 32, and either has
# to serve any number of experts with a choice: here more than the spare slots, as half of the experts have no slot and no pair.
@pytest.mark.parametrize("N,G,spr,k,T", [(16, 4, 5, 2, 15), (16, 4, 5, 2, 400), (200, 8, 28, 4, 700), (205, 8, 29, 4, 700), (200, 8, 29, 4, 700),
                                         (512, 17, 32, 1, 31), (512, 17, 32, 1, 32), (512, 32, 17, 8, 900), (480, 64, 8, 8, 900), (300, 16, 18, 3, 200),
                                         (300, 19, 16, 3, 200)])
def test_chain_of_few_spare_slots(oracle, N, G, spr, k, T):
    from paper_2512_09277_amd import api

    api.load()
    print(f"few N={N} G={G} spr={spr} k={k} T={T}", flush=True)
    rng = np.random.default_rng(N + G + T)
    there = np.sort(rng.permutation(N)[:N // 2])
    slots = [[] for _ in range(G)]
    for e in np.concatenate([rng.permutation(there), rng.permutation(there)]):            # two replicas of all or most
        free = [g for g in range(G) if len(slots[g]) < spr and e not in slots[g]]
        if free:
            slots[min(free, key=lambda g: len(slots[g]))].append(e)
    s2e = np.concatenate([(s + [-1] * spr)[:spr] for s in slots]).astype(np.int32)
    ids = np.stack([there[rng.permutation(there.size)[:k]] for _ in range(T)]).astype(np.int32)
    ref = oracle.route_metro(ids, s2e, N, G, spr)
    for rank in (0, G - 1):
        got, lists = api.metro_route_permute(dev(ids), dev(s2e), N, G, spr, rank)
        want = oracle.permute(ref["pair_slot"], rank, spr)
        assert int(got["err_flag"].item()) == 0
        for name in ("pair_slot", "expert_slot", "rank_active"):
            assert np.array_equal(got[name][0].cpu().numpy(), ref[name]), name
        n = int(want["n_pairs"])
        assert int(lists["n_pairs"].item()) == n
        assert np.array_equal(lists["group_offsets"].cpu().numpy(), want["group_offsets"])
        assert np.array_equal(lists["perm_pair"].cpu().numpy()[:n], want["perm_pair"][:n])
        assert np.array_equal(lists["pair_row"].cpu().numpy(), want["pair_row"])


@pytest.mark.parametrize("L,T", [(3, 1500), (58, 1024), (129, 700), (300, 300)])
def test_runs_of_many_layers(oracle, L, T):
    from paper_2512_09277_amd import api

    api.load()
    w = W.QWEN3_30B
    p = W.popularity(w.N, 1.0, L)
    s2e = W.placement(p, w.G, w.spr)
    ids = np.stack([W.topk_trace(p, T, w.k, 1000 + l) for l in range(L)])
    out = api.metro_route_token_balanced(dev(ids), dev(np.stack([s2e] * L)), w.N, w.G, w.spr)
    assert not out["err_flag"].any()
    for l in range(0, L, max(1, L // 7)):
        ref = oracle.route_token_balanced(ids[l], s2e, w.N, w.G, w.spr)
        assert np.array_equal(out["pair_slot"][l].cpu().numpy(), ref["pair_slot"]), l
        assert np.array_equal(out["rank_bitmap"][l].cpu().numpy().view(np.uint64), ref["rank_bitmap"]), l


@pytest.mark.parametrize("T", [1024, 4096])
def test_slots_written_over_the_ids(oracle, T):
    """pair_slot may be the id tensor itself."""
    from paper_2512_09277_amd import api

    api.load()
    w = W.QWEN3_30B
    p = W.popularity(w.N, 1.0, T)
    s2e, ids = W.placement(p, w.G, w.spr), W.topk_trace(p, T, w.k, T)
    for plain, fused, ref in ((api.metro_route, api.metro_route_permute, oracle.route_metro),
                              (api.metro_route_token_balanced, api.metro_route_token_balanced_permute,
                               oracle.route_token_balanced)):
        want = ref(ids, s2e, w.N, w.G, w.spr)["pair_slot"]
        for lists in (False, True):
            d = dev(ids)
            out = api.route_buffers(1, T, w.k, w.N, w.G, "cuda")
            out["pair_slot"] = d.unsqueeze(0)
            if lists:
                _, got = fused(d, dev(s2e), w.N, w.G, w.spr, 3, out=out)
                rows = oracle.permute(want, 3, w.spr)
                assert np.array_equal(got["pair_row"].cpu().numpy(), rows["pair_row"])
                assert np.array_equal(got["perm_pair"].cpu().numpy()[:rows["n_pairs"]], rows["perm_pair"])
            else:
                plain(d, dev(s2e), w.N, w.G, w.spr, out=out)
            assert np.array_equal(d.cpu().numpy(), want), lists


def routed(routing, T, place=None):
    """The fused call on T tokens, with `place` = (output, input, offset): that output in the input's memory, `offset` entries in;
    or "count": n_pairs as the last entry of group_offsets.
    Returns every output (on the host) and the oracle's arguments."""
    import torch

    from paper_2512_09277_amd import api

    w = W.QWEN3_30B
    p = W.popularity(w.N, 1.0, T)
    s2e, ids = W.placement(p, w.G, w.spr), W.topk_trace(p, T, w.k, T)
    inputs = dict(ids=dev(ids), s2e=dev(s2e))
    out, lists = api.route_buffers(1, T, w.k, w.N, w.G, "cuda"), api.permute_buffers(T, w.k, w.spr, "cuda")
    if place == "count":                                     # n_pairs is the last offset
        lists["n_pairs"] = lists["group_offsets"][w.spr:]
    elif place:
        name, host, offset = place
        into = out if name in out else lists
        old = into[name]
        words = old.numel() * old.element_size() // 4
        into[name] = inputs[host].view(-1)[offset:offset + words].view(old.dtype).view(old.shape)
    fused = api.metro_route_permute if routing == "metro" else api.metro_route_token_balanced_permute
    fused(inputs["ids"], inputs["s2e"], w.N, w.G, w.spr, 3, out=out, lists=lists)
    torch.cuda.synchronize()
    return {n: t.cpu().numpy() for n, t in {**out, **lists}.items()}, ids, s2e


# 8192 pairs: the ids of a single workgroup fit its registers; 8200 and 16384: they do not; 16: one run
@pytest.mark.parametrize("T,place", [(2, "count"), (2048, "count")] + [(T, (name, "ids", 0)) for T in (2, 1024, 1025, 2048) for name in ("pair_slot", "perm_pair", "pair_row")] +
                         [(1024, (name, host, offset)) for host in ("ids", "s2e") for offset in (0, 8)
                          for name in ("expert_slot", "rank_active", "rank_bitmap", "err_flag", "group_offsets", "n_pairs")])
@pytest.mark.parametrize("routing", ["metro", "token_balanced"])
def test_outputs_in_the_inputs_memory(oracle, routing, T, place):
    """An output in the memory of the ids or of the placement: every output as with memory of its own, at any batch size."""
    from paper_2512_09277_amd import api

    api.load()
    print(f"shared memory {routing} T={T} {place}", flush=True)
    w = W.QWEN3_30B
    got, ids, s2e = routed(routing, T, place)
    ref = (oracle.route_metro if routing == "metro" else oracle.route_token_balanced)(ids, s2e, w.N, w.G, w.spr)
    want = oracle.permute(ref["pair_slot"], 3, w.spr)
    assert not got["err_flag"].any()
    for name in ("pair_slot", "rank_active") + (("expert_slot",) if routing == "metro" else ()):
        assert np.array_equal(got[name][0], ref[name]), name
    assert np.array_equal(got["rank_bitmap"][0].view(np.uint64), ref["rank_bitmap"])
    n = want["n_pairs"]
    assert int(got["n_pairs"][0]) == n
    assert np.array_equal(got["group_offsets"], want["group_offsets"])
    assert np.array_equal(got["perm_pair"][:n], want["perm_pair"])
    assert np.array_equal(got["pair_row"], want["pair_row"])
