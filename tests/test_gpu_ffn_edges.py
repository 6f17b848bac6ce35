"""Grouped FFN at the sizes where its kernels change path or end inside a tile, every row against the CPU oracle.

Tolerance: max|gpu - ref| / max|ref|.  fp32: sums of n products in any order err by at most n * 2^-24 of the sum of
magnitudes, which for random signs is about sqrt(n) of the result's scale: below 1e-5 for n <= 2048.  bf16: two roundings
of 2^-9 relative (the intermediate and the output), 2e-2 over the tensor."""
import numpy as np
import pytest

from paper_2512_09277_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"bf16": 2e-2, "f32": 1e-5}


def dev(a):
    import torch

    t = torch.from_numpy(np.ascontiguousarray(a))
    return (t.view(torch.bfloat16) if a.dtype == np.uint16 else t).cuda()


def weights(a, pitch):
    """[slots, rows, K] on the device, rows `pitch` elements apart, the gap filled with NaN."""
    import torch

    t = dev(a)
    buf = torch.full((t.shape[0], t.shape[1], pitch), float("nan"), dtype=t.dtype, device="cuda")
    view = buf[:, :, :t.shape[2]]
    view.copy_(t)
    return view


def check(oracle, dtype, H, I, sizes, T=256, k=2, extra=0):
    from paper_2512_09277_amd import api

    api.load()
    print(f"edges {dtype} H={H} I={I} sizes={sizes}", flush=True)
    spr = len(sizes)
    rng = np.random.default_rng(H * 7 + I)
    pairs = rng.permutation(T * k)[:sum(sizes)]
    ps = np.full(T * k, -1, np.int32)
    ps[pairs] = np.repeat(np.arange(spr), sizes)
    ps = ps.reshape(T, k)
    x = W.activations(T, H, 5, dtype)
    w13, w2 = W.expert_weights(spr, H, I, 6, dtype)
    pm = api.moe_permute(dev(ps), 0, spr)
    up8 = lambda n: (n + 7) // 8 * 8 + extra  # noqa: E731
    y = api.moe_grouped_ffn(dev(x), pm["perm_pair"], pm["group_offsets"], k, weights(w13, up8(H)), weights(w2, up8(I)))
    ref = oracle.permute(ps, 0, spr)
    want = oracle.ffn(x, ref["perm_pair"], ref["group_offsets"], k, w13, w2)
    got = y[:ref["n_pairs"]].float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    err = np.abs(got - want).max() / np.abs(want).max()
    assert err <= TOL[dtype], err


# the last K step of either stage whole, one element short or long, shorter than a vector, a multiple of no vector; output
# columns ending inside a 16-row block and inside a vector; rows at the edges of the 16-row sub-tiles
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,I", [(1, 1), (3, 5), (7, 2), (4, 8), (8, 9), (9, 16), (31, 33), (32, 64), (63, 127), (65, 130),
                                 (129, 31), (250, 96), (257, 66), (1023, 255)])
def test_general_path_edges(oracle, dtype, H, I):
    check(oracle, dtype, H, I, [1, 16, 0, 17, 32, 33, 15, 65])


# matrix-core path: rows at the edges of every tile class (16, 32, 48, 64 in a launch cut into narrow tiles; 16 narrow, 64, 96, 128
# tall in the others; beyond one tile), K of 2 steps (two of the four waves without any) and of step counts that end inside
# the prefetch ring.  At 128 x 128 both stages, at 1152 x 256 gate/up are cut into narrow tiles; the others have tall ones.
@pytest.mark.parametrize("H,I", [(128, 128), (384, 640), (1152, 256), (2048, 1024), (4096, 2048)])
def test_matrix_path_edges(oracle, H, I):
    check(oracle, "bf16", H, I, [1, 15, 16, 17, 31, 32, 33, 0, 47, 48, 49, 63, 64, 65, 96, 97, 128, 129, 200], T=700,
          extra=128)


# the rule that cuts a launch, at 384 x 640 (20 gate/up column tiles of a narrow tile, 10 of a tall one): 12 | 13 tiles of 64 rows
# fill the CUs once; up to 38 the launch is narrow only if fewer than 17 tiles would be tall and more than a third as many small;
# past 38 tiles of 17 to 32 rows are narrow if fewer than 17 would be tall
@pytest.mark.parametrize("sizes", [[16] * 12, [16] * 13, [33] * 12, [33] * 13, [65] * 6 + [1], [5] * 20 + [64] * 16, [5] * 20 + [64] * 17,
                                   [1] * 5 + [40] * 15, [1] * 6 + [40] * 15, [16] * 38, [16] * 39, [16] * 10 + [64] * 28, [144] * 5,
                                   [5] * 30 + [24] * 7 + [32, 33, 40, 90], [5] * 22 + [24] * 17])
def test_cut_rule_edges(oracle, sizes):
    check(oracle, "bf16", 384, 640, sizes, T=1000)


# lists of tall tiles per XCD: 1, 2, 4, 7, 11 and 14 column tiles (fewer than the XCDs, no multiple of them), slots of one to sixteen
# tiles, empty ones between them, K of 2 and 4 steps (shorter than the prefetch ring) and of 14 and 22
@pytest.mark.parametrize("H,I", [(256, 128), (128, 256), (896, 512), (1408, 896)])
def test_tall_lists(oracle, H, I):
    check(oracle, "bf16", H, I, [0, 2000, 1, 0, 1500, 700, 65, 97, 33, 17, 0, 130, 128, 16, 300], T=2600)


# combine: vectors of 8 bf16 or 4 fp32 columns, k in registers (<= 8) or not, rows that are no whole vectors, pairs of other
# ranks.  Sums of k products in fp32 in the oracle's order: fp32 within k * 2^-24 of the sum of magnitudes, bf16 one rounding.
@pytest.mark.parametrize("dtype,tol", [("f32", 2e-6), ("bf16", 8e-3)])
@pytest.mark.parametrize("H,k", [(1, 1), (4, 3), (6, 8), (8, 8), (12, 9), (1028, 8), (2048, 12)])
def test_unpermute_edges(oracle, dtype, tol, H, k):
    from paper_2512_09277_amd import api

    api.load()
    T = 37
    rng = np.random.default_rng(H + k)
    row = np.full(T * k, -1, np.int32)
    here = np.flatnonzero(rng.random(T * k) < 0.4)
    row[here] = rng.permutation(here.size)
    y = W.activations(max(here.size, 1), H, 3, dtype)
    tw = W.gating_weights(T, k, 4)
    full = np.zeros((T * k, H), y.dtype)
    full[:y.shape[0]] = y
    out = api.moe_unpermute(dev(full), dev(row.reshape(T, k)), dev(tw))
    as_f64 = W.bf16_bits_to_f32(full).astype(np.float64) if dtype == "bf16" else full.astype(np.float64)
    want = oracle.unpermute(as_f64, row.reshape(T, k), tw)
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.abs(got - want).max() <= tol * max(np.abs(want).max(), 1e-30)


# the combine's workgroups on both sides of 1024 tokens: rows of less than a wave, of uneven turns, past 512 and 1024 vectors
@pytest.mark.parametrize("dtype,tol", [("f32", 2e-6), ("bf16", 8e-3)])
@pytest.mark.parametrize("T,H,k", [(1024, 40, 3), (1025, 40, 3), (1024, 7176, 2), (1025, 2600, 8), (1025, 4136, 9), (1100, 5208, 1)])
def test_unpermute_workgroups(oracle, dtype, tol, T, H, k):
    from paper_2512_09277_amd import api

    api.load()
    print(f"unpermute {dtype} T={T} H={H} k={k}", flush=True)
    rng = np.random.default_rng(T + H)
    row = np.full(T * k, -1, np.int32)
    here = np.flatnonzero(rng.random(T * k) < 0.2)
    row[here] = rng.permutation(here.size)
    y = W.activations(here.size, H, 3, dtype)
    tw = W.gating_weights(T, k, 4)
    out = api.moe_unpermute(dev(y), dev(row.reshape(T, k)), dev(tw))
    as_f64 = np.zeros((T * k, H))
    as_f64[:here.size] = W.bf16_bits_to_f32(y) if dtype == "bf16" else y
    want = oracle.unpermute(as_f64, row.reshape(T, k), tw)
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.abs(got - want).max() <= tol * max(np.abs(want).max(), 1e-30)


def test_unpermute_of_millions_of_tokens():
    """2^22 tokens whose rows would fill a workgroup of 1024 threads: more threads than one launch may have."""
    import torch

    from paper_2512_09277_amd import api

    api.load()
    T, H = 1 << 22, 8192
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 70 GB of device memory")
    out = torch.empty((T, H), dtype=torch.bfloat16, device="cuda")
    some = [0, 1, T // 2, T - 2, T - 1]
    out[some] = 7.0
    row = torch.full((T, 1), -1, dtype=torch.int32, device="cuda")
    row[T - 1] = 0
    y = torch.ones((1, H), dtype=torch.bfloat16, device="cuda")
    api.moe_unpermute(y, row, torch.full((T, 1), 2.0, device="cuda"), out=out)
    assert torch.equal(out[some].float().cpu(), torch.tensor([0.0, 0.0, 0.0, 0.0, 2.0])[:, None].expand(5, H))
    del out
    torch.cuda.empty_cache()


def test_activations_past_2_gib():
    """Tokens (first stage) and list rows (second) more than 2^31 bytes into their arrays, in tall and narrow tiles: addressed by unsigned
    32-bit offsets up to 4 GiB.  Against float64 products of the rows on the device."""
    import torch

    from paper_2512_09277_amd import api

    api.load()
    T, H, I, sizes = 1_200_000, 1024, 1024, [700, 9, 700]
    n = sum(sizes)
    print(f"past 2 GiB T={T} H={H} I={I} sizes={sizes}", flush=True)
    assert 2**31 < (T - n) * H * 2 and T * H * 2 < 2**32
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    tokens = torch.cat([torch.arange(T - 1000, T), torch.arange(n - 1000)]).cuda()[torch.randperm(n, generator=g, device="cuda")]
    x = torch.empty((T, H), dtype=torch.bfloat16, device="cuda")
    x[tokens] = torch.randn((n, H), generator=g, device="cuda").bfloat16()
    w13 = (0.02 * torch.randn((3, 2 * I, H), generator=g, device="cuda")).bfloat16()
    w2 = (0.02 * torch.randn((3, H, I), generator=g, device="cuda")).bfloat16()
    perm = torch.zeros((T,), dtype=torch.int32, device="cuda")
    perm[T - n:] = tokens.int()
    offsets = torch.tensor([T - n, T - n + sizes[0], T - sizes[2], T], dtype=torch.int32, device="cuda")     # the last rows of the list
    y = torch.empty((T, H), dtype=torch.bfloat16, device="cuda")
    api.moe_grouped_ffn(x, perm, offsets, 1, w13, w2, y_perm=y)
    begin = 0
    for slot, m in enumerate(sizes):
        h = torch.mm(x[tokens[begin:begin + m]].double(), w13[slot].double().t().contiguous())
        want = torch.mm(torch.nn.functional.silu(h[:, :I]) * h[:, I:], w2[slot].double().t().contiguous())
        got = y[T - n + begin:T - n + begin + m].double()
        err = ((got - want).abs().max() / want.abs().max()).item()
        assert err <= TOL["bf16"], (slot, err)
        begin += m
