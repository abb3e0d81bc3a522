"""GPU parity at the edges of the size rules that choose between kernel shapes, against the CPU oracle."""
import numpy as np
import pytest
import torch

import moe_workloads as W
import paper_2106_10715_amd as M
from oracle import moe_oracle as O
from paper_2106_10715_amd import harness as H
from test_gpu_stages import TOL, gpu_route, make_inputs, rel_l2, rounded, run_ffn
from tile_rows import N_CU, heights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f", [(64, 64),       # both products in 32 x 32 tiles with the reduction split over the waves
                                 (128, 4096),    # up-projection in 64 x 64 tiles
                                 (4096, 64)])    # down-projection in 64 x 64 tiles
def test_f32_expert_ffn_tile_shapes(d, f):
    counts = [0, 1, 31, 32, 33, 64, 65, 130]
    got, ref, offsets = run_ffn(sum(counts), d, f, len(counts), 1, "f32", counts, 0, seed=d + 3 * f)
    for e in range(len(counts)):
        lo, hi = offsets[e], offsets[e + 1]
        if hi > lo:
            # two chained fp32 sums of at most 4096 terms: rounding errors of 2^-24 add up like a random walk, 2^-24 * 64 = 4e-6
            assert rel_l2(got[lo:hi], ref[lo:hi]) <= 4e-6, f"expert {e}"


@pytest.mark.parametrize("T,d,E,k", [(4096, 64, 5, 2), (4097, 64, 5, 2), (4098, 128, 70, 3), (33, 192, 65, 2)])
def test_f32_gate_tokens_per_wave(T, d, E, k):
    x, Wg, b = make_inputs(T + E, T, d, E, "f32", bias=True)
    idx, w = gpu_route(M.MoeCfg.make(T, d, 64, E, k, "f32"), x, Wg, b, "f32")
    r = O.route(x, Wg, k, b, 1)
    assert np.array_equal(idx, r.idx)
    assert rel_l2(w, r.w) <= 1e-5


def test_f32_layer_without_copy_and_combine():
    """One expert per token: the layer reads its rows from x and writes them to y itself; the four calls give the same bytes."""
    rng = np.random.default_rng(5)
    T, d, f, E = 333, 128, 192, 5
    cfg = M.MoeCfg.make(T, d, f, E, 1, "f32")
    x, Wg, _ = make_inputs(9, T, d, E, "f32")
    ex = [tuple(rng.standard_normal(s).astype(np.float32) * 0.05 for s in ((d, f), (d, f), (f, d))) for _ in range(E)]
    packed = torch.empty((E, M.moe_expert_bytes(cfg)), dtype=torch.uint8, device="cuda")
    for e in range(E):
        M.moe_pack_weights(cfg, *(H.to_device(m, "f32") for m in ex[e]), packed[e])
    dx, dW = H.to_device(x, "f32"), H.to_device(Wg, "f32")
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    y = torch.full((T, d), float("nan"), device="cuda")
    M.moe_layer_forward(cfg, dx, dW, None, packed, None, y, ws)

    def ints(*n):
        return torch.empty(n, dtype=torch.int32, device="cuda")
    idx, w, counts, offsets, perm, inv = ints(T, 1), torch.empty((T, 1), device="cuda"), ints(E), ints(E + 1), ints(T), ints(T)
    Xp, Yp, y4 = torch.empty_like(dx), torch.empty_like(dx), torch.empty_like(dx)
    M.moe_route(cfg, dx, dW, None, idx, w, ws)
    M.moe_permute(cfg, dx, idx, counts, offsets, perm, inv, Xp, ws)
    M.moe_expert_ffn(cfg, Xp, offsets, packed, Yp, ws)
    M.moe_combine(cfg, Yp, inv, w, y4)
    torch.cuda.synchronize()
    assert torch.equal(y, y4)
    ref = O.layer_forward(x, Wg, lambda e: ex[e], E, 1, None, 1)[0]
    assert rel_l2(H.to_f64(y), ref) <= TOL["f32"]


@pytest.mark.parametrize("counts", [[1], [0, 16, 0], [17, 0], [5, 0, 9, 18], [32], [0, 15, 17], [33], [1] * 32, [28, 5]],
                         ids=lambda c: "x".join(map(str, c[:4])) + f"-{sum(c)}")
@pytest.mark.parametrize("d,f", [(64, 64), (192, 704), (1024, 576)])
def test_few_rows_expert_ffn(counts, d, f):
    """Blocks of 16 and 32 rows per expert, up to 16 rows in all (units of 16 columns) and more; one expert with 33 rows is past
    the limit of 32 rows per expert."""
    got, ref, offsets = run_ffn(sum(counts), d, f, len(counts), 1, "bf16", counts, d % 128 // 64, seed=sum(counts) + d)
    for e in range(len(counts)):
        lo, hi = offsets[e], offsets[e + 1]
        if hi > lo:
            assert rel_l2(got[lo:hi], ref[lo:hi]) <= TOL["bf16"], f"expert {e}"


# (a wave of the down-projection per compute unit at most and 64 steps or more: 14 in flight; 64, 65, 70 and 139 steps are rounds of 14 and 8, 9, 0 and 13 more. The last
# two are past the limit of steps, and of waves)
@pytest.mark.parametrize("counts,d,f", [([1], 4096, 4096), ([16], 256, 4160), ([3, 0, 13], 1024, 4480), ([1, 1, 1, 1], 1024, 8896), ([16], 256, 4032), ([1, 1, 1, 1, 1], 1024, 4096)],
                         ids=lambda c: str(c) if isinstance(c, int) else "x".join(map(str, c)))
def test_few_rows_long_down_projection(counts, d, f):
    got, ref, offsets = run_ffn(sum(counts), d, f, len(counts), 1, "bf16", counts, 0, seed=d + f)
    error = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert (error <= TOL["bf16"]).all(), f"row {error.argmax()}: {error.max():.3e}"


@pytest.mark.parametrize("T,k", [(1, 1), (7, 2), (30, 1), (21, 3)])
def test_few_rows_streamed_equals_resident(T, k):
    wl = W.Workload("few", T=T, d=256, f=384, E=6, k=k, dtype="bf16", seed=50 + T)
    L = H.build_layer(wl, host_copy=True)
    M.moe_layer_forward(L.cfg, L.x, L.Wg, L.bias, L.packed, None, L.y, L.ws)
    torch.cuda.synchronize()
    want = L.y.clone()
    ref = O.layer_forward(W.gen_x(wl), W.gen_gate(wl)[0], lambda e: W.gen_expert(wl, e), wl.E, k, None, wl.renorm)[0]
    assert rel_l2(H.to_f64(want), ref) <= TOL["bf16"]
    ctx = M.StreamCtx(L.cfg, L.host_packed, torch.empty((2, M.moe_expert_bytes(L.cfg)), dtype=torch.uint8, device="cuda"), 2)
    for _ in range(2):
        L.y.fill_(float("nan"))
        M.moe_layer_forward(L.cfg, L.x, L.Wg, L.bias, None, ctx, L.y, L.ws)
        torch.cuda.synchronize()
        assert torch.equal(L.y, want)
    ctx.close()


@pytest.mark.parametrize("T", [16320, 16321, 16449])      # 32 tokens per block, 64 with one in the last block, and a few more
@pytest.mark.parametrize("d,E,k,bias", [(64, 7, 2, True), (192, 45, 3, False)])
def test_gate_block_sizes(T, d, E, k, bias):
    x, Wg, b = make_inputs(T + E, T, d, E, "bf16", bias=bias)
    idx, w = gpu_route(M.MoeCfg.make(T, d, 64, E, k, "bf16"), x, Wg, b, "bf16")
    r = O.route(x, Wg, k, b, 1)
    assert np.array_equal(idx, r.idx)
    assert rel_l2(w, r.w) <= 1e-5


@pytest.mark.parametrize("T,E,k,renorm", [(70, 40, 3, 0), (40, 20, 1, 1)])
def test_gate_many_close_tokens_in_one_block(T, E, k, renorm):
    """Equal columns, and more of them than are evaluated one by one: every token of a block goes through the exact branches."""
    x, Wg, _ = make_inputs(T, T, 256, E, "bf16")
    Wg[:, 1::2] = Wg[:, 0::2]                       # pairs tie exactly
    Wg[:, E // 2:] = Wg[:, :1]                      # and half of the columns are one and the same
    idx, w = gpu_route(M.MoeCfg.make(T, 256, 64, E, k, "bf16", renorm), x, Wg, None, "bf16")
    r = O.route(x, Wg, k, None, renorm)
    assert np.array_equal(idx, r.idx)
    assert rel_l2(w, r.w) <= 1e-5


def expert_ffn_rows(counts, rows_of, d, f, dtype, act=0):
    """Yp per expert of a call in which expert e gets the first counts[e] of the rows rows_of(e)."""
    E, A = len(counts), sum(counts)
    rng = np.random.default_rng(d + f)
    ex = [tuple(rounded(rng.standard_normal(s) * 0.05, dtype) for s in ((d, f), (d, f), (f, d))) for _ in range(E)]
    cfg = M.MoeCfg.make(A, d, f, E, 1, dtype, 1, act)
    packed = H.pack_experts(W.Workload("t", A, d, f, E, 1, dtype, 0), cfg, experts=lambda e: ex[e])[0]
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    Xp = H.to_device(np.concatenate([rows_of(e)[:n] for e, n in enumerate(counts)]), dtype)
    Yp = torch.full_like(Xp, float("nan"))
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    M.moe_expert_ffn(cfg, Xp, torch.from_numpy(offsets).cuda(), packed, Yp, ws)
    torch.cuda.synchronize()
    return [Yp[offsets[e]:offsets[e + 1]] for e in range(E)]


@pytest.mark.parametrize("few,many", [([1, 0, 3], [300, 40, 270]), ([12, 4, 0], [33, 470, 9]), ([20, 40, 3], [257, 100, 240]),
                                      ([64, 0, 17], [200, 230, 130])])
@pytest.mark.parametrize("d,f,dtype", [(64, 64, "bf16"), (192, 704, "bf16"), (2112, 1088, "bf16"),
                                       (192, 4096, "f32"), (4096, 192, "f32")])      # up, down: split and wide tiles
def test_rows_have_the_same_bits_in_every_batch(d, f, dtype, few, many):
    """An expert's row gives the same bytes whatever else is in the batch, and so whichever kernel the batch size selects."""
    def rows_of(e):
        return rounded(np.random.default_rng(e).standard_normal((512, d)), dtype)
    small, large = expert_ffn_rows(few, rows_of, d, f, dtype), expert_ffn_rows(many, rows_of, d, f, dtype)
    for e in range(len(few)):
        n = min(few[e], many[e])
        assert torch.isfinite(small[e].float()).all() and torch.isfinite(large[e].float()).all()
        assert torch.equal(small[e][:n], large[e][:n]), f"expert {e}"


@pytest.mark.parametrize("d,E,k,renorm", [(1024, 7, 2, 0), (4160, 32, 2, 1), (2048, 60, 3, 0), (1024, 100, 2, 0), (1024, 200, 2, 1)])
def test_gate_does_not_depend_on_the_place_in_the_batch(d, E, k, renorm):
    """A token's experts and weights have the same bits in every place of every batch (8, 16, 32 and 64 tokens per block)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(d + E)
    x = torch.empty((16450, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    x[300:310] = x[5:15]                           # the same token in two places
    Wg = torch.empty((d, E), dtype=torch.bfloat16, device="cuda").normal_(0.0, d ** -0.5, generator=g)

    def route(x):
        cfg = M.MoeCfg.make(x.shape[0], d, 64, E, k, "bf16", renorm)
        idx = torch.full((x.shape[0], k), -7, dtype=torch.int32, device="cuda")
        w = torch.full((x.shape[0], k), float("nan"), device="cuda")
        M.moe_route(cfg, x, Wg, None, idx, w, torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        return idx, w
    idx, w = route(x)
    assert torch.equal(idx[300:310], idx[5:15]) and torch.equal(w[300:310], w[5:15])
    for part in (x[:1], x[:260], x[:4100], x[:8200]):
        i2, w2 = route(part)
        assert torch.equal(i2, idx[:len(part)]) and torch.equal(w2, w[:len(part)]), f"{len(part)} tokens"
    i2, w2 = route(torch.roll(x, 1037, dims=0))
    assert torch.equal(i2, torch.roll(idx, 1037, dims=0)) and torch.equal(w2, torch.roll(w, 1037, dims=0))


@pytest.mark.parametrize("T", [130, 4100, 8200, 16450])         # 8, 16, 32 and 64 tokens per block
@pytest.mark.parametrize("E", [8, 32, 80])
def test_gate_every_token_tied(T, E):
    """Every column twice: each token's best two tie exactly.  Then all columns equal: every token picks the first ones."""
    x, Wg, _ = make_inputs(T + E, T, 128, E // 2, "bf16")
    best, _ = gpu_route(M.MoeCfg.make(T, 128, 64, E // 2, 1, "bf16"), x, Wg, None, "bf16")
    idx, w = gpu_route(M.MoeCfg.make(T, 128, 64, E, 2, "bf16"), x, np.repeat(Wg, 2, axis=1), None, "bf16")
    assert np.array_equal(idx, 2 * best + np.array([0, 1]))
    assert (w == 0.5).all()
    idx, w = gpu_route(M.MoeCfg.make(T, 128, 64, E, 4, "bf16"), x, np.repeat(Wg[:, :1], E, axis=1), None, "bf16")
    assert np.array_equal(idx, np.tile(np.arange(4), (T, 1)))
    assert (w == 0.25).all()


@pytest.mark.parametrize("T,d,E,k", [(20, 4160, 32, 2), (20, 8256, 32, 1), (20, 4160, 64, 2), (20, 8256, 64, 3), (4100, 4160, 32, 2),
                                     (8200, 4160, 32, 1)])
def test_gate_long_rows(T, d, E, k):
    """More groups per wave than are requested ahead, column norms of more groups than are read ahead; columns that differ in one
    element by one unit in the last place, so that the error bound has to send their tokens to the exact branch."""
    x, Wg, _ = make_inputs(T + d, T, d, E, "bf16")
    Wg[:, E // 2:] = Wg[:, :E // 2]
    Wg[d - 1, E // 2:] *= 1 + 2.0 ** -7
    Wg = rounded(Wg, "bf16")
    idx, w = gpu_route(M.MoeCfg.make(T, d, 64, E, k, "bf16"), x, Wg, None, "bf16")
    r = O.route(x, Wg, k, None, 1)
    assert np.array_equal(idx, r.idx)
    assert rel_l2(w, r.w) <= 1e-5


@pytest.mark.parametrize("T,d,k,dtype", [(300, 2048, 3, "bf16"), (301, 2112, 4, "bf16"), (302, 4160, 5, "bf16"), (50, 1024, 2, "f32"),
                                         (51, 2112, 8, "f32"),       # one, two and four pieces of a row per thread
                                         (43000, 1088, 3, "bf16"), (16500, 4160, 2, "bf16"), (9000, 4160, 5, "bf16"),
                                         (165000, 1024, 1, "bf16"), (41000, 4160, 1, "bf16")])    # non-temporal sums; copies as well
def test_rows_out_and_back(T, d, k, dtype):
    """Batching and weighted sum, every row length and number of rows per token, against torch in fp64."""
    g = torch.Generator(device="cuda")
    g.manual_seed(T + d)
    cfg = M.MoeCfg.make(T, d, 64, 8, k, dtype)
    x = torch.empty((T, d), dtype=cfg.torch_dtype, device="cuda").normal_(generator=g)
    idx = torch.rand((T, 8), device="cuda", generator=g).topk(k, 1).indices.int()
    w = torch.rand((T, k), device="cuda", generator=g)

    def ints(*n):
        return torch.full(n, -1, dtype=torch.int32, device="cuda")
    counts, offsets, perm, inv = ints(8), ints(9), ints(T * k), ints(T * k)
    Xp = torch.full((T * k, d), float("nan"), dtype=cfg.torch_dtype, device="cuda")
    M.moe_permute(cfg, x, idx, counts, offsets, perm, inv, Xp, torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda"))
    order = idx.flatten().long().sort(stable=True).indices
    assert torch.equal(perm.long(), order)
    assert torch.equal(Xp, x[order // k])
    Yp = torch.empty_like(Xp).normal_(generator=g)
    y = torch.full_like(x, float("nan"))
    M.moe_combine(cfg, Yp, inv, w, y)
    ref = torch.zeros((T, d), dtype=torch.float64, device="cuda")
    for j in range(k):
        ref += w[:, j:j + 1].double() * Yp[inv.view(T, k)[:, j].long()].double()
    # k fp32 roundings of sums no larger than sum(w) max|Yp|, half a unit (2^-24) each; then one to the stored type, whose half unit
    # is 2^-8 of the value with the 8 significant bits of bf16 and 2^-24 with the 24 of fp32
    half = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -24
    fp32_sum = w.sum(1, keepdim=True).double() * Yp.abs().max().double() * (k * 2.0 ** -24)
    assert ((y.double() - ref).abs() <= fp32_sum + (ref.abs() + fp32_sum) * half).all()


# Limits of rows in all, by E x ceil(d / 256): 32 E below 86, 8 E up to 256, 2 E beyond (256 compute units).
@pytest.mark.parametrize("d,E,limit", [(320, 7, 224), (1024, 22, 176), (1024, 64, 512), (1024, 65, 130)])
@pytest.mark.parametrize("heavy", [1, 33, 64, 65, 128])
@pytest.mark.parametrize("over", [0, 1])
def test_few_rows_limits_and_crowded_experts(d, E, limit, heavy, over):
    """The last batch on the kernels for few rows and the first on the others, even and with many rows on one expert."""
    rest = limit + over - heavy
    counts = [rest // (E - 1) + (e <= rest % (E - 1)) for e in range(E)]
    counts[0] = heavy
    counts[1] += limit + over - sum(counts)
    got, ref, offsets = run_ffn(sum(counts), d, 128, E, 1, "bf16", counts, 0, seed=d + E + heavy)
    for e in range(E):
        lo, hi = offsets[e], offsets[e + 1]
        if hi > lo:
            assert rel_l2(got[lo:hi], ref[lo:hi]) <= TOL["bf16"], f"expert {e}"


@pytest.mark.parametrize("T,crowd", [(16, 1.0), (33, 1.0), (65, 1.0), (200, 1.0), (200, 0.2), (224, 1.0)])
def test_few_rows_gathered_equals_batched(T, crowd):
    """The layer looks its rows up in x; with nearly all tokens on one expert as with a few, the four calls give the same bytes."""
    d, f, E = 320, 192, 7
    rng = np.random.default_rng(T)
    cfg = M.MoeCfg.make(T, d, f, E, 1, "bf16")
    x, Wg, _ = make_inputs(T, T, d, E, "bf16")
    bias = np.zeros(E, dtype=np.float32)
    bias[3] = 5.0 * crowd
    ex = [tuple(rounded(rng.standard_normal(s) * 0.05, "bf16") for s in ((d, f), (d, f), (f, d))) for _ in range(E)]
    packed = H.pack_experts(W.Workload("t", T, d, f, E, 1, "bf16", 0), cfg, experts=lambda e: ex[e])[0]
    dx, dW, db = H.to_device(x, "bf16"), H.to_device(Wg, "bf16"), torch.from_numpy(bias).cuda()
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    y = torch.full_like(dx, float("nan"))
    M.moe_layer_forward(cfg, dx, dW, db, packed, None, y, ws)

    def ints(*n):
        return torch.empty(n, dtype=torch.int32, device="cuda")
    idx, w, counts, offsets, perm, inv = ints(T, 1), torch.empty((T, 1), device="cuda"), ints(E), ints(E + 1), ints(T), ints(T)
    Xp, Yp, y4 = torch.empty_like(dx), torch.empty_like(dx), torch.empty_like(dx)
    M.moe_route(cfg, dx, dW, db, idx, w, ws)
    M.moe_permute(cfg, dx, idx, counts, offsets, perm, inv, Xp, ws)
    M.moe_expert_ffn(cfg, Xp, offsets, packed, Yp, ws)
    M.moe_combine(cfg, Yp, inv, w, y4)
    torch.cuda.synchronize()
    assert torch.equal(y, y4)
    ref = O.layer_forward(x, Wg, lambda e: ex[e], E, 1, bias, 1)[0]
    assert rel_l2(H.to_f64(y), ref) <= TOL["bf16"]


def _four_calls(cfg, dx, dW, db, packed, ws):
    """(y of the four calls, y of the layer)"""
    A, E = cfg.T * cfg.k, cfg.E

    def ints(*n):
        return torch.empty(n, dtype=torch.int32, device="cuda")
    idx, w, counts, offsets, perm, inv = ints(cfg.T, cfg.k), torch.empty((cfg.T, cfg.k), device="cuda"), ints(E), ints(E + 1), ints(A), ints(A)
    Xp = torch.empty((A, cfg.d), dtype=dx.dtype, device="cuda")
    Yp, y4, y = torch.empty_like(Xp), torch.full_like(dx, float("nan")), torch.full_like(dx, float("nan"))
    M.moe_route(cfg, dx, dW, db, idx, w, ws)
    M.moe_permute(cfg, dx, idx, counts, offsets, perm, inv, Xp, ws)
    M.moe_expert_ffn(cfg, Xp, offsets, packed, Yp, ws)
    M.moe_combine(cfg, Yp, inv, w, y4)
    M.moe_layer_forward(cfg, dx, dW, db, packed, None, y, ws)
    torch.cuda.synchronize()
    return y4, y


def _tall_ffn(counts, d, f, E, T, want):
    """Experts of `counts` rows, and others without, in a call of at most T rows, whose tiles have up to `want` = (up, down, narrow units) rows: every expert against
    fp64, and the last 40 rows of every expert with the bits that they have in a call of their own (which the kernels for few rows take)."""
    assert torch.cuda.get_device_properties(0).multi_processor_count == N_CU and heights(T, d, f, E) == want and sum(counts) <= T
    x = _normal(T, d, seed=d + f).bfloat16()
    ex = [[(_normal(*s, seed=100 + 3 * e + i) * 0.05).bfloat16() for i, s in enumerate(((d, f), (d, f), (f, d)))] for e in range(len(counts))]
    cfg = M.MoeCfg.make(T, d, f, E, 1, "bf16")
    packed = torch.zeros((E, M.moe_expert_bytes(cfg)), dtype=torch.uint8, device="cuda")
    for e, matrices in enumerate(ex):
        M.moe_pack_weights(cfg, *matrices, packed[e])

    def run(rows, counts):
        n = rows.shape[0]
        cfg = M.MoeCfg.make(n, d, f, E, 1, "bf16")
        offsets = torch.tensor([0] + counts + [0] * (E - len(counts)), device="cuda").cumsum(0).int()
        Y = torch.full((n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        M.moe_expert_ffn(cfg, rows, offsets, packed, Y, torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        return Y
    got, lo = run(x, counts), 0
    for e, n in enumerate(counts):
        W_in, W_gate, W_out = (m.double() for m in ex[e])
        rows = x[lo:lo + n]
        ref = (torch.nn.functional.gelu(rows.double() @ W_gate) * (rows.double() @ W_in)) @ W_out
        error = (got[lo:lo + n].double() - ref).norm(dim=1) / ref.norm(dim=1)
        assert (error <= TOL["bf16"]).all(), f"expert {e}: row {error.argmax().item()} of {n}"
        few = min(n, 40)
        alone = run(rows[n - few:].clone(), [0] * e + [few])
        assert torch.equal(alone, got[lo + n - few:lo + n]), f"expert {e}: rows {n - few} to {n}"
        lo += n
    assert torch.isnan(got[lo:]).all()


# steps of 64 in the two reductions, 1 to 10 each: fewer than are requested ahead, rounds of four (three for 19 and 20 blocks) and what does not fill one
@pytest.mark.parametrize("up,down,E,T,narrow", [
    (1, 7, 256, 38400, True), (2, 6, 220, 44000, True), (3, 3, 120, 20400, True), (4, 8, 120, 20400, True), (5, 5, 160, 27200, True), (5, 2, 250, 42500, True),
    (6, 1, 250, 42500, True), (7, 7, 120, 24000, True), (8, 4, 120, 22800, True), (9, 10, 100, 20000, True), (10, 9, 100, 20000, True),
    (1, 2, 160, 44800, False), (2, 9, 200, 46000, False), (3, 5, 160, 48000, False), (5, 3, 100, 25000, False), (5, 10, 100, 25000, False), (6, 4, 100, 28000, False),
    (7, 7, 100, 28000, False), (8, 8, 100, 28000, False), (9, 6, 64, 17920, False), (10, 1, 160, 51200, False)])
def test_expert_ffn_every_tile_height(up, down, E, T, narrow):
    """Tiles of 1 to 20 blocks of 16 rows in both kernels, full and not, of experts with one, and of 11 to 20 where an expert has two or three."""
    _tall_ffn([16 * b - b % 3 for b in range(1, 21)] + [32 * b - 5 for b in range(11, 21)] + [321, 960], 64 * up, 64 * down, E, T, (320, 320, narrow))


@pytest.mark.parametrize("d,f", [(64, 576), (128, 832), (192, 1408), (256, 1408), (320, 1408), (384, 1408), (448, 1408)])
def test_gathered_tiles_equal_batched(d, f):
    """Rows looked up in x, tiles of 1 to 14 blocks, and of 8 and 14 where an expert has two: the layer gives the bytes of the four calls, whose tiles are others."""
    counts = [16 * b - b % 3 for b in range(1, 15)] + [225, 448, 0, 0, 0, 0]
    T, E = sum(counts), len(counts)
    assert heights(T, d, f, E, gather=True)[0] == 224 and T // E <= 160
    expert = torch.tensor([e for e, n in enumerate(counts) for _ in range(n)], device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    x = _normal(T, d, seed=d)
    x[:, :E] = 4.0 * torch.nn.functional.one_hot(expert[torch.randperm(T, generator=g, device="cuda")], E)
    cfg = M.MoeCfg.make(T, d, f, E, 1, "bf16")
    packed = torch.empty((E, M.moe_expert_bytes(cfg)), dtype=torch.uint8, device="cuda")
    for e in range(E):
        M.moe_pack_weights(cfg, *((_normal(*s, seed=70 + 3 * e + i) * 0.05).bfloat16() for i, s in enumerate(((d, f), (d, f), (f, d)))), packed[e])
    ws = torch.full((M.moe_workspace_bytes(cfg) // 2,), float("nan"), dtype=torch.bfloat16, device="cuda").view(torch.uint8)
    y4, y = _four_calls(cfg, x.bfloat16(), torch.eye(d, E, device="cuda").bfloat16(), None, packed, ws)
    assert torch.isfinite(y.float()).all()
    assert torch.equal(y, y4)


# one chunk, chunk edges, the last batch of one launch and the first of the chunked kernels
@pytest.mark.parametrize("A", [1, 63, 1023, 1024, 1025, 4099, 65535, 65536, 65537])
@pytest.mark.parametrize("E", [1, 33, 256])
@pytest.mark.parametrize("shift", [0, 1])               # idx at a 16-byte boundary and not
def test_batching_in_one_launch(A, E, shift):
    g = torch.Generator(device="cuda")
    g.manual_seed(A + E)
    buf = torch.empty(A + 4, dtype=torch.int32, device="cuda")
    idx = buf[shift:shift + A]
    idx.copy_((torch.rand(A, device="cuda", generator=g) ** 3 * (E + 2)).int() - 1)        # skewed, and some out of range: clamped
    _check_batching(idx, E)


def _check_batching(idx, E):
    A, e = idx.numel(), idx.long().clamp(0, E - 1)

    def ints(n):
        return torch.full((n,), -1, dtype=torch.int32, device="cuda")
    cfg = M.MoeCfg.make(A, 64, 64, E, 1, "bf16")
    counts, offsets, perm, inv = ints(E), ints(E + 1), ints(A), ints(A)
    M.moe_permute(cfg, None, idx.view(A, 1), counts, offsets, perm, inv, None, torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    order = e.sort(stable=True).indices
    assert torch.equal(perm.long(), order)
    assert torch.equal(inv.long()[order], torch.arange(A, device="cuda"))
    assert torch.equal(counts.long(), torch.bincount(e, minlength=E))
    assert offsets.tolist() == [0] + torch.cumsum(counts, 0).tolist()


# the sizes where the counting goes over to more histograms
@pytest.mark.parametrize("A", [8192, 8193, 32768, 32769, 65536])
@pytest.mark.parametrize("E,share", [(1, 1.0), (256, 1.0), (256, 0.5)])
def test_batching_with_one_dominant_expert(A, E, share):
    g = torch.Generator(device="cuda")
    g.manual_seed(A)
    idx = torch.randint(0, E, (A,), dtype=torch.int32, device="cuda", generator=g)
    idx[torch.rand(A, device="cuda", generator=g) < share] = E - 1
    _check_batching(idx, E)


@pytest.mark.parametrize("T,k", [(1, 1), (2, 8), (16, 1), (17, 1), (21, 3), (32, 2), (64, 1), (65, 1)])
@pytest.mark.parametrize("E,crowd", [(9, 0.0), (9, 8.0), (256, 0.0), (64, 3.0)])
@pytest.mark.parametrize("dtype,renorm", [("bf16", 1), ("bf16", 0), ("f32", 1)])
def test_layer_without_batching(T, k, E, crowd, dtype, renorm):
    """Up to 64 assignments the expert kernels find their rows in idx themselves: the bytes of the four calls, with experts of one row
    and with all rows on a few (up to 64 rows: two tiles of the fp32 kernel)."""
    d, f = 128, 192
    rng = np.random.default_rng(T + E)
    cfg = M.MoeCfg.make(T, d, f, E, k, dtype, renorm)
    x, Wg, _ = make_inputs(T, T, d, E, dtype)
    ex = [tuple(rounded(rng.standard_normal(s) * 0.05, dtype) for s in ((d, f), (d, f), (f, d))) for _ in range(min(E, 9))]
    packed = H.pack_experts(W.Workload("t", T, d, f, E, k, dtype, 0), cfg, experts=lambda e: ex[e % len(ex)])[0]
    bias = torch.zeros(E, device="cuda")
    bias[E // 2:E // 2 + k] = crowd
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    y4, y = _four_calls(cfg, H.to_device(x, dtype), H.to_device(Wg, dtype), bias, packed, ws)
    assert torch.isfinite(y.float()).all()
    assert torch.equal(y, y4)


# row blocks 1 to 4 and a second tile; narrow and wide blocks of columns in both products; quarters of the reduction of 0, 1 and more steps
@pytest.mark.parametrize("d,f", [(64, 64), (64, 4096), (2048, 128), (192, 8192)])
def test_f32_expert_ffn_row_blocks(d, f):
    counts = [1, 16, 17, 33, 48, 64, 65, 97, 129]
    got, ref, offsets = run_ffn(sum(counts), d, f, len(counts), 1, "f32", counts, 1, seed=d + f)
    for e in range(len(counts)):
        lo, hi = offsets[e], offsets[e + 1]
        # two chained sums; one addition of 2^-24 per 32 elements in each, and the rounding inside the instruction is of the same size
        assert rel_l2(got[lo:hi], ref[lo:hi]) <= 1e-6, f"expert {e}"


def test_f32_expert_ffn_large_and_infinite_values():
    """The parts of an infinity are no numbers: rows that hold one, or a NaN, and a row of large finite values."""
    d, f, E = 64, 128, 2
    rng = np.random.default_rng(0)
    ex = [tuple(rng.standard_normal(s).astype(np.float32) * 0.05 for s in ((d, f), (d, f), (f, d))) for _ in range(E)]
    cfg = M.MoeCfg.make(6, d, f, E, 1, "f32")
    packed = H.pack_experts(W.Workload("t", 6, d, f, E, 1, "f32", 0), cfg, experts=lambda e: ex[e])[0]
    x = rng.standard_normal((6, d)).astype(np.float32)
    x[1, 3], x[2, 5], x[3, 7] = np.inf, -np.inf, np.nan
    x[4] *= np.float32(1e18)                     # H about 1e36, finite
    Yp = torch.empty((6, d), device="cuda")
    M.moe_expert_ffn(cfg, torch.from_numpy(x).cuda(), torch.tensor([0, 5, 6], dtype=torch.int32, device="cuda"), packed, Yp,
                     torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    got = Yp.cpu().double()
    for r in range(6):
        W_in, W_gate, W_out = (torch.from_numpy(m).double() for m in ex[0 if r < 5 else 1])
        t = torch.from_numpy(x[r]).double()
        h = torch.nn.functional.gelu(t @ W_gate) * (t @ W_in)
        ref = h @ W_out
        if r in (1, 2, 3):
            assert torch.equal(torch.isnan(got[r]), torch.isnan(ref.float())) and torch.equal(torch.isinf(got[r]), torch.isinf(ref.float()))
        else:
            assert rel_l2(got[r].numpy(), ref.numpy()) <= 1e-6


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("E,k,renorm", [(6, 2, 1), (40, 1, 1), (40, 3, 0), (70, 2, 0), (1, 1, 1), (3, 3, 1), (12, 12, 0)])
@pytest.mark.parametrize("special", [float("inf"), float("-inf"), float("nan")])
def test_gate_infinite_logits_keep_the_fp32_order(E, k, renorm, special, dtype):
    """Tokens with an infinity or a NaN have no error bound and go through the exact branch.  There infinite logits are ordered as in fp32 (+inf first,
    equal ones by column), logits that are no numbers come with the smallest, experts stay in range and differ, and the other tokens of the block are
    what they are without them."""
    k = min(k, 8)
    x, Wg, _ = make_inputs(E, 20, 256, E, dtype)
    cfg = M.MoeCfg.make(20, 256, 64, E, k, dtype, renorm)
    idx0, w0 = gpu_route(cfg, x, Wg, None, dtype)
    y = x.copy()
    y[7, 100] = special
    idx, w = gpu_route(cfg, y, Wg, None, dtype)
    others = np.arange(20) != 7
    assert np.array_equal(idx[others], idx0[others]) and np.array_equal(w[others], w0[others])
    assert idx[7].min() >= 0 and idx[7].max() < E and len(set(idx[7].tolist())) == k
    if np.isinf(special):
        logit = Wg[100] * special
        assert np.array_equal(idx[7], np.argsort(-logit, kind="stable")[:k])
        Wg[100, E // 2 + 1:] = 0                     # infinity times zero
        idx, _ = gpu_route(cfg, y, Wg, None, dtype)
        some = np.argsort(-logit[:E // 2 + 1], kind="stable")[:k]
        some = some[logit[some] > 0]                 # the infinite ones; what comes after ranks with the logits that are no numbers
        assert np.array_equal(idx[7][:len(some)], some)
        assert idx[7].min() >= 0 and idx[7].max() < E and len(set(idx[7].tolist())) == k


@pytest.mark.parametrize("counts", [[700, 10, 300, 0, 257, 40, 600, 33, 513, 5, 270, 120], [330] * 7 + [90, 200], [350, 255, 256] * 3, [2000, 1, 1, 1]],
                         ids=lambda c: f"{len(c)}-{sum(c)}")
def test_expert_ffn_merged_work_list(counts):
    """Experts of several tiles among experts of one: 192 rows per expert and more, where the work list merges the two kinds."""
    _tall_ffn(counts, 384, 256, 100, 28000, (320, 320, False))


def test_three_million_rows_on_one_expert():
    """More rows on one expert than a 32-bit product of its tiles and blocks holds: every row is what it is in a batch of its own."""
    T, d, f = 3_000_000, 64, 64
    cfg = M.MoeCfg.make(T, d, f, 1, 1, "bf16")
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    x = torch.empty((T, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    ex = [torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.1, generator=g) for s in ((d, f), (d, f), (f, d))]
    packed = torch.empty((1, M.moe_expert_bytes(cfg)), dtype=torch.uint8, device="cuda")
    M.moe_pack_weights(cfg, *ex, packed[0])
    Wg = torch.zeros((d, 1), dtype=torch.bfloat16, device="cuda")
    y = torch.full_like(x, float("nan"))
    M.moe_layer_forward(cfg, x, Wg, None, packed, None, y, torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda"))
    part = 1 << 17
    small = M.MoeCfg.make(part, d, f, 1, 1, "bf16")
    ws, want = torch.empty(M.moe_workspace_bytes(small), dtype=torch.uint8, device="cuda"), torch.empty((part, d), dtype=torch.bfloat16, device="cuda")
    for lo in [*range(0, T - part, part), T - part]:
        M.moe_layer_forward(small, x[lo:lo + part], Wg, None, packed, None, want, ws)
        assert torch.equal(y[lo:lo + part], want), f"rows {lo}..{lo + part}"


def _f32_sums(x, W):
    """16 x W by the fp32 expert kernel (x [T, K], W [K, N], N <= K; column 0 of x and row 0 of W are used up: the gate is 16 exactly, GELU(16) = 16 in
    fp32, and the down-projection an identity), and the same in 64 bits."""
    (T, K), N = x.shape, W.shape[1]
    x, W, gate = x.clone(), W.clone(), torch.zeros_like(W)
    x[:, 0], W[0], gate[0] = 16.0, 0.0, 1.0
    cfg = M.MoeCfg.make(T, K, N, 1, 1, "f32")
    packed = torch.empty((1, M.moe_expert_bytes(cfg)), dtype=torch.uint8, device="cuda")
    M.moe_pack_weights(cfg, W, gate, torch.eye(N, K, device="cuda"), packed[0])
    Y = torch.full((T, K), float("nan"), device="cuda")
    M.moe_expert_ffn(cfg, x, torch.tensor([0, T], dtype=torch.int32, device="cuda"), packed, Y,
                     torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    return Y[:, :N], 16 * (x[:, 1:].double() @ W[1:].double())


def _normal(*shape, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.empty(shape, device="cuda").normal_(generator=g)


@pytest.mark.parametrize("K", [64, 512])
def test_f32_expert_ffn_single_products(K):
    """Rows with one value: the sum is one product, and right to half of its last bit (1/64 more for the part of the product that is left out and for
    the instruction's cutting off of the small parts)."""
    x, at = torch.zeros((200, K), device="cuda"), torch.arange(200, device="cuda") % (K - 1) + 1
    x[torch.arange(200, device="cuda"), at] = _normal(200, seed=1)
    got, ref = _f32_sums(x, _normal(K, 64, seed=2))
    assert ((got.double() - ref).abs() <= ref.abs() * 2.0 ** -24 * (1 + 2.0 ** -6)).all()


@pytest.mark.parametrize("value", [1 + 2.0 ** -7 - 2.0 ** -23, 1 + 2.0 ** -8 + 2.0 ** -17 - 2.0 ** -23, 1 / 3])
def test_f32_expert_ffn_equal_products(value):
    """63 times the same product: its error comes 63 times with one sign.  Two steps of 32 in two of the four quarters, each rounded three times to 2^-24 of
    at most the sum (inside the instruction, twice outside), and the sum of the two."""
    got, ref = _f32_sums(torch.full((20, 64), value, device="cuda"), torch.full((64, 64), value, device="cuda"))
    assert ((got.double() - ref).abs() <= ref.abs() * 2.0 ** -24 * 4).all()


@pytest.mark.parametrize("up,down", [(1e30, 1e-30), (3e37, 0.1), (1e10, 1e25)])
def test_f32_expert_ffn_large_values(up, down):
    """Operands and sums up to the upper end of fp32 are summed in 64 bits where the products of parts are infinite, else as any others."""
    got, ref = _f32_sums(_normal(70, 128, seed=5) * up, _normal(128, 64, seed=6) * down / 64)
    assert torch.isfinite(got).all()
    assert rel_l2(got.cpu().numpy(), ref.cpu().numpy()) <= 2.0 ** -22


def test_f32_expert_ffn_partial_sums_overflow():
    """Half of the products are 2e38 and half -2e38: the sum of a quarter, and of 32 products, is past the end of fp32, the whole is not.  A NaN, and
    an infinity (times the gate's zeros), stay in their rows."""
    x, W = torch.full((5, 64), 1e19, device="cuda"), torch.full((64, 64), 2e19, device="cuda")
    x[:, 32:] *= -1
    x[1, 40] = -0.96e19
    x[2, 3], x[3, 5] = float("inf"), float("nan")
    x[:, 33] = 0
    got, ref = _f32_sums(x, W)
    assert torch.equal(got[[0, 4]], torch.zeros_like(got[[0, 4]]))
    assert torch.isnan(got[2:4]).all()
    assert ((got[1].double() - ref[1]).abs() <= ref[1].abs() * 2.0 ** -23).all() and (ref[1] > 1e38).all()


@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** -112, 2.0 ** -125])
def test_f32_expert_ffn_small_values(scale):
    """Operands down to the lower end of fp32 (values 1 to 2 times the scale, last bit 2^-23 of it): a power of two changes no bit of the sums."""
    x, W = 1 + _normal(70, 128, seed=3).abs().remainder(1.0), 1 + _normal(128, 64, seed=4).abs().remainder(1.0)
    want = _f32_sums(x, W)[0]
    assert torch.equal(_f32_sums(x * scale, W)[0], want * scale)
    assert torch.equal(_f32_sums(x, W * scale)[0], want * scale)


def _ffn_by_expert(counts, d, f, seed):
    got, ref, offsets = run_ffn(sum(counts), d, f, len(counts), 1, "bf16", counts, 0, seed=seed)
    for e in range(len(counts)):
        lo, hi = offsets[e], offsets[e + 1]
        if hi > lo:
            assert rel_l2(got[lo:hi], ref[lo:hi]) <= TOL["bf16"], f"expert {e}"


# steps of the down-projection: 3, 4 + 1, 4 + 2, 4 + 3 (rounds of four, and what does not fill one)
@pytest.mark.parametrize("f", [192, 320, 384, 448])
def test_expert_ffn_every_tile_height_of_the_wide_down_projection(f):
    """32 experts x 16 column groups: tiles of 1 to 16 blocks in units of 64 columns and, with fewer than 192 rows per expert, the sorted list, where the
    up-projection has few items and so lower tiles and a list of its own."""
    counts = [16 * b - b % 3 for b in range(1, 17)] * 2
    up, down, narrow = heights(sum(counts), 4096, f, 32)
    assert up <= 96 and down == 256 and not narrow
    _ffn_by_expert(counts, 4096, f, seed=f)


def test_expert_ffn_tall_tiles_in_a_merged_work_list():
    """More than 224 rows per expert and a column group for every compute unit: the down-projection's tiles have 256 rows, experts of several
    among experts of one, beside an up-projection of tiles of 64."""
    counts = [700, 256, 513, 230, 257, 100, 768, 144, 260, 200, 300, 176, 512, 60, 1000, 0]
    assert heights(sum(counts), 4096, 192, 16) == (64, 256, False)
    _ffn_by_expert(counts, 4096, 192, seed=7)


@pytest.mark.parametrize("d,f", [(192, 640), (704, 320)])
def test_f32_rows_keep_their_bits_in_every_tile_height(d, f):
    """Blocks of 64, 32 and 16 rows, of all the columns and of half: a row has the same bits in a batch of 1500 rows as in short ones."""
    x = _normal(1500, d, seed=8)
    ex = [_normal(*s, seed=9 + i) * 0.05 for i, s in enumerate(((d, f), (d, f), (f, d)))]

    def run(rows):
        T = len(rows)
        cfg = M.MoeCfg.make(T, d, f, 1, 1, "f32")
        packed = torch.empty((1, M.moe_expert_bytes(cfg)), dtype=torch.uint8, device="cuda")
        M.moe_pack_weights(cfg, *ex, packed[0])
        Y = torch.full((T, d), float("nan"), device="cuda")
        M.moe_expert_ffn(cfg, rows, torch.tensor([0, T], dtype=torch.int32, device="cuda"), packed, Y,
                         torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        return Y
    want = run(x)
    assert torch.isfinite(want).all()
    for n in (1, 17, 40, 100, 333, 700):
        assert torch.equal(run(x[:n].clone()), want[:n]), f"{n} rows"


def test_expert_ffn_tiles_of_more_than_256_rows_in_long_reductions():
    """17 to 20 blocks of 16 rows, whose last sums lie in other registers than the rest, at their edges, alone and among several tiles of one expert, in 64 and 35 steps."""
    _tall_ffn([257, 272, 273, 288, 289, 304, 305, 320, 321, 576, 560, 960], 4096, 2240, 17, 5250, (320, 320, False))


@pytest.mark.parametrize("T,d,E,k,renorm", [(1, 64, 4, 1, 1), (7, 192, 4, 2, 0), (33, 320, 12, 3, 0), (70, 1088, 64, 2, 1), (50, 2112, 68, 1, 0), (20, 448, 256, 8, 0),
                                            (4099, 128, 8, 2, 0), (4100, 192, 100, 2, 1)])
def test_f32_gate_by_four_columns(T, d, E, k, renorm):
    """Gate matrices of a multiple of four columns, read four at a time: the experts are those of 64-bit arithmetic and the weights within the order of sums of d
    products (some d / 64 + 40 roundings of the logits, doubled); and an equal matrix 4, 8 or 12 bytes past a 16-byte boundary gives the same bits."""
    x, W = _normal(T, d, seed=21), _normal(d, E, seed=22) * d ** -0.5
    W[:, 1] = W[:, 0]                                # a tie in every token
    bias = 0.1 * _normal(E, seed=23)
    bias[1] = bias[0]
    cfg = M.MoeCfg.make(T, d, 64, E, k, "f32", renorm)
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    out = []
    for shift in (0, 1, 2, 3):
        Wg = torch.empty(d * E + shift, device="cuda")[shift:].view(d, E)
        Wg.copy_(W)
        assert Wg.data_ptr() % 16 == 4 * shift
        idx, w = torch.full((T, k), -1, dtype=torch.int32, device="cuda"), torch.empty((T, k), device="cuda")
        M.moe_route(cfg, x, Wg, bias, idx, w, ws)
        torch.cuda.synchronize()
        out.append((idx, w))
    logits = x.double() @ W.double() + bias.double()
    top = logits.sort(dim=1, descending=True, stable=True)
    assert torch.equal(out[0][0].long(), top.indices[:, :k])
    for idx, w in out[1:]:
        assert torch.equal(idx, out[0][0]) and torch.equal(w, out[0][1])
    want = top.values[:, :k].softmax(1) if renorm else (top.values[:, :k] - logits.logsumexp(1, keepdim=True)).exp()
    bound = 2 * (d / 64 + 40) * 2.0 ** -24 * float(x.norm(dim=1).max() * W.norm(dim=0).max()) + 1e-6
    assert ((out[0][1].double() - want).abs() <= bound * want).all()


# two quads of four terms per lane at most, and more: 1, 2, 4, 8, 16 and 32 lanes of four columns
@pytest.mark.parametrize("d,E", [(512, 4), (576, 4), (256, 8), (320, 8), (128, 12), (192, 12), (64, 32), (128, 32), (64, 64), (64, 100), (1088, 8)])
def test_f32_gate_keeps_its_bits_in_every_batch(d, E):
    """A wave per token with two or eight quads of terms requested at a time, with four from the third block per compute unit on, and four tokens per wave beyond 4096:
    the experts are those of 64-bit arithmetic, and a token has the same weights, bit for bit, in all of them."""
    T, k = 4101, 2
    x, W = _normal(T, d, seed=24), _normal(d, E, seed=25) * d ** -0.5
    out = []
    for n in (T, 4096, 2049, 2048, 5):
        cfg = M.MoeCfg.make(n, d, 64, E, k, "f32", 0)
        idx, w = torch.full((n, k), -1, dtype=torch.int32, device="cuda"), torch.empty((n, k), device="cuda")
        M.moe_route(cfg, x[:n], W, None, idx, w, torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        out.append((idx, w))
    logits = x.double() @ W.double()
    top = logits.sort(dim=1, descending=True, stable=True)
    assert torch.equal(out[0][0].long(), top.indices[:, :k])
    want = (top.values[:, :k] - logits.logsumexp(1, keepdim=True)).exp()
    bound = 2 * (d / 64 + 40) * 2.0 ** -24 * float(x.norm(dim=1).max() * W.norm(dim=0).max()) + 1e-6       # (the order of the sums, as above)
    assert ((out[0][1].double() - want).abs() <= bound * want).all()
    for idx, w in out[1:]:
        assert torch.equal(idx, out[0][0][:len(idx)]) and torch.equal(w, out[0][1][:len(w)])


@pytest.mark.parametrize("T,d,E,k,renorm", [(15570, 64, 33, 1, 1), (15571, 192, 64, 2, 0), (16400, 1088, 40, 3, 1), (33000, 576, 50, 2, 0)])
def test_gate_with_two_blocks_per_compute_unit(T, d, E, k, renorm):
    """Long batches on 33 to 64 experts: the experts are those of 64-bit arithmetic (two columns tie in every token, so close ones are in every block), and
    a token has the same weights, bit for bit, as in a short batch."""
    x, W = _normal(T, d, seed=31).bfloat16(), (_normal(d, E, seed=32) * d ** -0.5).bfloat16()
    W[:, E - 1] = W[:, E // 2]

    def route(x):
        n = x.shape[0]
        cfg = M.MoeCfg.make(n, d, 64, E, k, "bf16", renorm)
        idx, w = torch.full((n, k), -1, dtype=torch.int32, device="cuda"), torch.full((n, k), float("nan"), device="cuda")
        M.moe_route(cfg, x, W, None, idx, w, torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        return idx, w
    idx, w = route(x)
    logits = x.double() @ W.double()
    logits[:, E - 1] = logits[:, E // 2]             # (the same sum, whatever order the product above adds in)
    assert torch.equal(idx.long(), logits.sort(dim=1, descending=True, stable=True).indices[:, :k])
    for lo in (0, T // 2, T - 300):
        short = route(x[lo:lo + 300].clone())
        assert torch.equal(short[0], idx[lo:lo + 300]) and torch.equal(short[1], w[lo:lo + 300])


@pytest.mark.parametrize("T,d,E,k,renorm,gate", [(1, 64, 1, 1, 1, "topk"), (9, 512, 33, 2, 0, "topk"), (300, 448, 32, 1, 0, "topk"), (515, 320, 64, 3, 1, "topk"),
                                                 (4080, 128, 31, 2, 0, "topk"), (77, 512, 64, 1, 1, "hash"), (40, 64, 16, 1, 1, "hash"), (33, 576, 40, 2, 0, "topk")])
def test_gate_matrix_as_it_is(T, d, E, k, renorm, gate):
    """A gate that the call reads as it is, 2 bytes off any boundary, against the same gate packed: the same experts and the same bits, ties and all columns in
    reach included (d 576: the limit, packed by the call)."""
    cols = E if gate == "topk" else E.bit_length() - 1
    x, W = _normal(T, d, seed=41).bfloat16(), (_normal(d, cols, seed=42) * d ** -0.5).bfloat16()
    W[:, cols - 1] = W[:, 0]
    x[T // 2] = 0                                    # every column ties
    shifted = torch.empty(d * cols + 1, dtype=torch.bfloat16, device="cuda")[1:].view(d, cols)
    shifted.copy_(W)
    cfg = M.MoeCfg.make(T, d, 64, E, k, "bf16", renorm, 0, M.GATE_HASH if gate == "hash" else M.GATE_TOPK)
    block = torch.empty(M.moe_gate_bytes(cfg), dtype=torch.uint8, device="cuda")
    M.moe_pack_gate(cfg, W, block)
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    out = []
    for c, Wg in ((cfg, shifted), (cfg.with_packed_gate(True), block)):
        idx, w = torch.full((T, k), -1, dtype=torch.int32, device="cuda"), torch.full((T, k), float("nan"), device="cuda")
        M.moe_route(c, x, Wg, None, idx, w, ws)
        torch.cuda.synchronize()
        out.append((idx, w))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert out[0][0].min() >= 0 and out[0][0].max() < E and torch.isfinite(out[0][1]).all()


@pytest.mark.parametrize("T,E,d,f,crowd", [(2000, 16, 256, 10240, 700), (2000, 16, 256, 10240, 1500), (2500, 16, 64, 10240, 2449), (2560, 16, 1024, 4096, 2048)])
@pytest.mark.parametrize("mode", ["ascending", "greedy", "kept"])
def test_streamed_crowded_expert_equals_resident(T, E, d, f, crowd, mode):
    """A layer of few rows per expert, whose streamed experts look their rows up in x, with most of them on one: every row has the bytes of the resident call."""
    heavy = 5
    want = torch.tensor([heavy] * crowd + [e for i in range(T) for e in [i % E] if e != heavy][:T - crowd], device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(T + crowd)
    want = want[torch.randperm(T, generator=g, device="cuda")]
    x = _normal(T, d, seed=51)
    x[:, :E] = 4.0 * torch.nn.functional.one_hot(want, E)
    x, Wg = x.bfloat16(), torch.eye(d, E, device="cuda").bfloat16()
    cfg = M.MoeCfg.make(T, d, f, E, 1, "bf16")
    packed = torch.empty((E, M.moe_expert_bytes(cfg)), dtype=torch.uint8, device="cuda")
    for e in range(E):
        M.moe_pack_weights(cfg, *((_normal(*s, seed=60 + 3 * e + i) * 0.05).bfloat16() for i, s in enumerate(((d, f), (d, f), (f, d)))), packed[e])
    host = torch.empty(packed.shape, dtype=torch.uint8, pin_memory=True)
    host.copy_(packed)

    def run(ctx):
        ws = torch.full((M.moe_workspace_bytes(cfg) // 2,), float("nan"), dtype=torch.bfloat16, device="cuda").view(torch.uint8)
        y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        M.moe_layer_forward(cfg, x, Wg, None, None if ctx else packed, ctx, y, ws)
        torch.cuda.synchronize()
        return y
    resident = run(None)
    assert torch.isfinite(resident).all()
    K = 4
    ctx = M.StreamCtx(cfg, host, torch.empty((K, packed.shape[1]), dtype=torch.uint8, device="cuda"), K)
    if mode == "greedy":
        ctx.set_order(M.ORDER_GREEDY, 100.0, 2)
    if mode == "kept":
        ctx.keep_experts(True)
    for _ in range(2):
        y = run(ctx)
        wrong = (y.view(torch.int16) != resident.view(torch.int16)).any(1).sum().item()
        assert wrong == 0, f"{wrong} rows differ"
    ctx.close()
