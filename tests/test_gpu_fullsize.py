"""Parity at the full sizes of the measured configurations, in the launch configuration the bench
times (resident moe_layer_forward; host-streamed for the offload case).

What the layer computes is fixed by Section 2.1 (every token goes to the expert its gate picks, whose
output stands in for the FFN output), Section 6.2 (tokens batched by expert) and Table 1 (d_model 4096,
d_ff 10240, three matrices per expert).  Routing, counts, offsets and the permutation are compared with
the oracle in full and bit for bit.  At T 2048 / 8 experts and T 4096 / 32 experts (and the streamed
T 512 / T 8192 runs of the same layer) the WHOLE of Yp and y is compared with the fp64 oracle, expert by
expert: normalised L2 per expert segment, per row (worst row printed) and over the whole tensor.  At the
two large workloads the oracle evaluates the rows at every tile seam of a few experts (first and last
row of each row tile the kernel cuts the segment into, the start of the last 32-row block, random rows)
and whole tokens whose experts are among them; y is always checked against what the oracle makes of its
own Yp, weights and inverse permutation.  The fused entry point must reproduce the staged calls bit
for bit."""
import numpy as np
import pytest
import torch

import moe_workloads as W
import paper_2106_10715_amd as M
from oracle import moe_oracle as O
from paper_2106_10715_amd import harness as H
from tile_rows import heights

pytestmark = pytest.mark.gpu

TOL = 1e-2          # normalised L2 of bf16 outputs against the fp64 oracle on the same stored inputs


def rel_l2(got, ref):
    den = np.linalg.norm(ref)
    return float(np.linalg.norm(np.asarray(got, np.float64) - ref) / (den if den > 0 else 1.0))


def row_l2(got, ref):
    """Normalised L2 of every row."""
    den = np.linalg.norm(ref, axis=1)
    return np.linalg.norm(np.asarray(got, np.float64) - ref, axis=1) / np.where(den > 0, den, 1.0)


def staged(L):
    cfg, T, A = L.cfg, L.wl.T, L.wl.A
    t = lambda shape, dt: torch.empty(shape, dtype=dt, device="cuda")
    s = dict(idx=t((T, cfg.k), torch.int32), w=t((T, cfg.k), torch.float32), counts=t(cfg.E, torch.int32),
             offsets=t(cfg.E + 1, torch.int32), perm=t(A, torch.int32), inv=t(A, torch.int32),
             Xp=t((A, cfg.d), cfg.torch_dtype), Yp=t((A, cfg.d), cfg.torch_dtype), y=t((T, cfg.d), cfg.torch_dtype))
    M.moe_route(cfg, L.x, L.Wg, L.bias, s["idx"], s["w"], L.ws)
    M.moe_permute(cfg, L.x, s["idx"], s["counts"], s["offsets"], s["perm"], s["inv"], s["Xp"], L.ws)
    M.moe_expert_ffn(cfg, s["Xp"], s["offsets"], L.packed, s["Yp"], L.ws)
    M.moe_combine(cfg, s["Yp"], s["inv"], s["w"], s["y"])
    torch.cuda.synchronize()
    return s


def check_integers(wl, s, x, Wg, bias):
    """Gate and batching against the oracle, everything, bit for bit (weights to fp32 accuracy)."""
    r = O.route(x, Wg, wl.k, bias, wl.renorm)
    p = O.permute(x, r.idx, wl.E)
    print(f"\n[{wl.name}] min routing margin {r.margin.min():.3e}; counts max {p.counts.max()} min {p.counts.min()} "
          f"empty {(p.counts == 0).sum()}")
    assert np.array_equal(s["idx"].cpu().numpy(), r.idx)
    assert rel_l2(s["w"].cpu().numpy(), r.w) <= 1e-5
    assert np.array_equal(s["counts"].cpu().numpy(), p.counts)
    assert np.array_equal(s["offsets"].cpu().numpy(), p.offsets)
    assert np.array_equal(s["perm"].cpu().numpy(), p.perm)
    assert np.array_equal(s["inv"].cpu().numpy(), p.inv)
    rng = np.random.default_rng(wl.seed)
    rows = rng.choice(wl.A, size=min(wl.A, 1500), replace=False)
    assert np.array_equal(H.to_f64(s["Xp"][torch.from_numpy(rows).cuda()]), p.Xp[rows])
    if wl.n_dead:
        assert (p.counts == 0).sum() >= wl.n_dead
    return r, p


def oracle_whole_layer(wl, x, r, p):
    """Yp and y of the whole batch by the oracle, one expert's weights in memory at a time."""
    pool = W.make_pool()
    try:
        Yp = O.expert_ffn(p.Xp, p.offsets, lambda e: W.gen_expert(wl, e, pool))
    finally:
        pool.shutdown()
    return Yp, O.combine(Yp, p.inv, r.w)


def compare_whole(name, what, got, ref, offsets=None):
    """Whole tensor, every expert segment (if offsets are given) and every row within TOL; prints the worst."""
    total = rel_l2(got, ref)
    rows = row_l2(got, ref)
    worst = int(rows.argmax())
    msg = f"[{name}] {what}: whole tensor {total:.3e}, worst row {worst} {rows[worst]:.3e}"
    if offsets is not None:
        seg = [(rel_l2(got[lo:hi], ref[lo:hi]), e) for e, (lo, hi) in enumerate(zip(offsets[:-1], offsets[1:])) if hi > lo]
        msg += f", worst expert segment {max(seg)[1]} {max(seg)[0]:.3e}"
        assert max(seg)[0] <= TOL, msg
    print(msg)
    assert total <= TOL and rows[worst] <= TOL, msg


def check_whole(wl, L):
    """Every element of Yp and y against the oracle (the workloads the oracle finishes in seconds)."""
    x = W.gen_x(wl)
    Wg, bias = W.gen_gate(wl)
    s = staged(L)
    M.moe_layer_forward(L.cfg, L.x, L.Wg, L.bias, L.packed, None, L.y, L.ws)
    torch.cuda.synchronize()
    assert torch.equal(L.y, s["y"]), "fused entry point differs from the staged calls"
    r, p = check_integers(wl, s, x, Wg, bias)
    Yp_ref, y_ref = oracle_whole_layer(wl, x, r, p)
    compare_whole(wl.name, "Yp", H.to_f64(s["Yp"]), Yp_ref, p.offsets)
    compare_whole(wl.name, "y", H.to_f64(L.y), y_ref)
    return s


def seam_rows(n, limits):
    """Rows of an n-row expert segment at the seams of the kernels' tiling: for each limit, its blocks of 16 rows spread evenly over as few tiles as that many rows
    allow; first and last row of every tile, and the start of the last 32-row block."""
    out = {0, n - 1, (n - 1) // 32 * 32}
    for limit in limits:
        tiles, blocks = -(-n // limit), -(-n // 16)
        for t in range(tiles):
            lo, hi = ((i * (blocks // tiles) + min(i, blocks % tiles)) * 16 for i in (t, t + 1))
            out |= {lo, min(hi, n) - 1}
    return out


def check_sampled(wl, L, n_experts=4, random_rows=6, n_tokens=48):
    """The large workloads: integers in full; Yp on the seam rows and random rows of a few experts (the two
    heaviest, the lightest, random ones); y on whole tokens all of whose experts are among those, built from
    the oracle's own Yp rows, weights and inverse permutation."""
    rng = np.random.default_rng(wl.seed)
    x = W.gen_x(wl)
    Wg, bias = W.gen_gate(wl)
    s = staged(L)
    M.moe_layer_forward(L.cfg, L.x, L.Wg, L.bias, L.packed, None, L.y, L.ws)
    torch.cuda.synchronize()
    assert torch.equal(L.y, s["y"]), "fused entry point differs from the staged calls"
    assert bool(torch.isfinite(s["y"].float()).all())
    r, p = check_integers(wl, s, x, Wg, bias)

    live = np.nonzero(p.counts > 0)[0]
    by_load = live[np.argsort(-p.counts[live], kind="stable")]
    pick = [int(by_load[0]), int(by_load[1]), int(by_load[-1])]
    pick += [int(e) for e in rng.choice(live, size=min(len(live), n_experts), replace=False)]
    pick = sorted(set(pick))
    inv2 = p.inv.reshape(wl.T, wl.k)
    in_pick = np.isin(r.idx, pick).all(axis=1)
    toks = np.nonzero(in_pick)[0]
    toks = np.sort(rng.choice(toks, size=min(len(toks), n_tokens), replace=False))
    assert len(toks) > 0
    need = {e: set() for e in pick}
    for t in toks:
        for j in range(wl.k):
            need[int(r.idx[t, j])].add(int(inv2[t, j]))
    pool = W.make_pool()
    limits = set(heights(wl.T, wl.d, wl.f, wl.E, wl.k)[:2])
    Yp_ref = {}                                   # batched row -> oracle output row
    worst_row, n_rows = 0.0, 0
    try:
        for e in pick:
            lo, hi = int(p.offsets[e]), int(p.offsets[e + 1])
            rows = {lo + v for v in seam_rows(hi - lo, limits)} | {int(v) for v in rng.integers(lo, hi, size=random_rows)} | need[e]
            rows = np.array(sorted(rows))
            ref = O.expert_ffn_rows(p.Xp[rows], *W.gen_expert(wl, e, pool))
            got = H.to_f64(s["Yp"][torch.from_numpy(rows).cuda()])
            err = row_l2(got, ref)
            assert err.max() <= TOL, f"expert {e} ({hi - lo} rows): row {rows[err.argmax()] - lo} normalised L2 {err.max():.3e}"
            assert rel_l2(got, ref) <= TOL
            worst_row = max(worst_row, float(err.max()))
            n_rows += len(rows)
            Yp_ref.update({int(rw): ref[i] for i, rw in enumerate(rows)})
    finally:
        pool.shutdown()
    y_ref = np.zeros((len(toks), wl.d))
    for i, t in enumerate(toks):
        for j in range(wl.k):
            y_ref[i] += np.float64(r.w[t, j]) * Yp_ref[int(inv2[t, j])]
    y_got = H.to_f64(L.y[torch.from_numpy(toks).cuda()])
    y_err = row_l2(y_got, y_ref)
    assert y_err.max() <= TOL and rel_l2(y_got, y_ref) <= TOL
    print(f"[{wl.name}] {n_rows} Yp rows of experts {pick} (all tile seams): worst row {worst_row:.3e}; "
          f"{len(toks)} whole tokens of y against the oracle's own Yp: worst {y_err.max():.3e}")
    return s


@pytest.fixture(scope="module")
def c3_layer():
    L = H.build_layer(W.CONFIGS["c3"], host_copy=True)
    yield L
    del L
    torch.cuda.empty_cache()


def test_c2_resident_full_size():
    wl = W.CONFIGS["c2"]
    L = H.build_layer(wl)
    check_whole(wl, L)
    del L
    torch.cuda.empty_cache()


def test_c3_resident_full_size(c3_layer):
    check_whole(W.CONFIGS["c3"], c3_layer)


@pytest.mark.parametrize("name", ["c4a", "c4b"])
def test_c4_streamed_equals_resident_full_size(c3_layer, name):
    wl = W.CONFIGS[name]                        # same weights as c3 (same seed), other token counts
    base = c3_layer
    cfg = H.cfg_of(wl)
    xs = W.gen_x(wl)
    x = H.to_device(xs, wl.dtype)
    ws = torch.empty(M.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    y_res = torch.empty((wl.T, wl.d), dtype=torch.bfloat16, device="cuda")
    y_str = torch.full((wl.T, wl.d), float("nan"), dtype=torch.bfloat16, device="cuda")
    M.moe_layer_forward(cfg, x, base.Wg, None, base.packed, None, y_res, ws)
    slots = torch.empty((2, M.moe_expert_bytes(cfg)), dtype=torch.uint8, device="cuda")
    ctx = M.StreamCtx(cfg, base.host_packed, slots, 2)
    for _ in range(2):
        M.moe_layer_forward(cfg, x, base.Wg, None, None, ctx, y_str, ws)
        torch.cuda.synchronize()
        assert torch.equal(y_str, y_res)
    st = ctx.stats()
    print(f"\n[{wl.name}] streamed: {st['n_loaded']} experts, {st['bytes'] / st['copy_ms'] / 1e6:.1f} GB/s over the copy window")
    ctx.close()
    # and the streamed result is the layer's: every element of y against the oracle
    Wg, _ = W.gen_gate(wl)
    r = O.route(xs, Wg, 1)
    p = O.permute(xs, r.idx, wl.E)
    _, y_ref = oracle_whole_layer(wl, xs, r, p)
    compare_whole(wl.name, "y (streamed)", H.to_f64(y_str), y_ref)


def test_c5_zipf_top2_full_size():
    wl = W.CONFIGS["c5"]
    L = H.build_layer(wl)
    s = check_sampled(wl, L, n_experts=3)
    counts = s["counts"].cpu().numpy()
    assert counts.max() > 20 * max(1, counts[counts > 0].min())      # the load really is skewed
    del L
    torch.cuda.empty_cache()


def test_c6_token_throughput_regime_full_size():
    wl = W.CONFIGS["c6"]
    L = H.build_layer(wl)
    s = check_sampled(wl, L, n_experts=2)
    counts = s["counts"].cpu().numpy()
    assert counts.min() > 1500                                       # every expert is in the compute-bound regime
    del L
    torch.cuda.empty_cache()


def test_largest_batch_the_index_range_allows():
    """T*k*d_ff just below 2^31 (the library's documented limit) on the 32-expert layer: 209715 tokens, a ragged last
    block everywhere.  Integers in full, tile-seam rows and whole tokens against the oracle as for the other large workloads."""
    wl = W.CONFIGS["c3"].with_tokens((2 ** 31 - 1) // 10240)
    assert wl.T == 209715 and wl.T * wl.f < 2 ** 31 <= (wl.T + 1) * wl.f
    L = H.build_layer(wl)
    s = check_sampled(wl, L, n_experts=2, n_tokens=32)
    assert int(s["offsets"][-1]) == wl.T
    with pytest.raises(M.MoeError, match="2\\^31"):
        M.moe_workspace_bytes(H.cfg_of(wl.with_tokens(wl.T + 1)))
    del L, s
    torch.cuda.empty_cache()
