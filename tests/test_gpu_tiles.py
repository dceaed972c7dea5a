"""Kernel edges against the oracle: tile remainders, the smallest and the largest of a
kernel's range, and either side of a dispatch rule."""

import ctypes

import numpy as np
import pytest
import torch

from oracle import exfold_oracle as O
from paper_2608_24938_amd import exfold as X
from paper_2608_24938_amd import synth

from .gpu_common import TOL_Y, LayerPair, from_dev, logits_bound, per_token_rel_l2, sync, to_dev

pytestmark = pytest.mark.gpu


def _shape(d, inter, n, k, dtype="f32", shared=0, bias=False):
    return synth.LayerShape("edge", d=d, inter=inter, n_experts=n, top_k=k, dtype=dtype, shared_inter=shared,
                            router_bias=bias)


# Gram tiles of 16 rows: 16, 8, 5 (padded to 8), 3 (padded to 4) and 1 rows a token with ragged token
# counts; more than 16 rows a token (common mode: two tiles a side, the second ragged; nine tiles a side);
# a router bias that gives some experts no token and some several m-tiles of rows.
@pytest.mark.parametrize("n,k,m,mode", [(4, 1, 1, "corouted"), (20, 1, 33, "corouted"), (20, 3, 37, "corouted"),
                                        (24, 5, 131, "corouted"), (64, 8, 301, "corouted"),
                                        (40, 16, 50, "corouted"), (20, 2, 19, "common"), (17, 2, 70, "common"),
                                        (130, 2, 9, "common"), (256, 16, 40, "corouted")])
def test_calibration_at_tile_edges(n, k, m, mode):
    shape = _shape(256, 64, n, k, bias=True)
    lp = LayerPair(shape, seed=n + k)
    xs = synth.calibration_tokens(shape, m, seed=n + k)
    print(f"calibration edge: N={n} K={k} m={m} {mode}", flush=True)
    S, L, h, st = X.calibrate_projectors(lp.dev, to_dev(xs), mode=mode, with_stats=True)
    S2, L2, h2 = X.calibrate_projectors(lp.dev, to_dev(xs), mode=mode)
    sync()
    assert torch.equal(S, S2) and torch.equal(L, L2) and torch.equal(h, h2)
    rS, rL, rh, rst = O.calibrate(lp.ref, synth.widen(xs), k, lam=1e-3, clip=4.0, mode=mode)
    st = st.cpu().numpy()
    np.testing.assert_array_equal(st[..., 3], rst["n"])
    # the expert rows are float32 sums (about 1e-6 each); statistics and scalars are float64 from there
    tol = 1e-4
    for q, key in enumerate("AVC"):
        np.testing.assert_allclose(st[..., q], rst[key], rtol=tol, atol=tol * np.abs(rst[key]).max())
    np.testing.assert_allclose(S.cpu().numpy(), rS, rtol=tol, atol=tol * max(1.0, np.abs(rS).max()))
    obs = rst["n"] > 0
    np.testing.assert_array_equal(L.cpu().numpy()[~obs], rL[~obs])
    np.testing.assert_allclose(L.cpu().numpy()[obs], rL[obs], rtol=tol, atol=tol)
    np.testing.assert_allclose(h.cpu().numpy(), rh, rtol=tol)


SIMT, TILE, SKINNY, WIDE = range(4)


def _plan(d, inter, n, k, T, shared=0, dtype=X.BF16):
    """(kind, rows a tile, ranges of the reduction) of the gate/up and the down GEMM of moe_execute."""
    out = (ctypes.c_int32 * 10)()
    ly = X._Layer(d, inter, n, k, shared, dtype, 0, 0x10000, None, 0x10000, 0x10000, *[0x10000 if shared else None] * 2)
    rows, active = T * k + (T if shared else 0), min(n, T * k) + (1 if shared else 0)
    assert X.lib().exfold_gemm_plan(ctypes.byref(ly), rows, active, 256, out) == X.OK
    direct = k == 1 and not shared  # one row a token: the down reduction is not split
    return (out[0], out[1], out[3]), (out[5], out[6], 1 if direct else out[8])


def _execute(shape, T, ids, seed):
    """moe_execute on given routes against the oracle: the largest per-token error."""
    lp = LayerPair(shape, seed=seed)
    rng = np.random.default_rng(seed)
    w = rng.standard_normal(ids.shape).astype(np.float32)
    xs = synth.tokens(shape, T, seed=seed)
    print(f"execute: {shape.dtype} d={shape.d} I={shape.inter} N={shape.n_experts} routes={ids.shape}", flush=True)
    y = X.moe_execute(lp.dev, to_dev(xs), to_dev(ids), to_dev(w))
    sync()
    ref = O.moe_output(lp.ref, synth.widen(xs), ids, w)
    return per_token_rel_l2(from_dev(y), ref).max()


def _skewed(T, k, n, seed):
    """Route ids [T, k], half of them on expert 0 (ragged groups, some empty)."""
    rng = np.random.default_rng(seed)
    ids = rng.integers(0, n, size=(T, k)).astype(np.int32)
    ids[rng.random((T, k)) < 0.5] = 0
    return ids


# float32 tiles of 16, 32 and 64 rows: either side of 16 and 32 rows per busy expert, one
# row, ragged groups, the shared expert, a reduction of one step a wave (d 128, I 64) and a
# ragged last batch of steps (d 640: ten steps a wave; I 320: five).
@pytest.mark.parametrize("d,inter,n,k,shared,T,bm", [(128, 64, 5, 1, 0, 1, 16), (128, 64, 5, 2, 0, 40, 16),
                                                     (128, 64, 5, 2, 0, 41, 32), (640, 320, 5, 2, 320, 64, 32),
                                                     (640, 320, 5, 2, 320, 79, 64), (640, 320, 5, 2, 0, 80, 32),
                                                     (640, 320, 5, 2, 0, 81, 64), (256, 192, 3, 1, 192, 333, 64),
                                                     (1024, 576, 8, 2, 0, 1100, 64)])
def test_float32_tiles(d, inter, n, k, shared, T, bm):
    shape = _shape(d, inter, n, k, shared=shared)
    assert _plan(d, inter, n, k, T, shared, X.F32) == ((SIMT, bm, 1),) * 2
    assert _execute(shape, T, _skewed(T, k, n, T), seed=3) <= TOL_Y["f32"]


# More routes a token than the combine holds in registers (17 rows, the shared one among them): either side
# of that, bf16 rows and split float32 partials (I = 4096), a ragged last step of four.
@pytest.mark.parametrize("d,inter,n,k,shared,T,dtype", [
    (256, 64, 5, 16, 64, 3, "bf16"), (256, 64, 5, 17, 0, 3, "bf16"), (256, 64, 5, 17, 64, 3, "bf16"),
    (256, 64, 24, 18, 0, 9, "f32"), (1152, 192, 40, 33, 192, 7, "bf16"), (128, 4096, 4, 19, 0, 2, "bf16"),
    (128, 64, 256, 300, 0, 2, "f32")])
def test_execute_of_many_routes(d, inter, n, k, shared, T, dtype):
    ids = np.random.default_rng(k).integers(0, n, size=(T, k)).astype(np.int32)
    shape = _shape(d, inter, n, min(k, n, 16), dtype=dtype, shared=shared)
    assert _execute(shape, T, ids, seed=6) <= TOL_Y[dtype]


# float32 router: N <= 32 in the routing kernel up to 1024 tokens (8, 16 and 32 experts a
# build), 16 x 16 tiles beyond either limit.
@pytest.mark.parametrize("n,T,d", [(7, 1, 128), (13, 5, 1152), (32, 33, 640), (33, 17, 384), (32, 1024, 128),
                                   (32, 1025, 128), (6, 1031, 256)])
def test_float32_router_logits(n, T, d):
    shape = _shape(d, 64, n, 2, bias=True)
    lp = LayerPair(shape, seed=n)
    xs = synth.tokens(shape, T, seed=n)
    dbg = X.debug_buffers(lp.dev, T, "dense", 0, "cuda:0")
    print(f"router f32: N={n} T={T} d={d}", flush=True)
    X.moe_forward(lp.dev, to_dev(xs), "dense", debug=dbg)
    sync()
    got = dbg["logits"].cpu().numpy()
    ref = O.router_logits(xs, lp.ref.w_router, lp.ref.router_bias)
    assert np.all(np.abs(got.astype(np.float64) - ref) <= logits_bound(xs, lp.ref.w_router, lp.ref.router_bias, d))
    r_ids, _ = O.route(got, 2)
    np.testing.assert_array_equal(dbg["topk_ids"].cpu().numpy(), r_ids)


# Wide tiles: full tiles (129 to 256 rows of the last 256) and 128 x 512 tails (1 to 128 rows)
# either side of every 32-row block, reductions of two stages (d 128, gate/up only), eight (d 512)
# and split ones of even and odd lengths (I 2048 and 2816 in the last, partial round of the down
# projection), outputs straight to y (one route a token) and as bf16 rows.
@pytest.mark.parametrize("d,inter,k", [(128, 2048, 1), (512, 2048, 1), (512, 2816, 2), (1024, 1536, 2)])
def test_wide_tile_edges(d, inter, k):
    sizes = [129, 160, 161, 192, 193, 224, 225, 256, 257, 288, 289, 320, 321, 352, 353, 384, 1, 32, 33, 64, 65, 96,
             97, 128, 0, 700]
    sizes[-1] += sum(sizes) % k
    ids = np.random.default_rng(d).permutation(np.repeat(np.arange(len(sizes)), sizes)).astype(np.int32)
    ids = ids.reshape(-1, k)
    shape = _shape(d, inter, len(sizes), k, dtype="bf16")
    gu, dn = _plan(d, inter, len(sizes), k, ids.shape[0])
    assert gu[0] == WIDE and dn[0] == (WIDE if d % 512 == 0 else TILE)
    assert _execute(shape, ids.shape[0], ids, seed=4) <= TOL_Y["bf16"]


# Skinny tiles of 32 rows (gate/up up to 12 rows per busy expert, or 24 where there are at most four
# tiles a CU), of 64 (gate/up up to 24, down up to 48) and 64-row down tiles (up to 80), each case with the
# tiles it is there for: groups of 0, 1, 32, 33, 64, 65 and more rows; reductions that end in half a
# 128-column stage (I = 192, 320, 704), of one stage (I = 128) and below one (I = 64); one and several
# routes a token, the shared expert, a split down reduction (I = 4096; I = 1728 and 4160: ranges that end in
# half a stage).
_EDGES64 = [64, 65, 0, 33, 32, 1, 63, 2, 31, 0, 5, 0, 0, 0, 1, 0]


@pytest.mark.parametrize("d,inter,sizes,k,shared,gu,dn", [
    (256, 192, [1, 0, 32, 33, 0, 2, 4, 0], 1, 0, (SKINNY, 32, 1), (SKINNY, 32, 1)),
    (256, 192, [1, 0, 12, 33, 0, 24, 9, 1], 2, 192, (SKINNY, 32, 1), (SKINNY, 32, 1)),
    (128, 320, [64, 65, 0, 32, 33, 1, 3, 2], 1, 0, (TILE, 128, 1), (SKINNY, 64, 1)),
    (384, 704, [64, 65, 0, 32, 33, 1, 3, 2], 2, 0, (TILE, 128, 1), (SKINNY, 64, 1)),
    (128, 128, [40, 30, 20, 60], 2, 128, (TILE, 128, 1), (SKINNY, 64, 1)),
    (256, 64, [20, 10, 5, 1], 1, 0, (SKINNY, 32, 1), (TILE, 64, 1)),
    (256, 64, [20, 10, 5, 1], 2, 0, (SKINNY, 32, 1), (TILE, 64, 1)),
    (256, 320, [64, 65, 63, 128, 129, 1], 2, 0, (TILE, 128, 1), (TILE, 64, 1)),
    (640, 192, [64, 65, 63, 128, 20, 1], 1, 0, (TILE, 128, 1), (TILE, 64, 1)),
    (128, 4096, [3, 1, 0, 4], 2, 0, (SKINNY, 32, 1), (SKINNY, 32, 4)),
    (128, 4160, [40, 50, 33, 65], 2, 0, (TILE, 128, 1), (SKINNY, 64, 5)),
    (512, 1728, [47] * 34, 2, 0, (TILE, 128, 1), (SKINNY, 64, 3)),
    # 64-row gate/up tiles (more than four 32-column tiles a CU): one stage of d, three, the shared expert
    (128, 2112, _EDGES64, 1, 0, (SKINNY, 64, 1), (SKINNY, 32, 1)),
    (384, 2112, _EDGES64, 2, 0, (SKINNY, 64, 1), (SKINNY, 32, 3)),
    (256, 2048, _EDGES64 + [10] * 16, 2, 2048, (SKINNY, 64, 1), (SKINNY, 32, 2)),
    # more than two 128-column down tiles a CU: 64-row tiles from 21 rows on average, skinny at 20
    (2048, 128, [21] * 33, 1, 0, (SKINNY, 32, 1), (TILE, 64, 1)),
    (2048, 192, [20] * 33, 1, 0, (SKINNY, 32, 1), (SKINNY, 64, 1)),
    (4096, 64, [64, 1, 0, 65, 33] * 7, 2, 0, (TILE, 128, 1), (TILE, 64, 1))])
def test_streaming_tile_edges(d, inter, sizes, k, shared, gu, dn):
    ids = np.random.default_rng(inter).permutation(np.repeat(np.arange(len(sizes)), sizes)).astype(np.int32)
    ids = ids[: len(ids) // k * k].reshape(-1, k)
    assert _plan(d, inter, len(sizes), k, ids.shape[0], shared) == (gu, dn)
    shape = _shape(d, inter, len(sizes), k, dtype="bf16", shared=shared)
    assert _execute(shape, ids.shape[0], ids, seed=5) <= TOL_Y["bf16"]


# One-workgroup permutation and decode front end: up to 1, 4 and 8 slots a thread (either side of 1024
# and 4096 slots, the largest), a last wave with one slot, one expert with every slot, 256 experts.
@pytest.mark.parametrize("T,K,n,phase", [(1, 1, 3, "execute"), (65, 1, 256, "execute"), (128, 8, 128, "execute"),
                                         (1025, 1, 7, "execute"), (1024, 4, 256, "execute"),
                                         (128, 8, 128, "decode"), (129, 8, 40, "decode"), (512, 8, 64, "decode"),
                                         (513, 8, 64, "decode"), (512, 16, 256, "decode"), (1024, 8, 9, "decode"),
                                         (16, 16, 256, "decode"), (17, 2, 128, "decode")])
def test_one_workgroup_permutation(T, K, n, phase):
    shape = _shape(128, 64, n, K, dtype="bf16", bias=True)
    lp = LayerPair(shape, seed=n + K)
    x = to_dev(synth.tokens(shape, T, seed=n))
    print(f"permutation: T={T} K={K} N={n} {phase}", flush=True)
    if phase == "execute":
        ids = np.zeros((T, K), np.int32) if n == 7 else _skewed(T, K, n, T)
        dbg = {"offsets": torch.empty(n + 2, dtype=torch.int32, device="cuda:0"),
               "row_slot": torch.empty(T * K, dtype=torch.int32, device="cuda:0")}
        X.moe_execute(lp.dev, x, to_dev(ids), to_dev(np.ones((T, K), np.float32)), debug=dbg)
    else:
        S, L, h = synth.synthetic_tables(n, seed=n)
        budget = max(2, n // 4)
        dbg = X.debug_buffers(lp.dev, T, phase, budget, "cuda:0")
        X.moe_forward(lp.dev, x, phase, budget, to_dev(S), to_dev(L), to_dev(h), debug=dbg)
    sync()
    g = {k: v.cpu().numpy() for k, v in dbg.items()}
    if phase == "decode":
        pool, _ = O.select_decode_pool(g["topk_ids"], g["topk_w"], h, n, budget)
        assert g["pool"][: int(g["pool_size"][0])].tolist() == pool
        ids, f_w, _, _ = O.fold_decode(g["topk_ids"], g["topk_w"], pool, S, L, n)
        np.testing.assert_array_equal(g["fold_ids"], ids)
        np.testing.assert_array_equal(g["fold_w"].view(np.uint32), f_w.view(np.uint32))
    _, offsets, row_slot = O.permute_routes(ids, n)
    np.testing.assert_array_equal(g["offsets"][: n + 1], offsets)
    np.testing.assert_array_equal(g["row_slot"], row_slot)


# Prefill fold by pairs of routes (K <= 8) and by one lane a route (K > 8): either side of 8, one
# route, every route or one retained, equal losses and losses of either zero (the first route wins).
@pytest.mark.parametrize("K,kp,opts", [(1, 1, {}), (2, 1, {}), (7, 3, dict(loss_cap=0.5)), (8, 1, {}), (8, 7, {}),
                                       (8, 8, {}), (8, 4, dict(confidence=True, renorm=True)), (9, 4, {}),
                                       (9, 1, dict(loss_cap=0.25, renorm=True))])
def test_fold_either_side_of_eight_routes(K, kp, opts):
    rng = np.random.default_rng(10 * K + kp)
    T, N = 67, 24
    ids = np.stack([rng.permutation(N)[:K] for _ in range(T)]).astype(np.int32)
    w = rng.dirichlet(np.ones(K), size=T).astype(np.float32)
    S = rng.standard_normal((N, N)).astype(np.float32)
    L = rng.choice(np.array([0.0, -0.0, 0.25, 0.5, 1.0, 1e30], np.float32), size=(N, N))
    keep = O.select_prefill(ids, w, rng.random(N).astype(np.float32), kp)
    print(f"fold: K={K} K'={kp} {opts}", flush=True)
    out_ids, out_w = X.fold_gates("prefill", kp, to_dev(ids), to_dev(w), to_dev(S), to_dev(L),
                                  keep=to_dev(keep.astype(np.uint8)), **opts)
    sync()
    if opts:
        ref_ids, ref_w = O.fold_prefill_safeguarded(ids, w, keep, S, L, **opts)
    else:
        ref_ids, ref_w = O.fold_prefill(ids, w, keep, S, L)
    np.testing.assert_array_equal(out_ids.cpu().numpy(), ref_ids)
    np.testing.assert_array_equal(out_w.cpu().numpy().view(np.uint32), ref_w.view(np.uint32))


# The first minimum under strict `<`, as the oracle scans: a NaN loss (of either sign) is taken only as the
# first candidate and loses to nothing then, is never within a cap, and an infinite loss is an ordinary value.
@pytest.mark.parametrize("K,kp", [(2, 1), (3, 2), (8, 1), (8, 3), (8, 7), (9, 3), (16, 5)])
@pytest.mark.parametrize("opts", [{}, dict(loss_cap=0.5), dict(loss_cap=float("inf"), renorm=True)])
def test_fold_of_nan_and_infinite_losses(K, kp, opts):
    rng = np.random.default_rng(100 * K + kp)
    T, N = 131, 24
    ids = np.stack([rng.permutation(N)[:K] for _ in range(T)]).astype(np.int32)
    w = rng.dirichlet(np.ones(K), size=T).astype(np.float32)
    S = rng.standard_normal((N, N)).astype(np.float32)
    nan = np.float32("nan")
    L = rng.choice(np.array([nan, -nan, nan, np.inf, -np.inf, -0.0, 0.25, 0.5, 1.0], np.float32), size=(N, N))
    keep = O.select_prefill(ids, w, rng.random(N).astype(np.float32), kp)
    print(f"fold with NaN: K={K} K'={kp} {opts}", flush=True)
    out_ids, out_w = X.fold_gates("prefill", kp, to_dev(ids), to_dev(w), to_dev(S), to_dev(L),
                                  keep=to_dev(keep.astype(np.uint8)), **opts)
    sync()
    if opts:
        ref_ids, ref_w = O.fold_prefill_safeguarded(ids, w, keep, S, L, **opts)
    else:
        ref_ids, ref_w = O.fold_prefill(ids, w, keep, S, L)
    np.testing.assert_array_equal(out_ids.cpu().numpy(), ref_ids)
    np.testing.assert_array_equal(out_w.cpu().numpy().view(np.uint32), ref_w.view(np.uint32))


# Router of many tokens and a multiple of 128 experts: 64-row tiles, a ragged last one.
@pytest.mark.parametrize("T,n,d", [(1009, 128, 256), (1088, 256, 1024), (2049, 128, 512)])
def test_tiled_router_logits(T, n, d):
    shape = _shape(d, 64, n, 4, dtype="bf16", bias=True)
    lp = LayerPair(shape, seed=n)
    xs = synth.tokens(shape, T, seed=n)
    dbg = X.debug_buffers(lp.dev, T, "dense", 0, "cuda:0")
    print(f"router bf16: N={n} T={T} d={d}", flush=True)
    X.moe_forward(lp.dev, to_dev(xs), "dense", debug=dbg)
    sync()
    x = synth.widen(xs)
    ref = O.router_logits(x, lp.ref.w_router, lp.ref.router_bias)
    got = dbg["logits"].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= logits_bound(x, lp.ref.w_router, lp.ref.router_bias, d))
