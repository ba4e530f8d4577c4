"""Calls with few rows, which run on smaller tiles and their own side-down pass: the kernels a call takes must not
show in its results."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import zo_block as ob
from oracle import zo_oracle as zo
from paper_2605_28760_amd import binding as zb
from paper_2605_28760_amd import workloads as wl
from paper_2605_28760_amd.runner import DeviceBatch, DeviceWorkload
from zo_testlib import assert_close, oracle_layer, to_np

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _layer(seed, lens, seq_cand, m, n, r, R, act, bias):
    """One bf16 probe linear over sequences of the given lengths; candidates 0..5 = (+, -) of three directions,
    6 = centre."""
    rng = np.random.default_rng(seed)
    cu = np.zeros(len(lens) + 1, np.int32)
    cu[1:] = np.cumsum(lens)
    X = wl.as_bf16_values(rng.standard_normal((int(cu[-1]), n)).astype(np.float32))
    W = wl.as_bf16_values((rng.standard_normal((m, n)) / np.sqrt(n)).astype(np.float32))
    P = (rng.standard_normal((m, R)) * 1e-2).astype(np.float32) if R else None
    Vb = (rng.standard_normal((n, R)) * 1e-2).astype(np.float32) if R else None
    b = (rng.standard_normal(m) * 0.3).astype(np.float32) if bias else None
    layer = wl.Layer("layer", m, n, 6, W, act, P, Vb, R, X, b)
    return wl.Workload("small-calls", 9, "bf16", r, 0.25, cu, np.array(seq_cand, np.int32),
                       np.array([0, 0, 1, 1, 2, 2, -1], np.int32), np.array([1, -1, 1, -1, 1, -1, 0], np.float32),
                       np.arange(3, dtype=np.uint64) + np.uint64(77 + seed), [layer], False)


# (weight rows, row count of the small call): most of the tiles from 32x32 to 128x128, at the edges of the tile and of the
# weight rows, few K stages; the full batch takes the 256x256 kernel
@pytest.mark.parametrize("m,rows,full", [(520, 1, 16500), (520, 33, 16500), (512, 500, 16500), (504, 1000, 16500),
                                         (16384, 20, 700), (520, 1999, 16500), (512, 4000, 16500), (32768, 31, 400),
                                         (512, 8001, 16500)])
@pytest.mark.parametrize("n,r,R,act,bias", [(64, 16, 0, 0, False), (320, 33, 72, 1, True), (448, 4, 200, 2, False)])
@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_small_call_has_the_bits_of_a_large_one(m, rows, full, n, r, R, act, bias, out):
    if act == 2 and m % 16:
        m = (m + 15) // 16 * 16
    rng = np.random.default_rng(m + rows)
    # sequences of the small call first (ragged, all kinds, one empty), then filler of all kinds
    lens, left = [], rows
    while left > 0:
        lens.append(min(left, int(rng.integers(1, max(2, rows // 3 + 2)))))
        left -= lens[-1]
    lens.insert(len(lens) // 2, 0)
    keep = len(lens)
    left = full - rows
    while left > 0:
        lens.append(min(left, 300))
        left -= lens[-1]
    w = _layer(rows, lens, [i % 8 - 1 for i in range(len(lens))], m, n, r, R, act, bias)
    big = DeviceWorkload(w, DEV, out_dtype=out)
    order = np.arange(keep)[::-1].copy()   # the small call packs them the other way round
    sub = wl.subset_sequences(w, order)
    small = DeviceWorkload(sub, DEV, out_dtype=out)
    a = big.probe_linear(0)[torch.from_numpy(np.asarray(sub.meta["rows"])).to(DEV)]
    b = small.probe_linear(0)
    torch.cuda.synchronize()
    assert sub.T == rows and torch.equal(a, b)


@pytest.mark.parametrize("n,r,R,act,bias,out", [(2112, 33, 72, 1, True, "bf16"), (1088, 16, 0, 0, False, "f32"),
                                                (2368, 8, 130, 2, False, "bf16")])
def test_every_tile_has_the_bits_of_the_large_one(n, r, R, act, bias, out):
    """Each of the seven tiles, on widths that take every ring of stages round at least twice and end inside a stage of 256
    columns.  The row counts hold for 256 compute units: which tile each takes is asserted."""
    m, rows = 4112, [31, 64, 95, 161, 300, 447, 890]
    tile_of = zb.lib()["_ZN2zo15small_gemm_tileEii"]   # zo::small_gemm_tile(rows, weight rows)
    assert [tile_of(x, m) for x in rows] == list(range(7)) and tile_of(sum(rows), m) == -1
    lens, group = [], []
    for i, x in enumerate(rows):
        a = min(x // 2, 200)
        lens += [a, 0, x - a - 7, 7]
        group += [i] * 4
    w = _layer(n, lens, [i % 8 - 1 for i in range(len(lens))], m, n, r, R, act, bias)
    y = DeviceWorkload(w, DEV, out_dtype=out).probe_linear(0)
    for i, x in enumerate(rows):
        sub = wl.subset_sequences(w, np.flatnonzero(np.array(group) == i)[::-1].copy())
        got = DeviceWorkload(sub, DEV, out_dtype=out).probe_linear(0)
        torch.cuda.synchronize()
        assert sub.T == x and torch.equal(y[torch.from_numpy(np.asarray(sub.meta["rows"])).to(DEV)], got), "tile %d" % i
    some = np.r_[0:40, w.T - 40:w.T]
    want = oracle_layer(w, 0, w.layers[0].X, rows=some, out_dtype=out)
    # (a gated output is the product of two sums, each within 2e-2: d(ab)/ab = da/a + db/b)
    assert_close(to_np(y)[some], want, 4e-2 if act == 2 else 2e-2, "Y")


@pytest.mark.parametrize("n,r,R,act,bias,out", [(704, 33, 72, 1, True, "bf16"), (192, 16, 0, 0, False, "f32"),
                                                (64, 4, 0, 0, True, "bf16"), (1088, 8, 200, 2, False, "bf16")])
def test_tiles_of_160_weight_rows_have_the_bits_of_the_large_one(n, r, R, act, bias, out):
    """Both tiles of 160 weight rows (the waves' loads of their weights do not come out even there), the last one of fewer rows,
    on widths of fewer K stages than their rings hold, and with side state of more and of fewer than that.  The row counts hold
    for 256 compute units: which tile each takes is asserted."""
    m, rows = 5072, [897, 1990, 2113]
    tile_of = zb.lib()["_ZN2zo9gemm_tileEii"]   # zo::gemm_tile(rows, weight rows)
    assert [tile_of(x, m) for x in rows[:2]] == [7, 8] and tile_of(sum(rows), m) == -1
    lens, group = [], []
    for i, x in enumerate(rows):
        while x > 0:
            lens.append(min(x, 333))
            group.append(i)
            x -= lens[-1]
    w = _layer(n, lens, [i % 8 - 1 for i in range(len(lens))], m, n, r, R, act, bias)
    y = DeviceWorkload(w, DEV, out_dtype=out).probe_linear(0)
    for i in (0, 1):
        sub = wl.subset_sequences(w, np.flatnonzero(np.array(group) == i)[::-1].copy())
        got = DeviceWorkload(sub, DEV, out_dtype=out).probe_linear(0)
        torch.cuda.synchronize()
        assert sub.T == rows[i] and torch.equal(y[torch.from_numpy(np.asarray(sub.meta["rows"])).to(DEV)], got), "tile %d" % i
    some = np.r_[0:20, 880:910, w.T - 20:w.T]
    want = oracle_layer(w, 0, w.layers[0].X, rows=some, out_dtype=out)
    # (a gated output is the product of two sums, each within 2e-2: d(ab)/ab = da/a + db/b)
    assert_close(to_np(y)[some], want, 4e-2 if act == 2 else 2e-2, "Y")


@pytest.mark.parametrize("n", [64, 192, 640])
@pytest.mark.parametrize("m,rows,filler", [(4112, [300, 890], 1300), (5072, [897, 1990], 2113)])
def test_more_side_stages_than_the_ring_holds(n, m, rows, filler):
    """The four tiles with stages of 64 columns behind 9 side K tiles, more than any of their rings: no base column in the ring when
    the walk begins, and fewer base stages than the ring, as many, more."""
    tile_of = zb.lib()["_ZN2zo9gemm_tileEii"]   # zo::gemm_tile(rows, weight rows)
    assert [tile_of(x, m) for x in rows] == ([4, 6] if m == 4112 else [7, 8]) and tile_of(sum(rows) + filler, m) == -1
    lens, group = [], []
    for i, x in enumerate(rows + [filler]):
        while x > 0:
            lens.append(min(x, 70))
            group.append(i)
            x -= lens[-1]
    w = _layer(n + m, lens, [i % 8 - 1 for i in range(len(lens))], m, n, 33, 330, 0, True)
    y = DeviceWorkload(w, DEV, out_dtype="f32").probe_linear(0)
    for i in (0, 1):
        sub = wl.subset_sequences(w, np.flatnonzero(np.array(group) == i)[::-1].copy())
        got = DeviceWorkload(sub, DEV, out_dtype="f32").probe_linear(0)
        torch.cuda.synchronize()
        assert sub.T == rows[i] and torch.equal(y[torch.from_numpy(np.asarray(sub.meta["rows"])).to(DEV)], got), "tile %d" % i
    some = np.r_[0:20, rows[0] - 8:rows[0] + 8, w.T - 20:w.T]
    assert_close(to_np(y)[some], oracle_layer(w, 0, w.layers[0].X, rows=some, out_dtype="f32"), 2e-2, "Y")


# widths with and without whole groups of four columns, K slabs that end early, tiles of 32 and of 64 (the second row
# count of a pair takes the larger tile), a vocabulary that ends inside a tile and inside a wave's rows
@pytest.mark.parametrize("n,m,vocab,r,R,act", [(256, 256, 512, 4, 0, 0), (130, 200, 77, 3, 9, 1), (63, 96, 1000, 10, 0, 2),
                                               (388, 260, 65, 1, 33, 0)])
def test_fp32_call_on_either_tile_size(n, m, vocab, r, R, act):
    """fp32 results against the 64-bit oracle at rel 1e-5, and the rows of a call on the larger tiles bit-equal to a
    small call's."""
    lens = [1, 33, 0, 70, 16] + [250] * 28
    w = _layer(n + m, lens, [i % 8 - 1 for i in range(len(lens))], m, n, r, R, act, bool(R))
    rng = np.random.default_rng(vocab)
    m_out = m // 2 if act == 2 else m
    w.dtype, w.eps, w.chain = "f32", 1e-2, True
    w.X, w.layers[0].X = w.layers[0].X, None
    w.head = (rng.standard_normal((vocab, m_out)) / np.sqrt(m_out)).astype(np.float32)
    w.targets = rng.integers(-1, vocab, size=w.T).astype(np.int32)
    big = DeviceWorkload(w, DEV)
    big.step(update=False)
    want = oracle_layer(w, 0, w.X)
    assert_close(to_np(big.Y[0]), want, 1e-5, "Y")
    tok = zo.token_nll(to_np(big.Y[0]), w.head, w.targets)
    assert_close(to_np(big.tok_nll), tok, 1e-5, "tok_nll")
    sub = wl.subset_sequences(w, np.arange(5))
    small = DeviceWorkload(sub, DEV)
    small.step(update=False)
    torch.cuda.synchronize()
    for a, b in ((big.Y[0], small.Y[0]), (big.tok_nll, small.tok_nll)):
        assert torch.equal(a[:sub.T], b)
    assert torch.equal(big.seq_nll[:5], small.seq_nll)


# one and two directions, ranks below, at and above a block of 16 columns, with and without a bank, input widths that end inside
# a group of four, a block of 16 and a K slab, both tile sizes
@pytest.mark.parametrize("n,m,dirs,r,R", [(256, 256, 1, 4, 0), (130, 200, 2, 3, 0), (63, 96, 1, 16, 9), (300, 40, 1, 17, 0), (64, 64, 0, 1, 32),
                                          (5, 33, 1, 1, 1), (641, 52, 2, 16, 0)])
@pytest.mark.parametrize("long", [False, True])
def test_fp32_side_columns_have_the_same_bits_on_either_way(n, m, dirs, r, R, long):
    """Side columns computed along with the products, or by launches of their own: the latter are taken beyond 1024
    sequences, here empty ones among the others."""
    lens = [1, 33, 0, 70, 16, 2, 2, 2, 2] + ([250] * 80 if long else [])
    w = _layer(n * m, lens, [i % (2 * dirs + 2) - 1 for i in range(len(lens))], m, n, r, R, 0, True)
    w.dtype, w.eps, w.dir_seed = "f32", 1e-2, w.dir_seed[:dirs]
    w.cand_dir = np.append(np.repeat(np.arange(dirs, dtype=np.int32), 2), np.int32(-1))   # (+, -) of every direction, centre
    w.cand_sign = np.append(np.tile(np.array([1, -1], np.float32), dirs), np.float32(0))
    a = DeviceWorkload(w, DEV).probe_linear(0)
    empty = 1100
    w.cu_seqlens = np.concatenate([np.zeros(empty, np.int32), w.cu_seqlens])
    w.seq_cand = np.concatenate([np.arange(empty, dtype=np.int32) % (2 * dirs + 2) - 1, w.seq_cand]).astype(np.int32)
    b = DeviceWorkload(w, DEV).probe_linear(0)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    assert_close(to_np(b), oracle_layer(w, 0, w.layers[0].X), 1e-5, "Y")


@pytest.mark.parametrize("m,act", [(33, 1), (300, 0), (64, 2)])
def test_fp32_linear_of_inputs_without_columns(m, act):
    """Every row is act(bias), whatever the compute units' LDS holds (NaN, from a bf16 linear on whole tiles before)."""
    dirty = _layer(m, [256 * 64], [0], 4096, 192, 4, 0, 0, False)
    for l in dirty.layers:
        l.X, l.W = np.full_like(l.X, np.nan), np.full_like(l.W, np.nan)
    dirty = DeviceWorkload(dirty, DEV)
    lens, r = [5, 0, 70, 33, 2], 4
    cu = np.zeros(len(lens) + 1, np.int32)
    cu[1:] = np.cumsum(lens)
    T = int(cu[-1])
    b = DeviceBatch(cu, np.array([0, 1, -1, 2, 1], np.int32), np.array([0, 0, -1], np.int32), np.array([1, -1, 0], np.float32),
                    np.array([9], np.uint64), DEV)
    X, W, bias = torch.zeros(T, 1, device=DEV), torch.zeros(m, 1, device=DEV), torch.randn(m, device=DEV)
    m_out = m // 2 if act == 2 else m
    Y = torch.full((T, m_out), 7.0, device=DEV)
    n_ws = zb.zo_probe_linear_workspace_bytes(T, b.S, b.K, m, 0, r, 0, zb.ZO_F32)
    ws = torch.full((n_ws,), 255, device=DEV, dtype=torch.uint8)
    dirty.probe_linear(0)
    zb.zo_probe_linear(b.struct, X, 1, W, 1, bias, m, 0, zb.ZO_F32, r, 0.5, 2, None, act, Y, m_out, zb.ZO_F32, ws, n_ws)
    torch.cuda.synchronize()
    want = torch.relu(bias) if act == 1 else bias if act == 0 else torch.nn.functional.silu(bias[0::2]) * bias[1::2]
    assert_close(to_np(Y), np.broadcast_to(to_np(want), (T, m_out)), 1e-6, "Y")


# the larger tiles (which call takes which way is asserted, for 256 compute units): widths with and without whole groups of four,
# one to three blocks of 16 columns, with a bank, of a bank alone
@pytest.mark.parametrize("T,n,m,dirs,r,R", [(8100, 256, 256, 1, 4, 0), (6000, 130, 200, 2, 3, 0), (17000, 64, 64, 1, 16, 9),
                                            (5400, 100, 333, 3, 5, 0), (8100, 64, 256, 1, 4, 17), (16000, 63, 96, 0, 1, 32)])
def test_fp32_side_columns_of_larger_tiles_have_the_same_bits_on_either_way(T, n, m, dirs, r, R):
    rides = zb.lib()["_ZN2zo20f32_side_rides_alongEiiiiiiii"]   # zo::f32_side_rides_along(T, m, n, r, R, K, S, C)
    rides.restype = ctypes.c_bool
    lens = [1, 33, 0, 70, 16, 2] + [250] * ((T - 122) // 250) + [(T - 122) % 250]
    w = _layer(n * m, lens, [i % (2 * dirs + 2) - 1 for i in range(len(lens))], m, n, r, R, 0, True)
    w.dtype, w.eps, w.dir_seed = "f32", 1e-2, w.dir_seed[:dirs]
    w.cand_dir = np.append(np.repeat(np.arange(dirs, dtype=np.int32), 2), np.int32(-1))
    w.cand_sign = np.append(np.tile(np.array([1, -1], np.float32), dirs), np.float32(0))
    assert w.T == T and rides(T, m, n, r, R, dirs, len(lens), 2 * dirs + 1)
    a = DeviceWorkload(w, DEV).probe_linear(0)
    some = np.r_[0:130, T // 2:T // 2 + 70, T - 70:T]
    assert_close(to_np(a)[some], oracle_layer(w, 0, w.layers[0].X, rows=some), 1e-5, "Y")
    empty = 1100
    w.cu_seqlens = np.concatenate([np.zeros(empty, np.int32), w.cu_seqlens])
    w.seq_cand = np.concatenate([np.arange(empty, dtype=np.int32) % (2 * dirs + 2) - 1, w.seq_cand]).astype(np.int32)
    assert not rides(T, m, n, r, R, dirs, len(lens) + empty, 2 * dirs + 1)
    b = DeviceWorkload(w, DEV).probe_linear(0)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


@pytest.mark.parametrize("dirs,r,R", [(9, 3, 5), (16, 1, 0), (7, 17, 0)])
def test_fp32_rows_of_many_directions_in_one_block(dirs, r, R):
    """A side launch takes 16 rows at a time, and up to four directions among them in parallel: sequences of one and two rows
    over more directions than that, foreground and centre ones and an empty one among them."""
    lens = [1, 2, 1, 1, 0, 1, 2] * 30
    rng = np.random.default_rng(dirs)
    w = _layer(dirs, lens, rng.integers(-1, 2 * dirs + 1, len(lens)).tolist(), 40, 70, r, R, 0, False)
    w.dtype, w.eps, w.dir_seed = "f32", 1e-2, np.arange(dirs, dtype=np.uint64) + np.uint64(11)
    w.cand_dir = np.append(np.repeat(np.arange(dirs, dtype=np.int32), 2), np.int32(-1))
    w.cand_sign = np.append(np.tile(np.array([1, -1], np.float32), dirs), np.float32(0))
    assert max(len(set(np.repeat(w.seq_cand // 2, lens)[i:i + 16])) for i in range(0, w.T, 16)) > 4
    y = DeviceWorkload(w, DEV).probe_linear(0)
    assert_close(to_np(y), oracle_layer(w, 0, w.layers[0].X), 1e-5, "Y")


@pytest.mark.parametrize("n", [64, 256, 1000, 2048])
@pytest.mark.parametrize("K,r", [(1, 4), (4, 16)])
def test_fp32_side_term_alone_against_64_bits(n, K, r):
    """W = 0: the side term as it is summed along with the products (one direction) and in a launch of its own (four).  Rounding
    errors are independent, so their squares add: a rounding of a partial sum counts by its share of the sum, and is at most
    2^-24 (uniform: / sqrt(3) in the root mean square).  64 partial sums of the width, paired off, count n/64 / 2 + 6.5, the scale 1,
    a chain of r products (r + 1) / 2; one chain over the width would count n / 2."""
    m, T = 96, 1024
    cu = (np.arange(2 * K + 1) * (T // (2 * K))).astype(np.int32)
    seeds = np.arange(K, dtype=np.uint64) + np.uint64(300 + n)
    b = DeviceBatch(cu, np.arange(2 * K, dtype=np.int32), np.repeat(np.arange(K, dtype=np.int32), 2), np.tile(np.array([1, -1], np.float32), K), seeds, DEV)
    X = torch.randn(T, n, device=DEV, generator=torch.Generator(device=DEV).manual_seed(n))
    W, Y = torch.zeros(m, n, device=DEV), torch.empty(T, m, device=DEV)
    n_ws = zb.zo_probe_linear_workspace_bytes(T, b.S, b.K, m, n, r, 0, zb.ZO_F32)
    ws = torch.empty(n_ws, device=DEV, dtype=torch.uint8)
    zb.zo_probe_linear(b.struct, X, n, W, n, None, m, n, zb.ZO_F32, r, 0.5, 2, None, 0, Y, m, zb.ZO_F32, ws, n_ws)
    U, V = torch.empty(m, r, device=DEV), torch.empty(n, r, device=DEV)   # (the device's own factors: their rounding is not at issue)
    want = np.empty((T, m))
    x = X.cpu().numpy().astype(np.float64)
    for s in range(2 * K):
        zb.zo_factor_fill(int(seeds[s // 2]), 2, m, r, zb.ZO_F32, U)
        zb.zo_factor_fill(int(seeds[s // 2]), 3, n, r, zb.ZO_F32, V)
        u, v = (t.cpu().numpy().astype(np.float64) for t in (U, V))
        want[cu[s]:cu[s + 1]] = (0.5 - s % 2) * (x[cu[s]:cu[s + 1]] @ v) @ u.T
    err = np.linalg.norm(to_np(Y).astype(np.float64) - want) / np.linalg.norm(want)
    assert err <= 2.0 ** -24 / np.sqrt(3) * np.sqrt(n / 128 + 6.5 + 1 + (r + 1) / 2), err


@pytest.mark.parametrize("lens", [[1, 31, 32, 33, 64, 0, 96], [127, 128, 129], [160, 161, 255, 257, 1]])
@pytest.mark.parametrize("scale,grow", [(128 ** -0.5, 0.0), (-(128 ** -0.5), 0.0), (0.0, 0.0), (0.1, 0.02), (0.1, -0.02)])
def test_attention_at_the_edges_of_its_steps(lens, scale, grow):
    """Lengths around the 64 keys of a step, the 32 rows of a wave and the 128 of a workgroup; negative and zero
    scales; scores that grow along the sequence, so that the running maximum is raised again and again, or shrink, so
    that it never is.  Weights and outputs are bf16: 2e-2 as for every bf16 output here."""
    H, Hkv, dh = 4, 2, 128
    rng = np.random.default_rng(sum(lens))
    T = sum(lens)
    cu = np.zeros(len(lens) + 1, np.int32)
    cu[1:] = np.cumsum(lens)
    pos = np.concatenate([np.arange(n) for n in lens])[:, None]
    q = wl.as_bf16_values((rng.standard_normal((T, H * dh)) + (grow != 0)).astype(np.float32))
    k = wl.as_bf16_values((rng.standard_normal((T, Hkv * dh)) + grow * pos).astype(np.float32))
    v = wl.as_bf16_values(rng.standard_normal((T, Hkv * dh)).astype(np.float32))
    b = DeviceBatch(cu, np.full(len(lens), -1), np.zeros(0), np.zeros(0), np.zeros(0, np.uint64), DEV)
    dev = [torch.from_numpy(x).to(DEV, torch.bfloat16) for x in (q, k, v)]
    out = torch.empty((T, H * dh), device=DEV, dtype=torch.bfloat16)
    zb.zo_attention(b.struct, dev[0], H * dh, dev[1], Hkv * dh, dev[2], Hkv * dh, H, Hkv, dh, scale, zb.ZO_BF16, out, H * dh)
    assert_close(to_np(out), ob.attention(q, k, v, cu, H, Hkv, dh, scale, "bf16"), 2e-2, "attention")


# on both sides of the line between the one-launch side-down pass and the staged one, at widths whose ranges end inside and at the end of a batch of 256 columns, with 1, 2, 4 and 8 ranges
@pytest.mark.parametrize("n,r,R", [(64, 1, 0), (448, 48, 16), (1088, 16, 40), (2560, 8, 136), (5184, 70, 0), (20480, 4, 32)])
def test_side_term_on_either_pass(n, r, R):
    lens = [1, 17, 0, 40, 16, 5] + [200] * (12 if n > 10000 else 260 if n == 64 else 110)
    w = _layer(n, lens, [i % 8 - 1 for i in range(len(lens))], 64, n, r, R, 0, False)
    big = DeviceWorkload(w, DEV, out_dtype="f32")
    y = big.probe_linear(0)
    rows = np.r_[0:80, w.T - 80:w.T]
    assert_close(to_np(y)[rows], oracle_layer(w, 0, w.layers[0].X, out_dtype="f32")[rows], 2e-2, "Y")
    sub = wl.subset_sequences(w, np.array([5, 3, 1, 0, 2, 4]))
    b = DeviceWorkload(sub, DEV, out_dtype="f32").probe_linear(0)
    torch.cuda.synchronize()
    assert torch.equal(y[torch.from_numpy(np.asarray(sub.meta["rows"])).to(DEV)], b)


@pytest.mark.parametrize("vocab,d,pitch", [(300, 64, 64), (257, 192, 192), (70000, 128, 128), (600, 256, 256), (513, 320, 328),
                                           (257, 1024, 1024), (66000, 448, 2048)])
@pytest.mark.parametrize("scored", [1, 15, 127, 128, 129])
def test_few_scored_tokens_have_the_bits_of_a_full_call(vocab, d, pitch, scored):
    """Up to 128 scored tokens take a narrow token tile: 1 to 16 K tiles (its ring of three stages goes round up to
    five times), vocabularies that end one row into a tile, inside a wave's rows and past one round of workgroups; the last
    head spans more than 256 MB and is read by the streaming variant."""
    rng = np.random.default_rng(vocab + scored)
    T = 600
    cu = np.array([0, 100, 100, 350, T], np.int32)
    w = wl.Workload("few", 9, "bf16", 4, 1e-3, cu, np.array([0, 1, -1, 0], np.int32), np.zeros(2, np.int32),
                    np.array([1, -1], np.float32), np.arange(1, dtype=np.uint64), [], True,
                    wl.as_bf16_values(rng.standard_normal((T, d)).astype(np.float32)),
                    wl.as_bf16_values((rng.standard_normal((vocab, d)) / np.sqrt(d)).astype(np.float32)),
                    rng.integers(0, vocab, T).astype(np.int32), 0)
    g = DeviceWorkload(w, DEV)
    if pitch != d:
        wide = torch.zeros((vocab, pitch), device=DEV, dtype=torch.bfloat16)
        wide[:, :d] = g.head
        g.head = wide[:, :d]
    g.score(H=g.X)
    full = g.tok_nll.clone()
    keep = torch.from_numpy(np.sort(rng.choice(T, scored, replace=False))).to(DEV)
    few = torch.full_like(g.targets, -1)
    few[keep] = g.targets[keep]
    g.targets = few
    g.tok_nll.fill_(float("nan"))
    g.score(H=g.X)
    torch.cuda.synchronize()
    assert torch.equal(g.tok_nll[keep], full[keep])
    assert int((g.tok_nll != 0).sum()) <= scored and float(g.cand_cnt.sum()) <= scored
    assert_close(to_np(full), zo.token_nll(w.X, w.head, w.targets), 1e-4, "tok_nll", atol=1e-4)


@pytest.mark.parametrize("d", [64, 192, 320])
def test_some_hundred_scored_tokens_have_the_bits_of_a_full_call(d):
    """Several narrow token tiles (129 to 640 tokens against 274 vocabulary tiles: three to six rounds of 256 workgroups, the last
    tile of one token and of all), against the wide tiles that 1201 tokens take, with 1, 3 and 5 K tiles."""
    vocab, T = 70000, 1201
    rng = np.random.default_rng(d)
    cu = np.array([0, 100, 100, 750, T], np.int32)
    w = wl.Workload("some", 9, "bf16", 4, 1e-3, cu, np.array([0, 1, -1, 0], np.int32), np.zeros(2, np.int32),
                    np.array([1, -1], np.float32), np.arange(1, dtype=np.uint64), [], True,
                    wl.as_bf16_values(rng.standard_normal((T, d)).astype(np.float32)),
                    wl.as_bf16_values((rng.standard_normal((vocab, d)) / np.sqrt(d)).astype(np.float32)),
                    rng.integers(0, vocab, T).astype(np.int32), 0)
    g = DeviceWorkload(w, DEV)
    g.score(H=g.X)
    full, targets = g.tok_nll.clone(), g.targets
    some = np.r_[0:40, T - 40:T]
    assert_close(to_np(full)[some], zo.token_nll(w.X[some], w.head, w.targets[some]), 1e-4, "tok_nll", atol=1e-4)
    taken = zb.lib()["_ZN2zo18head_narrow_countsEiiii"]   # zo::head_narrow_counts(vocabulary tiles, workgroups, K, pitch), one bit per count
    taken.restype = ctypes.c_uint64
    assert [taken(274, 256, d, 2 * d) >> k & 1 for k in (2, 3, 5, 10)] == [1, 1, 1, 0]   # (10: the full call)
    for scored in (129, 256, 300, 640):
        keep = torch.from_numpy(np.sort(rng.choice(T, scored, replace=False))).to(DEV)
        g.targets = torch.full_like(targets, -1)
        g.targets[keep] = targets[keep]
        g.tok_nll.fill_(float("nan"))
        g.score(H=g.X)
        torch.cuda.synchronize()
        assert torch.equal(g.tok_nll[keep], full[keep]), scored
        assert int((g.tok_nll != 0).sum()) <= scored


@pytest.mark.parametrize("T", [129, 224, 256, 500, 896])
def test_scoring_every_token_on_narrow_tiles_has_the_bits_of_a_larger_call(T):
    """A vocabulary of 36 tiles: 2 to 7 narrow token tiles, all in one round of a grid larger than the wide tiles need, against wide
    ones (1500 tokens)."""
    vocab, d, full = 9100, 192, 1500
    taken, grid_of = zb.lib()["_ZN2zo18head_narrow_countsEiiii"], zb.lib()["_ZN2zo16head_gather_gridEiiii"]
    taken.restype = ctypes.c_uint64
    K, grid = (d, 2 * d), grid_of(T, 36, d, 2 * d)
    assert grid == 8 * (-(-36 * -(-T // 128) // 8)) and taken(36, grid, *K) >> -(-T // 128) & 1
    assert not taken(36, grid_of(full, 36, *K), *K) >> 12 & 1
    rng = np.random.default_rng(T)
    head = wl.as_bf16_values((rng.standard_normal((vocab, d)) / np.sqrt(d)).astype(np.float32))
    X = wl.as_bf16_values(rng.standard_normal((full, d)).astype(np.float32))
    targets = rng.integers(0, vocab, full).astype(np.int32)
    nll = []
    for n in (full, T):
        w = wl.Workload("all", 9, "bf16", 4, 1e-3, np.array([0, n // 3, n], np.int32), np.array([0, 1], np.int32), np.zeros(2, np.int32),
                        np.array([1, -1], np.float32), np.arange(1, dtype=np.uint64), [], True, X[:n], head, targets[:n], 0)
        g = DeviceWorkload(w, DEV)
        g.tok_nll.fill_(float("nan"))
        g.score(H=g.X)
        nll.append(g.tok_nll)
    torch.cuda.synchronize()
    assert torch.equal(nll[0][:T], nll[1])
    assert_close(to_np(nll[1])[-40:], zo.token_nll(X[T - 40:T], head, targets[T - 40:T]), 1e-4, "tok_nll", atol=1e-4)


@pytest.mark.parametrize("S,K", [(1025, 3), (1500, 70), (300, 70), (1024, 64)])
def test_tables_of_many_sequences_and_directions(S, K):
    """More than 1024 sequences (tables in global memory instead of LDS) and more than 64 directions (slot lists searched
    instead of a mask), many of them inside one token tile."""
    rng = np.random.default_rng(S + K)
    lens = rng.integers(0, 4, S)
    w = _layer(S, lens.tolist(), rng.integers(-1, 2 * K, S).tolist(), 64, 64, 4, 16, 0, False)
    w.cand_dir = np.repeat(np.arange(K, dtype=np.int32), 2)
    w.cand_sign = np.tile(np.array([1, -1], np.float32), K)
    w.dir_seed = np.arange(K, dtype=np.uint64) + np.uint64(5)
    y = DeviceWorkload(w, DEV, out_dtype="f32").probe_linear(0)
    assert_close(to_np(y), oracle_layer(w, 0, w.layers[0].X, out_dtype="f32"), 2e-2, "Y")


# 33 tiles and more have their tables built by threads or, where a tile has many sequences, by waves: on both sides of that line
# with few and with more than 64 directions, more sequences than are kept in LDS, more tiles than a workgroup has threads
@pytest.mark.parametrize("tiles,per_tile,K", [(33, 0.3, 3), (33, 1, 64), (33, 12, 65), (40, 30, 20), (64, 8, 70), (64, 3, 200), (64, 90, 3),
                                              (200, 30, 17), (200, 100, 16), (1030, 0.6, 2), (1090, 1.5, 90)])
def test_tables_of_many_token_tiles(tiles, per_tile, K):
    rng = np.random.default_rng(tiles + K)
    lens, rows = [], (tiles - 1) * 256 + 100
    mean = 256 / per_tile
    while rows > 0:
        lens.append(int(min(rows, rng.integers(0, 2 * mean + 1))))
        rows -= lens[-1]
    w = _layer(tiles, lens, rng.integers(-1, 2 * K + 1, len(lens)).tolist(), 64, 64, 4, 16, 0, False)
    w.cand_dir = np.append(np.repeat(np.arange(K, dtype=np.int32), 2), np.int32(-1))
    w.cand_sign = np.append(np.tile(np.array([1, -1], np.float32), K), np.float32(0))
    w.dir_seed = np.arange(K, dtype=np.uint64) + np.uint64(5)
    y = DeviceWorkload(w, DEV, out_dtype="f32").probe_linear(0)
    # rows of every tile: its first and last ones and some between
    some = np.unique(np.minimum(np.arange(tiles)[:, None] * 256 + np.array([0, 1, 77, 130, 255]), w.T - 1))
    want = oracle_layer(w, 0, w.layers[0].X, rows=some, out_dtype="f32")
    assert_close(to_np(y[torch.from_numpy(some).to(DEV)]), want, 2e-2, "Y")
    # and all rows against calls of a few tiles each
    cuts = np.searchsorted(w.cu_seqlens, np.arange(0, w.T, 5000))
    for a, b in list(zip(cuts, np.append(cuts[1:], len(lens))))[::max(1, len(cuts) // 8)]:
        if w.cu_seqlens[b] > w.cu_seqlens[a]:
            sub = wl.subset_sequences(w, np.arange(a, b))
            got = DeviceWorkload(sub, DEV, out_dtype="f32").probe_linear(0)
            assert torch.equal(got, y[int(w.cu_seqlens[a]):int(w.cu_seqlens[b])])


@pytest.mark.parametrize("n,R", [(64, 0), (2560, 40)])
def test_side_term_of_a_batch_changed_on_the_device(n, R):
    """The host's copies of the tables decide which side-down pass a call takes, never its result: a handle whose device tables were changed (one candidate sequence becomes 40) gives what a new handle gives."""
    lens = [5, 40, 1, 16, 17] * 8
    few = _layer(n, lens, [0] + [-1] * 39, 64, n, 20, R, 0, False)
    many = _layer(n, lens, [i % 7 for i in range(40)], 64, n, 20, R, 0, False)
    g = DeviceWorkload(few, DEV, out_dtype="f32")
    g.batch.seq_cand.copy_(torch.from_numpy(many.seq_cand))
    y = g.probe_linear(0)
    want = DeviceWorkload(many, DEV, out_dtype="f32").probe_linear(0)
    torch.cuda.synchronize()
    assert torch.equal(y, want)
    assert_close(to_np(y), oracle_layer(many, 0, many.layers[0].X, out_dtype="f32"), 2e-2, "Y")


@pytest.mark.parametrize("n,r,K,lens", [(448, 512, 24, [1] * 48), (128, 40, 80, [3, 0, 5] * 60), (64, 100, 3, [250, 12, 16, 1])])
def test_side_slots_of_high_ranks_and_many_directions(n, r, K, lens):
    """Slot lists of several hundred entries, more than 64 directions in a token tile, and items that lie in two tiles."""
    w = _layer(n + r, lens, [i % (2 * K) for i in range(len(lens))], 64, n, r, 16, 0, False)
    w.cand_dir = np.repeat(np.arange(K, dtype=np.int32), 2)
    w.cand_sign = np.tile(np.array([1, -1], np.float32), K)
    w.dir_seed = np.arange(K, dtype=np.uint64) + np.uint64(5)
    y = DeviceWorkload(w, DEV, out_dtype="f32").probe_linear(0)
    assert_close(to_np(y), oracle_layer(w, 0, w.layers[0].X, out_dtype="f32"), 2e-2, "Y")


@pytest.mark.parametrize("n,r,R,lens,K", [(64, 4, 0, [4] * 400, 64), (448, 20, 72, [5, 0, 61, 190, 40], 2), (64, 40, 9, [1] * 90, 30),
                                          (5184, 16, 16, [255, 2, 300, 17], 2)])
def test_side_images_are_cleared_where_they_are_used(n, r, R, lens, K):
    """A workspace full of NaN changes no result (every K tile in use is written whole), and the K tiles that the batch could
    have needed but does not use are left alone: with 400 sequences sorted by 64 directions, 42 of 207 are in use."""
    S = len(lens)
    w = _layer(n + r, lens, [i * 2 * K // S if i % 5 else -1 for i in range(S)], 64, n, r, R, 0, False)
    w.cand_dir = np.repeat(np.arange(K, dtype=np.int32), 2)
    w.cand_sign = np.tile(np.array([1, -1], np.float32), K)
    w.dir_seed = np.arange(K, dtype=np.uint64) + np.uint64(5)
    g = DeviceWorkload(w, DEV, out_dtype="f32")
    g.ws.zero_()
    want = g.probe_linear(0).clone()
    g.ws.fill_(255)
    got = g.probe_linear(0)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    assert_close(to_np(got), oracle_layer(w, 0, w.layers[0].X, out_dtype="f32"), 2e-2, "Y")
    if S == 400:
        assert int((g.ws == 255).sum()) > 160 * 256 * 64 * 2


@pytest.mark.parametrize("C,K", [(1, 1), (64, 64), (65, 40), (141, 70), (300, 130), (40, 200)])
@pytest.mark.parametrize("reduction", [0, 1])
def test_estimate_of_tables_of_any_length(C, K, reduction):
    """The candidate table is read 64 entries at a time by a workgroup per 64 directions: tables on both sides of that, in any
    order, with directions that lack a sign or have several candidates of one, centres and candidates without a token."""
    rng = np.random.default_rng(1000 * C + K)
    cand_dir = rng.permutation(np.arange(C) // 2 % K).astype(np.int32)
    cand_sign = rng.choice(np.array([1, -1, 0], np.float32), C, p=[0.45, 0.45, 0.1])
    cand_dir[cand_sign == 0] = -1
    cu = np.arange(C + 1, dtype=np.int32)
    b = DeviceBatch(cu, np.arange(C, dtype=np.int32), cand_dir, cand_sign, np.arange(K, dtype=np.uint64), DEV)
    cnt = rng.integers(0, 5, C).astype(np.int32)
    total = rng.uniform(0.5, 9.0, C).astype(np.float32)
    total[cnt == 0] = 0
    loss, grad = torch.full((C,), -7.0, device=DEV), torch.full((K,), -7.0, device=DEV)
    zb.zo_estimate(b.struct, torch.from_numpy(total).to(DEV), torch.from_numpy(cnt).to(DEV), 0.25, reduction, loss, grad)
    torch.cuda.synchronize()
    want_loss, want_grad = zo.estimate(zo.Batch(cu, np.arange(C, dtype=np.int32), cand_dir, cand_sign, np.arange(K, dtype=np.uint64)),
                                       total, cnt, 0.25, reduction)
    # a loss is one rounding (2^-24) from the quotient, a difference of two below 9 within three of 2^-24 * 9, doubled by 1 / (2 eps)
    assert np.all(np.abs(to_np(loss) - want_loss) <= 2.0 ** -24 * np.abs(want_loss))
    assert np.all(np.abs(to_np(grad) - want_grad) <= 2 * 3 * 9 * 2.0 ** -24)
    assert np.array_equal(to_np(grad) == 0, want_grad == 0)
