"""GPU parity of the paths a call is sent down by its sizes, at the sizes where each begins and ends.
Bit-exact against the CPU oracle, through the C ABI."""

import numpy as np
import pytest

from efs_gpu import Case, announce, assert_f32_equal, certify_randk, certify_topk, dev, host, order_certificate
from oracle import efsparse_oracle as O
from workloads.generate import to_bf16_bits

pytestmark = pytest.mark.gpu


def _messages(d, counts, seed):
    """Per worker counts[w] ascending distinct indices crowded into the first 1024 elements, the rest of
    each message after them, and values from denormals to the largest, signed zeros among them."""
    rng = np.random.default_rng(seed)
    W, K = len(counts), max(counts) + 37
    idx = np.empty((W, K), np.uint32)
    for w, n in enumerate(counts):
        idx[w, :n] = np.sort(rng.choice(1024, size=n, replace=False))
        idx[w, n:] = 1024 + np.sort(rng.choice(d - 1024, size=K - n, replace=False))
    val = (rng.standard_normal((W, K)) * 10.0 ** rng.uniform(-44, 37, (W, K))).astype(np.float32)
    val[rng.random((W, K)) < 0.1] = -0.0
    val[rng.random((W, K)) < 0.3] = np.float32(2.0 ** -149) * rng.integers(-9, 9)
    return idx, val


# entries of the first tile: one chunk of 64 less, exactly, more; marks on both sides of a chunk's edge;
# the packed form's most (4096) and one over; more workers than one group holds
@pytest.mark.parametrize("counts", [[1], [63], [64, 1], [65, 64, 63], [32, 32, 1], [0, 5, 0, 60, 1], [256] * 16,
                                    [256] * 15 + [257], [1024] * 5, [3] * 64, [2] * 65, [40, 0, 90] * 44],
                         ids=lambda c: f"{sum(c)}x{len(c)}")
def test_sparse_aggregate_tile_entries(counts):
    import paper_2009_09271_amd as E
    import torch
    announce("sparse aggregate tile", sum(counts), len(counts))
    d, W = 20011, len(counts)
    idx, val = _messages(d, counts, sum(counts) + W)
    K = idx.shape[1]
    c = Case([0, d], (K + 0.25) / d)
    assert c.K == K
    out = torch.empty(d, dtype=torch.float32, device="cuda")
    for average in (True, False):
        E.decompress_aggregate(c.L, E.EF_MSG_SPARSE, W, dev(idx.view(np.int32)), dev(val), out,
                               c.L.workspace(E.EF_OP_AGG_SPARSE, W), average)
        assert_f32_equal(out, O.decompress_aggregate_sparse(d, idx, val, average), f"average={average}")


# gaps between a message's entries, in tiles of 1024 elements: the last written by its entry's thread, by one
# wavefront and the first of each longer form, up to the last tile and past it; three messages whose range
# tables start at different places modulo 16 bytes
@pytest.mark.parametrize("last", [1, 33, 4096, 4097])
def test_sparse_aggregate_long_gaps(last):
    import paper_2009_09271_amd as E
    import torch
    announce("sparse aggregate gaps", last)
    gaps = [31, 32, 33, 34, 4095, 4096, 4097, 4098, 1]
    W, tiles = 3, sum(gaps) + last
    d = 1024 * tiles - 5
    assert (tiles + 1) % 4 != 0  # (tables of tiles + 1 words)
    rng = np.random.default_rng(last)
    idx = []
    for w in range(W):
        at = np.cumsum(rng.permutation(gaps)) - (w == 0)  # the tiles that hold entries
        idx.append(np.sort(np.concatenate([1024 * t + rng.choice(1000, 3, replace=False) for t in at])))
    idx = np.stack(idx).astype(np.uint32)
    K = idx.shape[1]
    val = rng.standard_normal((W, K)).astype(np.float32)
    c = Case([0, d], (K + 0.25) / d)
    assert c.K == K
    out = torch.empty(d, dtype=torch.float32, device="cuda")
    E.decompress_aggregate(c.L, E.EF_MSG_SPARSE, W, dev(idx.view(np.int32)), dev(val), out,
                           c.L.workspace(E.EF_OP_AGG_SPARSE, W))
    assert_f32_equal(out, O.decompress_aggregate_sparse(d, idx, val, True), f"gap to the end {last}")


# messages of a quarter of the elements and one entry more (chunks loaded by fours), tiles of 1 to 1024 entries
# of each worker among them, and more workers than one group holds
@pytest.mark.parametrize("W", [1, 5, 67])
@pytest.mark.parametrize("over", [0, 1])
def test_sparse_aggregate_full_messages(W, over):
    import paper_2009_09271_amd as E
    import torch
    d = 1024 * 9 + 200
    K = d // 4 + over
    assert (K > d // 4) == bool(over)
    announce("sparse aggregate full messages", W, K)
    rng = np.random.default_rng(W + over)
    idx = []
    for w in range(W):  # one tile sent whole, one entry in another, the rest at random
        whole, single = 1024 * (w % 7), 1024 * 8 + w % 200
        rest = np.setdiff1d(np.arange(d), np.r_[whole:whole + 1024, 1024 * 8:1024 * 9])
        idx.append(np.sort(np.r_[whole:whole + 1024, single, rng.choice(rest, K - 1025, replace=False)]))
    idx = np.stack(idx).astype(np.uint32)
    val = (rng.standard_normal((W, K)) * 10.0 ** rng.uniform(-3, 3, (W, K))).astype(np.float32)
    c = Case([0, d], (K + 0.25) / d)
    assert c.K == K
    out = torch.empty(d, dtype=torch.float32, device="cuda")
    E.decompress_aggregate(c.L, E.EF_MSG_SPARSE, W, dev(idx.view(np.int32)), dev(val), out,
                           c.L.workspace(E.EF_OP_AGG_SPARSE, W))
    assert_f32_equal(out, O.decompress_aggregate_sparse(d, idx, val, True), f"{W} workers, {K} entries")


def _certify_long_segment(c, before, acc, idx, val, e, seed, step):
    """One long segment after `before` segments of one element each and before more of them."""
    idx, n, k = host(idx).view(np.uint32).astype(np.int64), c.offs[before + 1] - before, c.ks[before]
    assert_f32_equal(val, acc[idx], "values")
    want = acc.copy()
    want[idx] = 0.0
    assert_f32_equal(e, want, "residual")
    assert np.array_equal(np.r_[idx[:before], idx[before + k:]], np.r_[np.arange(before), np.arange(before + n, c.d)])
    order_certificate(idx[before:before + k] - before, n, k, lambda a, b: ~O.randk_keys(n, before, seed, step, a, b), "long segment")


def _randk_route(sizes, density, extra=32.0):
    """The layout's random-k route by the library's rules: the select kernel's form ("small", "direct" lists in
    LDS, "lists" by a collection of their own, "big": rows' offsets over many workgroups), the expected undecided
    keys of the segment with the most of them, the bound on them that the forms are chosen by, and the rows."""
    rows, most, bound, at = 0, 0.0, 0.0, 0
    small = direct = True
    big = False
    for n in sizes:
        k = min(max(int(np.floor(density * n + 0.5)), 1), n)
        r = (at + n - 1) // 4096 - at // 4096 + 1
        w = min(k + 6 * k ** 0.5 + extra, n) - max(k - 6 * k ** 0.5 - extra, 0.0)
        b = w + 8 * w ** 0.5 + 16
        big |= k >= 1 << 20 or r > 16384
        direct &= r <= 8192 and b <= 8192
        small &= r <= 4096 and b <= 4096
        rows, most, bound, at = rows + r, max(most, w), max(bound, b), at + n
    return "big" if big else "small" if direct and small else "direct" if direct else "lists", most, bound, rows


# random-k on one segment, the select kernel's forms at the last sizes that take each and the first that do not:
# by rows (4096, 8192, 16384), by the bound on the undecided keys (4096, 8192), by k (2^20); lists in LDS and in
# global memory (over 8192 entries); the rows' offsets from one block of rows (2048) and from several
@pytest.mark.parametrize("d,k,form,edge", [
    (4096 * 4096, 16777, "small", None), (4096 * 4096 + 1, 16777, "direct", None),
    (1 << 20, 86828, "small", 4096), (1 << 20, 86829, "direct", 4096),
    (4096 * 4096, 86828, "small", 4096), (4096 * 8192, 33554, "direct", None), (4096 * 8192 + 1, 33554, "lists", None),
    (1 << 22, 382328, "direct", 8192), (1 << 22, 382329, "lists", 8192),
    (1 << 23, (1 << 20) - 1, "lists", None), (4096 * 2048, 1 << 20, "big", None), (4096 * 2048 + 1, 1 << 20, "big", None),
    (4096 * 16384, 671089, "lists", None), (4096 * 16384 + 5, 671089, "big", None)])
def test_randk_select_forms(d, k, form, edge):
    import paper_2009_09271_amd as E
    import torch
    announce("random-k forms", d, k, form)
    c = Case([0, d], (k + 0.25) / d)
    route, most, bound, rows = _randk_route([d], c.density)
    assert route == form and c.K == k
    assert edge is None or abs(bound - edge) < 0.05
    rng = np.random.default_rng(d % 1000)
    acc = rng.standard_normal(d, dtype=np.float32) + np.float32(0.0)  # (no -0: it leaves g + e as +0)
    e = torch.zeros(d, dtype=torch.float32, device="cuda")
    idx, val, ws = c.step("randk", acc, e, seed=77 + d, step=3)
    assert c.L.diag(ws, E.EF_OP_RANDK) == 0
    certify_randk(acc, c.offs, c.ks, host(idx), host(val), host(e), 77 + d, 3)


# random-k, 8 to 64 rows (the most) to a collecting wavefront: a segment of over 1024 rows between segments of
# one element each, so that wavefronts have rows of one segment and of several; the last with more than 2048
# rows to a block of the rows' offsets
@pytest.mark.parametrize("nrows,rw,main", [(32767, 8, 1100), (32768, 16, 1100), (65536, 32, 1100), (131072, 64, 1100),
                                           (2048 * 256 + 1, 64, 16385)])
def test_randk_rows_per_wavefront(nrows, rw, main):
    import paper_2009_09271_amd as E
    import torch
    announce("random-k rows per wavefront", nrows, rw)
    before, n = 4096 * 5, 4096 * main  # (the segments before: so many that the long one starts a tile)
    offs = np.r_[np.arange(before + 1), before + n + np.arange(nrows - before - main + 1)].tolist()
    density = 0.2 if main == 1100 else 0.01
    route, most, bound, rows = _randk_route(np.diff(offs).tolist(), density)
    assert route == ("lists" if main == 1100 else "big") and rows == nrows and bound > 8192
    want = 64
    while want > 1 and rows // want < 2048:
        want //= 2
    assert want == rw
    c = Case(offs, density)
    rng = np.random.default_rng(nrows)
    acc = rng.standard_normal(c.d, dtype=np.float32) + np.float32(0.0)
    e = torch.zeros(c.d, dtype=torch.float32, device="cuda")
    idx, val, ws = c.step("randk", acc, e, seed=nrows, step=1)
    assert c.L.diag(ws, E.EF_OP_RANDK) == 0
    _certify_long_segment(c, before, acc, idx, val, e, nrows, 1)


# random-k, a list in global memory of which more than 8192 entries lie where the k-th key is expected: the
# search over the whole list
def test_randk_band_too_wide():
    import paper_2009_09271_amd as E
    import torch
    d, k, extra = 1 << 22, 1000000, 990000.0
    announce("random-k band", d, k)
    c = Case([0, d], (k + 0.25) / d, tune={E.EF_TUNE_RANDK_EXTRA: extra})
    route, m, bound, rows = _randk_route([d], c.density, extra)
    need = m / 2  # (the window lies evenly about k)
    # the band's expected entries, six standard deviations and eight each way
    assert route == "lists" and c.K == k and 2 * (6 * (need * (1 - need / m)) ** 0.5 + 8) > 8192 + 3 * 8192 ** 0.5
    rng = np.random.default_rng(5)
    acc = rng.standard_normal(d, dtype=np.float32) + np.float32(0.0)
    e = torch.zeros(d, dtype=torch.float32, device="cuda")
    idx, val, ws = c.step("randk", acc, e, seed=21, step=2)
    assert c.L.diag(ws, E.EF_OP_RANDK) == 0
    certify_randk(acc, c.offs, c.ks, host(idx), host(val), host(e), 21, 2)


# random-k with every element undecided: 1088 rows whose 17 collecting wavefronts of 64 rows list them by
# wavefront, two in one sub-list, between segments of one element (which make the rows so many)
def test_randk_wide_lists_hold_two_wavefronts():
    import paper_2009_09271_amd as E
    import torch
    announce("random-k wide lists")
    before, n, nrows = 4096 * 5, 4096 * 1088, 131072
    offs = np.r_[np.arange(before + 1), before + n + np.arange(nrows - before - 1088 + 1)].tolist()
    c = Case(offs, 0.2, tune={E.EF_TUNE_RANDK_EXTRA: 1e9})
    rng = np.random.default_rng(3)
    acc = rng.standard_normal(c.d, dtype=np.float32) + np.float32(0.0)
    e = torch.zeros(c.d, dtype=torch.float32, device="cuda")
    idx, val, ws = c.step("randk", acc, e, seed=9, step=1)
    assert c.L.diag(ws, E.EF_OP_RANDK) == 0
    _certify_long_segment(c, before, acc, idx, val, e, 9, 1)


# top-k, a layout of several segments: +0 stored by the pass or by the emission (the densities on both sides of
# the rule; few samples above the threshold and many), segments sampled whole among them, and one of few
# magnitudes: its threshold is the smallest candidate key and shared by more elements than win, with
# candidates above it
@pytest.mark.parametrize("density", [0.004, 0.012, 0.013, 0.3])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_topk_residual_store(density, dtype):
    import paper_2009_09271_amd as E
    announce("top-k residual store", density, dtype)
    offs = np.cumsum([0, 4096 * 40 + 3, 5, 4096 * 9, 100000, 4096 * 3 + 1]).tolist()
    rng = np.random.default_rng(int(density * 1e4))
    g = rng.standard_normal(offs[-1], dtype=np.float32)
    o, n = offs[3], 100000
    g[o:o + n] = rng.integers(1, 4, n)
    g[o + rng.choice(n, 200, replace=False)] = rng.uniform(4, 8, 200)
    if dtype == "bf16":
        g16 = to_bf16_bits(g)
        g = (g16.astype(np.uint32) << 16).view(np.float32)
    import torch
    c = Case(offs, density)
    e0 = rng.standard_normal(offs[-1], dtype=np.float32)
    e0[o:o + n] = 0.0  # (the few magnitudes stay)
    acc = g + e0
    top = np.sort(np.abs(acc[o:o + n]))[::-1]
    T = top[c.ks[3] - 1]
    assert T == 3.0 and (top > T).sum() == 200 < c.ks[3] < (top >= T).sum()
    e = torch.from_numpy(e0.copy()).cuda()
    idx, val, ws = c.step("topk", g16 if dtype == "bf16" else g, e)
    assert not c.L.diag(ws, E.EF_OP_TOPK) & (E.DIAG_SLOW_PATH | E.DIAG_COUNT_MISMATCH)
    certify_topk(acc, c.offs, c.ks, host(idx), host(val), host(e))


def _topk_slot(d, density):
    """Static entries of a row of one sampled segment, by the library's rule at the smaller sample (a larger
    one expects fewer candidates and gives no more)."""
    k = int(np.floor(density * d + 0.5))
    ns = min(-(-16384 // 256), d // 256) * 256
    et = min(np.ceil(ns * k / d + 6 * (ns * k / d) ** 0.5 + 8) * d / ns, d) / -(-d // 4096)
    return min(4096, np.ceil((et + 4 * et ** 0.5 + 32) / 32) * 32)


# top-k with rows of every loudness: rows of no winner and rows whose winners alone exceed their static entries
# (a wavefront's chunks of 64, the overflow pool), with equal magnitudes, which at 0.7 are the threshold and
# more than win (their order kept by k_select, and by the rows from 2^20 winners on)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,density", [(4096 * 70 + 13, 0.0005), (4096 * 70 + 13, 0.012), (4096 * 70, 0.1), (4096 * 70 + 13, 0.7),
                                       (4096 * 520 + 1, 0.5), (4096 * 520 + 1, 0.7), (4096 * 16390, 0.03)])
def test_topk_crowded_rows(d, density, dtype):
    import paper_2009_09271_amd as E
    import torch
    announce("top-k crowded rows", d, density, dtype)
    c = Case([0, d], density)
    rng = np.random.default_rng(d % 997)
    g = rng.standard_normal(d, dtype=np.float32)
    for r in range(0, d // 4096, 7):  # every seventh row louder, by up to a factor of 64
        g[r * 4096:(r + 1) * 4096] *= np.float32(2.0 ** (r // 7 % 7))
    g[rng.random(d) < 0.2] = 0.25
    g += np.float32(0.0)  # (no -0: it leaves g + e as +0)
    if dtype == "bf16":
        g16 = to_bf16_bits(g)
        g = (g16.astype(np.uint32) << 16).view(np.float32)
    key = np.abs(g)
    T = np.partition(key, d - c.K)[d - c.K]
    above = np.add.reduceat((key > T).astype(np.int64), np.arange(0, d, 4096))  # (all of them candidates)
    assert density == 0.7 or above.max() > _topk_slot(d, density)
    assert density != 0.7 or (T == 0.25 and (key >= T).sum() > c.K)
    e = torch.zeros(d, dtype=torch.float32, device="cuda")
    idx, val, ws = c.step("topk", g16 if dtype == "bf16" else g, e)
    assert not c.L.diag(ws, E.EF_OP_TOPK) & (E.DIAG_SLOW_PATH | E.DIAG_COUNT_MISMATCH)
    certify_topk(g, c.offs, c.ks, host(idx), host(val), host(e))


# random-k in one batch: 256 select workgroups (one to a CU) and more (two to a CU), segments of one to 41 rows
@pytest.mark.parametrize("W", [16, 17])
def test_randk_batch_workgroups(W):
    import paper_2009_09271_amd as E
    import torch
    announce("random-k batch workgroups", W)
    offs = np.cumsum([0, 4096 * 40 + 3, 5, 4096, 70001, 1, 300] + [4097] * 10).tolist()
    c = Case(offs, 0.03)
    assert len(c.ks) == 16
    rng = np.random.default_rng(W)
    g = (rng.standard_normal((W, c.d), dtype=np.float32) + np.float32(0.0))
    gd, e = dev(g), torch.zeros((W, c.d), dtype=torch.float32, device="cuda")
    idx = torch.empty((W, c.K), dtype=torch.int32, device="cuda")
    val = torch.empty((W, c.K), dtype=torch.float32, device="cuda")
    ws, stride = E.batch_workspace(c.L, E.EF_OP_RANDK, W)
    seeds = [1000 + w for w in range(W)]
    E.ef_step_randk_batch(c.L, list(gd), list(e), seeds, 5, idx, val, ws, stride)
    for w in range(W):
        certify_randk(g[w], c.offs, c.ks, host(idx[w]), host(val[w]), host(e[w]), seeds[w], 5, f"worker {w}")
