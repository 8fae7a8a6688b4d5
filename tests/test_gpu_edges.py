"""Kernels at the sizes where their work split can go wrong: edges of
vectors, tiles and groups, remainders, views that start off a vector
boundary.  Same oracle and bounds as the kernel parity tests."""
import numpy as np
import pytest

from oracle import quant

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
DEV = "cuda"


def _srp():
    import paper_2106_12060_amd as srp
    return srp


def off_boundary(X, elements):
    """Contiguous device copy of X that starts `elements` past an allocation."""
    t = torch.from_numpy(np.ascontiguousarray(X))
    buf = torch.zeros(t.numel() + elements, dtype=t.dtype, device=DEV)
    buf[elements:] = t.reshape(-1).to(DEV)
    return buf[elements:].view(t.shape)


# groups of M = 4 ceil(256 / d) rows: fewer rows than a group, a remainder of
# rows, one column, widths around the 256-thread workgroup
@pytest.mark.parametrize("n,d,off", [(3, 60, 0), (1, 1, 1), (2049, 1, 0), (517, 3, 1), (1031, 255, 2),
                                     (64, 256, 0), (403, 257, 3), (4099, 131, 1)])
def test_staging_group_edges(n, d, off):
    srp = _srp()
    rng = np.random.default_rng(100 * n + d)
    grid = np.concatenate([quant._FP8_VALS, (quant._FP8_VALS[1:] + quant._FP8_VALS[:-1]) / 2])   # values and ties
    X = (rng.choice(grid, size=(n, d)) * rng.choice([-1.0, 1.0], size=(n, d)) *
         2.0 ** rng.integers(-3, 4, size=d)[None, :]).astype(np.float32)
    X[rng.random((n, d)) < 0.3] *= np.float32(1 + 2.0 ** -20)
    Xd = off_boundary(X, off)
    codes, scales = srp.srp_stage_fp8(Xd)
    ref, sc = quant.fp8_stage(X)
    np.testing.assert_array_equal(scales.cpu().numpy(), sc)
    np.testing.assert_array_equal(codes.cpu().numpy(), ref)
    np.testing.assert_array_equal(srp.srp_stage_bf16(Xd).float().cpu().numpy(), quant.bf16_round(X))
    Xb = off_boundary(quant.bf16_round(X).astype(np.float32), 0).to(torch.bfloat16)
    codes, scales = srp.srp_stage_fp8(Xb)
    ref, sc = quant.fp8_stage(Xb.double().cpu().numpy())
    np.testing.assert_array_equal(scales.cpu().numpy(), sc)
    np.testing.assert_array_equal(codes.cpu().numpy(), ref)


# blocks cut by rows (128) and by entries (4096), runs of empty rows, fewer
# rows than a block, column groups of 4, 8 and 16 lanes and two tiles of
# them, the widest matrix summed from the rows (2048 columns) and the first
# that takes the column copy, D gathered and (from 1024 / lanes rows a CU) in LDS
@pytest.mark.parametrize("n,d,nb,k,per_row,dt", [(1, 5, 1, 1, 3, np.float32), (63, 40, 2, 3, 35, np.float64),
                                                 (5000, 129, 2, 16, 12, np.float32), (4097, 2048, 1, 5, 90, np.float32),
                                                 (700, 2048, 1, 9, 1500, np.float64), (129, 1000, 2, 2, 30, np.float32),
                                                 (900, 2049, 2, 2, 40, np.float64), (20600, 2049, 1, 2, 4, np.float64),
                                                 (3000, 17, 1, 31, 0, np.float32),
                                                 (70001, 33, 2, 7, 4, np.float64), (40003, 50, 1, 27, 5, np.float32)])
def test_csr_products_edges(n, d, nb, k, per_row, dt):
    """Integer entries and directions: every sum is exact, so the products
    match bit for bit whatever the split."""
    from oracle import sparse as osp
    srp = _srp()
    rng = np.random.default_rng(n + d)
    blocks = []
    for _ in range(nb):
        counts = np.minimum(rng.poisson(per_row, n), d)
        counts[rng.random(n) < 0.2] = 0
        counts[n // 3: n // 3 + n // 4] = 0
        counts[-1] = min(d, 3 * per_row)
        ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
        cols = np.concatenate([np.sort(rng.choice(d, c, replace=False)) for c in counts]) if ptr[-1] else np.zeros(0)
        vals = rng.choice([-2.0, -1.0, 1.0, 2.0], size=int(ptr[-1])).astype(dt)
        blocks.append((ptr, cols.astype(np.int32), vals, d))
    Ws = [rng.integers(-3, 4, size=(d, k)).astype(np.float64) for _ in range(nb)]
    want = osp.pass_csr(blocks, Ws)
    on = [srp.Csr(*(torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in b[:3]), d) for b in blocks]
    wd = [torch.from_numpy(W).to(DEV) for W in Ws]
    got = srp.srp_gram_pass_csr(on[0], wd[0], *((on[1], wd[1]) if nb == 2 else ()))
    for g, w in zip(got, want):
        np.testing.assert_array_equal(g.cpu().numpy(), w)


@pytest.mark.parametrize("fault", ["decreasing", "repeat", "range", "negative", "end"])
def test_csr_structure_refused(fault):
    srp = _srp()
    n, d = 300, 50
    ptr = np.arange(0, 20 * n + 1, 20, dtype=np.int64)
    cols = np.tile(np.arange(0, 40, 2, dtype=np.int32), n)
    good = (ptr.copy(), cols.copy())
    r = 207
    if fault == "decreasing":
        ptr[r] = ptr[r + 1] + 5
    elif fault == "repeat":
        cols[20 * r + 17] = cols[20 * r + 16]
    elif fault == "range":
        cols[20 * r + 19] = d
    elif fault == "negative":
        cols[20 * r] = -1
    else:
        ptr[n] -= 1
    mk = lambda p, c: srp.Csr(torch.from_numpy(p).to(DEV), torch.from_numpy(c).to(DEV),
                              torch.ones(20 * n, device=DEV), d)
    W = torch.ones((d, 2), dtype=torch.float64, device=DEV)
    srp.srp_gram_pass_csr(mk(*good), W, mk(*good), W)
    for pair, name in (((mk(ptr, cols), mk(*good)), "A0"), ((mk(*good), mk(ptr, cols)), "A1")):
        with pytest.raises(srp.SrpError, match=name) as e:
            srp.srp_gram_pass_csr(pair[0], W, pair[1], W)
        assert e.value.code == srp.SRP_EINVAL


# blocks of 4, 8 and 16 rows at their last and first widths (32, 33, 64, 65
# and 128 tiles of 16 columns), a tile with one column, views just wide
# enough, rows off every 16-byte boundary, fewer rows than a block or a pair
# of blocks, an odd last block, short data on smaller blocks, direction
# groups with and without whole tiles, uneven views on either side of the
# producers' limit, more than the memory-side cache holds
@pytest.mark.parametrize("n,d0,d1,k,off", [(1, 64, 49, 1, 0), (3, 513, 0, 20, 1), (17, 49, 0, 16, 3),
                                           (8209, 256, 256, 16, 0), (8200, 257, 256, 9, 1), (9001, 512, 0, 17, 2),
                                           (9001, 513, 511, 14, 3), (2047, 1024, 0, 20, 0), (2049, 1025, 0, 3, 1),
                                           (1777, 1024, 1024, 10, 0), (1779, 1023, 1017, 7, 2), (777, 2048, 0, 19, 0),
                                           (640, 1500, 500, 10, 0), (3001, 99, 1201, 5, 3),
                                           (70003, 999, 2, 4, 0), (70001, 1000, 0, 12, 1)])
def test_gram_pass_block_edges(n, d0, d1, k, off):
    srp = _srp()
    rng = np.random.default_rng(n + d0 + d1)
    A = [rng.standard_normal((n, d), dtype=np.float32) for d in (d0, d1) if d]
    W = [rng.standard_normal((d, k)) for d in (d0, d1) if d]
    if d1 >= 49 and n > 2:
        A[1][n // 2, 33] = np.inf   # touches row 33 of J_1 and the products with P_1, nothing else
    D = [off_boundary(a, off + 1 - i) if off else off_boundary(a, 0) for i, a in enumerate(A)]
    out = srp.srp_gram_pass(D[0], torch.from_numpy(W[0]).to(DEV), *([D[1], torch.from_numpy(W[1]).to(DEV)] if d1 else []))
    Q = [a.astype(np.float64) for a in A]
    with np.errstate(invalid="ignore"):
        P = np.concatenate([a @ w for a, w in zip(Q, W)], axis=1)
        Pabs = np.concatenate([np.abs(a) @ np.abs(w) for a, w in zip(Q, W)], axis=1)
        ref, mag = [a.T @ P for a in Q], [np.abs(a).T @ Pabs for a in Q]
    for g, r, m in zip(out, ref, mag):
        g = g.cpu().numpy()
        ok = np.isfinite(r)
        assert np.array_equal(np.isfinite(g), ok)
        bound = (d0 + d1 + n + 2) * 2.0 ** -24 * m[ok]
        assert np.all(np.abs(g[ok] - r[ok]) <= bound)


# two views whose tiles are one more than their columns fill: the last of
# 129 (FP32, BF16 data) and of 57 (FP64)
@pytest.mark.parametrize("d0,d1,dt,comp", [(1985, 63, "f32", "f32"), (1025, 1023, "bf16", "f32"), (449, 447, "f64", "f64"),
                                           (833, 63, "f32", "f64")])
def test_gram_pass_one_tile_more(d0, d1, dt, comp):
    srp = _srp()
    rng = np.random.default_rng(d0)
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16, "f64": torch.float64}[dt]
    n, k = 701, 8
    A = [torch.from_numpy(rng.standard_normal((n, d))).to(tdt).to(DEV) for d in (d0, d1)]
    W = [rng.standard_normal((d, k)) for d in (d0, d1)]
    out = srp.srp_gram_pass(A[0], torch.from_numpy(W[0]).to(DEV), A[1], torch.from_numpy(W[1]).to(DEV), compute=comp)
    Q = [a.double().cpu().numpy() for a in A]
    P = np.concatenate([a @ w for a, w in zip(Q, W)], axis=1)
    Pabs = np.concatenate([np.abs(a) @ np.abs(w) for a, w in zip(Q, W)], axis=1)
    u = 2.0 ** -53 if comp == "f64" else 2.0 ** -24
    for g, q in zip(out, Q):
        assert np.all(np.abs(g.cpu().numpy() - q.T @ P) <= (d0 + d1 + n + 2) * u * (np.abs(q).T @ Pabs))


# BF16 products on whole numbers (P fits 8 bits, sums 24: every step exact):
# 16 and 8 rows a block at their last and first widths (32, 34, 64, 66 and
# 128 tiles), rows of 2, 4 and 6 columns past a 16-byte piece, rows off 16-byte
# boundaries, views that end half way into a 32-column tile, fewer rows than
# a block, an odd last block, one direction and sixteen
@pytest.mark.parametrize("n,d0,d1,k,off", [(3, 128, 0, 1, 0), (17, 256, 256, 16, 2), (1200, 258, 250, 5, 2),
                                           (2001, 514, 0, 16, 4), (2047, 500, 524, 9, 2), (1999, 526, 500, 7, 6),
                                           (4099, 1024, 1024, 16, 0), (4100, 2048, 0, 3, 0), (2501, 1006, 130, 10, 2),
                                           (9, 1500, 484, 8, 4), (70001, 2046, 0, 2, 2)])
def test_gram_pass_bf16_block_edges(n, d0, d1, k, off):
    srp = _srp()
    rng = np.random.default_rng(n + d0 + d1)
    A = [rng.integers(-1, 2, size=(n, d)).astype(np.float32) for d in (d0, d1) if d]
    W = [rng.integers(-1, 2, size=(d, k)).astype(np.float64) for d in (d0, d1) if d]
    if d1 and n > 2:
        A[1][n // 2, 40] = np.inf
    D = []
    for a in A:
        buf = torch.zeros(a.size + off, dtype=torch.bfloat16, device=DEV)
        buf[off:] = torch.from_numpy(a).reshape(-1).to(DEV)
        D.append(buf[off:].view(a.shape))
    out = srp.srp_gram_pass(D[0], torch.from_numpy(W[0]).to(DEV), *([D[1], torch.from_numpy(W[1]).to(DEV)] if d1 else []),
                            compute="bf16")
    with np.errstate(invalid="ignore"):
        P = np.concatenate([a.astype(np.float64) @ w for a, w in zip(A, W)], axis=1)
        ref = [a.T.astype(np.float64) @ P for a in A]
    assert np.max(np.abs(P[np.isfinite(P)])) <= 256
    for g, r in zip(out, ref):
        g = g.cpu().numpy()
        ok = np.isfinite(r)
        assert np.array_equal(np.isfinite(g), ok)
        np.testing.assert_array_equal(g[ok], r[ok])


# one diagonal block, a block with one column more and with one less, column
# blocks of R^-1 with one, two, three and four 64-row blocks to add
@pytest.mark.parametrize("d", [1, 63, 64, 65, 127, 129, 193, 256, 321])
def test_sketch_factor_block_edges(d):
    srp = _srp()
    rng = np.random.default_rng(d)
    A = rng.standard_normal((2 * d + 3, d))
    R, Rinv = srp.srp_sketch_factor(torch.from_numpy(A).to(DEV), 0.5)
    R, Rinv = R.cpu().numpy(), Rinv.cpu().numpy()
    G = A.T @ A + 0.5 * np.eye(d)
    assert not np.tril(R, -1).any() and not np.tril(Rinv, -1).any()
    # backward error of the factor: (d + 1) u |R|^T |R|, and of the Gram: n u |A|^T |A|
    u = 2.0 ** -53
    assert np.all(np.abs(R.T @ R - G) <= 4 * (3 * d + 8) * u * (np.abs(R).T @ np.abs(R) + np.abs(A).T @ np.abs(A)))
    # residual of the triangular inverse, formed by blocks: d u |R^-1| |R| |R^-1| |R|
    W = np.abs(Rinv) @ np.abs(R)
    assert np.all(np.abs(Rinv @ R - np.eye(d)) <= 4 * (d + 8) * u * (W @ W))


@pytest.mark.parametrize("d,col", [(64, 63), (150, 64), (150, 149), (200, 130)])
def test_sketch_factor_bad_pivot_in_any_block(d, col):
    srp = _srp()
    A = np.random.default_rng(d).standard_normal((2 * d, d))
    A[:, col] = 0.0
    with pytest.raises(srp.SrpError) as e:
        srp.srp_sketch_factor(torch.from_numpy(A).to(DEV), 0.0)
    assert e.value.code == srp.SRP_ENOTSPD


# one bucket of more rows than a sorting workgroup holds and than a chunk it
# compares with, more buckets than rows, rows of less than a wave of 16-byte
# pieces and the first of more, a rest of columns, several column chunks, rows
# off vector boundaries, data past the memory-side cache; every row added in
# ascending order in the sketch's type, so bit for bit
@pytest.mark.parametrize("n,d,s,dt,off", [(9001, 70, 1, "f32", 1), (5, 3, 9, "f64", 0), (2500, 127, 1, "f64", 1),
                                          (2049, 128, 2, "f64", 1), (1025, 255, 1, "f32", 0), (4097, 257, 40, "f32", 3),
                                          (1500, 511, 3, "bf16", 0), (1024, 1031, 8, "bf16", 1), (300, 2049, 3, "f32", 2),
                                          (130, 4099, 2, "bf16", 1), (34001, 2001, 900, "f32", 1)])
def test_countsketch_bucket_edges(n, d, s, dt, off):
    from oracle import sketch as osk
    srp = _srp()
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16, "f64": torch.float64}[dt]
    X = torch.from_numpy(np.random.default_rng(n + d).standard_normal((n, d), dtype=np.float32)).to(tdt)
    buf = torch.zeros(n * d + off, dtype=tdt, device=DEV)
    buf[off:] = X.reshape(-1).to(DEV)
    out = srp.srp_countsketch(buf[off:].view(n, d), s, 77).cpu().numpy()
    h, g = osk.countsketch_hash(n, s, 77)
    cols = np.unique(np.r_[0:min(d, 20), max(0, d - 20):d])
    acc = np.float64 if dt == "f64" else np.float32
    ref = np.zeros((s, cols.size), dtype=acc)
    np.add.at(ref, h, g.astype(acc)[:, None] * X[:, torch.from_numpy(cols)].to(torch.float64 if dt == "f64" else torch.float32).numpy())
    np.testing.assert_array_equal(out[:, cols], ref)


# the window around the threshold: whole key range, all rows, one row, lists
# that overflow (selection over all keys instead), one chunk, the most chunks
@pytest.mark.parametrize("n,s", [(2, 1), (2, 2), (100, 128), (1024, 512), (1024, 1), (3000, 2048), (4096, 4096),
                                 (65536, 30000), (200000, 4000), (200000, 262144), (1 << 20, 1), (1 << 20, 20000),
                                 (1 << 20, 500000)])
@pytest.mark.parametrize("seed", [0, 987654321])
def test_srht_row_sample_edges(n, s, seed):
    from oracle import sketch as osk
    srp = _srp()
    rows = srp.srp_srht_rows(n, s, seed).cpu().numpy()
    np.testing.assert_array_equal(rows, osk.srht_rows(osk.srht_padded_rows(n), s, seed))


def poison_lds():
    """Leaves quiet NaNs of both precisions all over every CU's LDS: a pass
    over rows that hold nothing else, more row blocks than workgroups."""
    srp = _srp()
    bits = torch.full((16 * 2048, 896), 0x7FFFFFFF7FFFFFFF, dtype=torch.int64, device=DEV)
    srp.srp_gram_pass(bits.view(torch.float64), torch.ones((896, 16), dtype=torch.float64, device=DEV), compute="f64")


# views whose last tile reaches past the row's pitch (the last row's into what
# follows the block), or past the columns that are staged (2048 in FP32); the
# first view's last tile ends inside the second's columns
@pytest.mark.parametrize("d0,d1,dt,comp", [(63, 65, "f64", "f64"), (100, 27, "f64", "f64"), (127, 65, "bf16", "f64"),
                                           (35, 29, "f32", "f32"), (30, 33, "bf16", "f32"), (1985, 63, "f32", "f32"),
                                           (1023, 1025, "bf16", "f32"), (831, 65, "f32", "f64")])
def test_gram_pass_reads_only_its_columns(d0, d1, dt, comp):
    """Whole numbers (exact in every precision here), after a call that
    filled LDS with NaNs; then an infinity in the second view's first column,
    which must reach P_1 and J_1's first row only."""
    srp = _srp()
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16, "f64": torch.float64}[dt]
    n, k = 70, 3
    rng = np.random.default_rng(d0)
    A = [rng.choice([-1.0, 1.0], size=(n, d)) for d in (d0, d1)]
    W = [rng.choice([-1.0, 1.0], size=(d, k)) for d in (d0, d1)]
    for planted in (False, True):
        if planted:
            A[1][n // 2, 0] = np.inf
        with np.errstate(invalid="ignore"):
            P = np.concatenate([a @ w for a, w in zip(A, W)], axis=1)
            ref = [a.T @ P for a in A]
        D = [torch.from_numpy(a).to(tdt).to(DEV) for a in A]
        Wd = [torch.from_numpy(w).to(DEV) for w in W]
        poison_lds()
        out = srp.srp_gram_pass(D[0], Wd[0], D[1], Wd[1], compute=comp)
        for g, r in zip(out, ref):
            np.testing.assert_array_equal(g.cpu().numpy(), r)


# widths that end in each way inside a 16-byte piece and a tile, blocks of 4,
# 8 and 16 rows, one and two views
@pytest.mark.parametrize("n,d0,d1,k", [(5000, 301, 203, 8), (9000, 250, 0, 12), (4500, 333, 335, 16), (9001, 1000, 0, 19),
                                       (9000, 998, 500, 7), (700, 66, 79, 2), (40, 2047, 0, 20), (33, 1500, 484, 8)])
def test_gram_pass_row_keeps_to_its_columns(n, d0, d1, k):
    """Whole numbers with an infinity in the first and in the last column of
    single rows, one of them a block's first: it reaches the sums of its own
    row's products only."""
    srp = _srp()
    assert srp.srp_gram_pass_kernel("f32", "f32", d0, d1, k).startswith("k_pass_quad")
    rng = np.random.default_rng(n + d0)
    for r, c in ((32, 0), (17, 0), (n - 1, 0), (15, -1)):
        A = [rng.choice([-1.0, 1.0], size=(n, d)).astype(np.float32) for d in (d0, d1) if d]
        W = [rng.choice([-1.0, 1.0], size=(d, k)) for d in (d0, d1) if d]
        A[-1][r, c] = np.inf
        with np.errstate(invalid="ignore"):
            P = np.concatenate([a.astype(np.float64) @ w for a, w in zip(A, W)], axis=1)
            ref = [a.T.astype(np.float64) @ P for a in A]
        D = [torch.from_numpy(a).to(DEV) for a in A]
        Wd = [torch.from_numpy(w).to(DEV) for w in W]
        out = srp.srp_gram_pass(D[0], Wd[0], *((D[1], Wd[1]) if d1 else ()))
        for g, q in zip(out, ref):
            np.testing.assert_array_equal(g.cpu().numpy(), q)


# the shapes of test_gram_pass_block_edges on whole numbers whose sums are
# exact in FP32: a row or a column left out or read twice anywhere changes the
# result
@pytest.mark.parametrize("n,d0,d1,k,off", [(1, 64, 49, 1, 0), (3, 513, 0, 20, 1), (17, 49, 0, 16, 3),
                                           (8209, 256, 256, 16, 0), (8200, 257, 256, 9, 1), (9001, 512, 0, 17, 2),
                                           (9001, 513, 511, 14, 3), (2047, 1024, 0, 20, 0), (2049, 1025, 0, 3, 1),
                                           (1777, 1024, 1024, 10, 0), (1779, 1023, 1017, 7, 2), (777, 2048, 0, 19, 0),
                                           (640, 1500, 500, 10, 0), (3001, 99, 1201, 5, 3), (70003, 999, 50, 4, 0),
                                           (70003, 999, 2, 4, 0), (70001, 1000, 0, 12, 1), (5003, 700, 600, 14, 1)])
def test_gram_pass_block_edges_exact(n, d0, d1, k, off):
    srp = _srp()
    rng = np.random.default_rng(n + d0 + d1)
    A = [rng.integers(-1, 2, size=(n, d)).astype(np.float32) for d in (d0, d1) if d]
    W = [rng.choice([-1.0, 1.0], size=(d, k)) for d in (d0, d1) if d]
    for a in A:   # the last rows and every view's first and last columns take part
        a[-32:] = rng.choice([-1.0, 1.0], size=a[-32:].shape)
        a[:, [0, -1]] = rng.choice([-1.0, 1.0], size=(n, 2))
    P = np.concatenate([a.astype(np.float64) @ w for a, w in zip(A, W)], axis=1)
    assert np.abs(P).sum(axis=0).max() < 2 ** 24   # bounds every partial sum
    D = [off_boundary(a, off + 1 - i) if off else off_boundary(a, 0) for i, a in enumerate(A)]
    Wd = [torch.from_numpy(w).to(DEV) for w in W]
    out = srp.srp_gram_pass(D[0], Wd[0], *((D[1], Wd[1]) if d1 else ()))
    for g, a in zip(out, A):
        np.testing.assert_array_equal(g.cpu().numpy(), a.T.astype(np.float64) @ P)


def call_us(f):
    """Fastest of twenty calls (each waits for its work), in us."""
    import time
    f()
    best = float("inf")
    for _ in range(20):
        t = time.perf_counter()
        f()
        best = min(best, time.perf_counter() - t)
    return 1e6 * best


# fewer rows than a group and a remainder of rows on either side of the width
# (64 columns a CU) from which a column's maximum is taken by one lane
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("n,d", [(3, 16383), (7, 16383), (3, 16384), (7, 16389), (66, 16384), (1, 100003), (5, 100003)])
def test_fp8_staging_of_wide_rows(n, d, dt):
    srp = _srp()
    X = torch.from_numpy(np.random.default_rng(n * d).standard_normal((n, d), dtype=np.float32))
    X[-1, ::3] *= 1000.0   # the maximum of these columns lies in the last row
    X = X.to(torch.bfloat16 if dt == "bf16" else torch.float32)
    codes, scales = srp.srp_stage_fp8(X.to(DEV))
    ref, sc = quant.fp8_stage(X.double().numpy() if dt == "bf16" else X.numpy())
    np.testing.assert_array_equal(scales.cpu().numpy(), sc)
    np.testing.assert_array_equal(codes.cpu().numpy(), ref)


@pytest.mark.parametrize("n", [7, 8])
def test_fp8_staging_of_wide_rows_costs_no_more(n):
    """A few wide rows, with and without a remainder past the last group,
    against as many elements in rows of 1000: scales and codes are as many
    bytes again, and the calls' fixed cost is most of either."""
    srp = _srp()
    X = torch.randn(8_000_000, device=DEV)
    wide, tall = X[:n * 1_000_000].view(n, -1), X[:n * 1_000_000].view(-1, 1000)
    assert call_us(lambda: srp.srp_stage_fp8(wide)) < 2.5 * call_us(lambda: srp.srp_stage_fp8(tall))


# the largest windows (half of the rows), chunks whose whole keys are listed;
# and seeds for which the smallest of 1024 keys lies past the window (found by
# searching), where the selection over all keys runs
@pytest.mark.parametrize("n,s,seed", [(1 << 20, 1 << 19, 3), (1 << 20, 131072, 4), (1 << 19, 262144, 5), (262144, 131072, 6),
                                      (1024, 512, 7), (2048, 1500, 8), (32768, 16384, 9), (65536, 32768, 10),
                                      (1024, 1, 4990599), (1000, 1, 6866827)])
def test_srht_row_sample_windows(n, s, seed):
    from oracle import sketch as osk
    srp = _srp()
    rows = srp.srp_srht_rows(n, s, seed).cpu().numpy()
    np.testing.assert_array_equal(rows, osk.srht_rows(osk.srht_padded_rows(n), s, seed))


def test_srht_row_sample_of_many_rows_costs_no_more():
    """Half of 2^20 rows: 125 times the rows written, and the keys read as
    often as for 4000 of them; either call is a few launches."""
    srp = _srp()
    many, few = (call_us(lambda: srp.srp_srht_rows(1 << 20, s, 5)) for s in (1 << 19, 4000))
    assert many < 4 * few


def csr_rows(n, d, per_row, bad=None):
    """n rows of per_row entries, column c in [c d / per_row, (c + 1) d / per_row); `bad` replaces the last index."""
    lo = (torch.arange(per_row, device=DEV) * d) // per_row
    width = torch.diff(torch.cat([lo, torch.tensor([d], device=DEV)]))
    idx = (lo + (torch.rand((n, per_row), device=DEV) * width).long().clamp(max=width - 1)).to(torch.int32).reshape(-1)
    if bad is not None:
        idx[-1] = bad
    vals = torch.randint(1, 4, (n * per_row,), device=DEV).to(torch.float32)
    return _srp().Csr(torch.arange(n + 1, device=DEV, dtype=torch.int64) * per_row, idx, vals, d)


def test_csr_structure_check_of_long_rows_costs_no_more():
    """As many entries in a few long rows as in many short ones; a bad last
    index ends the call after the check."""
    srp = _srp()
    def refused(A):
        with pytest.raises(srp.SrpError):
            srp.srp_countsketch_csr(A, 64, 1)
    few, many = csr_rows(1000, 8000, 4000, bad=-1), csr_rows(40000, 8000, 100, bad=8000)
    assert call_us(lambda: refused(few)) < 2 * call_us(lambda: refused(many))


# a row that ends at, one before and one after a whole step of the long rows' loop
@pytest.mark.parametrize("length", [15, 16, 17, 112, 113, 127, 128, 129, 241, 700])
def test_csr_structure_faults_in_a_long_row(length):
    srp = _srp()
    n, d = 9, 800
    cols = np.tile(np.arange(length, dtype=np.int32), n)
    ptr = np.arange(0, n * length + 1, length, dtype=np.int64)
    mk = lambda c: srp.Csr(torch.from_numpy(ptr).to(DEV), torch.from_numpy(c).to(DEV), torch.ones(n * length, device=DEV), d)
    srp.srp_countsketch_csr(mk(cols), 8, 1)
    for at in sorted({0, 1, 15, 16, length // 2, length - 2, length - 1} & set(range(length))):
        for value in {-1, d, cols[at - 1] if at else -7}:
            bad = cols.copy()
            bad[4 * length + at] = value
            with pytest.raises(srp.SrpError):
                srp.srp_countsketch_csr(mk(bad), 8, 1)


def test_csr_products_of_few_long_rows_cost_no_more():
    """A million entries in 1000 rows against the same number in 50000: the
    row ranges follow the entries, not the rows alone."""
    srp = _srp()
    W = torch.ones((2000, 8), dtype=torch.float64, device=DEV)
    few, many = csr_rows(1000, 2000, 1000), csr_rows(50000, 2000, 20)
    assert call_us(lambda: srp.srp_gram_pass_csr(few, W, few, W)) < 2.5 * call_us(lambda: srp.srp_gram_pass_csr(many, W, many, W))


# both sides of the rule that sums A^T P from the rows or from the column copy:
# few entries for a block's columns and many, P of one, two and four tiles
@pytest.mark.parametrize("n,d,per_row,k", [(300000, 1000, 2, 64), (300000, 2000, 8, 32), (300000, 2000, 30, 16),
                                           (300000, 1000, 2, 16), (66000, 2048, 40, 33), (66000, 2048, 3, 64)])
def test_csr_products_on_either_route(n, d, per_row, k):
    srp = _srp()
    A = csr_rows(n, d, per_row)
    W = torch.randint(-3, 4, (d, k), device=DEV).to(torch.float64)
    J, _ = srp.srp_gram_pass_csr(A, W)
    dense = torch.zeros((n, d), dtype=torch.float64, device=DEV)
    dense.scatter_(1, A.col_idx.view(n, per_row).long(), A.values.view(n, per_row).double())
    assert torch.equal(J, dense.t().contiguous() @ (dense @ W))   # whole numbers: exact whatever the order


def test_csr_solve_iterations_take_the_faster_route():
    """Two entries a row in 2000 columns: an iteration with eight times the
    directions is bound by the same few entries."""
    srp = _srp()
    X, Y = csr_rows(300000, 2000, 2), csr_rows(300000, 2000, 2)
    opt = srp.srp_default_options(max_iter=40, warm_start_iters=4)
    def iteration(k):
        infos = [srp.cca_solve_csr(X, Y, k, 0.1, 0.1, 6000, tol=1e-30, options=opt)[3] for _ in range(4)]
        return min(i["ms_iterate"] / i["iterations"] for i in infos)
    assert iteration(16) < 2.5 * iteration(2)


def test_countsketch_of_few_bf16_rows_costs_no_more():
    """More buckets than rows: the sketch's FP32 stores are the work, the same
    for BF16 and FP32 rows."""
    srp = _srp()
    A = torch.randn((119, 9427), device=DEV)
    B = A.to(torch.bfloat16)
    assert call_us(lambda: srp.srp_countsketch(B, 11602, 5)) < 1.35 * call_us(lambda: srp.srp_countsketch(A, 11602, 5))


# the first steps' products by the GEMM: one such step (the last column block
# of a single column), three, and the largest without
@pytest.mark.parametrize("d", [7105, 7300, 7104])
def test_sketch_factor_large(d):
    srp = _srp()
    A = torch.randn((d + 70, d), device=DEV, dtype=torch.float64)
    R, Rinv = srp.srp_sketch_factor(A, 1.0)
    assert not torch.tril(R, -1).any() and not torch.tril(Rinv, -1).any()
    G = A.t().contiguous() @ A + torch.eye(d, device=DEV, dtype=torch.float64)
    # bounds of test_sketch_factor_block_edges
    u = 2.0 ** -53
    Ra, Aa = R.abs(), A.abs()
    bound = 4 * (3 * d + 8) * u * (Ra.t().contiguous() @ Ra + Aa.t().contiguous() @ Aa)
    assert torch.all((R.t().contiguous() @ R - G).abs() <= bound)
    W = Rinv.abs() @ Ra
    assert torch.all((Rinv @ R - torch.eye(d, device=DEV, dtype=torch.float64)).abs() <= 4 * (d + 8) * u * (W @ W))


def test_fp8_staging_of_an_infinity():
    """The column's scale is the largest power of two that 448 leaves finite
    one step down; finite entries vanish beside it, the infinity saturates and
    the other columns are as without it."""
    srp = _srp()
    X = np.random.default_rng(0).standard_normal((700, 40)).astype(np.float32)
    ref, sc = quant.fp8_stage(X)
    X[333, 7] = np.inf
    codes, scales = srp.srp_stage_fp8(torch.from_numpy(X).to(DEV))
    codes, scales = codes.cpu().numpy(), scales.cpu().numpy()
    other = np.arange(40) != 7
    np.testing.assert_array_equal(scales[other], sc[other])
    np.testing.assert_array_equal(codes[:, other], ref[:, other])
    assert scales[7] == 2.0 ** 1016
    assert codes[333, 7] & 0x7F == 0x7E and not np.delete(codes[:, 7], 333).any()


# the streamed pass of two views with many directions: the same with its rows
@pytest.mark.parametrize("n,d0,d1,k", [(5003, 701, 598, 14), (33, 1500, 484, 10), (900, 1023, 1018, 16), (17, 1600, 79, 12)])
def test_gram_pass_streamed_row_keeps_to_its_columns(n, d0, d1, k):
    assert _srp().srp_gram_pass_kernel("f32", "f32", d0, d1, k) == "k_pass_dma"
    srp = _srp()
    rng = np.random.default_rng(n + d0)
    for v, r, c in ((0, 8, 0), (0, 11, 0), (1, 16, 0), (1, 9, 1), (0, n - 1, 0), (1, 15, -1)):
        A = [rng.choice([-1.0, 1.0], size=(n, d)).astype(np.float32) for d in (d0, d1)]
        W = [rng.choice([-1.0, 1.0], size=(d, k)) for d in (d0, d1)]
        A[v][r, c] = np.inf
        with np.errstate(invalid="ignore"):
            P = np.concatenate([a.astype(np.float64) @ w for a, w in zip(A, W)], axis=1)
            ref = [a.T.astype(np.float64) @ P for a in A]
        D = [torch.from_numpy(a).to(DEV) for a in A]
        Wd = [torch.from_numpy(w).to(DEV) for w in W]
        for g, q in zip(srp.srp_gram_pass(D[0], Wd[0], D[1], Wd[1]), ref):
            np.testing.assert_array_equal(g.cpu().numpy(), q)


# FP64 CCA whose last tile ends past the rows' pitch, after a call that filled
# LDS with NaNs: the products of every iteration and of the finish, whose
# rotation and signs follow from them, are those of the data alone
@pytest.mark.parametrize("dx,dy", [(9, 177), (63, 65), (39, 152)])
def test_cca_solve_after_nans_in_lds(dx, dy):
    from oracle import direct, metrics
    srp = _srp()
    rng = np.random.default_rng(dx)
    n, k, lam = 4000, 3, 1e-2
    Z = rng.standard_normal((n, 6))
    X = Z @ rng.standard_normal((6, dx)) + rng.standard_normal((n, dx))
    Y = Z @ rng.standard_normal((6, dy)) + rng.standard_normal((n, dy))
    sig_true, _, _ = direct.cca_direct(X, Y, lam, lam)
    Xd, Yd = torch.from_numpy(X).to(DEV), torch.from_numpy(Y).to(DEV)
    poison_lds()
    U, V, sig, info = srp.cca_solve(Xd, Yd, k, lam, lam, 4 * dy, tol=1e-10, options=srp.srp_default_options(max_iter=2000))
    Uh, Vh = U.cpu().numpy(), V.cpu().numpy()
    assert info["status"] == 0
    assert metrics.cca_rel_objective_error(Uh, Vh, X, Y, lam, lam, sig_true) < 1e-10
    assert max(metrics.constraint_residual(Uh, X, lam), metrics.constraint_residual(Vh, Y, lam)) < 1e-11
