"""Batches: products of several vectors from the packed codes on the matrix cores, at the edges
of their tiles.  Integer-valued vectors, so every output is exact (sums of at most 14336 products
of magnitude 8 stay far below 2^24) and the reference is the oracle's dense definition."""
import numpy as np
import pytest

import oracle
import rsr_inputs as gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
rsr = pytest.importorskip("paper_2603_27462_amd")
DEV = "cuda:0"


def _matrix(kind, rows, cols, seed):
    return gen.binary_matrix(rows, cols, 0.6, seed) if kind == rsr.RSR_BINARY else gen.ternary_matrix(rows, cols, 0.35, seed)


def _check(h, M, batch, bf16, pad, seed, distinct=None):
    """Vectors pad elements apart beyond their length (odd pads: rows of v off every alignment);
    `distinct`: how many different vectors, repeated in a fixed order, to keep the oracle quick."""
    rows, cols = M.shape
    distinct = min(batch, distinct or batch)
    vi = np.stack([gen.integer_f32(cols, seed=seed + i) for i in range(distinct)])
    order = np.random.default_rng(seed).permutation(np.arange(batch) % distinct)
    vbuf = torch.full((batch, cols + pad), float("nan"), dtype=torch.bfloat16 if bf16 else torch.float32, device=DEV)
    vbuf[:, :cols] = torch.from_numpy(vi).to(DEV).to(vbuf.dtype)[torch.from_numpy(order).to(DEV)]
    out = torch.full((batch, rows + 3), -5.0, dtype=torch.float32, device=DEV)
    rsr.rsr_matvec_ex(h, vbuf[:, :cols], scale=-2.0, out=out[:, :rows])
    got = out.cpu().numpy()
    assert np.all(got[:, rows:] == -5.0)                     # nothing past the rows
    want = np.stack([oracle.dense_matvec(M, x.astype(np.float64), -2.0) for x in vi])
    assert np.array_equal(got[:, :rows].astype(np.float64), want[order])


# one workgroup holds 32 rows x 32 vectors, eight waves share the columns in tiles of 256
@pytest.mark.parametrize("kind,rows,cols,k,batch,bf16,pad", [
    (rsr.RSR_BINARY, 1, 1, 1, 4, True, 0),
    (rsr.RSR_TERNARY_FUSED, 31, 7, 2, 5, False, 1),
    (rsr.RSR_TERNARY_2PASS, 33, 255, 4, 31, True, 3),
    (rsr.RSR_BINARY, 32, 257, 8, 32, False, 1),
    (rsr.RSR_TERNARY_FUSED, 65, 2049, 5, 33, True, 1),
    (rsr.RSR_DENSE_TERNARY_P2, 48, 1791, 0, 63, False, 0),
    (rsr.RSR_BINARY, 50, 2305, 6, 64, True, 0),
    (rsr.RSR_TERNARY_FUSED, 40, 14336, 8, 17, True, 0),
    (rsr.RSR_TERNARY_2PASS, 20, 32766, 6, 9, False, 2)])
def test_columns_split_over_waves(kind, rows, cols, k, batch, bf16, pad):
    M = _matrix(kind, rows, cols, 300 + rows + cols)
    _check(rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), k, kind), M, batch, bf16, pad, rows)


# 16 vectors or 32 per workgroup, one to four row groups, and waves that share rows instead of columns
# when there are few tiles of columns: sizes on both sides of every choice
@pytest.mark.parametrize("kind,rows,cols,k,batch,bf16,pad", [
    (rsr.RSR_DENSE_TERNARY_P2, 320 * 16, 300, 0, 5, True, 0), (rsr.RSR_BINARY, 320 * 16 + 1, 520, 8, 16, False, 1),
    (rsr.RSR_DENSE_TERNARY_P2, 640 * 16 + 1, 1025, 0, 16, True, 3), (rsr.RSR_BINARY, 640 * 16 - 15, 257, 6, 7, False, 0),
    (rsr.RSR_TERNARY_FUSED, 60001, 299, 6, 6, True, 1), (rsr.RSR_BINARY, 33333, 700, 8, 13, False, 0),
    (rsr.RSR_DENSE_TERNARY_P2, 8209, 1100, 0, 17, False, 1), (rsr.RSR_BINARY, 16400, 260, 8, 32, True, 0),
    (rsr.RSR_TERNARY_2PASS, 30011, 303, 8, 25, False, 3), (rsr.RSR_DENSE_TERNARY_P2, 4097, 2100, 0, 97, True, 0),
    (rsr.RSR_BINARY, 1500, 1999, 8, 300, False, 1), (rsr.RSR_DENSE_TERNARY_P2, 40001, 513, 0, 18, True, 1),
    (rsr.RSR_DENSE_TERNARY_P2, 512 * 16, 2817, 0, 5, False, 1), (rsr.RSR_BINARY, 512 * 16 + 3, 2817, 8, 5, False, 1),
    (rsr.RSR_DENSE_TERNARY_P2, 512 * 16 + 3, 2820, 0, 9, True, 1)])
def test_split_shapes(kind, rows, cols, k, batch, bf16, pad):
    M = _matrix(kind, rows, cols, 1100 + cols)
    _check(rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), k, kind), M, batch, bf16, pad, cols, distinct=4)


# one workgroup holds 128 rows x 128 vectors
@pytest.mark.parametrize("kind,rows,cols,k,batch,bf16,pad", [
    (rsr.RSR_TERNARY_FUSED, 128 * 24, 256, 4, 128 * 8, True, 0),
    (rsr.RSR_BINARY, 128 * 24 + 1, 255, 8, 128 * 8 + 1, False, 1),
    (rsr.RSR_DENSE_TERNARY_P2, 128 * 33 - 17, 777, 0, 128 * 7 - 1, True, 1),
    (rsr.RSR_TERNARY_2PASS, 128 * 100 - 1, 33, 6, 129, False, 0),
    (rsr.RSR_BINARY, 128 * 193, 40, 8, 65, True, 5),
    # eight waves up to 256 workgroups, four beyond
    (rsr.RSR_DENSE_TERNARY_P2, 128 * 128 - 5, 513, 0, 33, True, 1), (rsr.RSR_BINARY, 128 * 160 - 1, 767, 8, 120, False, 1),
    (rsr.RSR_TERNARY_FUSED, 128 * 64, 1024, 8, 512, True, 0), (rsr.RSR_DENSE_TERNARY_P2, 128 * 85, 290, 0, 300, False, 3),
    (rsr.RSR_BINARY, 128 * 86, 300, 8, 300, False, 0)])
def test_tiles_of_rows_and_vectors(kind, rows, cols, k, batch, bf16, pad):
    M = _matrix(kind, rows, cols, 500 + cols)
    _check(rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), k, kind), M, batch, bf16, pad, cols, distinct=40)


@pytest.mark.parametrize("kind,rows,cols,k", [(rsr.RSR_BINARY, 77, 300, 6), (rsr.RSR_BINARY, 90, 200, 8),
                                              (rsr.RSR_TERNARY_2PASS, 45, 513, 7),
                                              (rsr.RSR_TERNARY_FUSED, 203, 1500, 8)])
def test_codes_after_loading_and_after_a_new_matrix(kind, rows, cols, k):
    """The packed codes of a handle made from bytes, and of a handle whose matrix was replaced."""
    M = _matrix(kind, rows, cols, 8)
    h = rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), k, kind)
    _check(rsr.rsr_deserialize(rsr.rsr_serialize(h)), M, 6, True, 1, 4)
    M2 = M[::-1].copy()          # rows in another order: the streams keep their lengths' bounds
    try:
        rsr.rsr_preprocess_into(h, torch.from_numpy(M2).to(DEV))
    except rsr.RsrError as e:
        assert e.code == 3       # other blocks may not fit the layout of the first matrix
        return
    _check(h, M2, 6, False, 0, 5)


# up to four vectors: 1, 2, 4, 8 or 16 waves share the columns of 16 rows (1, 2, 4, 8 or 24 tiles of
# 256 columns and more), steps of one, two or four tiles
@pytest.mark.parametrize("cols", [1, 256, 257, 768, 1025, 2047, 2305, 5888, 6145, 14336, 32766])
@pytest.mark.parametrize("kind,rows,batch,bf16,pad", [
    (rsr.RSR_DENSE_TERNARY_P2, 17, 1, True, 0), (rsr.RSR_DENSE_TERNARY_P2, 65, 1, False, 0),
    (rsr.RSR_BINARY, 15, 2, True, 1), (rsr.RSR_TERNARY_FUSED, 33, 3, False, 1),
    (rsr.RSR_TERNARY_2PASS, 16, 4, True, 0), (rsr.RSR_BINARY, 40, 4, False, 3)])
def test_few_vectors(kind, rows, batch, bf16, pad, cols):
    M = _matrix(kind, rows, cols, 700 + rows + cols)
    _check(rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), 5, kind), M, batch, bf16, pad, rows)


# up to 256 columns and many rows: waves go through several row groups (the last one short), and
# 32 or 64 vectors share a workgroup; sizes on both sides of where these kernels start
@pytest.mark.parametrize("kind,rows,cols,batch,bf16,pad", [
    (rsr.RSR_DENSE_TERNARY_P2, 159999, 9, 1, False, 0), (rsr.RSR_DENSE_TERNARY_P2, 160001, 256, 1, False, 0),
    (rsr.RSR_DENSE_TERNARY_P2, 500007, 30, 1, True, 0), (rsr.RSR_BINARY, 65537, 251, 3, False, 1),
    (rsr.RSR_BINARY, 140001, 64, 4, True, 3), (rsr.RSR_TERNARY_2PASS, 65536, 17, 2, True, 0),
    (rsr.RSR_TERNARY_FUSED, 5, 1, 5, False, 1), (rsr.RSR_BINARY, 70001, 255, 16, False, 0),
    (rsr.RSR_BINARY, 1047, 200, 9, True, 1), (rsr.RSR_TERNARY_2PASS, 33001, 100, 13, False, 2),
    (rsr.RSR_TERNARY_FUSED, 10001, 256, 17, False, 1), (rsr.RSR_BINARY, 16384, 33, 32, True, 0),
    (rsr.RSR_BINARY, 70003, 129, 65, False, 1), (rsr.RSR_DENSE_TERNARY_P2, 40000, 7, 128, True, 0),
    (rsr.RSR_BINARY, 16385, 255, 33, True, 3)])
def test_tables(kind, rows, cols, batch, bf16, pad):
    M = _matrix(kind, rows, cols, 900 + cols)
    _check(rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), 8, kind), M, batch, bf16, pad, cols, distinct=5)


def test_stacked_table():
    """Sibling tables in one launch; every layer starts a new row group."""
    Ms = [_matrix(rsr.RSR_DENSE_TERNARY_P2, r, 40, 60 + r) for r in (100001, 17, 99999)]
    h = rsr.rsr_preprocess_stacked([torch.from_numpy(M).to(DEV) for M in Ms], 0, rsr.RSR_DENSE_TERNARY_P2)
    v = gen.integer_f32(40, seed=3)
    outs = rsr.rsr_matvec_stacked(h, torch.from_numpy(v).to(DEV), [1.0, -2.0, 0.5])
    for M, out, scale in zip(Ms, outs, (1.0, -2.0, 0.5)):
        assert np.array_equal(out.cpu().numpy().astype(np.float64), oracle.dense_matvec(M, v.astype(np.float64), scale))


@pytest.mark.parametrize("kind,rows,cols", [(rsr.RSR_TERNARY_FUSED, 203, 1500), (rsr.RSR_BINARY, 5000, 130)])
def test_library_chosen_height_after_loading(kind, rows, cols):
    """k = 0: however the handle multiplies single vectors, its copy made from bytes does the same,
    bit for bit; bytes without that field (written before it existed) are still read."""
    M = _matrix(kind, rows, cols, 21)
    h = rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), 0, kind)
    blob = rsr.rsr_serialize(h)
    h2 = rsr.rsr_deserialize(blob)
    assert rsr.rsr_kernel_name(h2) == rsr.rsr_kernel_name(h)
    v = torch.from_numpy(gen.normal_f32(cols, seed=8)).to(DEV)
    assert torch.equal(rsr.rsr_matvec(h, v), rsr.rsr_matvec(h2, v))
    old = np.concatenate([blob[:120], blob[128:]])      # the field is the header's last
    old[4:8].view(np.int32)[0] = 2
    old[112:120].view(np.int64)[0] -= 8
    for handle in (h, h2, rsr.rsr_deserialize(old)):
        for batch in (1, 3, 40):
            _check(handle, M, batch, True, 1, 30 + batch)


@pytest.mark.parametrize("kind,rows,cols,k", [(rsr.RSR_BINARY, 1, 1, 1), (rsr.RSR_BINARY, 33, 257, 1), (rsr.RSR_BINARY, 100, 70, 15),
                                              (rsr.RSR_TERNARY_2PASS, 47, 1030, 5), (rsr.RSR_TERNARY_2PASS, 31, 9000, 12),
                                              (rsr.RSR_TERNARY_FUSED, 90, 600, 10), (rsr.RSR_TERNARY_FUSED, 35, 20000, 3),
                                              (rsr.RSR_TERNARY_2PASS, 18, 32766, 7)])
def test_codes_rebuilt_from_the_artifacts(kind, rows, cols, k):
    """Blocks that straddle row groups, several per group, one longer than all rows; one word per column
    from one column to the widest; sparse and crowded pattern spaces."""
    for M in (_matrix(kind, rows, cols, 31), np.zeros((rows, cols), np.int8)):
        h = rsr.rsr_deserialize(rsr.rsr_serialize(rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), k, kind)))
        _check(h, M, 600 if rows < 20 else 90, False, 0, 3, distinct=4)


def test_loading_needs_no_room_for_the_matrix():
    """A table of a GiB of entries is loaded with half a GiB to spare beyond the handle's own buffers
    (1.1 GiB)."""
    rows, cols = 1 << 22, 256
    M = torch.empty((rows, cols), dtype=torch.int8, device=DEV)
    for at in range(0, rows, 1 << 20):
        M[at:at + (1 << 20)] = torch.rand((1 << 20, cols), device=DEV) < 0.4
    h = rsr.rsr_preprocess(M, 8, rsr.RSR_BINARY)
    del M
    v = torch.randint(-8, 9, (20, cols), device=DEV).float()
    want = rsr.rsr_matvec_ex(h, v)
    blob = rsr.rsr_serialize(h)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    rsr.rsr_destroy(h)
    own = torch.cuda.mem_get_info()[0] - before
    assert own > 1 << 30
    hog = torch.empty(torch.cuda.mem_get_info()[0] - own - (1 << 29), dtype=torch.uint8, device=DEV)
    try:
        h = rsr.rsr_deserialize(blob)
    finally:
        del hog
        torch.cuda.empty_cache()
    assert torch.equal(rsr.rsr_matvec_ex(h, v), want)
    rsr.rsr_destroy(h)


@pytest.mark.parametrize("kind,rows,cols,k", [(rsr.RSR_BINARY, 50, 300, 6), (rsr.RSR_BINARY, 40, 90, 8),
                                              (rsr.RSR_TERNARY_2PASS, 45, 513, 7), (rsr.RSR_TERNARY_FUSED, 203, 700, 5)])
def test_artifacts_of_no_matrix_are_refused(kind, rows, cols, k):
    """A byte string whose permutation or boundaries are damaged: RSR_EINVAL, not a handle whose single
    vectors and batches are products of different matrices."""
    M = _matrix(kind, rows, cols, 12)
    blob = rsr.rsr_serialize(rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), k, kind))
    nb, P = -(-rows // k), (3 if kind == rsr.RSR_TERNARY_FUSED else 2) ** k
    pi_at, off_at = 128, 128 + 2 * nb * cols

    def damaged(change):
        bad = blob.copy()
        change(bad[pi_at:off_at].view(np.uint16).reshape(nb, cols),
               bad[off_at:off_at + 4 * nb * (P + 1)].view(np.uint32).reshape(nb, P + 1))
        assert not np.array_equal(bad, blob)
        with pytest.raises(rsr.RsrError) as e:
            rsr.rsr_deserialize(bad)
        assert e.value.code == 1

    def twice(pi, off): pi[nb - 1, cols // 2] = pi[nb - 1, cols // 2 - 1]
    def too_wide(pi, off): pi[nb // 2, 3] = cols
    def far_too_wide(pi, off): pi[nb // 2, 3] = 65535
    def first_boundary(pi, off): off[0, 0] = 1
    def last_boundary(pi, off): off[nb - 1, P] = cols - 1
    def falling(pi, off): off[nb // 2, P // 2] = off[nb // 2, P // 2 + 1] + 1
    def beyond(pi, off): off[1, P // 2:P] = 0xfffffff0
    def absent_rows(pi, off): off[nb - 1, :P] = 0       # every column has the last code: all digits set
    changes = [twice, too_wide, far_too_wide, first_boundary, last_boundary, falling, beyond]
    if rows % k:
        changes.append(absent_rows)
    for change in changes:
        damaged(change)
    if kind == rsr.RSR_TERNARY_2PASS:                   # M+ as M- too: entries in both
        bad = blob.copy()
        h = rsr.rsr_deserialize(blob)
        one = [np.concatenate([rsr.rsr_get_perm(h, p).astype(np.uint16).view(np.uint8).ravel(),
                               rsr.rsr_get_offsets(h, p).view(np.uint8).ravel()]) for p in (0, 1)]
        at = blob.tobytes().index(one[1].tobytes())
        bad[at:at + one[0].size] = one[0]
        with pytest.raises(rsr.RsrError) as e:
            rsr.rsr_deserialize(bad)
        assert e.value.code == 1
    _check(rsr.rsr_deserialize(blob), M, 90, True, 0, 7, distinct=4)


# few rows: every vector has workgroups of its own and the sums of a single product, bit for bit
@pytest.mark.parametrize("kind,rows,cols,k,batch,bf16,pad", [
    (rsr.RSR_TERNARY_FUSED, 64, 14336, 8, 32, False, 0), (rsr.RSR_TERNARY_FUSED, 64, 14336, 8, 30, False, 1),
    (rsr.RSR_BINARY, 200, 9000, 8, 8, False, 8), (rsr.RSR_TERNARY_2PASS, 99, 20000, 8, 20, True, 0),
    (rsr.RSR_TERNARY_2PASS, 99, 20000, 8, 20, True, 3), (rsr.RSR_TERNARY_FUSED, 40, 7001, 10, 18, False, 0),
    (rsr.RSR_BINARY, 10, 32766, 8, 300, False, 0), (rsr.RSR_BINARY, 300, 14336, 5, 2, False, 0),
    (rsr.RSR_BINARY, 512, 14336, 8, 2, True, 0), (rsr.RSR_BINARY, 512, 14336, 8, 4, True, 8),
    (rsr.RSR_BINARY, 8, 200, 8, 40, False, 1), (rsr.RSR_TERNARY_FUSED, 3, 17, 4, 17, False, 0)])
def test_batches_of_few_rows(kind, rows, cols, k, batch, bf16, pad):
    M = _matrix(kind, rows, cols, 1300 + cols)
    h = rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), k, kind)
    _check(h, M, batch, bf16, pad, cols, distinct=6)
    v = torch.zeros((batch, cols + pad), device=DEV)
    v[:, :cols] = torch.from_numpy(np.stack([gen.normal_f32(cols, seed=i) for i in range(batch)])).to(DEV)
    v = v.to(torch.bfloat16 if bf16 else torch.float32)[:, :cols]
    got = rsr.rsr_matvec_ex(h, v, scale=0.5)
    for i in range(batch):
        assert torch.equal(got[i], rsr.rsr_matvec_ex(h, v[i], scale=0.5)), i


def _from_codes(h):
    """The same handle with its single vectors multiplied from the packed codes, as k = 0 may choose
    by timing (the last field of the header of its bytes)."""
    blob = rsr.rsr_serialize(h)
    blob[120:128].view(np.int64)[0] = 1
    return rsr.rsr_deserialize(blob)


# one of the vectors has infinite or NaN elements: every kernel of the matrix cores
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("kind,rows,cols,batch", [
    (rsr.RSR_TERNARY_FUSED, 1200, 1500, 1), (rsr.RSR_BINARY, 170000, 30, 1), (rsr.RSR_TERNARY_2PASS, 500100, 9, 1),
    (rsr.RSR_TERNARY_FUSED, 3001, 700, 3), (rsr.RSR_TERNARY_2PASS, 1200, 300, 9), (rsr.RSR_BINARY, 601, 520, 20),
    (rsr.RSR_TERNARY_FUSED, 12790, 300, 180), (rsr.RSR_BINARY, 12800, 290, 290),
    (rsr.RSR_BINARY, 65540, 100, 3), (rsr.RSR_TERNARY_2PASS, 3000, 201, 11),
    (rsr.RSR_TERNARY_FUSED, 17000, 256, 25), (rsr.RSR_BINARY, 17001, 63, 60)])
def test_infinities_and_nan(kind, rows, cols, batch, bf16):
    """Rows with no entry in those columns keep their values, and so do the other vectors."""
    M = _matrix(kind, rows, cols, 17)
    h = rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), 2, kind)
    if batch == 1:
        h = _from_codes(h)
        assert "few" in rsr.rsr_kernel_name(h, int(bf16))
    v = np.stack([gen.integer_f32(cols, seed=40 + i) for i in range(min(batch, 5))])[np.arange(batch) % min(batch, 5)]
    want = np.stack([oracle.dense_matvec(M, x.astype(np.float64), 0.5) for x in v[:5]])[np.arange(batch) % min(batch, 5)]
    hit = batch // 2
    for columns in ({1: np.inf}, {0: -np.inf, cols - 1: np.inf}, {cols // 2: np.nan}):
        x = v.copy()
        x[hit, list(columns)] = 0.0
        y = want.copy()
        y[hit] = oracle.dense_matvec(M, x[hit].astype(np.float64), 0.5)
        for j, bad in columns.items():
            x[hit, j] = bad
            with np.errstate(invalid="ignore"):
                y[hit] = np.where(M[:, j] != 0, y[hit] + M[:, j] * np.float64(bad), y[hit])
        xd = torch.from_numpy(x).to(DEV).to(torch.bfloat16 if bf16 else torch.float32)
        got = rsr.rsr_matvec_ex(h, xd if batch > 1 else xd[0], scale=0.5).cpu().numpy().reshape(batch, rows)
        assert np.array_equal(got.astype(np.float64), y, equal_nan=True), columns
        assert np.isfinite(got[hit]).any() or not (M[:, list(columns)] == 0).all(axis=1).any()


@pytest.mark.parametrize("kind,rows,cols,k,batch", [
    (rsr.RSR_TERNARY_FUSED, 64, 14336, 8, 20),      # few rows: block patterns
    (rsr.RSR_TERNARY_FUSED, 5000, 700, 8, 4), (rsr.RSR_BINARY, 5000, 700, 8, 20),
    (rsr.RSR_BINARY, 17000, 100, 8, 60), (rsr.RSR_DENSE_TERNARY_P2, 25700, 300, 0, 300)])
def test_batches_in_a_graph(kind, rows, cols, k, batch):
    """Captured and replayed several times, with new vectors in the same buffer and other work between."""
    M = _matrix(kind, rows, cols, 3)
    h = rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), k, kind)
    v = torch.zeros((batch, cols), device=DEV)
    out = torch.zeros((batch, rows), device=DEV)
    rsr.rsr_matvec_ex(h, v, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rsr.rsr_matvec_ex(h, v, out=out)
    for i in range(4):
        v.copy_(torch.randint(-8, 9, (batch, cols), device=DEV))
        want = rsr.rsr_matvec_ex(h, v)
        out.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), i
    assert np.array_equal(want[1].cpu().numpy().astype(np.float64),
                          oracle.dense_matvec(M, v[1].cpu().numpy().astype(np.float64)))


# 5 to 16 vectors, two or four row groups of 16 per workgroup: both sides of every limit
@pytest.mark.parametrize("groups,tiles,batch,bf16,G", [
    (512, 13, 5, False, 2), (513, 13, 5, False, 4), (536, 12, 16, False, 2), (537, 12, 7, False, 4), (640, 11, 6, False, 2),
    (641, 11, 6, False, 4), (536, 13, 9, True, 2), (537, 13, 9, True, 4), (640, 12, 9, True, 2), (640, 13, 8, True, 2),
    (641, 20, 8, True, 4)])
def test_row_groups_of_a_workgroup(groups, tiles, batch, bf16, G):
    rows, cols = 16 * groups - 9, 256 * tiles - 3
    M = _matrix(rsr.RSR_BINARY, rows, cols, groups + tiles)
    h = rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), 8, rsr.RSR_BINARY)
    name = "k_packed_split<%s, 1, 1, %d, false>" % ("unsigned short" if bf16 else "float", G)
    assert rsr.rsr_batch_kernel_name(h, int(bf16), batch) == name
    _check(h, M, batch, bf16, 1, cols, distinct=4)


# two or four row groups per wave: both sides of every rule, a last workgroup with fewer groups, ragged rows and columns
@pytest.mark.parametrize("kind,rows,cols,batch,bf16,kernel", [
    (rsr.RSR_DENSE_TERNARY_P2, 256 * 16, 6200, 4, True, "few"), (rsr.RSR_DENSE_TERNARY_P2, 256 * 16 + 1, 6200, 4, True, "tall"),
    (rsr.RSR_BINARY, 256 * 16 + 17, 6145, 2, False, "tall"), (rsr.RSR_DENSE_TERNARY_P2, 512 * 16 + 35, 6401, 3, False, "tall"),
    (rsr.RSR_DENSE_TERNARY_P2, 256 * 16 + 40, 14336, 1, False, "tall"), (rsr.RSR_DENSE_TERNARY_P2, 512 * 16, 2049, 1, False, "few"),
    (rsr.RSR_DENSE_TERNARY_P2, 512 * 16 + 1, 2049, 1, False, "tall"), (rsr.RSR_TERNARY_FUSED, 513 * 16 + 3, 2300, 4, False, "tall"),
    (rsr.RSR_BINARY, 768 * 16 + 2, 3000, 3, True, "tall"), (rsr.RSR_DENSE_TERNARY_P2, 1024 * 16 + 1, 3400, 2, True, "few"),
    (rsr.RSR_DENSE_TERNARY_P2, 769 * 16 + 5, 1100, 1, False, "few"), (rsr.RSR_BINARY, 2050 * 16 + 9, 300, 2, False, "tall"),
    (rsr.RSR_DENSE_TERNARY_P2, 800 * 16 - 3, 511, 4, True, "tall"), (rsr.RSR_DENSE_TERNARY_P2, 60000, 2500, 1, True, "few"),
    (rsr.RSR_DENSE_TERNARY_P2, 1281 * 16 - 1, 1300, 1, False, "tall"), (rsr.RSR_DENSE_TERNARY_P2, 1536 * 16 + 1, 1100, 1, False, "few"),
    (rsr.RSR_DENSE_TERNARY_P2, 768 * 16 + 1, 1024, 1, False, "tall"), (rsr.RSR_DENSE_TERNARY_P2, 896 * 16, 1200, 2, False, "few"),
    (rsr.RSR_DENSE_TERNARY_P2, 896 * 16 + 1, 1200, 3, True, "tall"), (rsr.RSR_BINARY, 1536 * 16, 515, 4, True, "few"),
    (rsr.RSR_DENSE_TERNARY_P2, 1536 * 16 + 1, 700, 2, True, "tall"), (rsr.RSR_DENSE_TERNARY_P2, 768 * 16, 11500, 1, False, "few"),
    (rsr.RSR_DENSE_TERNARY_P2, 768 * 16 - 7, 11000, 1, False, "tall<float, 2, 1, 16, 2, 4>"),
    (rsr.RSR_DENSE_TERNARY_P2, 576 * 16, 4000, 3, False, "tall<float, 2, 4, 8, 2, 1>"),
    (rsr.RSR_DENSE_TERNARY_P2, 576 * 16 + 1, 4000, 2, False, "tall<float, 2, 4, 8, 4, 1>"),
    (rsr.RSR_DENSE_TERNARY_P2, 768 * 16, 2560, 4, False, "tall<float, 2, 4, 8, 2, 1>"),
    (rsr.RSR_BINARY, 768 * 16 + 1, 2560, 4, False, "tall<float, 1, 4, 8, 4, 1>"),
    (rsr.RSR_BINARY, 577 * 16, 4090, 2, False, "tall<float, 1, 4, 8, 4, 1>"),
    (rsr.RSR_BINARY, 700 * 16 - 5, 4461, 3, False, "tall<float, 1, 4, 8, 2, 1>"),
    (rsr.RSR_DENSE_TERNARY_P2, 1536 * 16 - 1, 1020, 1, False, "tall<float, 2, 1, 4, 2, 4>"),
    (rsr.RSR_DENSE_TERNARY_P2, 1536 * 16 + 1, 1020, 1, False, "few<float, 2, 1, 4>"),
    (rsr.RSR_DENSE_TERNARY_P2, 1857 * 16, 843, 1, False, "tall<float, 2, 1, 4, 2, 4>")])
def test_several_row_groups_per_wave(kind, rows, cols, batch, bf16, kernel):
    M = _matrix(kind, rows, cols, 77 + cols)
    h = rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), 4, kind)
    assert rsr.rsr_batch_kernel_name(h, int(bf16), batch).startswith("k_packed_" + kernel)
    _check(h, M, batch, bf16, 3, cols)
    v = torch.ones((batch, cols), device=DEV, dtype=torch.bfloat16 if bf16 else torch.float32)
    v[batch - 1, cols // 2] = float("inf")
    got = rsr.rsr_matvec_ex(h, v).cpu().numpy()
    want = np.repeat(M.sum(axis=1, dtype=np.float32)[None], batch, axis=0)
    hit = M[:, cols // 2] != 0
    want[-1, hit] = np.inf * M[hit, cols // 2]
    if kind == rsr.RSR_DENSE_TERNARY_P2:        # every entry is multiplied; the planes of an infinity are inf and NaN
        assert np.isnan(got[-1, ~hit]).all() and not np.isfinite(got[-1]).any()
        got, want = got[:-1], want[:-1]
    assert np.array_equal(got, want)


# sixteen waves, bf16: two row groups where the last round of 512 is more than half full; four tiles staged for 36 to 64
@pytest.mark.parametrize("groups,tiles,batch,kernel", [
    (256, 35, 2, "few<unsigned short, 2, 4, 16>"), (255, 36, 3, "tall<unsigned short, 2, 4, 16, 1, 4>"),
    (17, 64, 4, "tall<unsigned short, 2, 4, 16, 1, 4>"), (256, 65, 4, "few<unsigned short, 2, 4, 16>"),
    (257, 24, 4, "tall<unsigned short, 2, 4, 16, 2, 2>"), (512, 36, 4, "tall<unsigned short, 2, 4, 16, 2, 4>"),
    (513, 24, 4, "few<unsigned short, 2, 4, 16>"), (768, 36, 2, "few<unsigned short, 2, 4, 16>"),
    (769, 25, 3, "tall<unsigned short, 2, 4, 16, 2, 2>"), (1025, 24, 2, "few<unsigned short, 2, 4, 16>"),
    (1281, 24, 3, "tall<unsigned short, 2, 4, 16, 2, 2>"), (1281, 36, 2, "few<unsigned short, 2, 4, 16>")])
def test_sixteen_waves(groups, tiles, batch, kernel):
    rows, cols = 16 * groups - 5, 256 * tiles - 7
    M = _matrix(rsr.RSR_DENSE_TERNARY_P2, rows, cols, groups + tiles)
    h = rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), 0, rsr.RSR_DENSE_TERNARY_P2)
    assert rsr.rsr_batch_kernel_name(h, rsr.RSR_BF16, batch) == "k_packed_" + kernel
    _check(h, M, batch, True, 3, cols)


# one float32 vector and one-bit codes, eight waves: a CU holds three workgroups of one row group, or two of two
@pytest.mark.parametrize("groups,tiles,kernel", [
    (520, 8, "few"), (611, 10, "few"), (768, 23, "few"), (769, 8, "tall"), (1024, 12, "tall"), (1025, 8, "tall"), (1025, 9, "few"),
    (1280, 16, "few"), (1281, 16, "tall"), (1281, 15, "few"), (1536, 15, "few"), (1537, 10, "tall")])
def test_one_bit_codes_with_eight_waves(groups, tiles, kernel):
    rows, cols = 16 * groups - 3, 256 * tiles - 11
    M = _matrix(rsr.RSR_BINARY, rows, cols, groups + tiles)
    h = _from_codes(rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), 8, rsr.RSR_BINARY))
    assert rsr.rsr_kernel_name(h, rsr.RSR_F32).startswith("k_packed_%s<float, 1, 1, 8" % kernel)
    per = 2 if kernel == "tall" else 1
    workgroups, threads, lds = rsr.rsr_launch_shape(h, rsr.RSR_F32)
    assert (workgroups, threads) == ((groups + per - 1) // per, 512) and lds > 0
    _check(h, M, 1, False, 1, cols)


def test_stacked_layers_with_several_row_groups_per_wave():
    """Layers begin inside a workgroup's groups."""
    rows, cols = (3001, 17, 5000, 2003), 2500
    Ms = [_matrix(rsr.RSR_DENSE_TERNARY_P2, r, cols, 90 + r) for r in rows]
    h = rsr.rsr_preprocess_stacked([torch.from_numpy(M).to(DEV) for M in Ms], 0, rsr.RSR_DENSE_TERNARY_P2)
    v = gen.integer_f32(cols, seed=5)
    outs = rsr.rsr_matvec_stacked(h, torch.from_numpy(v).to(DEV), [1.0, -2.0, 0.5, 4.0])
    for M, out, scale in zip(Ms, outs, (1.0, -2.0, 0.5, 4.0)):
        assert np.array_equal(out.cpu().numpy().astype(np.float64), oracle.dense_matvec(M, v.astype(np.float64), scale))
