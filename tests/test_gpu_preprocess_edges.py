"""Preprocessing at the edges of its kernels: columns around a wave, a workgroup and the widest
matrix that is sorted as (code, column) pairs; block heights around the sorting steps of five bits;
groups around the length that the whole workgroup copies.  The artifacts must be the oracle's bit
for bit, and an integer-valued vector must come out exact."""
import numpy as np
import pytest

import oracle
import rsr_inputs as gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
rsr = pytest.importorskip("paper_2603_27462_amd")
DEV = "cuda:0"
KINDS = {rsr.RSR_BINARY: oracle.BINARY, rsr.RSR_TERNARY_2PASS: oracle.TERNARY_2PASS,
         rsr.RSR_TERNARY_FUSED: oracle.TERNARY_FUSED}


def _check(M, k, kind):
    h = rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), k, kind)
    for n, p in enumerate(oracle.preprocess(M, k, KINDS[kind]).passes):
        assert np.array_equal(rsr.rsr_get_perm(h, n), p.pi)
        assert np.array_equal(rsr.rsr_get_offsets(h, n), p.off)
    vi = gen.integer_f32(M.shape[1], seed=3)
    got = rsr.rsr_matvec(h, torch.from_numpy(vi).to(DEV)).cpu().numpy()
    assert np.array_equal(got.astype(np.float64), oracle.dense_matvec(M, vi.astype(np.float64)))


@pytest.mark.parametrize("cols", [3, 63, 65, 257, 511, 513, 4097, 18432, 18433])
@pytest.mark.parametrize("kind,k", [(rsr.RSR_BINARY, 5), (rsr.RSR_TERNARY_FUSED, 7)])
def test_column_counts(kind, k, cols):
    M = gen.binary_matrix(2 * k + 1, cols, 0.4, cols) if kind == rsr.RSR_BINARY else \
        gen.ternary_matrix(2 * k + 1, cols, 0.4, cols)
    _check(M, k, kind)


# workgroups of 512 and of 1024 threads: by the columns, and by the number of blocks
@pytest.mark.parametrize("rows,cols", [(512, 2561), (513, 2561), (512, 2560), (513, 10240), (513, 10241), (515, 18432)])
def test_blocks_that_have_a_cu_to_themselves(rows, cols):
    _check(gen.ternary_matrix(rows, cols, 0.4, rows + cols), 2, rsr.RSR_TERNARY_FUSED)


@pytest.mark.parametrize("kind,k", [(rsr.RSR_BINARY, 1), (rsr.RSR_BINARY, 6), (rsr.RSR_BINARY, 11),
                                    (rsr.RSR_TERNARY_2PASS, 10), (rsr.RSR_TERNARY_FUSED, 1),
                                    (rsr.RSR_TERNARY_FUSED, 3), (rsr.RSR_TERNARY_FUSED, 4),
                                    (rsr.RSR_TERNARY_FUSED, 10)])
def test_block_heights(kind, k):
    M = gen.binary_matrix(3 * k, 1000, 0.5, k) if kind == rsr.RSR_BINARY else gen.ternary_matrix(3 * k, 1000, 0.4, k)
    _check(M, k, kind)


@pytest.mark.parametrize("length", [63, 64, 65, 700])
def test_long_groups(length):
    """Every pattern group of a block has about `length` columns."""
    for kind, k in ((rsr.RSR_BINARY, 4), (rsr.RSR_TERNARY_FUSED, 8)):
        base = gen.binary_matrix(k, 9, 0.5, 5) if kind == rsr.RSR_BINARY else gen.ternary_matrix(k, 9, 0.3, 5)
        M = np.ascontiguousarray(np.repeat(base, length, axis=1)[:, np.random.default_rng(1).permutation(9 * length)])
        _check(M, k, kind)


@pytest.mark.parametrize("cols", [64, 129, 4100, 18433])
@pytest.mark.parametrize("patterns", [1, 2, 5])
def test_positions_of_a_wave_that_share_a_digit(patterns, cols):
    """Few distinct columns: in every sorting step a wave takes many positions of one digit one 64
    after the other, each 64 counting on from where the last ones ended."""
    k = 7
    base = gen.ternary_matrix(k, patterns, 0.3, patterns)
    M = np.ascontiguousarray(base[:, np.random.default_rng(cols).integers(0, patterns, cols)])
    _check(M, k, rsr.RSR_TERNARY_FUSED)


def test_more_blocks_than_one_launch_holds():
    """8388700 blocks of one row: 512 threads each are more than the 2^32 a launch can have.  (Stacked,
    because a matrix of four columns alone takes the narrow layout.)"""
    rows = (1 << 32) // 512 + 92
    M = (torch.rand((rows, 4), device=DEV) < 0.5).to(torch.int8)
    v = torch.tensor([1.0, 2.0, 4.0, 8.0], device=DEV)
    h = rsr.rsr_preprocess_stacked([M], 1, rsr.RSR_BINARY)
    out, = rsr.rsr_matvec_stacked(h, v)
    assert torch.equal(out, M.float() @ v)
    rsr.rsr_destroy(h)


@pytest.mark.parametrize("cols", [7, 66, 4097, 18435])
def test_empty_groups_in_a_row(cols):
    """Codes 8, 9 and 10 apart, and far apart: up to eight boundaries are one thread's, more the wave's."""
    k = 12
    codes = np.array([0, 8, 17, 27, 28, 29, 500, 509, 4000, 4094])[np.random.default_rng(cols).integers(0, 10, cols)]
    M = ((codes[None, :] >> np.arange(k)[:, None]) & 1).astype(np.int8)
    _check(M, k, rsr.RSR_BINARY)
    _check(np.concatenate([M, np.zeros_like(M)])[:k + 1], k, rsr.RSR_BINARY)


# strips of 8 to 32 entries, alike or not over the waves of a block; 3 to 16 waves, odd numbers among them
@pytest.mark.parametrize("kind,k,cols", [
    (rsr.RSR_BINARY, 3, 700), (rsr.RSR_BINARY, 3, 1700), (rsr.RSR_TERNARY_FUSED, 5, 2300), (rsr.RSR_BINARY, 7, 4100),
    (rsr.RSR_BINARY, 9, 9000), (rsr.RSR_TERNARY_FUSED, 5, 9000), (rsr.RSR_TERNARY_FUSED, 7, 14336),
    (rsr.RSR_TERNARY_2PASS, 6, 20000), (rsr.RSR_TERNARY_2PASS, 8, 32766), (rsr.RSR_BINARY, 12, 32766)])
def test_strip_lengths(kind, k, cols):
    M = gen.binary_matrix(2 * k + 1, cols, 0.5, cols) if kind == rsr.RSR_BINARY else \
        gen.ternary_matrix(2 * k + 1, cols, 0.4, cols)
    _check(M, k, kind)
