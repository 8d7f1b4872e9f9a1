"""Every kernel that multiplies from packed codes, by name: the case says which instantiation it is meant
to run and the library says which one it takes, so that a change of a rule cannot empty a case.

float32 vectors are split into three bf16 planes of 8 bits.  Their elements here are odd integers of up to
20 bits in 16 columns and zeros elsewhere: all three planes carry bits, and as no sum reaches 2^24, of
whatever part of the columns or planes, every result is exact in any order.  bf16 vectors are
integers of magnitude 8.  Reference: the oracle's dense definition."""
import numpy as np
import pytest

import oracle
import rsr_inputs as gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
rsr = pytest.importorskip("paper_2603_27462_amd")
DEV = "cuda:0"
DENSE, BINARY, FUSED = rsr.RSR_DENSE_TERNARY_P2, rsr.RSR_BINARY, rsr.RSR_TERNARY_FUSED


def _planes_vector(cols, seed):
    rng = np.random.default_rng(seed)
    x = np.zeros(cols, np.float32)
    at = rng.choice(cols, min(cols, 16), replace=False)
    x[at] = (2 * rng.integers(1 << 17, 1 << 18, at.size) + 1) * rng.choice([-1, 1], at.size)
    return x


def _without_last_plane(x):
    """x without the bits below its 16 most significant ones."""
    top = (x.view(np.uint32) & 0xffff0000).view(np.float32)
    middle = ((x - top).view(np.uint32) & 0xffff0000).view(np.float32)
    return top + middle


CASES = [
    # few: 1, 2, 4, 8 or 16 waves on the columns
    (DENSE, 1040, 200, 1, "k_packed_few<%s, 2, 1, 1>"), (BINARY, 500, 500, 1, "k_packed_few<%s, 1, 1, 2>"),
    (BINARY, 500, 1500, 1, "k_packed_few<%s, 1, 1, 4>"), (DENSE, 1041, 3000, 1, "k_packed_few<%s, 2, 1, 8>"),
    (FUSED, 333, 9001, 1, "k_packed_few<%s, 2, 1, 16>"), (BINARY, 4099, 700, 3, "k_packed_few<%s, 1, 4, 2>"),
    (FUSED, 3001, 1100, 4, "k_packed_few<%s, 2, 4, 4>"), (DENSE, 77, 6500, 2, "k_packed_few<%s, 2, 4, 16>"),
    # split: 16 or 32 vectors, one to four row groups, waves on columns or on rows
    (DENSE, 1003, 2100, 9, "k_packed_split<%s, 2, 1, 1, false>"), (DENSE, 6001, 2100, 9, "k_packed_split<%s, 2, 1, 2, false>"),
    (DENSE, 14330, 2100, 16, "k_packed_split<%s, 2, 1, 4, false>"), (BINARY, 14001, 2300, 13, "k_packed_split<%s, 1, 1, 4, false>"),
    (DENSE, 1003, 2100, 30, "k_packed_split<%s, 2, 2, 2, false>"), (DENSE, 14330, 2100, 30, "k_packed_split<%s, 2, 2, 4, false>"),
    (DENSE, 60001, 300, 10, "k_packed_split<%s, 2, 1, 4, true>"),
    # tables: up to 256 columns
    (DENSE, 500100, 250, 1, "k_table_few<%s, 2, 1>"), (BINARY, 500001, 256, 1, "k_table_few<%s, 1, 1>"),
    (DENSE, 65601, 200, 3, "k_table_few<%s, 2, 4>"), (BINARY, 70001, 256, 4, "k_table_few<%s, 1, 4>"),
    (DENSE, 2003, 222, 11, "k_table_few<%s, 2, 16>"), (BINARY, 3005, 256, 16, "k_table_few<%s, 1, 16>"),
    (DENSE, 17001, 256, 25, "k_table_many<%s, 2, 1>"), (BINARY, 17003, 251, 32, "k_table_many<%s, 1, 1>"),
    (DENSE, 17005, 199, 60, "k_table_many<%s, 2, 2>"), (BINARY, 17007, 256, 100, "k_table_many<%s, 1, 2>"),
]
BY_TYPE = [
    (BINARY, 40000, 513, 24, True, "k_packed_split<float, 1, 2, 4, true>"),
    (BINARY, 40000, 513, 24, False, "k_packed_split<unsigned short, 1, 2, 2, true>"),
    # tiles of 128 rows and vectors: eight waves up to 256 workgroups, four beyond; rows and vectors ragged
    (DENSE, 12797, 601, 250, True, "k_packed_tile<float, 2, 2, 2>"), (BINARY, 12798, 777, 249, True, "k_packed_tile<float, 1, 2, 2>"),
    (DENSE, 25597, 513, 251, True, "k_packed_tile<float, 2, 1, 2>"), (BINARY, 25590, 290, 250, True, "k_packed_tile<float, 1, 1, 2>"),
    (FUSED, 9001, 1030, 250, False, "k_packed_tile<unsigned short, 2, 2, 1>"),
    (BINARY, 9003, 1029, 255, False, "k_packed_tile<unsigned short, 1, 2, 1>"),
    (FUSED, 25599, 300, 253, False, "k_packed_tile<unsigned short, 2, 1, 2>"),
    (BINARY, 25593, 517, 250, False, "k_packed_tile<unsigned short, 1, 1, 2>"),
]


@pytest.mark.parametrize("kind,rows,cols,batch,wide,kernel", [
    (kind, rows, cols, batch, wide, name % ("float" if wide else "unsigned short"))
    for kind, rows, cols, batch, name in CASES for wide in (True, False)] + BY_TYPE)
def test_exact_with_all_planes(kind, rows, cols, batch, wide, kernel):
    M = gen.binary_matrix(rows, cols, 0.6, rows) if kind == BINARY else gen.ternary_matrix(rows, cols, 0.35, rows)
    h = rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), 2, kind)
    if batch == 1 and kind != DENSE:        # as k = 0 may choose by timing: the last field of the header
        blob = rsr.rsr_serialize(h)
        blob[120:128].view(np.int64)[0] = 1
        h = rsr.rsr_deserialize(blob)
    assert rsr.rsr_batch_kernel_name(h, rsr.RSR_F32 if wide else rsr.RSR_BF16, batch) == kernel
    distinct = min(batch, 6)
    x = np.stack([_planes_vector(cols, 50 + i) if wide else gen.integer_f32(cols, seed=50 + i) for i in range(distinct)])
    want = np.stack([oracle.dense_matvec(M, r.astype(np.float64)) for r in x])
    if wide:
        assert not np.array_equal(oracle.dense_matvec(M, _without_last_plane(x[0]).astype(np.float64)), want[0])
    order = np.random.default_rng(1).permutation(np.arange(batch) % distinct)
    v = torch.from_numpy(x[order]).to(DEV).to(torch.float32 if wide else torch.bfloat16)
    got = rsr.rsr_matvec_ex(h, v if batch > 1 else v[0]).cpu().numpy().reshape(batch, rows)
    assert np.array_equal(got.astype(np.float64), want[order])


def test_every_kernel_family_is_a_case():
    names = {c[-1].split("<")[0] for c in CASES + BY_TYPE}
    assert names == {"k_packed_few", "k_packed_split", "k_packed_tile", "k_table_few", "k_table_many"}
