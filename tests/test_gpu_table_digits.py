"""One vector on a table of up to 256 columns: the digits of the vector's elements, in one set or, where elements are
less than 2^-55 of the largest, in several.  Reference: the matrix product in float64.  Every row's error is bounded by
roundings of partial sums, none of them larger than twice the row's sum of |m| |v|: six of the digits' planes of a set, and
one per further set, of five at most."""
import numpy as np
import pytest

import rsr_inputs as gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
rsr = pytest.importorskip("paper_2603_27462_amd")
DEV = "cuda:0"
ROWS = 240003            # at least as many as the rule asks for, and no whole number of row groups


def _handle(kind, M):
    h = rsr.rsr_preprocess(torch.from_numpy(M).to(DEV), 6, kind)
    if kind != rsr.RSR_DENSE_TERNARY_P2:        # as k = 0 may choose by timing: the last field of the header
        blob = rsr.rsr_serialize(h)
        blob[120:128].view(np.int64)[0] = 1
        h = rsr.rsr_deserialize(blob)
    assert rsr.rsr_kernel_name(h, rsr.RSR_BF16).startswith("k_table_few")
    assert rsr.rsr_kernel_name(h, rsr.RSR_F32).startswith("k_table_few")
    return h


def _vectors(cols, rng):
    normal = rng.standard_normal(cols)
    # the largest at 2^20, the smallest at the last binade that fits, with all 24 bits used
    wide = (rng.integers(1 << 23, 1 << 24, cols) | 1) * 2.0 ** -23 * 2.0 ** rng.integers(20 - 55, 21, cols)
    wide[0], wide[-1] = 2.0 ** 20 * (2 - 2.0 ** -23), 2.0 ** -35 * (1 + 2.0 ** -23)
    below = np.zeros(cols)                      # an element at the end of the digits' range
    below[cols // 2] = 2.0 ** -36 * 1.5
    below[0] = 2.0 ** 20
    every = (rng.integers(1 << 23, 1 << 24, cols) | 1) * 2.0 ** -23 * 2.0 ** rng.integers(-126, 120, cols)
    top = normal * 2.0 ** 118                   # sums near the largest float32
    yield "normal", normal, 6
    yield "wide", wide * rng.choice([-1, 1], cols), 6
    yield "below", below, 10
    yield "every exponent", every * rng.choice([-1, 1], cols), 10
    yield "zero", np.zeros(cols), 0
    yield "subnormal", np.round(normal * 64) * 2.0 ** -149, 6
    yield "top", top, 6


@pytest.mark.parametrize("kind,cols", [(rsr.RSR_BINARY, 1), (rsr.RSR_BINARY, 129), (rsr.RSR_BINARY, 256),
                                       (rsr.RSR_TERNARY_FUSED, 31), (rsr.RSR_DENSE_TERNARY_P2, 255),
                                       (rsr.RSR_TERNARY_2PASS, 256)])
def test_one_vector(kind, cols):
    rng = np.random.default_rng(cols)
    M = gen.binary_matrix(ROWS, cols, 0.6, cols) if kind == rsr.RSR_BINARY else gen.ternary_matrix(ROWS, cols, 0.35, cols)
    h = _handle(kind, M)
    Md = torch.from_numpy(M).to(DEV).double()
    for name, x, roundings in _vectors(cols, rng):
        for dtype in (torch.float32, torch.bfloat16):
            if name == "subnormal" and dtype == torch.bfloat16:
                continue                        # (a bf16 has no bits there)
            v = torch.from_numpy(x).to(DEV).to(dtype)
            got = rsr.rsr_matvec_ex(h, v, scale=0.5).double()
            want = 0.5 * (Md @ v.double())
            bound = 0.5 * 2 * roundings * 2.0 ** -24 * (Md.abs() @ v.double().abs()) + 2.0 ** -149
            assert bool(((got - want).abs() <= bound).all()), (name, dtype)


@pytest.mark.parametrize("kind", [rsr.RSR_BINARY, rsr.RSR_DENSE_TERNARY_P2])
@pytest.mark.parametrize("top", [20, 126])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_elements_below_the_digits_of_the_largest(kind, top, dtype):
    """Rows that take one small element and not the largest give that element, every bit of it."""
    cols = 40
    M = gen.binary_matrix(ROWS, cols, 0.2, 5) if kind == rsr.RSR_BINARY else gen.ternary_matrix(ROWS, cols, 0.8, 5)
    h = _handle(kind, M)
    last = 2.0 ** (-23 if dtype == torch.float32 else -7)
    x = np.zeros(cols)
    x[7] = 2.0 ** top
    # the last digit of the largest is 2^(top - 78), and elements from 2^(top - 55) on have all their bits above it
    small = {3: top - 55, 0: top - 56, 11: top - 79, 25: top - 110, 38: top - 112, 39: max(top - 245, -125)}
    for col, e in small.items():
        x[col] = 2.0 ** e * (1 + last)
    v = torch.from_numpy(x).to(DEV).to(dtype)
    assert np.array_equal(v.double().cpu().numpy(), x)
    got = rsr.rsr_matvec_ex(h, v).double().cpu().numpy()
    used = np.array([7] + list(small))
    single = (M[:, used] != 0).sum(axis=1) == 1
    for col in small:
        rows = single & (M[:, col] != 0)
        assert rows.sum() > 100 and np.array_equal(got[rows], M[rows, col] * x[col]), col


@pytest.mark.parametrize("kind", [rsr.RSR_BINARY, rsr.RSR_TERNARY_FUSED, rsr.RSR_DENSE_TERNARY_P2])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_elements_that_are_not_finite(kind, bad):
    cols = 200
    M = gen.binary_matrix(ROWS, cols, 0.6, 3) if kind == rsr.RSR_BINARY else gen.ternary_matrix(ROWS, cols, 0.35, 3)
    h = _handle(kind, M)
    x = gen.integer_f32(cols)
    x[77] = bad
    got = rsr.rsr_matvec_ex(h, torch.from_numpy(x).to(DEV)).cpu().numpy()
    hit = M[:, 77] != 0
    if kind == rsr.RSR_DENSE_TERNARY_P2:
        assert np.isnan(got[~hit]).all()
    else:
        x[77] = 0
        assert np.array_equal(got[~hit], (M.astype(np.float32) @ x)[~hit])
    assert not np.isfinite(got[hit]).any()


def test_stacked_layers():
    rows, cols = (120001, 17, 150002), 250
    Ms = [gen.ternary_matrix(r, cols, 0.35, r) for r in rows]
    h = rsr.rsr_preprocess_stacked([torch.from_numpy(M).to(DEV) for M in Ms], 0, rsr.RSR_DENSE_TERNARY_P2)
    x = gen.integer_f32(cols)
    for dtype in (torch.float32, torch.bfloat16):
        outs = rsr.rsr_matvec_stacked(h, torch.from_numpy(x).to(DEV).to(dtype), [1.0, -2.0, 4.0])
        for M, s, out in zip(Ms, (1.0, -2.0, 4.0), outs):
            assert np.array_equal(out.cpu().numpy(), s * (M.astype(np.float32) @ x))
