"""The matrix-core variant (half and int8 plans) against the CPU oracle: every tile shape at the
edges of its tiles, slabs and 16-byte chunks, small integers so that any order gives the same bits."""
import numpy as np
import pytest

from oracle import ref
from paper_2008_11849_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import check, run_spmm, run_spmm_strided  # noqa: E402
from paper_2008_11849_amd import sparsert as sp  # noqa: E402

# (rows, 16-column tiles) of every kernel
TILES = [(128, 8), (64, 8), (128, 4), (64, 4), (32, 4), (32, 2), (16, 4), (48, 4), (96, 8)]


def _opts(t):
    return dict(kernel=sp.KERNEL_SPEC, spec_mode=sp.SPEC_MFMA, spec_rows=t[0], spec_tiles=t[1])


def _ints(rng, M, K, density, dtype):
    mask = rng.random((M, K)) < density
    vals = (rng.integers(1, 4, size=(M, K)) * rng.choice([-1, 1], size=(M, K))).astype(dtype)
    return synth.csr_from_mask(vals, mask)


@pytest.mark.parametrize("dtype", [np.float16, np.int8])
@pytest.mark.parametrize("tile", TILES)
def test_spmm_at_the_edges_of_its_tiles(tile, dtype):
    rng = np.random.default_rng(7)
    for M, K, N in ((1, 1, 16), (130, 64, 17), (15, 127, 64), (97, 129, 129), (33, 700, 71), (200, 257, 200), (64, 32, 128)):
        csr = _ints(rng, M, K, 0.3 if K < 300 else 0.1, dtype)
        B = rng.integers(-4, 5, size=(K, N)).astype(dtype)
        want = ref.spmm(M, K, N, csr.row_ptr, csr.col_idx, csr.vals, B)[0]
        got, info = run_spmm(csr, B, **_opts(tile))
        assert info["spec_mode"] == sp.SPEC_MFMA and info["spec_rows"] == tile[0]
        assert np.array_equal(got.astype(np.float64), want), (M, K, N)
        got, pad_ok, _ = run_spmm_strided(csr, np.stack([B, -B]), N + 5, N + 3, **_opts(tile))
        assert pad_ok and np.array_equal(got.astype(np.float64), np.stack([want, -want])), (M, K, N)


@pytest.mark.parametrize("dtype", [np.float16, np.int8])
@pytest.mark.parametrize("tile", [(32, 2), (64, 4), (96, 8)])
def test_many_tiles_are_dealt_once_each(tile, dtype):
    """Tile counts that split unevenly over parts and XCDs; rows of C in whole 128-byte lines and not; every element is
    written (the result starts as NaN or a pattern) and by the right tile."""
    rng = np.random.default_rng(5)
    for M, K, N in ((tile[0] * 13 + 5, 40, 16 * tile[1] * 11 + 7), (tile[0] * 17, 300, 48), (70, 300, 16 * tile[1] * 17), (tile[0] * 9, 64, 16 * tile[1] * 8)):
        csr = _ints(rng, M, K, 0.2, dtype)
        B = rng.integers(-4, 5, size=(K, N)).astype(dtype)
        want = ref.spmm(M, K, N, csr.row_ptr, csr.col_idx, csr.vals, B)[0]
        for ldc in (N + 32, (N + 127) // 64 * 64):   # the second: a multiple of 128 bytes for either type, with a gap behind N
            got, pad_ok, _ = run_spmm_strided(csr, np.stack([B, -B]), N, ldc, **_opts(tile))
            assert pad_ok and np.array_equal(got.astype(np.float64), np.stack([want, -want])), (M, K, N, ldc)


@pytest.mark.parametrize("tile", [TILES[0], TILES[5]])
def test_half_values_subnormals_and_non_finite_operands(tile):
    case = synth.config("c2", np.float16)
    Cref, S = ref.spmm(512, 512, 196, case.csr.row_ptr, case.csr.col_idx, case.csr.vals, case.B)
    got, _ = run_spmm(case.csr, case.B, **_opts(tile))
    check(got, Cref, S, np.float16, gate_relative=True)
    rng = np.random.default_rng(9)
    csr = _ints(rng, 150, 300, 0.1, np.float16)
    B = rng.integers(-4, 5, size=(300, 200)).astype(np.float16) * np.float16(2.0 ** -24)      # subnormal operands and results
    want = ref.spmm(150, 300, 200, csr.row_ptr, csr.col_idx, csr.vals, B)[0]
    assert np.array_equal(run_spmm(csr, B, **_opts(tile))[0].astype(np.float64), want)
    # an infinity or NaN only reaches the rows that have a weight for it, zeros of A do not spread it
    B = rng.integers(-4, 5, size=(300, 200)).astype(np.float16)
    B[7, 3], B[7, 199], B[120, 64], B[299, 130] = np.inf, -np.inf, np.nan, np.inf
    base, _ = run_spmm(csr, B, kernel=sp.KERNEL_ROWS)
    got, _ = run_spmm(csr, B, **_opts(tile))
    assert np.isnan(base).any() and np.isfinite(base[:, 3]).any()
    assert np.array_equal(got, base, equal_nan=True)


@pytest.mark.parametrize("tile", TILES)
def test_a_non_finite_operand_changes_its_own_columns_only(tile):
    """Every other column keeps its bits, also where two waves store it (the last 16-byte chunk of a row overlaps the
    one before if N is no multiple of 8), and a column's value does not depend on how many others are redone."""
    rng = np.random.default_rng(11)
    M, K = 150, 701
    vals = rng.standard_normal((M, K)).astype(np.float16)
    mask = rng.random((M, K)) < 0.25
    csr = synth.csr_from_mask(vals, mask)
    for N in (201, 131, 21):
        B = rng.standard_normal((K, N)).astype(np.float16)
        clean, _ = run_spmm(csr, B, **_opts(tile))
        rows, _ = run_spmm(csr, B, kernel=sp.KERNEL_ROWS, split_threshold=1 << 30)   # sums in the order of the nonzeros
        for columns in ((N - 9,), (N - 1,), (0, 5, N - 8, N - 3), tuple(range(0, N, 2)), tuple(range(N))):
            X = B.copy()
            X[3, list(columns)] = np.inf
            got, _ = run_spmm(csr, X, **_opts(tile))
            others = np.setdiff1d(np.arange(N), columns)
            assert np.array_equal(got[:, others].view(np.uint16), clean[:, others].view(np.uint16)), (N, columns[:4])
            want = np.where(mask[:, 3:4], np.copysign(np.float16(np.inf), vals[:, 3:4]), rows[:, list(columns)])
            assert np.array_equal(got[:, list(columns)], want), (N, columns[:4])


def test_plan_round_trip_and_refusals():
    csr = synth.int8_csr(70, 200, 0.8, 3)
    B = synth.int8_dense(200, 100, 4)
    want = ref.spmm(70, 200, 100, csr.row_ptr, csr.col_idx, csr.vals, B)[0]
    plan = sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, 70, 200, 100, **_opts(TILES[4]))
    again = sp.load(plan.save())
    Bd = torch.from_numpy(B).cuda()
    for p in (plan, again):
        C = torch.zeros(70, 100, dtype=torch.int32, device="cuda")
        sp.spmm(p, Bd.data_ptr(), C.data_ptr(), torch.cuda.current_stream().cuda_stream)
        assert np.array_equal(C.cpu().numpy().astype(np.float64), want)
    for N, kw in ((100, dict(spec_rows=24)), (15, dict())):   # no such tile; fewer columns than a chunk
        with pytest.raises(sp.SparseRTError):
            sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, 70, 200, N, host_only=True, kernel=sp.KERNEL_SPEC, spec_mode=sp.SPEC_MFMA, **kw)
