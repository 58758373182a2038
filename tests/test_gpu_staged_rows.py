"""The row-walk kernel that stages B through LDS against the CPU oracle: small integers, so that any order
gives the same bits; column tiles with idle lanes and a ragged last one, chunks with a remainder, row groups
with empty slots, empty and full rows, batches and row pitches."""
import numpy as np
import pytest

from oracle import ref
from paper_2008_11849_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import run_spmm, run_spmm_strided  # noqa: E402
from paper_2008_11849_amd import sparsert as sp  # noqa: E402

# M, K, N, density, batch, row pitches beyond N; which kernels (V, rows per wave) of fp32, half and int8 it is
CASES = [
    (2049, 200, 196, 0.3, 4, 0, "44", True, False),
    (2100, 333, 516, 0.2, 1, 0, "24", True, True),
    (2100, 130, 1030, 0.2, 1, 0, "44", True, False),
    (1030, 300, 2052, 0.15, 1, 4, "28", True, True),
    (4000, 90, 2000, 0.1, 1, 0, "44", True, True),
    (4096, 1500, 788, 0.1, 1, 0, "44", True, True),
    (2000, 1000, 500, 0.3, 4, 0, "44", True, False),
    (1500, 200, 516, 0.3, 3, 4, "44", True, True),     # batches with a row pitch, of every type
    (1030, 300, 772, 0.3, 3, 8, "44", True, True),
]


@pytest.mark.parametrize("dtype", [np.float32, np.float16, np.int8])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:3])))
def test_spmm_against_the_oracle(case, dtype):
    M, K, N, density, batch, pad, shape, half, int8 = case
    rng = np.random.default_rng(M + N)
    mask = rng.random((M, K)) < density
    mask[5:40] = False
    mask[41] = True
    vals = (rng.integers(1, 3, size=(M, K)) * rng.choice([-1, 1], size=(M, K))).astype(dtype)
    csr = synth.csr_from_mask(vals, mask)
    opts = dict(kernel=sp.KERNEL_ROWS)
    B = rng.integers(-2, 3, size=(batch, K, N)).astype(dtype)
    plan = sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, M, K, N, batch=batch, ldb=N + pad, ldc=N + pad, host_only=True, **opts)
    staged = "staged_rows_kernel" in plan.kernel_name()
    assert staged == (True if dtype == np.float32 else half if dtype == np.float16 else int8)
    if dtype == np.float32:
        assert "<float, %s, %s>" % tuple(shape) in plan.kernel_name()
    want = np.stack([ref.spmm(M, K, N, csr.row_ptr, csr.col_idx, csr.vals, b)[0] for b in B])
    got, pad_ok, _ = run_spmm_strided(csr, B, N + pad, N + pad, **opts) if pad else (run_spmm(csr, B, **opts)[0], True, None)
    assert pad_ok and np.array_equal(got.astype(np.float64), want)


@pytest.mark.parametrize("dtype", [np.float32, np.float16, np.int8])
@pytest.mark.parametrize("M,K,N,lengths", [(4096, 600, 788, 22), (4096, 2400, 784, 8), (2049, 256, 784, 6)])
def test_shares_of_every_length(M, K, N, lengths, dtype):
    """Eights (fours, where shares are short) in a loop and four or two at the end: rows with 0 to lengths - 1 nonzeros in every
    50 columns; longer than a loop's step where they are not short."""
    rng = np.random.default_rng(K)
    mask = (np.arange(K)[None, :] % 50 * 7 + np.arange(M)[:, None]) % 50 < (np.arange(M) % lengths)[:, None]
    mask[-3:, :K - 1] |= lengths == 22
    vals = (rng.integers(1, 3, size=(M, K)) * rng.choice([-1, 1], size=(M, K))).astype(dtype)
    csr = synth.csr_from_mask(vals, mask)
    plan = sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, M, K, N, kernel=sp.KERNEL_ROWS, host_only=True)
    assert "staged_rows_kernel" in plan.kernel_name()
    assert ("StagedShortArgs" in plan.kernel_name()) == (dtype == np.float32 and lengths < 22)
    B = rng.integers(-1, 2, size=(K, N)).astype(dtype)
    want = ref.spmm(M, K, N, csr.row_ptr, csr.col_idx, csr.vals, B)[0]
    assert np.array_equal(run_spmm(csr, B, kernel=sp.KERNEL_ROWS)[0].astype(np.float64), want)


def test_non_finite_operands_stay_where_they_are():
    M, K, N = 2100, 333, 516
    rng = np.random.default_rng(3)
    mask = rng.random((M, K)) < 0.2
    csr = synth.csr_from_mask(rng.integers(1, 4, size=(M, K)).astype(np.float32), mask)
    B = rng.integers(-4, 5, size=(K, N)).astype(np.float32)
    places = ((7, 3), (332, 515), (0, 0), (103, 64))
    for k, n in places:
        B[k, n] = np.inf if k % 2 else np.nan
    got, _ = run_spmm(csr, B, kernel=sp.KERNEL_ROWS)
    for k, n in places:
        assert np.array_equal(~np.isfinite(got[:, n]), mask[:, k])
    assert (~np.isfinite(got)).sum() == mask[:, [k for k, _ in places]].sum()


@pytest.mark.parametrize("dtype", [np.float16, np.int8])
def test_rows_that_do_not_end_on_four_bytes_stay_on_the_plain_kernel(dtype):
    rng = np.random.default_rng(4)
    M, K, N = 2100, 333, 517
    csr = synth.csr_from_mask(np.ones((M, K), dtype=dtype), rng.random((M, K)) < 0.3)
    plan = sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, M, K, N, kernel=sp.KERNEL_ROWS, host_only=True)
    assert "staged" not in plan.kernel_name()
    B = rng.integers(-2, 3, size=(K, N)).astype(dtype)
    want = ref.spmm(M, K, N, csr.row_ptr, csr.col_idx, csr.vals, B)[0]
    assert np.array_equal(run_spmm(csr, B, kernel=sp.KERNEL_ROWS)[0].astype(np.float64), want)


def test_the_tuner_times_the_staged_kernel_beside_the_plain_one():
    M, K, N = 2048, 256, 256
    rng = np.random.default_rng(6)
    csr = synth.csr_from_mask(np.ones((M, K), dtype=np.float32), rng.random((M, K)) < 0.5)
    B = torch.from_numpy(rng.integers(-2, 3, size=(K, N)).astype(np.float32)).cuda()
    C = torch.empty(M, N, device="cuda")
    plan, entries = sp.tune(csr.row_ptr, csr.col_idx, csr.vals, M, K, N, B.data_ptr(), C.data_ptr(),
                            torch.cuda.current_stream().cuda_stream, kernel=sp.KERNEL_ROWS)
    assert all(e["agrees"] == 1 for e in entries)
    assert sorted({e["vec"] for e in entries}) == [0, 1, 2, 4] and sum(e["vec"] == 0 for e in entries) == 1
    for e in entries:   # the fields of an entry make its plan again
        again = sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, M, K, N, kernel=sp.KERNEL_ROWS, vec=e["vec"], split_threshold=e["split_threshold"], host_only=True)
        assert ("staged_rows_kernel" in again.kernel_name()) == (e["vec"] == 0)
