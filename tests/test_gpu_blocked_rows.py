"""The row-walk kernel that keeps a block of rows in registers, against the CPU oracle: small integers, so that any order gives
the same bits; column tiles with idle lanes and a ragged last one, blocks with empty slots, groups of columns that fillers
complete, parts with no group of columns, one and two, empty and long rows, the fewest rows and columns, batches and row pitches."""
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

ROWS = dict(kernel=sp.KERNEL_ROWS)


def _csr(M, K, density, seed, skewed):
    """Rows 5 to 39 empty, row 41 full; skewed: a tenth of the rows holds most of the nonzeros."""
    rng = np.random.default_rng(seed)
    p = np.full(M, density)
    if skewed:
        p[:] = density / 4
        p[rng.permutation(M)[:M // 10]] = min(1.0, density * 7.5)
    mask = rng.random((M, K)) < p[:, None]
    mask[5:40] = False
    mask[41] = True
    vals = (rng.integers(1, 3, size=(M, K)) * rng.choice([-1, 1], size=(M, K))).astype(np.float32)
    return synth.csr_from_mask(vals, mask)


# M, K, N, density, batch, row pitches beyond N, skewed; waves of a workgroup
CASES = [
    (1613, 951, 80, 0.06, 4, 0, True, 4),       # one tile, 40 of 64 lanes
    (153, 3470, 2328, 0.144, 1, 0, False, 4),   # few rows, a long K
    (448, 2212, 2617, 0.05, 1, 3, False, 4),    # an odd N, rows of B and C that begin anywhere
    (1344, 700, 925, 0.14, 4, 0, False, 4),     # full blocks, a ragged last tile
    (2664, 1500, 198, 0.076, 4, 5, False, 8),
    (2816, 630, 128, 0.16, 1, 0, True, 4),      # blocks of sixteen rows
    (186, 3320, 2062, 0.1, 4, 0, False, 8),
    (64, 1500, 2400, 0.12, 4, 0, False, 4),     # the fewest rows
    (3000, 3000, 49, 0.1, 4, 0, False, 8),      # the fewest columns
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:3])))
def test_spmm_against_the_oracle(case):
    M, K, N, density, batch, pad, skewed, waves = case
    csr = _csr(M, K, density, M + N, skewed)
    B = np.random.default_rng(N).integers(-2, 3, size=(batch, K, N)).astype(np.float32)
    plan = sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, M, K, N, batch=batch, ldb=N + pad, ldc=N + pad, host_only=True, **ROWS)
    assert plan.kernel_name() == f"void sparsert::blocked_rows_kernel<{waves}>(sparsert::BlockedArgs)"
    want = np.stack([ref.spmm(M, K, N, csr.row_ptr, csr.col_idx, csr.vals, b)[0] for b in B])
    got, pad_ok, _ = run_spmm_strided(csr, B, N + pad, N + pad, **ROWS) if pad else (run_spmm(csr, B, **ROWS)[0], True, None)
    assert pad_ok and np.array_equal(got.astype(np.float64), want)


@pytest.mark.parametrize("columns", [0, 1, 2, 40, 160])
def test_parts_with_few_groups_of_columns(columns):
    """Four waves share the columns that a block has nonzeros in, sixteen to a group: none, one or two of the waves have a column at all,
    each has one group, each has two."""
    M, K, N, batch = 300, 300, 640, 64
    rng = np.random.default_rng(columns)
    mask = np.zeros((M, K), dtype=bool)
    mask[:, np.linspace(1, K - 1, columns).astype(int)] = rng.random((M, columns)) < min(0.19, 1.75 / max(1, columns))
    csr = synth.csr_from_mask(rng.choice([-2.0, -1.0, 1.0, 2.0], size=(M, K)).astype(np.float32), mask)
    B = rng.integers(-2, 3, size=(batch, K, N)).astype(np.float32)
    plan = sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, M, K, N, batch=batch, host_only=True, **ROWS)
    assert plan.kernel_name() == "void sparsert::blocked_rows_kernel<4>(sparsert::BlockedArgs)"
    want = np.stack([ref.spmm(M, K, N, csr.row_ptr, csr.col_idx, csr.vals, b)[0] for b in B])
    assert np.array_equal(run_spmm(csr, B, **ROWS)[0].astype(np.float64), want)


def test_non_finite_operands_stay_where_they_are():
    """What only fills a layer up multiplies zero by an operand, into a sum that nobody reads."""
    M, K, N = 1344, 700, 925
    csr = _csr(M, K, 0.1, 3, True)
    rows = np.repeat(np.arange(M), np.diff(csr.row_ptr))
    mask = np.zeros((M, K), dtype=bool)
    mask[rows, csr.col_idx] = True
    B = np.random.default_rng(4).integers(-4, 5, size=(4, K, N)).astype(np.float32)
    places = ((7, 3), (332, 515), (0, 0), (699, 924), (103, 64))
    for k, n in places:
        B[:, k, n] = np.inf if k % 2 else np.nan
    assert "blocked" in sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, M, K, N, batch=4, host_only=True, **ROWS).kernel_name()
    got, _ = run_spmm(csr, B, **ROWS)
    for b in got:
        for k, n in places:
            assert np.array_equal(~np.isfinite(b[:, n]), mask[:, k])
        assert (~np.isfinite(b)).sum() == mask[:, [k for k, _ in places]].sum()


def test_saved_plans_and_graph_replays():
    M, K, N = 448, 2212, 2616
    csr = _csr(M, K, 0.05, 9, False)
    plan = sp.load(sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, M, K, N, **ROWS).save())
    assert plan.info()["blocked_rows"] > 0
    rng = np.random.default_rng(5)
    B = torch.empty(K, N, device="cuda")
    C = torch.empty(M, N, device="cuda")
    B.zero_()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        sp.spmm(plan, B.data_ptr(), C.data_ptr(), torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        b = rng.integers(-2, 3, size=(K, N)).astype(np.float32)
        B.copy_(torch.from_numpy(b))
        C.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().numpy().astype(np.float64), ref.spmm(M, K, N, csr.row_ptr, csr.col_idx, csr.vals, b)[0])
    plan.destroy()
