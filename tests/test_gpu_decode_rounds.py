"""GPU parity of the 3-to-16-token decode kernel where a workgroup's tiles are
summed in rounds (their partials do not all fit in LDS), and where K is split
over workgroups with each segment's x in registers."""

import numpy as np
import pytest

import pq_inputs as pi
from oracle import pq_oracle as orc
from gpu_util import assert_close, sample_rows, to_dev, to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
fasq = pytest.importorskip("paper_2605_04084_amd")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fasq.lib()
    yield
    torch.cuda.synchronize()


def exact_problem(rng, M, K, N, d, C, bits):
    """Signed one-hot codewords and ternary activations: exact in any order."""
    cb = pi.signed_one_hot_codebook(C, d, rng)
    ids = rng.integers(0, C, size=(N, K // d))
    return pi.ternary_x(rng, M, K), pi.pack_indices(ids, bits), cb


ROUNDS = [
    # M, K, N, d, C, bits: more tiles per workgroup than partials fit
    (16, 4096, 20481, 2, 256, 8),      # six tiles, the last one of a single row
    (16, 2048, 50000, 4, 256, 8),      # two row groups per workgroup
    (13, 4096, 50000, 4, 4096, 12),
    (16, 4096, 70000, 2, 256, 8),      # more than two rounds
]


@pytest.mark.parametrize("case", ROUNDS)
def test_rounds_of_tiles(case):
    M, K, N, d, C, bits = case
    print(f"[case] decode rounds {case}", flush=True)
    assert fasq.plan("gemv", M, K, N, bits, d, C).endswith(", 0, 0, 1>"), fasq.plan("gemv", M, K, N, bits, d, C)
    rng = np.random.default_rng(sum(case))
    x, idx, cb = exact_problem(rng, M, K, N, d, C, bits)
    y = to_np(fasq.pq_gemv(to_dev(x), to_dev(idx), bits, d, to_dev(cb))).astype(np.float64)
    assert np.isfinite(y).all()
    rows = np.unique(np.concatenate([sample_rows(N, 300), np.arange(N - 40, N)]))
    assert np.array_equal(y[:, rows], orc.pq_linear(x, idx, bits, d, cb, rows=rows))


def test_rounds_in_a_grouped_launch_give_the_bits_of_single_calls():
    rng = np.random.default_rng(21)
    M, K, d, C, bits = 16, 4096, 2, 256, 8
    x = pi.draw_x(rng, M, K)
    probs = [pi.draw_problem(rng, 1, K, N, d, C, bits) for N in (14336, 14300)]
    ys = fasq.pq_gemv_batched(to_dev(x), [to_dev(p.idx) for p in probs], bits, d, [to_dev(p.codebook) for p in probs])
    for p, y in zip(probs, ys):
        one = fasq.pq_gemv(to_dev(x), to_dev(p.idx), bits, d, to_dev(p.codebook))
        assert torch.equal(y.view(torch.int16), one.view(torch.int16))
        rows = sample_rows(p.N, 100)
        assert_close(to_np(y)[:, rows].astype(np.float64), orc.pq_linear(x, p.idx, bits, d, p.codebook, rows=rows), "group")


SEGMENTS = [
    # M, K, N, d, C, bits, segments
    (16, 14336, 4096, 2, 256, 8, 4),
    (12, 14336, 1030, 2, 256, 8, 4),
    (16, 9216, 3328, 2, 256, 8, 4),
    (5, 14336, 77, 4, 256, 8, 4),
    (12, 14336, 2000, 4, 4096, 12, 4),
    (9, 8192, 20000, 2, 256, 8, 2),     # rounds within the segments
]


@pytest.mark.parametrize("case", SEGMENTS)
def test_segments_with_x_in_registers(case):
    M, K, N, d, C, bits, nseg = case
    print(f"[case] decode segments {case}", flush=True)
    need = fasq.gemv_ex_workspace_bytes(M, K, N, bits, d, C, 0)
    assert need == nseg * M * N * 4
    rng = np.random.default_rng(sum(case))
    x, idx, cb = exact_problem(rng, M, K, N, d, C, bits)
    rows = sample_rows(N, 200)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda:0")  # NaN partials before the call
    y = to_np(fasq.pq_gemv_ex(to_dev(x), to_dev(idx), bits, d, to_dev(cb), workspace=ws)).astype(np.float64)
    assert np.isfinite(y).all()
    assert np.array_equal(y[:, rows], orc.pq_linear(x, idx, bits, d, cb, rows=rows))
    p = pi.draw_problem(rng, M, K, N, d, C, bits)
    y = to_np(fasq.pq_gemv_ex(to_dev(p.x), to_dev(p.idx), bits, d, to_dev(p.codebook), workspace=ws)).astype(np.float64)
    assert_close(y[:, rows], orc.pq_linear(p.x, p.idx, bits, d, p.codebook, rows=rows), str(case))


def test_a_workspace_too_small_for_the_segments_takes_the_gemm():
    """From 12 tokens on a workspace that holds the GEMM's K split but not the
    decode kernel's segments gives the GEMM's bits; one byte less than that
    gives the decode kernel's without a split; the full one its segments."""
    rng = np.random.default_rng(31)
    M, K, N, d, C, bits = 16, 14336, 5000, 2, 256, 8
    need, gemm_need = (f(M, K, N, bits, d, C, *a) for f, a in ((fasq.gemv_ex_workspace_bytes, (0,)),
                                                               (fasq.gemm_ex_workspace_bytes, ())))
    assert need == 4 * M * N * 4 and 0 < gemm_need < need
    p = pi.draw_problem(rng, M, K, N, d, C, bits)
    args = (to_dev(p.x), to_dev(p.idx), bits, d, to_dev(p.codebook))

    def call(nbytes):
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda:0")
        return fasq.pq_gemv_ex(*args, workspace=ws).view(torch.int16)

    rows = sample_rows(N, 200)
    ref = orc.pq_linear(p.x, p.idx, bits, d, p.codebook, rows=rows)
    for nbytes in (need, gemm_need, gemm_need - 1):
        assert_close(to_np(call(nbytes).view(torch.float16))[:, rows].astype(np.float64), ref, f"workspace {nbytes}")
    assert torch.equal(call(gemm_need), fasq.pq_gemm_ex(*args).view(torch.int16))
    assert torch.equal(call(gemm_need - 1), fasq.pq_gemv(*args).view(torch.int16))


SLABS = [
    # M, K, N, d, C, bits: one to several units per wave and slab, masked columns
    (5, 17216, 261, 4, 256, 8),
    (7, 10944, 4600, 4, 256, 8),
    (8, 14080, 33000, 4, 256, 8),
    (13, 19200, 1209, 8, 256, 8),
    (10, 11648, 20500, 8, 256, 8),
]


@pytest.mark.parametrize("case", SLABS)
def test_slabs_of_long_rows(case):
    M, K, N, d, C, bits = case
    print(f"[case] decode slabs {case}", flush=True)
    assert fasq.plan("gemv", M, K, N, bits, d, C).endswith(", 1, 1>"), fasq.plan("gemv", M, K, N, bits, d, C)
    rng = np.random.default_rng(sum(case))
    x, idx, cb = exact_problem(rng, M, K, N, d, C, bits)
    y = to_np(fasq.pq_gemv(to_dev(x), to_dev(idx), bits, d, to_dev(cb))).astype(np.float64)
    rows = np.unique(np.concatenate([sample_rows(N, 100), np.arange(N - 20, N)]))
    assert np.array_equal(y[:, rows], orc.pq_linear(x, idx, bits, d, cb, rows=rows))
