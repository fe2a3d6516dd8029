"""GPU parity of the prefill GEMM for codebooks gathered from global memory:
every tile, id width and sub-vector length, ragged M and N, fewer K chunks
than its pipeline holds, and the K split."""

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


CASES = [
    # M, K, N, d, C, bits, tile
    (17, 64, 8193, 4, 65536, 16, "64, 32"),       # one K chunk
    (64, 1024, 257, 4, 65536, 16, "64, 32"),
    (33, 2048, 100, 4, 20001, 16, "64, 32"),      # codebook of no whole 16-byte words
    (250, 192, 4096, 2, 40000, 16, "128, 32"),
    (511, 448, 4096, 4, 65536, 16, "256, 32"),    # the K = 7 chunks end inside the pipeline
    (500, 640, 4090, 8, 65536, 16, "256, 32"),
    (300, 128, 3000, 1, 65536, 16, "256, 32"),
    (1000, 128, 4000, 4, 65536, 16, "256, 64"),
    (1000, 128, 4000, 8, 9000, 16, "256, 64"),
    (900, 128, 4000, 1, 65536, 16, "256, 64"),
    (130, 256, 1030, 2, 250, 8, None),
    (600, 192, 3000, 1, 100, 8, None),
    (70, 128, 2000, 4, 1001, 12, None),           # odd id counts per thread: half-byte starts
    (600, 128, 4000, 4, 1001, 12, None),
    (40, 192, 900, 2, 1001, 12, None),
    (300, 64, 2000, 1, 1001, 12, None),
]


@pytest.mark.parametrize("case", CASES)
def test_gather_gemm(case):
    M, K, N, d, C, bits, tile = case
    print(f"[case] gather gemm {case}", flush=True)
    plan = fasq.plan("gemm", M, K, N, bits, d, C)
    assert plan.startswith(f"k_gemm_gather<{bits}, {d}, {tile or ''}"), plan
    rng = np.random.default_rng(sum(case[:6]))
    # signed one-hot codewords and ternary activations: exact in any order
    cb = pi.signed_one_hot_codebook(C, d, rng)
    ids = rng.integers(0, C, size=(N, K // d))
    x = pi.ternary_x(rng, M, K)
    idx = pi.pack_indices(ids, bits)
    xd, idd, cbd = to_dev(x), to_dev(idx), to_dev(cb)
    rows = sample_rows(N, 128)
    ref = orc.pq_linear(x, idx, bits, d, cb, rows=rows)
    for call in (fasq.pq_gemm, fasq.pq_gemm_ex):  # the second splits K where tiles leave CUs idle
        y = to_np(call(xd, idd, bits, d, cbd)).astype(np.float64)
        assert np.isfinite(y).all()
        assert np.array_equal(y[:, rows], ref)
    p = pi.draw_problem(rng, M, K, N, d, C, bits)
    y = to_np(fasq.pq_gemm_ex(to_dev(p.x), to_dev(p.idx), bits, d, to_dev(p.codebook))).astype(np.float64)
    assert_close(y[:, rows], orc.pq_linear(p.x, p.idx, bits, d, p.codebook, rows=rows), str(case))


def test_gather_gemm_splits_k_with_a_workspace():
    # 4096 x 4096 at 64 tokens: 128 tiles, two K ranges
    assert fasq.gemm_ex_workspace_bytes(64, 4096, 4096, 16, 4, 65536) == 2 * 64 * 4096 * 4
    assert fasq.gemv_ex_workspace_bytes(64, 4096, 4096, 16, 4, 65536, 0) == 2 * 64 * 4096 * 4
    assert fasq.gemm_ex_workspace_bytes(512, 4096, 4096, 16, 4, 65536) == 0
