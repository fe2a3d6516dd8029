"""GPU parity of the prefill GEMM for codebooks gathered from global memory:
every tile, id width and sub-vector length, ragged M and N, fewer K chunks
than its pipeline holds and several turns of it, and the K split."""

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
    (100, 1088, 70, 4, 65536, 16, "64, 32"),      # few ids
    (250, 192, 4096, 2, 40000, 16, "128, 32"),
    (511, 448, 4096, 4, 65536, 16, "256, 32"),    # the K = 7 chunks end inside the pipeline
    (500, 640, 4090, 8, 65536, 16, "256, 32"),
    (300, 128, 3000, 1, 65536, 16, "256, 32"),
    (1000, 128, 4000, 4, 65536, 16, "256, 64"),
    (1000, 192, 4000, 8, 9000, 16, "256, 64"),
    (900, 128, 4000, 1, 65536, 16, "256, 64"),
    (1100, 256, 16500, 4, 65536, 16, "256, 64"),  # several rounds of workgroups
    (130, 256, 1030, 2, 250, 8, "64, 32"),
    (600, 192, 3000, 1, 100, 8, "256, 64"),
    (70, 256, 2000, 4, 1001, 12, "64, 32"),       # odd id counts per thread: half-byte starts
    (600, 320, 2000, 4, 1001, 12, "256, 32"),
    (40, 192, 900, 2, 1001, 12, "64, 32"),
    (300, 64, 2000, 1, 1001, 12, "128, 32"),
    # turns of the ring: chunk counts of several turns and a remainder, for every tile
    (64, 2112, 1000, 4, 65536, 16, "64, 32"),
    (256, 2112, 4096, 4, 65536, 16, "128, 32"),
    (512, 2240, 4096, 4, 65536, 16, "256, 32"),
    (1000, 2112, 4000, 4, 65536, 16, "256, 64"),
    (200, 2368, 1030, 4, 251, 8, "64, 32"),
    (300, 2112, 3000, 1, 251, 8, "256, 32"),
    (250, 2304, 4000, 4, 1001, 12, "128, 32"),    # whole turns
    (1000, 2176, 4000, 2, 4095, 12, "256, 64"),
]


@pytest.mark.parametrize("case", CASES)
def test_gather_gemm(case):
    M, K, N, d, C, bits, tile = case
    print(f"[case] gather gemm {case}", flush=True)
    plan = fasq.plan("gemm", M, K, N, bits, d, C)
    assert plan.startswith(f"k_gemm_gather<{bits}, {d}, {tile}"), plan
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


def test_which_calls_gather():
    """Codebooks in global memory take the gather kernel, small and large
    calls alike, except for cheap codewords (d = 8, or a book of the L1's size
    from d = 2 on) in the 256 x 256 tile, with few K values in small tiles, or with
    a few more where the gather tiles need another round of workgroups."""
    def gathers(*c):
        M, K, N, d, C, bits = c
        return fasq.plan("gemm", M, K, N, bits, d, C).startswith("k_gemm_gather<")
    for M in (2048, 2049):
        assert gathers(M, 4096, 4096, 4, 65536, 16) and gathers(M, 4096, 14336, 4, 65536, 16)
    assert gathers(40, 64, 30, 4, 65536, 16) and gathers(40, 64, 12000, 1, 251, 8)
    assert not gathers(40, 128, 900, 8, 9000, 16) and gathers(40, 192, 900, 8, 9000, 16)
    assert not gathers(145, 64, 500, 2, 4095, 12) and gathers(145, 64, 11847, 2, 4095, 12)
    assert not gathers(40, 128, 900, 4, 251, 8) and gathers(40, 192, 900, 4, 251, 8)
    assert not gathers(340, 256, 10761, 4, 251, 8) and gathers(340, 320, 10761, 4, 251, 8)
    assert not gathers(3148, 2432, 9324, 4, 251, 8)


def call_us(M, K, N, d, C, bits, calls=20):
    rng = np.random.default_rng(M + K)
    p = pi.draw_problem(rng, M, K, N, d, C, bits)
    args = (to_dev(p.x), to_dev(p.idx), bits, d, to_dev(p.codebook))
    y = fasq.pq_gemm(*args)
    best = float("inf")
    for _ in range(5):
        torch.cuda._sleep(2_000_000)  # the launches reach the GPU back to back
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(calls):
            fasq.pq_gemm(*args, out=y)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / calls)
    return best


@pytest.mark.parametrize("d,C,bits", [(1, 65536, 16), (2, 65536, 16), (1, 4095, 12)])
def test_few_chunks_gather_no_more_than_they_hold(d, C, bits):
    """One chunk of K reads about a ninth of nine chunks' codewords; the
    pipeline's prologue and its clamped steps must not read them all the same."""
    few, nine = (call_us(40, K, 12000, d, C, bits) for K in (64, 576))
    print(f"[time] d={d} C={C}: 1 chunk {few:.1f} us, 9 chunks {nine:.1f} us", flush=True)
    assert few <= 0.5 * nine


@pytest.mark.parametrize("M,K,N,d,C,bits", [(70, 704, 130, 4, 65536, 16), (300, 192, 3000, 1, 251, 8)])
def test_infinities_and_nan_reach_only_their_outputs(M, K, N, d, C, bits):
    rng = np.random.default_rng(M + K)
    cb = pi.signed_one_hot_codebook(C, d, rng)
    ids = rng.integers(3, C, size=(N, K // d))
    ids[5, 0], ids[N - 1, K // d - 1], ids[7, 3] = 0, 1, 2
    cb[0], cb[1], cb[2] = np.inf, -np.inf, np.nan
    x = pi.ternary_x(rng, M, K)
    x[1, K - 1], x[M - 1, 0], x[M // 2, 9] = np.inf, -np.inf, np.nan
    idx = pi.pack_indices(ids, bits)
    with np.errstate(invalid="ignore"):
        ref = orc.pq_linear(x, idx, bits, d, cb)
    assert fasq.plan("gemm", M, K, N, bits, d, C).startswith("k_gemm_gather<")
    y = to_np(fasq.pq_gemm(to_dev(x), to_dev(idx), bits, d, to_dev(cb))).astype(np.float64)
    assert np.array_equal(y, ref, equal_nan=True)
