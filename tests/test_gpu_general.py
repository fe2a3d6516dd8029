"""GPU parity of the general kernels (the calls no tuned kernel takes) at the
edges of their spans, runs and tiles, and at pointers of any alignment."""

import numpy as np
import pytest

import pq_inputs as pi
from oracle import pq_oracle as orc
from gpu_util import assert_close, to_dev, to_np

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


def at_offset(a, offset):
    """The bytes of ``a`` on the device, ``offset`` bytes past an aligned address."""
    raw = torch.zeros(a.nbytes + 64, dtype=torch.uint8, device="cuda:0")
    raw[offset:offset + a.nbytes] = torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).reshape(-1)).cuda()
    return raw, raw.data_ptr() + offset


CASES = [
    # M, K, N, d, C, bits, per subspace, byte offsets of x, ids and codebook
    (1, 3, 1, 3, 2, 8, False, (0, 0, 0)),
    (16, 128, 16, 2, 256, 8, True, (2, 1, 4)),      # one whole span, one tile
    (17, 126, 17, 2, 256, 8, False, (2, 1, 2)),     # a span two short, second tiles of one
    (33, 130, 31, 1, 64, 8, True, (0, 3, 2)),       # a span and two values
    (49, 1516, 40, 4, 256, 8, False, (0, 0, 0)),
    (64, 2176, 33, 4, 500, 12, True, (0, 0, 0)),    # more spans than waves
    (65, 264, 50, 8, 300, 12, True, (8, 1, 16)),    # runs of six id bytes
    (130, 300, 270, 6, 100, 16, False, (2, 0, 0)),
    (5, 384, 20, 2, 3000, 16, True, (0, 0, 2)),     # codewords off their alignment
    (40, 384, 4500, 2, 256, 8, True, (0, 0, 0)),    # three token tiles per workgroup
    (20, 35, 9, 5, 4096, 12, False, (0, 1, 0)),     # odd 12-bit rows
    (3, 99, 1000, 3, 256, 8, True, (0, 0, 0)),      # runs of ten codewords, few features per workgroup
    (18, 312, 30, 24, 90, 12, False, (0, 0, 0)),    # one codeword per run
    (7, 200, 33, 40, 50, 8, False, (0, 1, 2)),      # codewords longer than a run
    (2, 350, 20, 35, 700, 16, True, (2, 0, 0)),
    (17, 3, 1, 3, 2, 8, False, (0, 0, 0)),          # the smallest sizes with more tokens than the row kernel takes
    (9, 99, 1000, 3, 256, 8, True, (0, 0, 0)),
]

# a wave per feature: few values per lane (one round of sub-vectors and more,
# whole and not), a second block of tokens, odd 12-bit rows, any alignment
ROWS = [
    # M, K, N, d, C, bits, per subspace, byte offsets of x, ids and codebook
    (1, 1, 1, 1, 1, 8, False, (0, 0, 0)),
    (1, 64, 5, 1, 256, 8, False, (2, 1, 2)),
    (2, 65, 7, 1, 300, 12, True, (2, 1, 2)),
    (8, 130, 3, 1, 300, 12, False, (0, 0, 0)),
    (16, 14, 2, 1, 512, 12, True, (0, 0, 2)),
    (9, 5, 4, 1, 4096, 12, False, (0, 1, 0)),
    (1, 110, 478, 5, 100, 8, False, (0, 0, 0)),
    (1, 336, 848, 6, 4096, 12, False, (2, 1, 2)),
    (3, 96, 2000, 3, 256, 8, True, (0, 0, 0)),
    (7, 35, 30, 5, 5000, 16, False, (2, 0, 2)),
    (1, 16, 3000, 2, 16, 8, True, (0, 3, 0)),
    (3, 16, 9, 4, 90, 8, False, (2, 0, 0)),
    (1, 144, 33, 9, 70, 12, True, (0, 1, 2)),
]


def test_small_calls_take_the_row_kernel(monkeypatch):
    """The kernel of the few-value calls, and the sizes from which the matrix
    cores are faster (its time grows with rounds x d x tokens)."""
    monkeypatch.setenv("FASQ_FORCE_PATH", "generic")
    rows = [fasq.plan("gemv", M, K, N, bits, d, C).startswith("k_pq_generic_rows<") for M, K, N, d, C, bits, *_ in ROWS]
    assert all(rows), rows
    for M, K, N, bits, d, C in [(4, 112, 1529, 8, 4, 256), (8, 6, 36, 16, 6, 5000), (1, 130, 9000, 8, 5, 256),
                                (17, 3, 1, 8, 3, 2), (1, 4096, 100, 8, 2, 256), (1, 24, 20000, 12, 6, 1000)]:
        assert not fasq.plan("gemv", M, K, N, bits, d, C).startswith("k_pq_generic_rows<"), (M, K, N, bits, d)


@pytest.mark.parametrize("case", CASES + ROWS)
def test_general_kernel_matches_oracle(case, monkeypatch):
    M, K, N, d, C, bits, per, (ox, oi, oc) = case
    print(f"[case] general {case}", flush=True)
    monkeypatch.setenv("FASQ_FORCE_PATH", "generic")
    rng = np.random.default_rng(sum(case[:6]))
    S = K // d
    books = pi.draw_codebook(rng, (S if per else 1) * C, d).reshape(-1, C, d)
    ids = pi.draw_ids(rng, N, S, C)
    x = pi.draw_x(rng, M, K)
    idx = pi.pack_indices(ids, bits)
    keep_x, xp = at_offset(x, ox)
    keep_i, ip = at_offset(idx, oi)
    keep_c, cp = at_offset(books, oc)
    y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    if per:
        st = fasq.gemv_ex_raw(xp, M, K, N, ip, bits, d, cp, C, C * d, y.data_ptr(), 0, 0, stream)
        ref = orc.lut_accumulate(x, books, ids.T)
    else:
        st = fasq.gemm_raw(xp, M, K, N, ip, bits, d, cp, C, y.data_ptr(), stream)
        ref = orc.pq_linear(x, idx, bits, d, books[0])
    assert st == 0, fasq.last_error()
    assert_close(to_np(y).astype(np.float64), ref, str(case))


def test_general_kernel_is_exact_on_small_integers(monkeypatch):
    """Signed one-hot codewords and ternary activations: every partial sum is
    a small integer, so any order gives the oracle's bits."""
    monkeypatch.setenv("FASQ_FORCE_PATH", "generic")
    rng = np.random.default_rng(4)
    M, K, N, d, C, bits = 35, 516, 70, 3, 60, 8
    books = np.stack([pi.signed_one_hot_codebook(C, d, rng) for _ in range(K // d)])
    ids = rng.integers(0, C, size=(N, K // d))
    x = pi.ternary_x(rng, M, K)
    y = to_np(fasq.pq_gemv_ex(to_dev(x), to_dev(pi.pack_indices(ids, bits)), bits, d, to_dev(books)))
    assert np.array_equal(y.astype(np.float64), orc.lut_accumulate(x, books, ids.T))


@pytest.mark.parametrize("case", [(37, 1516, 40, 4, 256, 8), (18, 99, 70, 3, 256, 8), (20, 130, 31, 1, 64, 8),
                                  (20, 160, 30, 40, 90, 12), (2, 65, 7, 1, 300, 12), (33, 264, 50, 8, 300, 12)])
@pytest.mark.parametrize("per", [False, True])
def test_infinities_and_nan_reach_only_their_outputs(case, per, monkeypatch):
    """Non-finite codewords and activations, also beside the zeros that fill a
    run past the row's end: the oracle's outputs, infinities and NaN included."""
    monkeypatch.setenv("FASQ_FORCE_PATH", "generic")
    M, K, N, d, C, bits = case
    rng = np.random.default_rng(sum(case) + per)
    S = K // d
    books = np.stack([pi.signed_one_hot_codebook(C, d, rng) for _ in range(S if per else 1)])
    ids = rng.integers(3, C, size=(N, S))
    ids[N // 2, 0], ids[N - 1, S - 1], ids[0, S // 2] = 0, 1, 2
    books[:, 0], books[:, 1], books[:, 2] = np.inf, -np.inf, np.nan
    x = pi.ternary_x(rng, M, K)
    x[0, K - 1], x[M - 1, 0] = np.inf, -np.inf
    if M > 2:
        x[M // 2, K // 2] = np.nan
    idx = pi.pack_indices(ids, bits)
    with np.errstate(invalid="ignore"):
        ref = orc.lut_accumulate(x, books, ids.T) if per else orc.pq_linear(x, idx, bits, d, books[0])
    cb = to_dev(books if per else books[0])
    y = to_np(fasq.pq_gemv_ex(to_dev(x), to_dev(idx), bits, d, cb)).astype(np.float64)
    assert np.array_equal(y, ref, equal_nan=True)
