"""GPU parity of the k-means encoder (fasq_pq_encode) against the CPU oracle.

The encoder's arithmetic is fully defined (fp32 distances without fused
multiply-add, lowest index on ties, exact cluster sums, fp64 division, one
fp16 rounding), so the codebook and the ids must match the oracle bit for bit.
"""

import numpy as np
import pytest

import pq_inputs as pi
from oracle import pq_encode as enc
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


def gpu_encode(w, d, bits, init, iters):
    cb, idx = fasq.pq_encode(to_dev(w), d, bits, to_dev(init), iters)
    return to_np(cb), to_np(idx)


def check_encode(w, d, C, bits, init, iters, label):
    cb_ref, ids_ref = enc.kmeans_encode(w, d, init, iters)
    cb, idx = gpu_encode(w, d, bits, init, iters)
    assert np.array_equal(cb.view(np.uint16), cb_ref.view(np.uint16)), f"{label}: codebook"
    ids = orc.unpack_indices(idx, w.shape[1] // d, bits, C)
    assert np.array_equal(ids, ids_ref), f"{label}: ids ({int((ids != ids_ref).sum())} differ)"
    return cb, idx


CASES = [
    # N, K, d, C, bits, iters
    (256, 512, 2, 256, 8, 5),     # cluster sums gathered in LDS per workgroup
    (128, 512, 4, 4096, 12, 3),   # one LDS table of cluster sums per workgroup
    (256, 512, 4, 20000, 16, 2),  # codebook in four LDS tiles
    (64, 256, 8, 256, 8, 4),
    (100, 300, 3, 50, 8, 3),      # every distance, d = 3 padded to 4
    (33, 64, 1, 16, 8, 6),
    (50, 36, 4, 9, 12, 4),        # odd 12-bit rows (pad nibble)
    (40, 64, 2, 64, 8, 0),        # no update: ids against the starting codebook
]


@pytest.mark.parametrize("case", CASES)
def test_encode_matches_oracle_bit_exact(case):
    N, K, d, C, bits, iters = case
    print(f"[case] encode {case}", flush=True)
    rng = np.random.default_rng(sum(case))
    w = pi.draw_weights(rng, N, K)
    init = pi.subvectors_at(w, d, pi.init_point_ids(rng, N * K // d, C))
    check_encode(w, d, C, bits, init, iters, str(case))


# The edges of the assignment paths: every distance up to 64 codewords, the
# matrix cores beyond (blocks of 8 codewords per lane up to 512, of 16 after;
# one LDS tile of the codebook up to 5376 codewords at d = 3 and 4, several
# after), padded d, point counts that fill no tile, and cluster sums in one
# LDS table, in ranges of clusters, and in global memory.
EDGES = [
    # N, K, d, C, bits, iters
    (31, 64, 2, 64, 8, 2),
    (31, 64, 2, 65, 8, 2),
    (1, 300, 3, 100, 8, 2),         # fewer points than one workgroup takes
    (257, 100, 5, 512, 12, 2),
    (257, 100, 5, 513, 12, 2),
    (100, 704, 11, 300, 12, 2),
    (64, 512, 16, 257, 12, 2),
    (300, 200, 1, 9000, 16, 2),
    (120, 256, 4, 5376, 16, 2),
    (120, 256, 4, 5377, 16, 2),
    (700, 400, 4, 60000, 16, 1),    # more clusters than the LDS tables take
    (1100, 1024, 2, 256, 8, 1),     # four point tiles per wave
]


@pytest.mark.parametrize("case", EDGES)
def test_encode_path_edges_match_oracle_bit_exact(case):
    N, K, d, C, bits, iters = case
    print(f"[case] encode edge {case}", flush=True)
    rng = np.random.default_rng(100 + sum(case))
    w = pi.draw_weights(rng, N, K)
    points = N * K // d
    # more codewords than points: the rest are drawn
    init = pi.subvectors_at(w, d, pi.init_point_ids(rng, points, min(C, points)))
    init = np.concatenate([init, pi.draw_codebook(rng, C - len(init), d)]) if len(init) < C else init
    check_encode(w, d, C, bits, np.ascontiguousarray(init), iters, str(case))


@pytest.mark.parametrize("d,C,bits", [(1, 300, 12), (2, 256, 8), (3, 1000, 12), (4, 4096, 12), (4, 6000, 16), (8, 600, 12)])
@pytest.mark.parametrize("values", ["lattice", "sparse", "alike", "subnormal"])
def test_encode_ties_go_to_the_lowest_index(values, d, C, bits):
    """Exact ties between codewords of different blocks and tiles: values on a
    coarse lattice, mostly zero weights with repeated codewords, all codewords
    alike, and fp16 subnormals (whose distances differ by single units)."""
    rng = np.random.default_rng(d * C + len(values))
    N, K = 48, 24 * d
    if values == "subnormal":
        w = (rng.integers(-9, 10, (N, K)) * 2.0 ** -24).astype(np.float16)
        init = (rng.integers(-9, 10, (C, d)) * 2.0 ** -24).astype(np.float16)
    else:
        w = (rng.integers(-3, 4, (N, K)) * 0.25).astype(np.float16)
        if values == "sparse":
            w[rng.random((N, K)) < 0.7] = 0
        init = (rng.integers(-3, 4, (C, d)) * 0.25).astype(np.float16)
        if values == "alike":
            init[:] = np.float16(0.5)
    check_encode(w, d, C, bits, init, 1, f"{values} d={d} C={C}")


def test_encode_never_picks_a_non_finite_codeword():
    """A codeword with an infinity or a NaN is at no finite distance; the
    others are chosen as if it were not there."""
    rng = np.random.default_rng(11)
    d, bits = 4, 16
    w = pi.draw_weights(rng, 64, 256)
    for C in (50, 300, 6000):
        init = pi.draw_codebook(rng, C, d)
        bad = init.copy()
        bad[::3, 0] = np.inf
        bad[1::5, 3] = np.nan
        bad[2::7, 1] = -np.inf
        keep = np.isfinite(bad).all(1)
        ids_ref = np.flatnonzero(keep)[enc.assign(w.reshape(-1, d), init[keep])]
        _, idx = gpu_encode(w, d, bits, bad, 0)
        assert np.array_equal(orc.unpack_indices(idx, 64, bits, C).reshape(-1), ids_ref), C


def test_encode_is_deterministic_and_accepts_in_place_init():
    rng = np.random.default_rng(7)
    N, K, d, C, bits = 512, 1024, 2, 256, 8
    w = to_dev(pi.draw_weights(rng, N, K))
    init = to_dev(pi.subvectors_at(to_np(w), d, pi.init_point_ids(rng, N * K // d, C)))
    a_cb, a_idx = fasq.pq_encode(w, d, bits, init, 4)
    b_cb, b_idx = fasq.pq_encode(w, d, bits, init, 4)
    assert torch.equal(a_cb.view(torch.int16), b_cb.view(torch.int16))
    assert torch.equal(a_idx, b_idx)
    # init_codebook == codebook: the encoder updates the buffer in place
    buf = init.clone()
    idx = torch.empty_like(a_idx)
    ws = torch.empty(fasq.encode_workspace_bytes(N, K, d, C), dtype=torch.uint8, device=w.device)
    st = fasq.encode_raw(w.data_ptr(), N, K, d, C, bits, buf.data_ptr(), 4, buf.data_ptr(), idx.data_ptr(),
                         ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert st == 0, fasq.last_error()
    assert torch.equal(buf.view(torch.int16), a_cb.view(torch.int16))
    assert torch.equal(idx, a_idx)


def test_means_on_fp16_halfway_points_and_subnormals():
    """Cluster means that fall exactly halfway between fp16 neighbours (ties
    to even) and means in the fp16 subnormal range."""
    rng = np.random.default_rng(9)
    d, C, bits = 1, 64, 8
    vals = []
    for k in range(C // 2):
        a = np.float16(1.0 + k / 64)
        b = np.nextafter(a, np.float16(4.0))
        vals += [a, b]                       # mean halfway between a and b
    for k in range(C // 2):
        vals += [np.float16((k + 1) * 2.0 ** -24), np.float16((k + 2) * 2.0 ** -24)]  # subnormal means
    pts = np.array(vals, dtype=np.float16)
    w = np.repeat(pts, 4).reshape(-1, 8)     # each value four times: same means
    init = np.unique(pts)[:C].reshape(-1, 1)
    init = np.concatenate([init, np.full((C - len(init), 1), 100.0, np.float16)]).astype(np.float16)
    check_encode(w, d, C, bits, init, 3, "halfway")


def test_encoded_layer_runs_through_the_matmul():
    """Encode dense weights, then y = x . W_hat^T from the encoding agrees with
    the oracle on the oracle's encoding (they are the same bits)."""
    rng = np.random.default_rng(10)
    N, K, d, C, bits = 512, 2048, 2, 256, 8
    w = pi.draw_weights(rng, N, K)
    init = pi.subvectors_at(w, d, pi.init_point_ids(rng, N * K // d, C))
    cb, idx = check_encode(w, d, C, bits, init, 6, "layer")
    x = pi.draw_x(rng, 1, K)
    y = to_np(fasq.pq_gemv(to_dev(x), to_dev(idx), bits, d, to_dev(cb))).astype(np.float64)
    assert_close(y, orc.pq_linear(x, idx, bits, d, cb), "encoded layer")
    # quantization error of the layer output against the dense fp16 weights, for the record
    dense = x.astype(np.float64) @ w.astype(np.float64).T
    print(f"[encode] layer rel error vs dense weights: {orc.relative_l2(y, dense):.3f}", flush=True)


def nearest(w, d, cb):
    """The defined assignment on the GPU by plain torch: fp32 differences,
    squares and sums rounded one by one, the lowest index on ties."""
    points, c = w.view(-1, d).float(), cb.float()
    order = torch.arange(len(c), device=w.device, dtype=torch.int32)
    out = torch.empty(len(points), dtype=torch.int64, device=w.device)
    block = max(1, (1 << 26) // len(c))
    for b in range(0, len(points), block):
        p = points[b:b + block]
        dist = torch.zeros((len(p), len(c)), device=w.device)
        for i in range(d):
            diff = p[:, i:i + 1] - c[None, :, i]
            dist += diff * diff
        dist[~(dist < float("inf"))] = float("inf")  # a non-finite codeword is never chosen
        near = dist == dist.amin(1, keepdim=True)
        out[b:b + block] = torch.where(near, order, len(c)).amin(1).long()
    return out


def weights(values, N, K, d):
    """Weights whose nearest codeword the matrix-core pass decides (normal) or
    leaves open: a large common offset, half of the sub-vectors pruned (the
    starting codewords repeat zero), values on a lattice."""
    g = torch.Generator(device="cuda").manual_seed(N + K + d)
    w = torch.randn((N, K), generator=g, device="cuda") * 0.02
    if values == "offset":
        w = w + 0.5
    elif values == "pruned":
        keep = torch.rand((N * K // d, 1), generator=g, device="cuda") < 0.5
        w = (w.view(-1, d) * keep).view(N, K)
    elif values == "lattice":
        w = (w / 0.01).round() * 0.01
    return w.half()


def first_codewords(w, d, C):
    points = w.view(-1, d)
    return points[torch.linspace(0, len(points) - 1, C, device="cuda").long()].contiguous()


# four point tiles per wave (from 524288 points on) and one, codebooks of one
# LDS tile (blocks of 8 and of 16 codewords) and of several, padded d
OPEN = [
    # N, K, d, C, bits
    (1031, 1024, 1, 300, 12),      # point count that fills no tile
    (520, 1024, 1, 4096, 12),
    (1040, 1024, 2, 256, 8),
    (1037, 1030, 2, 1000, 12),
    (1100, 1536, 3, 100, 8),
    (2100, 1024, 4, 4096, 12),     # the 12-bit format's codebook
    (2080, 1024, 4, 6000, 16),     # two LDS tiles
    (4201, 1024, 8, 257, 12),
    (4200, 2048, 16, 520, 12),
    (100, 1000, 2, 300, 12),
    (64, 1024, 4, 20000, 16),
    (90, 704, 11, 300, 12),
]


@pytest.mark.parametrize("values", ["normal", "offset", "pruned", "lattice"])
@pytest.mark.parametrize("case", OPEN)
def test_points_left_open_by_the_matrix_cores(case, values):
    N, K, d, C, bits = case
    print(f"[case] encode open {case} {values}", flush=True)
    K = K // d * d
    w = weights(values, N, K, d)
    init = first_codewords(w, d, C)
    if values == "lattice":
        init[C // 3] = float("inf")  # codewords staged as zeros
        init[C // 2, 0] = float("nan")
    ref = nearest(w, d, init)
    _, idx = fasq.pq_encode(w, d, bits, init, 0)
    ids = orc.unpack_indices(to_np(idx), K // d, bits, C).reshape(-1)
    assert np.array_equal(ids, ref.cpu().numpy()), int((ids != ref.cpu().numpy()).sum())


@pytest.mark.parametrize("d,C,bits", [(1, 300, 12), (2, 256, 8), (4, 512, 12), (4, 6000, 16)])
def test_whole_blocks_of_codewords_at_no_distance(d, C, bits):
    """Runs of codewords whose distances are all NaN (a NaN component, or
    infinities of weight and codeword) among points whose every distance is
    evaluated: they are passed over like single ones."""
    N, K = 300, 1024
    w = weights("pruned", N, K, d)
    init = first_codewords(w, d, C)
    init[16:40] = float("nan")
    init[64:96] = float("inf")
    init[C - 20:] = float("nan")
    w[7] = float("inf")  # at no finite distance from any codeword
    ref = nearest(w, d, init)
    _, idx = fasq.pq_encode(w, d, bits, init, 0)
    ids = orc.unpack_indices(to_np(idx), K // d, bits, C).reshape(-1)
    assert np.array_equal(ids, ref.cpu().numpy()), int((ids != ref.cpu().numpy()).sum())


def encode_ms(w, d, bits, init, calls=20):
    ws = torch.empty(fasq.encode_workspace_bytes(*w.shape, d, len(init)), dtype=torch.uint8, device="cuda")
    best = float("inf")
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(calls):
            fasq.pq_encode(w, d, bits, init, 0, workspace=ws)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / calls)
    return best


@pytest.mark.parametrize("d,C,values", [(1, 256, "pruned"), (1, 1024, "offset"), (2, 256, "offset"), (2, 256, "pruned"),
                                        (4, 512, "pruned"), (8, 256, "pruned")])
def test_open_points_cost_no_more_than_every_distance(d, C, values):
    """Where the matrix-core pass leaves most points open, the encoder must not
    take longer than evaluating every distance, which it does for codebooks
    of up to 64 codewords: C / 64 times such a call (and a quarter, for the
    pass itself and the spread of a timing)."""
    N, K = 2048, 2048
    w = weights(values, N, K, d)
    every = encode_ms(w, d, 8, first_codewords(w, d, 64)) * (C / 64)
    took = encode_ms(w, d, 12 if C > 256 else 8, first_codewords(w, d, C))
    print(f"[time] d={d} C={C} {values}: {took * 1e3:.0f} us, every distance {every * 1e3:.0f} us", flush=True)
    assert took <= 1.25 * every
