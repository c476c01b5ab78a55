"""GPU parity: the HIP library, called through its C ABI, against the float64 CPU oracle on the
same seeded inputs.

Bar: per group, max|gpu - oracle| / max|oracle| <= 1e-5 for the float32 outputs; status words,
survivor handling and located adversary sets bit-exact.
"""
import numpy as np
import pytest

from oracle import approxifer_oracle as orc
from paper_2109_09868_amd import synthetic as syn
from parity_cases import (TOL, ILL_POSED_FUZZ_ALL, ILL_POSED_FUZZ_BYZANTINE, ILL_POSED_RAGGED, assert_rounding_ties,
                          fuzz_all_cases, fuzz_byzantine_cases, group_err, ragged_decode_case, rational_tolerance,
                          well_posed)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2109_09868_amd import binding
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.load()                      # raises if the HIP library was not built: no fallback
    return torch, binding, torch.device("cuda:0")


# --------------------------------------------------------------------------------------
# encoder
# --------------------------------------------------------------------------------------
def test_encode_tiny_workload(gpu):
    torch, binding, dev = gpu
    w = syn.WORKLOADS["tiny"]
    alpha, beta = orc.chebyshev_nodes(w.K, w.W)
    X = syn.queries(w)
    coded = binding.approxifer_encode(torch.from_numpy(X).to(dev), alpha, beta)
    err = group_err(coded.cpu().numpy(), orc.encode(X, alpha, beta))
    assert err.max() <= TOL, err.max()


@pytest.mark.parametrize("K,N,D,G", [
    (1, 2, 5, 2), (2, 3, 1000, 3), (3, 5, 4100, 2), (5, 9, 1023, 3), (7, 16, 2048, 2), (12, 20, 4 * 700, 3),
    (16, 24, 4 * 300 + 4, 2), (17, 21, 777, 2), (32, 48, 4 * 513, 2), (33, 40, 258, 1), (64, 128, 4 * 260, 2),
    (8, 12, 3, 5), (12, 20, 1, 4),
    # K > 16 with 16-byte rows: the matrix-core kernel; K % 4 != 0, N % 16 != 0, ragged column tiles
    (17, 21, 4 * 100, 3), (20, 33, 4 * 65, 2), (22, 16, 4 * 64, 2), (24, 36, 4 * 700 + 4, 2), (31, 47, 4 * 3, 3),
    (32, 48, 4 * 1024, 2), (47, 100, 4 * 129, 1), (63, 127, 4 * 77, 2), (64, 65, 4 * 64, 1), (18, 2, 4 * 50, 2),
    # 8 <= K <= 16 with N >= 2K + 4 and full 64-column blocks: the matrix-core kernel; neighbours stay on the vector kernel
    (8, 24, 4 * 64 * 3, 2), (12, 28, 4 * 128, 2), (16, 36, 4 * 64, 2), (9, 24, 4 * 64 * 2, 2), (8, 20, 4 * 64, 3),
    (8, 19, 4 * 64, 3), (8, 24, 4 * 70, 2), (7, 24, 4 * 64, 2), (13, 128, 4 * 64, 1),
    # matrix-core kernel over the flattened (group, column) numbering: short ragged rows
    (12, 28, 784, 5), (8, 24, 4 * 50, 3), (20, 30, 4 * 70, 3), (32, 48, 4 * 10, 7), (17, 20, 4 * 1, 9),
    # residency caps: K = 1, 2, 4 run with many more waves per CU
    (1, 2, 4 * 64 * 40, 3), (2, 3, 4 * 64 * 33, 3), (4, 6, 4 * 64 * 21, 2),
    # short ragged rows (D % 4 != 0, D <= 128) take 4-byte accesses for every column; 129 and up: 128-bit + tail
    (8, 12, 30, 700), (12, 20, 7, 300), (8, 24, 126, 40), (20, 30, 127, 9), (33, 40, 5, 11), (8, 12, 129, 40), (12, 28, 130, 9),
])
def test_encode_shapes_with_ragged_tails(gpu, K, N, D, G):
    torch, binding, dev = gpu
    rng = np.random.default_rng(1000 * K + N)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.standard_normal((G, K, D)).astype(np.float32)
    coded = binding.approxifer_encode(torch.from_numpy(X).to(dev), alpha, beta)
    err = group_err(coded.cpu().numpy(), orc.encode(X, alpha, beta))
    assert err.max() <= TOL, err.max()


@pytest.mark.parametrize("K,N,D,G,off_in,off_out", [
    (6, 10, 1000, 2, 1, 3), (6, 10, 1003, 3, 0, 0), (6, 10, 1001, 2, 1, 2), (12, 20, 4 * 64 * 3 + 2, 2, 3, 1),
    (8, 24, 4 * 64 * 2 + 1, 2, 2, 2), (20, 30, 4 * 64 + 3, 2, 1, 1), (33, 40, 4 * 64 * 2, 1, 3, 3), (3, 5, 2, 4, 1, 1),
    (8, 12, 30, 50, 1, 2), (12, 20, 127, 6, 3, 1), (8, 12, 30, 50, 2, 2), (5, 7, 126, 9, 0, 2),
])
def test_encode_unaligned_pointers_and_canaries(gpu, K, N, D, G, off_in, off_out):
    # rows that are only 4-byte aligned (odd row length and/or offset base pointers): 128-bit accesses through the
    # 4-byte-aligned vector type plus a 4-byte tail; nothing outside the output tensor may be touched
    torch, binding, dev = gpu
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = np.random.default_rng(5 + D).uniform(0, 1, (G, K, D)).astype(np.float32)
    flat_in = torch.zeros(G * K * D + off_in + 5, dtype=torch.float32, device=dev)
    flat_in[off_in:off_in + G * K * D] = torch.from_numpy(X).to(dev).reshape(-1)
    q = flat_in[off_in:off_in + G * K * D].view(G, K, D)
    flat_out = torch.full((G * N * D + off_out + 9,), 7.5, dtype=torch.float32, device=dev)
    c = flat_out[off_out:off_out + G * N * D].view(G, N, D)
    binding.approxifer_encode(q, alpha, beta, coded=c)
    err = group_err(c.cpu().numpy(), orc.encode(X, alpha, beta))
    assert err.max() <= TOL
    assert torch.all(flat_out[:off_out] == 7.5) and torch.all(flat_out[off_out + G * N * D:] == 7.5)


@pytest.mark.parametrize("K,N", [(1, 2), (5, 8), (16, 20), (8, 24), (12, 28), (20, 24), (33, 64)])
@pytest.mark.parametrize("off_in,off_out", [(0, 0), (3, 0), (0, 6), (1, 13)])
def test_encode_tiles_of_whole_sectors(gpu, K, N, off_in, off_out):
    # rows that are no whole 64-byte sectors: one tile up to 63 vectors of a row, then 60 a tile less one for the last; row
    # ends of every remainder, rows just above and below a tile more, phases of every row from the base's and the length's
    torch, binding, dev = gpu
    alpha, beta = orc.chebyshev_nodes(K, N)
    for D in (129, 130, 160, 250, 251, 252, 253, 254, 299, 300, 473, 475, 476, 477, 714, 717, 960, 2047, 2050):
        G = 3
        X = np.random.default_rng(D).uniform(0, 1, (G, K, D)).astype(np.float32)
        flat_in = torch.full((G * K * D + off_in + 5,), float("nan"), dtype=torch.float32, device=dev)
        flat_in[off_in:off_in + G * K * D] = torch.from_numpy(X).to(dev).reshape(-1)
        flat_out = torch.full((G * N * D + off_out + 40,), 7.5, dtype=torch.float32, device=dev)
        c = flat_out[off_out:off_out + G * N * D].view(G, N, D)
        binding.approxifer_encode(flat_in[off_in:off_in + G * K * D].view(G, K, D), alpha, beta, coded=c)
        got, ref = c.cpu().numpy(), orc.encode(X, alpha, beta)
        # every element: K roundings of weights and products, the weights' absolute sum times the largest query (below 1)
        bound = (K + 2) * 2.0 ** -23 * np.abs(orc.encode(np.eye(K)[None], alpha, beta)).sum(axis=2).max()
        assert np.abs(got - ref).max() <= bound, (D, np.abs(got - ref).max(), bound)
        assert torch.all(flat_out[:off_out] == 7.5) and torch.all(flat_out[off_out + G * N * D:] == 7.5), D


@pytest.mark.parametrize("K,N,D,G", [
    (4, 6, 260, 6200), (8, 12, 1004, 900), (12, 28, 1004, 520), (14, 35, 156, 3000), (1, 9, 388, 2100),    # 16-byte pieces
    (24, 48, 204, 2100), (20, 26, 2036, 240), (33, 40, 1004, 420),
    (6, 12, 252, 4000), (3, 5, 792, 1296), (8, 20, 776, 1600), (14, 35, 136, 2400), (5, 8, 2052, 500), (1, 2, 1484, 4000),
    (4, 16, 141, 700), (1, 2, 275, 4200), (9, 12, 203, 700), (11, 26, 218, 1400), (16, 20, 387, 330), (20, 24, 161, 40),   # ragged rows
])
def test_encode_gives_the_same_bits_in_calls_of_every_size(gpu, K, N, D, G):
    # the number of groups decides between the tiles of whole sectors and the kernels that move rows as they come, and between
    # vector and matrix cores: the same float32 multiply-adds in the same order everywhere
    torch, binding, dev = gpu
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = torch.rand((G, K, D), generator=torch.Generator(device=dev).manual_seed(D), device=dev)
    whole = torch.full((G, N, D), float("nan"), device=dev)
    binding.approxifer_encode(X, alpha, beta, coded=whole)
    for g0, n in [(0, 1), (1, 7), (G // 2, min(G // 4, 600)), (G - 1, 1)]:
        part = torch.full((n, N, D), float("nan"), device=dev)
        binding.approxifer_encode(X[g0:g0 + n].clone(), alpha, beta, coded=part)      # from a 16-byte address again
        assert torch.equal(part, whole[g0:g0 + n]), (g0, n)
    bound = (K + 2) * 2.0 ** -23 * np.abs(orc.encode(np.eye(K)[None], alpha, beta)).sum(axis=2).max()
    for g in (0, G - 1):
        assert np.abs(whole[g].cpu().numpy() - orc.encode(X[g:g + 1].cpu().numpy(), alpha, beta)[0]).max() <= bound


@pytest.mark.parametrize("K,N,D,few,many", [(9, 12, 203, 3, 700), (11, 26, 1004, 2, 900), (14, 18, 141, 4, 800), (17, 23, 1008, 2, 40),
                                            (22, 30, 501, 2, 40), (33, 41, 64, 2, 600)])
def test_encode_of_an_infinity_in_the_last_query_is_that_infinity(gpu, K, N, D, few, many):
    # numbers of queries that are no multiple of the matrix cores' four: what fills them up counts for nothing, and the kernels
    # with and without matrix cores, between which the number of groups decides, answer the same
    torch, binding, dev = gpu
    alpha, beta = orc.chebyshev_nodes(K, N)
    weight = orc.encode(np.eye(K)[None], alpha, beta)[0][:, K - 1]
    rows = np.abs(weight) > 1e-6
    sign = torch.from_numpy(np.sign(weight[rows]).astype(np.float32)).to(dev)
    for G in (few, many):
        X = torch.rand((G, K, D), generator=torch.Generator(device=dev).manual_seed(G), device=dev)
        plain = binding.approxifer_encode(X, alpha, beta)
        X[:, K - 1, 5::7] = float("inf")
        coded = binding.approxifer_encode(X, alpha, beta)
        keep = torch.ones(D, dtype=torch.bool, device=dev)
        keep[5::7] = False
        assert torch.equal(coded[:, :, keep], plain[:, :, keep])
        got = coded[:, torch.from_numpy(rows).to(dev)][:, :, 5::7]
        assert bool((got == (sign * float("inf"))[None, :, None]).all()), G


@pytest.mark.parametrize("rows", [14397, 14398, 14399, 14400, 14401, 16798, 47999])
def test_rows_of_many_full_tiles_are_written_to_their_end(gpu, rows):
    # from 60 tiles a row on a row can be whole tiles of sixty vectors, and the last one still has to keep a lane for the shift;
    # the encoders' vector and matrix-core tiles and the decoder's, output rows of all four phases of a 16-byte piece
    torch, binding, dev = gpu
    rng = np.random.default_rng(rows)
    for K, N, S, off in [(3, 5, 1, 0), (3, 5, 1, 2), (12, 17, 4, 0), (12, 17, 4, 1), (20, 30, 6, 0), (20, 30, 6, 3)]:
        alpha, beta = orc.chebyshev_nodes(K, N)
        X = rng.uniform(0, 1, (2, K, rows)).astype(np.float32)
        flat = torch.full((off + 2 * N * rows + 40,), float("nan"), dtype=torch.float32, device=dev)
        c = flat[off:off + 2 * N * rows].view(2, N, rows)
        binding.approxifer_encode(torch.from_numpy(X).to(dev), alpha, beta, coded=c)
        # as for the short rows above: K roundings of weights and products
        bound = (K + 2) * 2.0 ** -23 * np.abs(orc.encode(np.eye(K)[None], alpha, beta)).sum(axis=2).max()
        assert np.all(np.abs(c.cpu().numpy() - orc.encode(X, alpha, beta)) <= bound), (K, off)
        assert torch.isnan(flat[:off]).all() and torch.isnan(flat[off + 2 * N * rows:]).all()
        Y = rng.standard_normal((2, N, rows)).astype(np.float32)
        mask = np.ones((2, N), np.uint8)
        mask[:, rng.choice(N, S, replace=False)] = 0
        flat = torch.full((off + 2 * K * rows + 40,), float("nan"), dtype=torch.float32, device=dev)
        out = flat[off:off + 2 * K * rows].view(2, K, rows)
        binding.approxifer_decode(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta, S, 1, out=out)
        ref, _ = orc.decode(Y, mask, alpha, beta, S, 1)
        # one rounding to float32, float64 sums before it
        assert np.all(np.abs(out.cpu().numpy() - ref) <= 2.0 ** -24 * np.abs(ref) + 1e-12 * np.abs(Y).max()), (K, off)
        assert torch.isnan(flat[:off]).all() and torch.isnan(flat[off + 2 * K * rows:]).all()


def test_encode_node_coincidence_passes_query_through(gpu):
    torch, binding, dev = gpu
    alpha, beta = orc.chebyshev_nodes(2, 5)
    beta = beta.copy()
    beta[1], beta[3] = alpha[0], alpha[1]
    X = np.random.default_rng(6).standard_normal((3, 2, 600)).astype(np.float32)
    coded = binding.approxifer_encode(torch.from_numpy(X).to(dev), alpha, beta).cpu().numpy()
    assert np.array_equal(coded[:, 1], X[:, 0]) and np.array_equal(coded[:, 3], X[:, 1])
    assert group_err(coded, orc.encode(X, alpha, beta)).max() <= TOL
    # K=6, N=9: beta_2 and alpha_1 are both cos(pi/4) straight from the node formulas
    alpha, beta = orc.chebyshev_nodes(6, 9)
    X = np.random.default_rng(7).standard_normal((2, 6, 64)).astype(np.float32)
    coded = binding.approxifer_encode(torch.from_numpy(X).to(dev), alpha, beta).cpu().numpy()
    assert group_err(coded, orc.encode(X, alpha, beta)).max() <= TOL


def test_encode_constant_queries_and_replication(gpu):
    torch, binding, dev = gpu
    alpha, beta = orc.chebyshev_nodes(12, 20)
    v = np.random.default_rng(8).uniform(0, 1, 512).astype(np.float32)
    X = np.broadcast_to(v, (2, 12, 512)).copy()
    coded = binding.approxifer_encode(torch.from_numpy(X).to(dev), alpha, beta).cpu().numpy()
    assert np.max(np.abs(coded - v)) <= 4e-7
    alpha, beta = orc.chebyshev_nodes(1, 4)
    coded = binding.approxifer_encode(torch.from_numpy(X[:, :1]).to(dev).contiguous(), alpha, beta).cpu().numpy()
    assert np.array_equal(coded, np.broadcast_to(v, (2, 4, 512)))


@pytest.mark.timeout(600)
def test_encode_cifar_full_size(gpu):
    torch, binding, dev = gpu
    w = syn.WORKLOADS["cifar"]
    alpha, beta = orc.chebyshev_nodes(w.K, w.W)
    X = syn.queries(w, threads=16)
    coded = binding.approxifer_encode(torch.from_numpy(X).to(dev), alpha, beta).cpu().numpy()
    worst = 0.0
    for g0 in range(0, w.G, 256):
        worst = max(worst, group_err(coded[g0:g0 + 256], orc.encode(X[g0:g0 + 256], alpha, beta)).max())
    assert worst <= TOL, worst


def _full_size_encode_sampled(gpu, name, sample):
    """Full-size launch (the configuration the benchmark times).  The groups in `sample` are compared
    element by element; every group is compared on a strided sample of feature columns that includes
    the first and last columns."""
    torch, binding, dev = gpu
    w = syn.WORKLOADS[name]
    alpha, beta = orc.chebyshev_nodes(w.K, w.W)
    X = syn.queries(w, threads=16)
    dX = torch.from_numpy(X).to(dev)
    coded = binding.approxifer_encode(dX, alpha, beta)
    torch.cuda.synchronize()
    for g in sample:
        ref = orc.encode(X[g:g + 1], alpha, beta)
        err = group_err(coded[g:g + 1].cpu().numpy(), ref)
        assert err.max() <= TOL, (g, err.max())
    # every group: a strided sample of feature columns (first, last, and a ragged stride)
    cols = np.unique(np.concatenate([np.arange(0, w.D, 4099), [w.D - 1, w.D - 2, 1]]))
    sub = coded[:, :, torch.from_numpy(cols).to(dev)].cpu().numpy()
    ref = orc.encode(X[:, :, cols], alpha, beta)
    err = group_err(sub, ref)
    assert err.max() <= TOL, err.max()


@pytest.mark.timeout(900)
def test_encode_imagenet_full_size_sampled(gpu):
    _full_size_encode_sampled(gpu, "imagenet", [0, 1, 255, 511])


@pytest.mark.timeout(900)
def test_encode_text_full_size_sampled(gpu):
    _full_size_encode_sampled(gpu, "text", [0, 513, 1023])


@pytest.mark.timeout(900)
def test_encode_text_k32_full_size_sampled(gpu):
    _full_size_encode_sampled(gpu, "text_k32", [0, 1023])


def _full_size_encode_every_element(gpu, name, chunk):
    """Full-size launch (the configuration the benchmark times), EVERY element of every group compared with the
    oracle, `chunk` groups at a time (the oracle's float64 copy of a chunk is what bounds host memory)."""
    import sys
    torch, binding, dev = gpu
    w = syn.WORKLOADS[name]
    alpha, beta = orc.chebyshev_nodes(w.K, w.W)
    dX = torch.empty((w.G, w.K, w.D), dtype=torch.float32, device=dev)
    for g0 in range(0, w.G, chunk):
        dX[g0:g0 + chunk] = torch.from_numpy(syn.queries(w, g0, min(g0 + chunk, w.G), threads=16)).to(dev)
    coded = binding.approxifer_encode(dX, alpha, beta)          # one launch over all G groups
    torch.cuda.synchronize()
    del dX
    worst = 0.0
    for g0 in range(0, w.G, chunk):
        g1 = min(g0 + chunk, w.G)
        ref = orc.encode(syn.queries(w, g0, g1, threads=16), alpha, beta)
        worst = max(worst, group_err(coded[g0:g1].cpu().numpy(), ref).max())
        print("%s encode: groups %d..%d of %d compared, worst %.3g" % (name, g0, g1, w.G, worst), flush=True)
        sys.stdout.flush()
        assert worst <= TOL, (g0, worst)


@pytest.mark.timeout(1200)
def test_encode_imagenet_full_size_every_element(gpu):
    _full_size_encode_every_element(gpu, "imagenet", 32)


@pytest.mark.timeout(1200)
def test_encode_text_full_size_every_element(gpu):
    _full_size_encode_every_element(gpu, "text", 64)


@pytest.mark.timeout(1200)
def test_encode_text_k32_full_size_every_element(gpu):
    _full_size_encode_every_element(gpu, "text_k32", 32)


# --------------------------------------------------------------------------------------
# decoder
# --------------------------------------------------------------------------------------
def _decode_both(gpu, Y, mask, alpha, beta, S, mode):
    torch, binding, dev = gpu
    out, st = binding.approxifer_decode(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta, S, mode)
    ref, st_ref = orc.decode(Y, mask, alpha, beta, S, mode)
    return out.cpu().numpy(), st.cpu().numpy(), ref, st_ref


@pytest.mark.parametrize("mode", [0, 1])
def test_decode_tiny_workload(gpu, mode):
    w = syn.WORKLOADS["tiny"]
    alpha, beta = orc.chebyshev_nodes(w.K, w.W)
    Y = syn.model_apply(w, syn.model_params(w), orc.encode(syn.queries(w), alpha, beta))
    out, st, ref, st_ref = _decode_both(gpu, Y, syn.masks(w), alpha, beta, w.S, mode)
    assert np.array_equal(st, st_ref) and np.all(st == 0)
    assert group_err(out, ref).max() <= TOL


@pytest.mark.parametrize("K,N,S,C,G", [
    (1, 2, 1, 1, 3), (2, 3, 1, 7, 4), (4, 9, 0, 260, 3), (5, 100, 10, 33, 2), (12, 20, 8, 1003, 2),
    (16, 24, 6, 2, 9), (32, 48, 12, 2, 5), (64, 128, 0, 12, 2), (64, 128, 60, 5, 2), (9, 70, 3, 516, 2),
    # the packed small-shape kernel at and just past its limits (K, survivors, classes <= 16, N <= 64)
    (16, 20, 4, 16, 9), (16, 64, 48, 16, 5), (16, 20, 3, 16, 5), (16, 20, 4, 17, 5), (13, 15, 2, 11, 131), (3, 64, 61, 1, 7),
    (1, 5, 4, 16, 6), (12, 13, 1, 10, 4099),
    # .. and its 32-survivor tile: 17 to 32 survivors, and one more
    (16, 24, 6, 2, 1031), (8, 24, 4, 10, 300), (16, 64, 32, 16, 9), (16, 40, 8, 16, 5), (3, 34, 2, 5, 70), (11, 18, 0, 13, 66),
    # .. and its (32 queries, 64 survivors) tile, two groups per workgroup
    (32, 48, 12, 2, 1025), (20, 30, 4, 4, 301), (32, 64, 0, 16, 7), (17, 40, 4, 9, 50), (8, 60, 4, 10, 21), (32, 34, 2, 16, 3),
])
@pytest.mark.parametrize("mode", [0, 1])
def test_decode_shapes(gpu, K, N, S, C, G, mode):
    rng = np.random.default_rng(K * 131 + N * 7 + S)
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        mask[g, rng.permutation(N)[: N - S]] = 1
    Y[mask == 0] = np.nan                                  # rows of stragglers must never be read
    out, st, ref, st_ref = _decode_both(gpu, Y, mask, alpha, beta, S, mode)
    assert np.all(st == 0) and np.array_equal(st, st_ref)
    assert np.all(np.isfinite(out))
    assert group_err(out, ref).max() <= TOL


@pytest.mark.parametrize("K,N,S,C,G", [(3, 6, 1, 280, 8300), (7, 12, 4, 132, 16500), (12, 20, 8, 1000, 4200),
                                       (16, 70, 10, 260, 8200), (9, 14, 0, 4 * 64 * 2 + 4, 5600)])
@pytest.mark.parametrize("mode", [0, 1])
def test_decode_streaming_kernel(gpu, K, N, S, C, G, mode):
    # 16-byte rows and K <= 16: one wave keeps all K accumulator rows; many groups, ragged last tiles, a rejected mask
    # and per-group straggler counts among the groups
    torch, binding, dev = gpu
    rng = np.random.default_rng(K * 977 + C)
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        mask[g, rng.permutation(N)[: N - S]] = 1
    mask[7, np.nonzero(mask[7])[0][0]] = 0                 # one survivor too few
    Y[mask == 0] = np.nan
    out = torch.full((G, K, C), -3.0, dtype=torch.float32, device=dev)
    Yd, md = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    _, st = binding.approxifer_decode(Yd, md, alpha, beta, S, mode, out=out)
    ref, st_ref = orc.decode(Y, mask, alpha, beta, S, mode)
    o, s = out.cpu().numpy(), st.cpu().numpy()
    assert np.array_equal(s, st_ref) and s[7] == 1 and s.sum() == 1
    assert np.all(o[7] == -3.0)
    good = s == 0                                          # every accepted group is compared: none of these seeds
    assert good.sum() == G - 1                             # draws a mask whose weights float64 cannot decide
    assert group_err(o[good], ref[good]).max() <= TOL
    # per-group straggler counts: the same masks, read off group by group
    out2, st2 = binding.approxifer_decode(Yd, md, alpha, beta, binding.S_FROM_MASK, mode)
    ref2, _ = orc.decode(Y[:64], mask[:64], alpha, beta, None, mode)
    assert np.all(st2.cpu().numpy() == 0)
    assert group_err(out2.cpu().numpy()[:64], ref2).max() <= TOL


@pytest.mark.parametrize("K,N,S,C,G,off_in,off_out", [
    (12, 20, 8, 1001, 3, 0, 0), (8, 12, 4, 101, 40, 1, 3), (5, 9, 2, 4 * 64 + 1, 7, 2, 1), (16, 70, 10, 4 * 64 * 2 + 3, 3, 3, 2),
    (7, 12, 4, 256, 9, 1, 1), (3, 6, 1, 5, 600, 0, 1), (20, 30, 4, 131, 5, 1, 2), (8, 12, 4, 4 * 130 + 2, 300, 0, 0),
])
def test_decode_rows_that_are_only_4_byte_aligned(gpu, K, N, S, C, G, off_in, off_out):
    # class counts that are not a multiple of four and/or offset tensors: 128-bit accesses through the 4-byte-aligned
    # vector type, the last partial vector of a row float by float; nothing outside the output tensor may be touched
    torch, binding, dev = gpu
    rng = np.random.default_rng(C * 7 + K)
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        mask[g, rng.permutation(N)[: N - S]] = 1
    Y[mask == 0] = np.nan
    flat_in = torch.zeros(G * N * C + off_in + 5, dtype=torch.float32, device=dev)
    flat_in[off_in:off_in + G * N * C] = torch.from_numpy(Y).to(dev).reshape(-1)
    flat_out = torch.full((G * K * C + off_out + 9,), -77.0, dtype=torch.float32, device=dev)
    preds = flat_in[off_in:off_in + G * N * C].view(G, N, C)
    out = flat_out[off_out:off_out + G * K * C].view(G, K, C)
    _, st = binding.approxifer_decode(preds, torch.from_numpy(mask).to(dev), alpha, beta, S, 1, out=out)
    ref, st_ref = orc.decode(Y, mask, alpha, beta, S, 1)
    assert np.array_equal(st.cpu().numpy(), st_ref) and np.all(st_ref == 0)
    assert group_err(out.cpu().numpy(), ref).max() <= TOL
    host = flat_out.cpu().numpy()
    assert np.all(host[:off_out] == -77.0) and np.all(host[off_out + G * K * C:] == -77.0)


def test_decode_bad_masks_leave_rows_untouched(gpu):
    torch, binding, dev = gpu
    K, N, S, C = 3, 7, 2, 40
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = np.random.default_rng(3).standard_normal((4, N, C)).astype(np.float32)
    mask = np.ones((4, N), np.uint8)
    mask[0, [1, 5]] = 0                    # good
    mask[1, [1]] = 0                       # one too many
    mask[2, [0, 1, 2]] = 0                 # one too few
    mask[3, [2, 6]] = 0
    mask[3, 0] = 200                       # any non-zero byte counts as returned
    out = torch.full((4, K, C), -5.0, dtype=torch.float32, device=dev)
    out, st = binding.approxifer_decode(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta, S,
                                        0, out=out)
    ref, st_ref = orc.decode(Y, mask, alpha, beta, S, 0)
    out = out.cpu().numpy()
    assert list(st.cpu().numpy()) == [0, 1, 1, 0] == list(st_ref)
    assert np.all(out[1] == -5.0) and np.all(out[2] == -5.0)
    assert group_err(out[[0, 3]], ref[[0, 3]]).max() <= TOL
    # status pointer may be NULL
    import ctypes
    a = np.ascontiguousarray(alpha); b = np.ascontiguousarray(beta)
    dp = ctypes.POINTER(ctypes.c_double)
    dY, dm = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    out2 = torch.zeros((4, K, C), dtype=torch.float32, device=dev)
    rc = binding.load().approxifer_decode(dY.data_ptr(), dm.data_ptr(), out2.data_ptr(), None, 4, K, N, S, C,
                                          a.ctypes.data_as(dp), b.ctypes.data_as(dp), 0,
                                          torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0 and group_err(out2.cpu().numpy()[[0, 3]], ref[[0, 3]]).max() <= TOL


@pytest.mark.parametrize("mode", [0, 1])
def test_decode_at_surviving_worker_nodes_returns_their_rows(gpu, mode):
    K, N, S, C = 4, 8, 3, 64
    _, beta = orc.chebyshev_nodes(K, N)
    F = [0, 2, 3, 6, 7]
    mask = np.zeros((2, N), np.uint8)
    mask[:, F] = 1
    Y = np.random.default_rng(4).standard_normal((2, N, C)).astype(np.float32)
    out, st, ref, _ = _decode_both(gpu, Y, mask, beta[F][:K], beta, S, mode)
    assert np.array_equal(out, Y[:, F[:K]])


def test_decode_ill_conditioned_worker_index_signs(gpu):
    # worker-index signs lose Berrut's alternation once workers are missing; search seeded masks for
    # the largest Lebesgue constants at the imagenet shape and decode exactly those groups
    K, N, S, C = 12, 20, 8, 96
    alpha, beta = orc.chebyshev_nodes(K, N)
    rng = np.random.default_rng(12)
    cands = []
    for _ in range(4000):
        F = np.sort(rng.permutation(N)[: N - S])
        leb = np.abs(orc.decode_weights(alpha, beta, F, 0)).sum(axis=1).max()
        cands.append((leb, tuple(F)))
    cands.sort(reverse=True)
    worst = cands[:32]
    assert worst[0][0] > 1e3
    mask = np.zeros((32, N), np.uint8)
    for g, (_, F) in enumerate(worst):
        mask[g, list(F)] = 1
    Y = (3 * rng.standard_normal((32, N, C))).astype(np.float32)
    out, st, ref, _ = _decode_both(gpu, Y, mask, alpha, beta, S, 0)
    assert np.all(st == 0)
    assert group_err(out, ref).max() <= TOL


@pytest.mark.timeout(600)
@pytest.mark.parametrize("mode", [0, 1])
def test_decode_cifar_full_size(gpu, mode):
    w = syn.WORKLOADS["cifar"]
    alpha, beta = orc.chebyshev_nodes(w.K, w.W)
    params = syn.model_params(w)
    Y = np.empty((w.G, w.W, w.C), np.float32)
    for g0 in range(0, w.G, 512):
        Y[g0:g0 + 512] = syn.model_apply(w, params, orc.encode(syn.queries(w, g0, g0 + 512, threads=16), alpha, beta))
    out, st, ref, st_ref = _decode_both(gpu, Y, syn.masks(w), alpha, beta, w.S, mode)
    assert np.all(st == 0) and np.array_equal(st, st_ref)
    assert group_err(out, ref).max() <= TOL


@pytest.mark.timeout(600)
@pytest.mark.parametrize("mode", [0, 1])
def test_decode_imagenet_full_size(gpu, mode):
    w = syn.WORKLOADS["imagenet"]
    alpha, beta = orc.chebyshev_nodes(w.K, w.W)
    Y = syn.iid_logits(w)
    out, st, ref, st_ref = _decode_both(gpu, Y, syn.masks(w), alpha, beta, w.S, mode)
    assert np.all(st == 0) and np.array_equal(st, st_ref)
    assert group_err(out, ref).max() <= TOL


@pytest.mark.timeout(600)
@pytest.mark.parametrize("name", ["text", "text_k32"])
def test_decode_text_full_size(gpu, name):
    # the hosted model here is mean-pool + linear, an affine map, so f(coded query) equals the
    # oracle's encoding of the pooled queries (the basis functions sum to one); the pooled tensor
    # is 128 times smaller than the queries, which keeps this test's host work small
    w = syn.WORKLOADS[name]
    alpha, beta = orc.chebyshev_nodes(w.K, w.W)
    params = syn.model_params(w)
    T, E = w.query_shape
    small = syn.scaled(w, query_shape=(1, E))
    pooled = syn.queries(small, threads=16)                                  # stands for the token mean
    Y = syn.model_apply(small, params, orc.encode(pooled, alpha, beta))
    for mode in (0, 1):
        out, st, ref, st_ref = _decode_both(gpu, Y, syn.masks(w), alpha, beta, w.S, mode)
        assert np.all(st == 0) and np.array_equal(st, st_ref)
        assert group_err(out, ref).max() <= TOL


# --------------------------------------------------------------------------------------
# fused decoder + top-1
# --------------------------------------------------------------------------------------
def _top1_both(gpu, Y, mask, alpha, beta, S, mode):
    torch, binding, dev = gpu
    top1, score, st = binding.approxifer_decode_top1(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev),
                                                     alpha, beta, S, mode)
    ref_top1, ref_score, st_ref = orc.decode_top1(Y, mask, alpha, beta, S, mode)
    return top1.cpu().numpy(), score.cpu().numpy(), st.cpu().numpy(), ref_top1, ref_score, st_ref


def _assert_top1(Y, mask, alpha, beta, S, mode, top1, score, st, ref_top1, ref_score, st_ref):
    assert np.array_equal(st, st_ref)
    good = st_ref == 0
    # both sides take the decision on float64 values; where the oracle's top two are further apart than
    # float64 rounding of the contraction can explain the indices must be identical
    out, _ = orc.decode(Y, mask, alpha, beta, S, mode)
    top2 = np.sort(out, axis=-1)[..., -2:] if out.shape[-1] > 1 else np.stack([out[..., 0] - 1, out[..., 0]], -1)
    clear = ((top2[..., 1] - top2[..., 0]) > 1e-9 * np.abs(out).max(axis=-1)) & good[:, None]
    assert np.array_equal(top1[clear], ref_top1[clear])
    assert clear[good].mean() > 0.999
    same = (top1 == ref_top1) & good[:, None]
    scale = np.abs(ref_score[good]).max()
    assert np.max(np.abs(score[same] - ref_score[same])) <= TOL * scale


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("name", ["tiny", "imagenet"])
def test_decode_top1_workloads(gpu, name, mode):
    w = syn.WORKLOADS[name]
    alpha, beta = orc.chebyshev_nodes(w.K, w.W)
    if name == "tiny":
        Y = syn.model_apply(w, syn.model_params(w), orc.encode(syn.queries(w), alpha, beta))
    else:
        Y = syn.iid_logits(w)
    mask = syn.masks(w)
    _assert_top1(Y, mask, alpha, beta, w.S, mode, *_top1_both(gpu, Y, mask, alpha, beta, w.S, mode))


@pytest.mark.parametrize("K,N,S,C,G", [(1, 2, 1, 1, 3), (2, 3, 1, 7, 4), (5, 100, 10, 33, 2), (12, 20, 8, 1003, 2),
                                       (16, 20, 4, 16, 9), (16, 64, 48, 16, 5), (13, 15, 2, 11, 131), (8, 9, 1, 10, 1030),
                                       (32, 48, 12, 2, 5), (64, 128, 0, 12, 2), (9, 70, 3, 516, 2), (8, 9, 1, 10, 300),
                                       (16, 24, 6, 2, 300), (8, 24, 4, 10, 131), (16, 64, 32, 16, 9), (16, 40, 7, 16, 5),
                                       (32, 48, 12, 2, 300), (20, 30, 4, 4, 301), (32, 64, 0, 16, 7), (17, 40, 3, 9, 50), (8, 60, 4, 10, 21),
                                       # few groups, thousands of classes: one workgroup per quad of queries
                                       (8, 12, 4, 5000, 3), (5, 9, 2, 4099, 2), (12, 20, 8, 20004, 2), (30, 40, 6, 4100, 2)])
def test_decode_top1_shapes_and_bad_masks(gpu, K, N, S, C, G):
    torch, binding, dev = gpu
    rng = np.random.default_rng(K + 3 * N + S)
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        mask[g, rng.permutation(N)[: N - S]] = 1
    if S > 0:
        mask[G - 1, np.nonzero(mask[G - 1] == 0)[0][0]] = 1          # one survivor too many in the last group
    Y[mask == 0] = np.nan
    top1 = torch.full((G, K), -9, dtype=torch.int32, device=dev)
    score = torch.full((G, K), -9.0, dtype=torch.float32, device=dev)
    t, sc, st = binding.approxifer_decode_top1(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta,
                                               S, 1, top1=top1, score=score)
    ref = orc.decode_top1(Y, mask, alpha, beta, S, 1)
    t, sc, st = t.cpu().numpy(), sc.cpu().numpy(), st.cpu().numpy()
    _assert_top1(Y, mask, alpha, beta, S, 1, t, sc, st, *ref)
    if S > 0:
        assert st[G - 1] == 1 and np.all(t[G - 1] == -9) and np.all(sc[G - 1] == -9.0)
    # score pointer may be NULL
    t2, none, _ = binding.approxifer_decode_top1(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta,
                                                 S, 1, want_score=False)
    assert none is None and np.array_equal(t2.cpu().numpy()[st == 0], t[st == 0])


def test_decode_top1_exact_ties_take_smallest_class(gpu):
    K, N, C = 4, 6, 12
    alpha, beta = orc.chebyshev_nodes(K, N)
    rng = np.random.default_rng(2)
    base = rng.standard_normal((3, N, 1)).astype(np.float32)
    Y = np.repeat(base, C, axis=2)                       # every class column identical -> all decoded values tie
    Y[..., 7] += 2.0
    Y[..., 9] = Y[..., 7]                                # classes 7 and 9 tie
    mask = np.ones((3, N), np.uint8)
    top1, score, st, ref_top1, ref_score, _ = _top1_both(gpu, Y, mask, alpha, beta, 0, 0)
    assert np.array_equal(top1, ref_top1)
    assert set(np.unique(top1)) <= {0, 7}


@pytest.mark.parametrize("K,N,S,C,exact", [
    (8, 9, 1, 1, True), (8, 9, 1, 2, True), (12, 28, 2, 10, True), (17, 33, -1, 15, True), (4, 12, 4, 16, True),
    (8, 12, 4, 17, True), (12, 20, 8, 100, True), (16, 24, -1, 1283, True),
    (8, 70, 10, 40, False), (20, 30, 2, 40, False),       # the kernels for more workers or more queries
])
def test_decode_top1_of_predictions_that_are_not_numbers(gpu, K, N, S, C, exact):
    # A worker that answered may return NaN or infinities, in every class or in some: the answer is a class all the same.
    # NaN never wins; a query without any value above -inf gets class 0.  The rule is applied to what approxifer_decode
    # makes of the same predictions (`exact` off: a row of NaN and -inf only may also give the first -inf).
    torch, binding, dev = gpu
    G = 48
    rng = np.random.default_rng(1000 * K + C)
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        late = S if S >= 0 else int(rng.integers(0, N - 1))
        order = rng.permutation(N)
        mask[g, order[late:]] = 1
        w = order[late]                                   # it answered
        kind = g % 8
        some = rng.permutation(C)[: (C + 1) // 2]
        if kind == 0:
            Y[g, w] = np.nan
        elif kind == 1:
            Y[g, w, some] = np.nan
        elif kind == 2:
            Y[g, w] = -np.inf
        elif kind == 3:
            Y[g, w] = np.inf
        elif kind == 4:
            Y[g, w], Y[g, w, some] = -np.inf, np.nan
        elif kind == 5:
            Y[g, w], Y[g, w, some] = np.inf, np.nan
        elif kind == 6:
            Y[g, w, some] = -np.inf
        else:
            Y[g, w, 0] = np.nan
    Yd, md = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    out, st = binding.approxifer_decode(Yd, md, alpha, beta, S, 1)
    top1, score, st1 = binding.approxifer_decode_top1(Yd, md, alpha, beta, S, 1)
    out, st, top1, score, st1 = (t.cpu().numpy() for t in (out, st, top1, score, st1))
    assert np.all(st == 0) and np.all(st1 == 0)
    assert np.all((top1 >= 0) & (top1 < C))
    above = out > -np.inf                                 # False for NaN
    none = ~above.any(-1)
    assert none.any() and (C == 1 or (~none).any())
    ranked = np.where(above, out.astype(np.float64), -np.inf)
    best = ranked.argmax(-1)
    srt = np.sort(ranked, axis=-1)
    with np.errstate(invalid="ignore"):
        clear = np.ones(none.shape, bool) if C == 1 else ~(srt[..., -1] - srt[..., -2] <= 1e-6 * np.abs(srt[..., -1]))
    clear |= np.isinf(srt[..., -1])                       # equal infinities: the first
    pick = clear & ~none
    assert np.array_equal(top1[pick], best[pick])
    assert np.array_equal(score[pick], ranked.max(-1)[pick].astype(np.float32))
    only_nan = np.isnan(out).all(-1)
    assert np.all(top1[none if exact else only_nan] == 0)
    assert not np.any(score[none] > -np.inf)


@pytest.mark.parametrize("K,N,S,C,G", [
    (8, 12, 4, 100, 2048), (8, 12, 4, 100, 2047), (8, 12, 4, 104, 2048),     # short rows: from 2048 groups on
    (16, 24, -1, 40, 2050), (6, 9, 2, 20, 2100),
    (4, 7, 1, 77, 8192), (6, 9, -1, 78, 5462), (8, 9, 1, 79, 4095),          # rows that are only 4-byte aligned
    (10, 17, 7, 256, 256), (10, 17, 7, 256, 255), (15, 21, 6, 192, 400),     # K = 9..16: from 1024 tiles on
    (12, 20, 8, 1000, 512), (12, 20, 8, 1000, 513), (14, 25, 11, 108, 600),  # .. up to 8192
])
def test_decode_tiles_on_both_sides_of_their_rule(gpu, K, N, S, C, G):
    # Query nodes that are worker nodes (6 of 9, 10 of 17, 15 of 21, ..), straggler counts off the masks, groups without
    # any answer and with one too many; answers that did not come hold NaN.  Forty groups and the last against the oracle.
    torch, binding, dev = gpu
    rng = np.random.default_rng(7 * K + C + G)
    alpha, beta = orc.chebyshev_nodes(K, N)
    order = rng.random((G, N)).argsort(1).argsort(1)
    late = np.full((G, 1), S) if S >= 0 else rng.integers(0, N - 1, (G, 1))
    mask = (order >= late).astype(np.uint8)
    mask[1] = 0
    if S > 0:
        mask[2] = 1
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    poisoned = np.where(mask[:, :, None] != 0, Y, np.float32(np.nan))
    out = torch.full((G, K, C), -3.0, dtype=torch.float32, device=dev)
    out, st = binding.approxifer_decode(torch.from_numpy(poisoned).to(dev), torch.from_numpy(mask).to(dev), alpha, beta, S, 1, out=out)
    out, st = out.cpu().numpy(), st.cpu().numpy()
    some = np.unique(np.concatenate([[0, 1, 2, 3, G - 1], rng.integers(0, G, 36)]))
    ref, st_ref = orc.decode(Y[some], mask[some], alpha, beta, S, 1)
    assert np.array_equal(st[some], st_ref) and st[1] == 1 and (S <= 0 or st[2] == 1)
    good = st_ref == 0
    assert np.all(out[some][~good] == -3.0) and np.isfinite(out[st == 0]).all()
    assert group_err(out[some][good], ref[good]).max() <= TOL


@pytest.mark.parametrize("K,N,S,C,G", [
    (8, 12, 4, 1100, 40), (10, 17, 7, 1283, 33), (16, 24, -1, 1283, 21),     # tiles: a second pass over the columns
    (15, 21, 6, 68, 70), (6, 9, -1, 19, 90), (3, 6, 1, 126, 50),
    (4, 7, 1, 130, 60), (4, 7, 1, 132, 60), (3, 5, 2, 750, 90),              # K <= 4: 4-byte rows longer than 128 leave the tiles
    (7, 13, 6, 133, 4095), (7, 13, 6, 133, 4096),
])
def test_decode_top1_tiles_on_both_sides_of_their_rule(gpu, K, N, S, C, G):
    torch, binding, dev = gpu
    rng = np.random.default_rng(11 * K + C + G)
    alpha, beta = orc.chebyshev_nodes(K, N)
    order = rng.random((G, N)).argsort(1).argsort(1)
    late = np.full((G, 1), S) if S >= 0 else rng.integers(0, N - 1, (G, 1))
    mask = (order >= late).astype(np.uint8)
    mask[1] = 0
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    Y[0, mask[0].nonzero()[0], C - 1] += 50.0             # the last class wins: every survivor says so
    poisoned = np.where(mask[:, :, None] != 0, Y, np.float32(np.nan))
    top1, score, st = binding.approxifer_decode_top1(torch.from_numpy(poisoned).to(dev), torch.from_numpy(mask).to(dev), alpha, beta, S, 1)
    top1, score, st = (t.cpu().numpy() for t in (top1, score, st))
    some = np.unique(np.concatenate([[0, 1, 2, G - 1], rng.integers(0, G, 36)]))
    ref = orc.decode_top1(Y[some], mask[some], alpha, beta, S, 1)
    assert st[1] == 1 and np.all(top1[1] == -1) and np.all(top1[0] == C - 1)
    _assert_top1(Y[some], mask[some], alpha, beta, S, 1, top1[some], score[some], st[some], *ref)


@pytest.mark.parametrize("K,N,S,C", [(2, 3, 1, 10), (4, 7, 1, 16), (7, 13, 3, 1), (8, 9, 1, 10), (10, 17, -1, 10), (12, 28, 4, 3),
                                     (16, 33, 0, 2), (20, 41, 21, 5), (32, 64, 12, 2)])
def test_decode_small_classes_four_rows_or_one_to_a_group(gpu, K, N, S, C):
    # Up to 2048 groups a group's queries are split over four rows of lanes: the same bits either way.
    torch, binding, dev = gpu
    G = 2300
    rng = np.random.default_rng(K * N + C)
    alpha, beta = orc.chebyshev_nodes(K, N)
    order = rng.random((G, N)).argsort(1).argsort(1)
    late = np.full((G, 1), S) if S >= 0 else rng.integers(0, N - 1, (G, 1))
    mask = (order >= late).astype(np.uint8)
    mask[3] = 0
    Y = np.where(mask[:, :, None] != 0, rng.standard_normal((G, N, C)), np.nan).astype(np.float32)
    Yd, md = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    whole = binding.approxifer_decode(Yd, md, alpha, beta, S, 1) + binding.approxifer_decode_top1(Yd, md, alpha, beta, S, 1)
    for n in (1, 2048):
        part = binding.approxifer_decode(Yd[:n], md[:n], alpha, beta, S, 1) + binding.approxifer_decode_top1(Yd[:n], md[:n], alpha, beta, S, 1)
        for a, b in zip(whole, part):
            assert np.array_equal(a[:n].cpu().numpy(), b.cpu().numpy())
    assert whole[1][3] == 1 and torch.all(whole[1][torch.arange(G, device=dev) != 3] == 0)


@pytest.mark.parametrize("K,N,S,C,G", [(6, 9, 2, 10, 40), (15, 21, -1, 16, 2100), (6, 9, 2, 20, 2100), (10, 17, 7, 256, 256),
                                       (13, 27, 11, 192, 400), (6, 9, 1, 77, 5500)])
def test_decode_query_on_an_answered_workers_node_is_that_workers_row(gpu, K, N, S, C, G):
    # .. bit for bit, and whatever the other workers returned: one of them returns NaN and infinities.
    torch, binding, dev = gpu
    rng = np.random.default_rng(K * N + C)
    alpha, beta = orc.chebyshev_nodes(K, N)
    j_of, w_of = np.nonzero(alpha[:, None] == beta[None, :])
    assert len(j_of) > 0
    order = rng.random((G, N)).argsort(1).argsort(1)
    late = np.full((G, 1), S) if S >= 0 else rng.integers(0, N - 2, (G, 1))
    mask = (order >= late).astype(np.uint8)
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    other = int([w for w in range(N) if w not in set(w_of)][0])
    Y[:, other, 0::3] = np.nan
    Y[:, other, 1::3] = np.inf
    out, st = binding.approxifer_decode(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta, S, 1)
    top1, score, _ = binding.approxifer_decode_top1(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta, S, 1)
    out, top1, score = out.cpu().numpy(), top1.cpu().numpy(), score.cpu().numpy()
    assert torch.all(st == 0)
    for j, w in zip(j_of, w_of):
        came = mask[:, w] != 0
        assert came.any()
        assert np.array_equal(out[came, j], Y[came, w])
        assert np.array_equal(top1[came, j], Y[came, w].argmax(-1)) and np.array_equal(score[came, j], Y[came, w].max(-1))


@pytest.mark.parametrize("K,N,S,C,few,many", [(17, 18, 0, 50, 5, 450), (20, 41, 3, 50, 5, 450), (33, 34, 1, 90, 5, 450),
                                              (27, 28, 0, 130, 5, 300)])
def test_decode_beyond_sixteen_queries_is_the_same_in_calls_of_every_size(gpu, K, N, S, C, few, many):
    # A query on an answered worker's node, while another worker returns NaN and infinities: a group's values and classes do
    # not depend on how many groups the call has, nor on whether the classes are decided with the decoding or after it.
    torch, binding, dev = gpu
    rng = np.random.default_rng(K * N)
    alpha, beta = orc.chebyshev_nodes(K, N)
    if not np.isin(alpha, beta).any():
        beta[N // 2] = alpha[K // 2]
    mask = np.ones((many, N), np.uint8)
    mask[:, 1:1 + S] = 0
    Y = rng.standard_normal((many, N, C)).astype(np.float32)
    Y[:, N - 1, 0::3] = np.nan
    Y[:, N - 1, 1::3] = np.inf
    Yd, md = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    whole = binding.approxifer_decode(Yd, md, alpha, beta, S, 1)[0]
    part = binding.approxifer_decode(Yd[:few], md[:few], alpha, beta, S, 1)[0]
    # one rounding to float32 each, float64 sums before it
    assert torch.allclose(whole[:few], part, rtol=2.0 ** -23, atol=1e-12 * 10, equal_nan=True)
    for values in (whole, part):
        fused = binding.approxifer_decode_top1(Yd[:len(values)], md[:len(values)], alpha, beta, S, 1)
        after = binding.approxifer_top1(values)
        assert torch.equal(fused[0], after[0])
        assert torch.allclose(fused[1], after[1], rtol=2.0 ** -23, atol=1e-12 * 10)


@pytest.mark.parametrize("K,N,S,C,few,many", [
    (10, 17, 7, 1027, 400, 800), (9, 14, 0, 253, 500, 1039), (11, 16, 2, 130, 2000, 2100), (13, 15, 1, 301, 20, 2500),
    (21, 31, 2, 35, 3, 401), (24, 26, 1, 63, 3, 401), (26, 29, 0, 33, 5, 420), (18, 20, 2, 70, 5, 420),
])
def test_decode_is_the_same_in_calls_of_every_size(gpu, K, N, S, C, few, many):
    # the number of groups decides which kernel decodes them
    torch, binding, dev = gpu
    alpha, beta = orc.chebyshev_nodes(K, N)
    gen = torch.Generator(device=dev).manual_seed(K * C)
    Y = torch.randn((many, N, C), generator=gen, device=dev)
    mask = (torch.rand((many, N), generator=gen, device=dev).argsort(1).argsort(1) >= S).to(torch.uint8)
    whole, status = binding.approxifer_decode(Y, mask, alpha, beta, S, 1)
    part, _ = binding.approxifer_decode(Y[:few].clone(), mask[:few].clone(), alpha, beta, S, 1)
    assert torch.all(status == 0)
    # one rounding to float32 each, float64 sums before it
    assert torch.allclose(whole[:few], part, rtol=2.0 ** -23, atol=1e-12 * 10)
    some = [0, few - 1, many - 1]
    ref, _ = orc.decode(Y[some].cpu().numpy(), mask[some].cpu().numpy(), alpha, beta, S, 1)
    assert np.all(np.abs(whole[some].cpu().numpy() - ref) <= 2.0 ** -24 * np.abs(ref) + 1e-12 * 10)


@pytest.mark.parametrize("K,N,S,C,few,many", [
    (12, 16, 2, 1000, 200, 520), (12, 16, 0, 1000, 300, 1030), (10, 40, 2, 404, 250, 300), (10, 34, 0, 404, 700, 1030),
    (16, 20, 1, 96, 1700, 1720), (14, 15, 1, 250, 1000, 1030), (21, 24, 1, 1903, 40, 50), (36, 40, 0, 1100, 50, 60),
    (40, 44, 2, 50, 250, 520), (36, 45, 2, 360, 200, 300), (50, 60, 2, 18, 700, 1030), (20, 26, 0, 33, 500, 600),
])
def test_class_decision_is_the_same_in_calls_of_every_size(gpu, K, N, S, C, few, many):
    # the number of groups decides which kernel decides the classes, and with how many waves to a group
    torch, binding, dev = gpu
    alpha, beta = orc.chebyshev_nodes(K, N)
    gen = torch.Generator(device=dev).manual_seed(K * C)
    Y = torch.randn((many, N, C), generator=gen, device=dev)
    Y[:, :, 7] = Y[:, :, 11] = 50.0 * (torch.arange(many, device=dev) % 2)[:, None]     # ties in every other group
    mask = (torch.rand((many, N), generator=gen, device=dev).argsort(1).argsort(1) >= S).to(torch.uint8)
    whole = binding.approxifer_decode_top1(Y, mask, alpha, beta, S, 1)
    part = binding.approxifer_decode_top1(Y[:few].clone(), mask[:few].clone(), alpha, beta, S, 1)
    assert torch.all(whole[2] == 0) and torch.all(whole[0][1::2] == 7)
    assert torch.equal(whole[0][:few], part[0])
    assert torch.allclose(whole[1][:few], part[1], rtol=2.0 ** -23, atol=1e-12 * 50)    # float64 sums, rounded once
    some = [0, few - 1, many - 1]
    ref, _ = orc.decode(Y[some].cpu().numpy(), mask[some].cpu().numpy(), alpha, beta, S, 1)
    top = ref.max(axis=2)
    assert np.all(np.abs(whole[1][some].cpu().numpy() - top) <= 2.0 ** -24 * np.abs(top) + 1e-12 * 50)


# --------------------------------------------------------------------------------------
# Byzantine decoder
# --------------------------------------------------------------------------------------
def _byzantine_inputs(w):
    alpha, beta = orc.chebyshev_nodes(w.K, w.W)
    params = syn.model_params(w)
    clean = np.empty((w.G, w.W, w.C), np.float32)
    for g0 in range(0, w.G, 512):
        g1 = min(g0 + 512, w.G)
        clean[g0:g1] = syn.model_apply(w, params, orc.encode(syn.queries(w, g0, g1, threads=16), alpha, beta))
    mask = syn.masks(w)
    adv_true = syn.adversaries(w, mask)
    return alpha, beta, syn.corrupt(w, clean, adv_true), mask, adv_true


def _byz_both(gpu, Y, mask, alpha, beta, S, A, mode=0):
    torch, binding, dev = gpu
    out, adv, st = binding.approxifer_decode_byzantine(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev),
                                                       alpha, beta, S, A, mode)
    ref, adv_ref, st_ref = orc.decode_byzantine(Y, mask, alpha, beta, S, A, mode)
    return out.cpu().numpy(), adv.cpu().numpy(), st.cpu().numpy(), ref, adv_ref, st_ref


@pytest.mark.timeout(600)
def test_byzantine_workload_full_size(gpu):
    w = syn.WORKLOADS["byzantine"]
    alpha, beta, Y, mask, adv_true = _byzantine_inputs(w)
    out, adv, st, ref, adv_ref, st_ref = _byz_both(gpu, Y, mask, alpha, beta, w.S, w.A)
    assert np.all(st == 0) and np.array_equal(st, st_ref)
    assert adv.dtype == np.int32 and np.array_equal(adv, adv_ref)          # bit-exact index sets
    assert np.array_equal(adv, adv_true)                                   # and they are the planted ones
    assert group_err(out, ref).max() <= TOL


@pytest.mark.parametrize("K,A,S,N,C,G", [
    (2, 1, 0, 6, 3, 16), (3, 2, 2, 12, 10, 16), (12, 1, 0, 26, 10, 8), (12, 2, 0, 28, 10, 8), (12, 3, 0, 30, 10, 8),
    (8, 2, 6, 26, 10, 8), (8, 2, 4, 24, 1000, 3), (8, 2, 0, 64, 6, 3), (16, 4, 0, 40, 4, 4), (4, 1, 3, 13, 17, 8),
    # every register-tile size of the projected kernel, odd numbers of available workers, K + A = 16, one class
    (2, 1, 0, 22, 5, 8), (8, 2, 0, 40, 7, 6), (13, 3, 1, 33, 3, 4), (3, 1, 0, 9, 6, 8), (5, 2, 2, 23, 4, 8),
    (1, 1, 0, 48, 2, 4), (6, 1, 0, 14, 1, 16), (14, 2, 0, 48, 9, 3), (9, 1, 5, 54, 12, 3), (15, 2, 0, 36, 4, 3),
    # class tiles of 32 and 64, several tiles with a ragged last one, many groups (one wave per group)
    (8, 2, 4, 24, 20, 6), (8, 2, 4, 24, 40, 6), (5, 1, 0, 12, 150, 4), (3, 1, 1, 9, 6, 4200),
])
def test_byzantine_exactly_rational_predictions(gpu, K, A, S, N, C, G):
    # a linear hosted model makes the coded predictions exactly rational in beta (Theorem 1): the
    # planted adversaries must come back, identical to the oracle's
    rng = np.random.default_rng(K * 100 + A * 10 + S)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, 96))
    Mf = rng.standard_normal((96, C)) / 10
    clean = (orc.encode(X, alpha, beta) @ Mf).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    adv_true = np.zeros((G, A), np.int32)
    Y = clean.copy()
    for g in range(G):
        avail = np.sort(rng.permutation(N)[: N - S])
        mask[g, avail] = 1
        ok = avail[np.abs(beta[avail]) > 1e-9]             # a node equal to 0 cannot be located (Q(0) = 1)
        adv_true[g] = np.sort(rng.permutation(ok)[:A])
        Y[g, adv_true[g]] += (10 * clean.std() * rng.standard_normal((A, C))).astype(np.float32)
    out, adv, st, ref, adv_ref, st_ref = _byz_both(gpu, Y, mask, alpha, beta, S, A)
    assert np.all(st == 0)
    assert np.array_equal(adv, adv_ref)
    if K + A <= 16:                                        # beyond that float32-rounded data no longer separates cleanly
        assert np.array_equal(adv, adv_true)
    assert group_err(out, ref).max() <= TOL


@pytest.mark.parametrize("locator", [2, 1])
@pytest.mark.parametrize("K,A,N,C,G", [(8, 2, 24, 1000, 5), (12, 2, 30, 257, 6), (4, 1, 12, 4003, 3), (2, 1, 8, 20001, 2),
                                       (8, 2, 60, 300, 3)])
def test_byzantine_many_classes_few_groups(gpu, K, A, N, C, G, locator):
    # with few groups and many classes several workgroups share a group and meet through atomics in the caller's
    # workspace (all three kernels: the last shape has up to 60 available workers, Algorithm 2's LDS kernel):
    # per-group straggler counts, a rejected mask among the groups (its rows and located workers must stay
    # untouched), twice in a row on the same buffers
    torch, binding, dev = gpu
    entry = binding.approxifer_decode_byzantine if locator == 2 else binding.approxifer_decode_byzantine_homogeneous
    rng = np.random.default_rng(K * 1000 + C)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, 40))
    clean = (orc.encode(X, alpha, beta) @ (rng.standard_normal((40, C)) / 6)).astype(np.float32)
    M = K + A
    mask = np.zeros((G, N), np.uint8)
    Y = clean.copy()
    adv_true = np.full((G, A), -7, np.int32)
    for g in range(G):
        cnt = 2 * M - 1 if g == 1 else int(rng.integers(2 * M, N + 1))     # group 1: one worker too few
        avail = np.sort(rng.permutation(N)[:cnt])
        mask[g, avail] = 1
        if g != 1:
            ok = avail[np.abs(beta[avail]) > 1e-9]
            adv_true[g] = np.sort(rng.permutation(ok)[:A])
            Y[g, adv_true[g]] += (10 * clean.std() * rng.standard_normal((A, C))).astype(np.float32)
    ref, adv_ref, st_ref = orc.decode_byzantine(Y, mask, alpha, beta, None, A, 1, locator)
    out = torch.full((G, K, C), -3.0, dtype=torch.float32, device=dev)
    adv = torch.full((G, A), -7, dtype=torch.int32, device=dev)
    Yd, md = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    for _ in range(2):
        _, _, st = entry(Yd, md, alpha, beta, binding.S_FROM_MASK, A, 1, out=out, adv=adv)
        o, a, s = out.cpu().numpy(), adv.cpu().numpy(), st.cpu().numpy()
        assert np.array_equal(s, st_ref) and s[1] == 1 and s.sum() == 1
        assert np.all(o[1] == -3.0) and np.all(a[1] == -7)
        good = s == 0
        assert np.array_equal(a[good], adv_ref[good]) and np.array_equal(a[good], adv_true[good])
        assert group_err(o[good], ref[good]).max() <= TOL


@pytest.mark.parametrize("entry", ["approxifer_decode_byzantine", "approxifer_decode_byzantine_homogeneous"])
@pytest.mark.parametrize("K,A,N,C,G", [(8, 2, 24, 1000, 5), (3, 1, 10, 4003, 3), (8, 2, 60, 300, 3)])
def test_byzantine_workspace_through_the_c_abi(gpu, entry, K, A, N, C, G):
    # the raw C ABI with a workspace of the size approxifer_workspace_bytes() gives: the classes of a group are spread
    # over several workgroups that meet there.  The workspace and every output sit between canaries; the workspace
    # arrives full of garbage; output rows of a rejected group keep their contents.  Then the same call with
    # NULL / 0, with a workspace one byte short, and with a misaligned one: one workgroup per group, and the same
    # bits in every output.
    import ctypes
    torch, binding, dev = gpu
    lib = binding.load()
    rng = np.random.default_rng(K * 31 + C)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, 40))
    clean = (orc.encode(X, alpha, beta) @ (rng.standard_normal((40, C)) / 6)).astype(np.float32)
    M = K + A
    mask = np.zeros((G, N), np.uint8)
    Y = clean.copy()
    for g in range(G):
        cnt = 2 * M - 1 if g == 1 else int(rng.integers(2 * M, N + 1))     # group 1: one worker too few
        avail = np.sort(rng.permutation(N)[:cnt])
        mask[g, avail] = 1
        ok = avail[np.abs(beta[avail]) > 1e-9]
        bad = np.sort(rng.permutation(ok)[:A])
        Y[g, bad] += (10 * clean.std() * rng.standard_normal((A, C))).astype(np.float32)
    locator = orc.LOCATOR_ALGORITHM_2 if entry == "approxifer_decode_byzantine" else orc.LOCATOR_ALGORITHM_1
    ref, adv_ref, st_ref = orc.decode_byzantine(Y, mask, alpha, beta, None, A, 1, locator)
    need = binding.approxifer_workspace_bytes(G, K, N, binding.S_FROM_MASK, A, C)
    assert need >= 4 * (N + 1) * G                               # these shapes are shared between workgroups
    dp = ctypes.POINTER(ctypes.c_double)
    a64, b64 = np.ascontiguousarray(alpha), np.ascontiguousarray(beta)
    Yd, md = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    pad = 64

    def framed(n_elems, dtype, fill):
        buf = torch.full((n_elems + 2 * pad,), fill, dtype=dtype, device=dev)
        return buf, buf[pad:pad + n_elems]

    def call(ws_ptr, ws_bytes):
        out_buf, out = framed(G * K * C, torch.float32, -3.0)
        adv_buf, adv = framed(G * A, torch.int32, -7)
        st_buf, st = framed(G, torch.int32, -9)
        rc = getattr(lib, entry)(Yd.data_ptr(), md.data_ptr(), out.data_ptr(), adv.data_ptr(), st.data_ptr(), G, K, N,
                                 binding.S_FROM_MASK, A, C, a64.ctypes.data_as(dp), b64.ctypes.data_as(dp), 1,
                                 ws_ptr, ctypes.c_size_t(ws_bytes), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert rc == 0
        for buf, fill in ((out_buf, -3.0), (adv_buf, -7), (st_buf, -9)):
            assert torch.all(buf[:pad] == fill) and torch.all(buf[-pad:] == fill)
        return out.view(G, K, C).cpu().numpy(), adv.view(G, A).cpu().numpy(), st.cpu().numpy()

    ws_buf = torch.randint(-2 ** 31, 2 ** 31 - 1, (need // 4 + 2 * pad,), dtype=torch.int32, device=dev)
    before = ws_buf.clone()
    ws = ws_buf[pad:pad + need // 4]
    o, a, s = call(ws.data_ptr(), need)
    assert torch.equal(ws_buf[:pad], before[:pad]) and torch.equal(ws_buf[-pad:], before[-pad:])
    assert np.array_equal(s, st_ref) and s[1] == 1 and s.sum() == 1
    assert np.all(o[1] == -3.0) and np.all(a[1] == -7)
    good = s == 0
    assert np.array_equal(a[good], adv_ref[good])
    assert group_err(o[good], ref[good]).max() <= TOL
    o2, a2, s2 = call(ws.data_ptr(), need)                      # again, on the workspace the first call left behind
    assert np.array_equal(o2, o) and np.array_equal(a2, a) and np.array_equal(s2, s)
    for ptr, nbytes in ((None, 0), (ws.data_ptr(), 4 * (N + 1) * G - 1), (ws.data_ptr() + 1, need - 1), (None, need)):
        o3, a3, s3 = call(ptr, nbytes)
        assert np.array_equal(o3, o) and np.array_equal(a3, a) and np.array_equal(s3, s)


@pytest.mark.parametrize("mode", [0, 1])
def test_byzantine_sign_modes_and_bad_masks(gpu, mode):
    torch, binding, dev = gpu
    w = syn.scaled(syn.WORKLOADS["byzantine"], G=64)
    alpha, beta, Y, mask, adv_true = _byzantine_inputs(w)
    mask[5, np.nonzero(mask[5])[0][0]] = 0                 # one survivor too few
    mask[9, np.nonzero(mask[9] == 0)[0][0]] = 1            # one too many
    out = torch.full((w.G, w.K, w.C), -3.0, dtype=torch.float32, device=dev)
    adv = torch.full((w.G, w.A), -7, dtype=torch.int32, device=dev)
    out, adv, st = binding.approxifer_decode_byzantine(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev),
                                                       alpha, beta, w.S, w.A, mode, out=out, adv=adv)
    ref, adv_ref, st_ref = orc.decode_byzantine(Y, mask, alpha, beta, w.S, w.A, mode)
    out, adv, st = out.cpu().numpy(), adv.cpu().numpy(), st.cpu().numpy()
    assert np.array_equal(st, st_ref) and st[5] == 1 and st[9] == 1 and st.sum() == 2
    assert np.all(out[[5, 9]] == -3.0) and np.all(adv[[5, 9]] == -7)
    good = st == 0
    assert np.array_equal(adv[good], adv_ref[good]) and np.array_equal(adv[good], adv_true[good])
    assert group_err(out[good], ref[good]).max() <= TOL


@pytest.mark.parametrize("K,A,N,C,G", [(12, 2, 28, 10, 257), (8, 2, 24, 10, 5), (4, 1, 12, 1, 7), (2, 1, 9, 3, 10),
                                       (6, 2, 20, 5, 1), (12, 3, 30, 6, 33), (3, 1, 30, 15, 6), (14, 2, 32, 9, 4), (14, 2, 48, 7, 9),
                                       # enough groups for four of them to share a workgroup; group counts 4 does not divide
                                       (12, 2, 28, 10, 1367), (4, 1, 12, 1, 4099), (2, 1, 9, 3, 4101), (5, 2, 16, 6, 2050),
                                       (3, 1, 30, 15, 1025)])
@pytest.mark.parametrize("mode", [0, 1])
def test_byzantine_no_stragglers_groups_share_one_factorisation(gpu, K, A, N, C, G, mode):
    # Section 4.2, "Byzantine-Robustness": S = 0.  With a workspace the node set is factorised once per call and, when
    # a group's classes do not fill whole rounds of four, several groups share a workgroup.  Odd group counts, one
    # class, a group that is not full (bad by the S = 0 contract) in the middle; against the oracle, and bit for
    # bit against the same call without a workspace (one workgroup and one factorisation per group).
    torch, binding, dev = gpu
    rng = np.random.default_rng(1000 * K + 10 * C + G)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, 64))
    Mf = rng.standard_normal((64, C)) / 8
    Y = (orc.encode(X, alpha, beta) @ Mf).astype(np.float32)
    mask = np.ones((G, N), np.uint8)
    adv_true = np.zeros((G, A), np.int32)
    ok = np.nonzero(np.abs(beta) > 1e-9)[0]
    for g in range(G):
        adv_true[g] = np.sort(rng.permutation(ok)[:A])
        Y[g, adv_true[g]] += (10 * Y.std() * rng.standard_normal((A, C))).astype(np.float32)
    bad = G // 2 if G >= 3 else -1
    if bad >= 0:
        mask[bad, 1] = 0
    Yd, md = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    res = {}
    for name, ws in (("shared", None), ("alone", binding.NO_WORKSPACE)):
        out = torch.full((G, K, C), -3.0, dtype=torch.float32, device=dev)
        adv = torch.full((G, A), -7, dtype=torch.int32, device=dev)
        out, adv, st = binding.approxifer_decode_byzantine(Yd, md, alpha, beta, 0, A, mode, out=out, adv=adv, workspace=ws)
        res[name] = (out.cpu().numpy(), adv.cpu().numpy(), st.cpu().numpy())
    assert binding.approxifer_workspace_bytes(G, K, N, 0, A, C) > 0
    for a, b in zip(res["shared"], res["alone"]):
        assert np.array_equal(a, b)
    out, adv, st = res["shared"]
    ref, adv_ref, st_ref = orc.decode_byzantine(Y, mask, alpha, beta, 0, A, mode)
    assert np.array_equal(st, st_ref) and st.sum() == (1 if bad >= 0 else 0)
    if bad >= 0:
        assert st[bad] == 1 and np.all(out[bad] == -3.0) and np.all(adv[bad] == -7)
    good = st == 0
    assert np.array_equal(adv[good], adv_ref[good]) and np.array_equal(adv[good], adv_true[good])
    assert group_err(out[good], ref[good]).max() <= TOL


@pytest.mark.parametrize("K,A,N,C", [(12, 2, 28, 10), (8, 2, 20, 10), (6, 2, 18, 3), (12, 3, 32, 15), (13, 3, 33, 10), (15, 1, 40, 10),
                                     (6, 2, 32, 7), (8, 2, 20, 16), (12, 2, 28, 40)])
@pytest.mark.parametrize("entry", ["approxifer_decode_byzantine", "approxifer_decode_byzantine_homogeneous"])
def test_byzantine_same_bits_with_and_without_workspace_where_picks_hang_on_rounding(gpu, K, A, N, C, entry):
    # Fewer liars than A, none at all, softmax answers: which innocent workers go is decided by the last bits of the fits,
    # so that a factorisation that differs in rounding between the two ways shows up as another located set.
    torch, binding, dev = gpu
    decode = getattr(binding, entry)
    G = 300 if entry == "approxifer_decode_byzantine" else 60
    rng = np.random.default_rng(K + C)
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = orc.encode(rng.uniform(0, 1, (G, K, 32)), alpha, beta) @ (rng.standard_normal((32, C)) / 6)
    one = Y.copy()
    one[:, 0] += 5 * rng.standard_normal((G, C))
    soft = np.exp(3 * Y) / np.exp(3 * Y).sum(-1, keepdims=True)
    md = torch.ones((G, N), dtype=torch.uint8, device=dev)
    for data in (Y, one, soft, rng.standard_normal(Y.shape)):
        Yd = torch.from_numpy(data.astype(np.float32)).to(dev)
        with_ws = decode(Yd, md, alpha, beta, 0, A, 1)
        without = decode(Yd, md, alpha, beta, 0, A, 1, workspace=binding.NO_WORKSPACE)
        for a, b in zip(with_ws, without):
            assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())


@pytest.mark.parametrize("K,N,S,C,G", [
    (1, 2, 0, 1, 1), (4, 16, 3, 16, 17), (5, 17, 4, 3, 33), (6, 9, 2, 10, 16), (8, 9, 1, 10, 257), (12, 28, 9, 15, 5),
    (16, 33, 15, 2, 31), (17, 48, 12, 5, 18), (24, 64, 30, 16, 3), (32, 64, 0, 7, 15), (32, 48, 12, 2, 40), (9, 32, -1, 10, 50),
])
@pytest.mark.parametrize("mode", [0, 1])
def test_decode_small_classes_sixteen_groups_to_a_workgroup(gpu, K, N, S, C, G, mode):
    # Edges of the row kernel: register counts of K, chunks of sixteen workers, the last workgroup partly filled, query
    # nodes that are worker nodes (6 of 9, 5 of 17, ..), answers that did not come hold NaN; decode and fused top-1.
    torch, binding, dev = gpu
    rng = np.random.default_rng(91 * K + N + C)
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        late = S if S >= 0 else int(rng.integers(0, N - 1))
        mask[g, rng.permutation(N)[late:]] = 1
    if G > 2:
        mask[1] = 0                                       # bad: nobody answered
    poisoned = np.where(mask[:, :, None] != 0, Y, np.float32(np.nan))
    Yd, md = torch.from_numpy(poisoned).to(dev), torch.from_numpy(mask).to(dev)
    out = torch.full((G, K, C), -3.0, dtype=torch.float32, device=dev)
    out, st = binding.approxifer_decode(Yd, md, alpha, beta, S, mode, out=out)
    top1, score, st1 = binding.approxifer_decode_top1(Yd, md, alpha, beta, S, mode)
    out, st, top1, score, st1 = (t.cpu().numpy() for t in (out, st, top1, score, st1))
    ref, st_ref = orc.decode(Y, mask, alpha, beta, S, mode)
    assert np.array_equal(st, st_ref) and np.array_equal(st1, st_ref)
    good = st == 0
    assert np.all(out[~good] == -3.0) and np.all(top1[~good] == -1)
    ok = good & np.isfinite(ref).all(axis=(1, 2)) & (np.abs(ref).max(axis=(1, 2)) < 1e6)   # printed signs can meet a pole
    assert ok.sum() >= good.sum() // 2
    assert group_err(out[ok], ref[ok]).max() <= TOL
    assert np.array_equal(score[ok], out[ok].max(-1))
    srt = np.sort(ref, axis=-1)
    clear = ok[:, None] & (np.ones((G, K), bool) if C == 1 else srt[..., -1] - srt[..., -2] > 1e-9 * np.abs(srt).max(-1))
    assert np.array_equal(top1[clear], ref.argmax(-1)[clear])


@pytest.mark.parametrize("K,A,S,N,C", [
    (8, 2, 4, 24, 10),      # the byzantine workload: one row block of workers more than answer
    (8, 2, 9, 30, 15),      # many more workers than answer; the most classes a staged tile takes
    (2, 1, 3, 9, 1), (3, 1, 38, 48, 2), (6, 2, 4, 21, 7), (12, 2, 4, 32, 4), (14, 2, 1, 33, 10), (15, 1, 5, 37, 3),
    (6, 1, 2, 17, 16),      # one class too many for the tile: the workgroup-per-group kernel
    (2, 1, 20, 26, 12), (8, 2, 19, 44, 10), (12, 2, 12, 40, 10),     # many more workers than answer: by rule one or the other
    (15, 1, 0, 40, 10), (4, 2, 0, 30, 7),                            # no stragglers, more rows of U than a row of lanes
    (6, 2, -1, 24, 10),     # straggler counts read off the masks
])
@pytest.mark.parametrize("locator", [orc.LOCATOR_ALGORITHM_2, orc.LOCATOR_ALGORITHM_1])
def test_byzantine_groups_packed_into_workgroups(gpu, K, A, S, N, C, locator):
    # Four, two or one group(s) to a workgroup, by the number of groups: the same bits each way, a bad group in between,
    # the first groups against the oracle.  Several shapes have a query node that is a worker's node.
    torch, binding, dev = gpu
    G, G_ref, mode = 2700, 24, (K + C) % 2
    rng = np.random.default_rng(77 * K + N)
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = (orc.encode(rng.uniform(0, 1, (G, K, 32)), alpha, beta) @ (rng.standard_normal((32, C)) / 6)).astype(np.float32)
    sd = Y.std()
    mask = np.zeros((G, N), np.uint8)
    adv_true = np.zeros((G, A), np.int32)
    for g in range(G):
        late = S if S >= 0 else int(rng.integers(0, N - 2 * (K + A) + 1))
        order = rng.permutation(N)
        mask[g, order[late:]] = 1
        adv_true[g] = np.sort([w for w in order[late:] if abs(beta[w]) > 1e-9][:A])
        Y[g, adv_true[g]] += (10 * sd * rng.standard_normal((A, C))).astype(np.float32)
        Y[g, mask[g] == 0] = np.nan                      # an answer that did not come is not looked at
    mask[5] = 0
    Yd, md = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    res = {}
    for n_groups in (2700, 1500, 40):
        out = torch.full((n_groups, K, C), -3.0, dtype=torch.float32, device=dev)
        adv = torch.full((n_groups, A), -7, dtype=torch.int32, device=dev)
        decode = binding.approxifer_decode_byzantine if locator == orc.LOCATOR_ALGORITHM_2 else binding.approxifer_decode_byzantine_homogeneous
        got = decode(Yd[:n_groups], md[:n_groups], alpha, beta, S, A, mode, out=out, adv=adv)
        res[n_groups] = [t.cpu().numpy() for t in got]
    for n_groups in (1500, 40):
        for whole, part in zip(res[2700], res[n_groups]):
            assert np.array_equal(whole[:n_groups], part)
    out, adv, st = [x[:G_ref] for x in res[2700]]
    Yz = np.where(mask[:G_ref, :, None] != 0, Y[:G_ref], 0.0).astype(np.float32)
    ref, adv_ref, st_ref = orc.decode_byzantine(Yz, mask[:G_ref], alpha, beta, S, A, mode, locator=locator)
    assert np.array_equal(st, st_ref) and st[5] == 1 and st.sum() == 1
    assert np.all(out[5] == -3.0) and np.all(adv[5] == -7)
    good = (st == 0) & np.array([np.array_equal(a, b) for a, b in zip(adv_ref, adv_true[:G_ref])])
    assert good.sum() >= (G_ref - 1 if C >= 7 else 1)     # one class may hold an answer that is hardly wrong
    assert np.array_equal(adv[good], adv_ref[good])
    assert group_err(out[good], ref[good]).max() <= TOL


def test_byzantine_nonlinear_model_votes(gpu):
    # softmax outputs are not rational in beta: Algorithm 2's fit is a genuine least-squares problem
    # and single classes may disagree.  The GPU must reproduce the oracle's vote wherever the oracle's
    # own vote is not a near tie.
    K, A, S, N, C, G = 4, 1, 2, 12, 10, 128
    rng = np.random.default_rng(77)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, 48))
    Mf = rng.standard_normal((48, C))
    z = orc.encode(X, alpha, beta) @ Mf
    clean = (np.exp(z) / np.exp(z).sum(-1, keepdims=True)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    Y = clean.copy()
    for g in range(G):
        avail = np.sort(rng.permutation(N)[: N - S])
        mask[g, avail] = 1
        bad = rng.permutation(avail)[:A]
        Y[g, bad] += rng.standard_normal((A, C)).astype(np.float32)
    out, adv, st, ref, adv_ref, _ = _byz_both(gpu, Y, mask, alpha, beta, S, A)
    clear = np.zeros(G, bool)
    for g in range(G):
        _, _, counts = orc.locate(Y[g], np.nonzero(mask[g])[0], beta, K, A)
        top = np.sort(counts)[::-1]
        clear[g] = top[A - 1] - top[A] >= 2
    assert clear.sum() >= G // 2
    assert np.array_equal(adv[clear], adv_ref[clear])
    same = np.all(adv == adv_ref, axis=1)
    assert same.mean() >= 0.97
    assert_rounding_ties(Y, mask, beta, K, A, adv, adv_ref)             # the rest differ on float64 ties only
    assert group_err(out[same], ref[same]).max() <= TOL


@pytest.mark.parametrize("real", [0, 1])
def test_byzantine_fewer_real_adversaries_than_A(gpu, real):
    # the decoder is configured for A = 2 adversaries but fewer workers actually lie ("at most E", Section 2).
    # Every fitted Q still vanishes at the real ones, so they must be among the located; the remaining picks
    # are innocent workers, whose removal costs nothing.  The sets must equal the oracle's wherever its own vote
    # is decisive, and the decoded values must equal the oracle's decode over the same survivors.
    torch, binding, dev = gpu
    K, A, S, N, C, G = 8, 2, 4, 24, 10, 96
    rng = np.random.default_rng(50 + real)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, 96))
    Mf = rng.standard_normal((96, C)) / 10
    clean = (orc.encode(X, alpha, beta) @ Mf).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    Y = clean.copy()
    truth = []
    for g in range(G):
        avail = np.sort(rng.permutation(N)[: N - S])
        mask[g, avail] = 1
        bad = np.sort(rng.permutation(avail)[:real])
        truth.append(set(int(b) for b in bad))
        Y[g, bad] += (10 * clean.std() * rng.standard_normal((real, C))).astype(np.float32)
    out, adv, st, ref, adv_ref, st_ref = _byz_both(gpu, Y, mask, alpha, beta, S, A, 1)
    assert np.all(st == 0) and np.array_equal(st, st_ref)
    decisive = np.zeros(G, bool)
    for g in range(G):
        assert truth[g] <= set(adv[g].tolist()) and truth[g] <= set(adv_ref[g].tolist())
        assert len(set(adv[g].tolist())) == A and np.all(mask[g, adv[g]] == 1) and np.all(np.diff(adv[g]) > 0)
        _, _, counts = orc.locate(Y[g], np.nonzero(mask[g])[0], beta, K, A)
        top = np.sort(counts)[::-1]
        decisive[g] = top[A - 1] - top[A] >= 2
    same = np.all(adv == adv_ref, axis=1)
    assert np.all(same[decisive]) and same.mean() >= 0.9
    assert_rounding_ties(Y, mask, beta, K, A, adv, adv_ref)             # rank-deficient fits: every class is a tie
    assert group_err(out[same], ref[same]).max() <= TOL
    for g in np.nonzero(~same)[0]:                          # decode parity given the kernel's own survivor set
        m2 = mask[g:g + 1].copy()
        m2[0, adv[g]] = 0
        ref_g, _ = orc.decode(Y[g:g + 1], m2, alpha, beta, S + A, 1)
        assert group_err(out[g:g + 1], ref_g).max() <= TOL


@pytest.mark.parametrize("entry", ["approxifer_decode_byzantine", "approxifer_decode_byzantine_homogeneous"])
@pytest.mark.parametrize("K,A,S,N,C", [(8, 2, 4, 24, 10), (12, 2, 0, 28, 10), (3, 1, 0, 64, 5), (18, 2, 0, 44, 3)])
def test_byzantine_degenerate_predictions(gpu, K, A, S, N, C, entry):
    # rank-deficient fits: all-zero predictions, the same constant everywhere, identical classes, one available
    # worker holding NaN.  No located set is "right" here; what must hold: every group is decoded, the located
    # workers are distinct available workers in ascending order, and -- the weights sum to one -- constants
    # decode to themselves whoever was dropped
    torch, binding, dev = gpu
    G = 6
    rng = np.random.default_rng(K + N)
    alpha, beta = orc.chebyshev_nodes(K, N)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        mask[g, rng.permutation(N)[: N - S]] = 1
    Y = np.zeros((G, N, C), np.float32)
    Y[1] = 2.5                                                  # constant
    Y[2] = rng.standard_normal((N, 1)).astype(np.float32)      # every class the same column
    Y[3] = 1e30                                                 # huge constant
    Y[4] = rng.standard_normal((N, C)).astype(np.float32)
    Y[4, np.nonzero(mask[4])[0][3]] = np.nan                    # a worker that returns NaN
    Y[5] = rng.standard_normal((N, C)).astype(np.float32) * 1e-30
    out, adv, st = getattr(binding, entry)(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta, S,
                                           A, 1)
    out, adv, st = out.cpu().numpy(), adv.cpu().numpy(), st.cpu().numpy()
    assert np.all(st == 0)
    for g in range(G):
        assert np.all(np.diff(adv[g]) > 0) and np.all(mask[g, adv[g]] == 1)
    assert np.all(out[0] == 0.0)
    assert np.max(np.abs(out[1] - 2.5)) <= 2.5e-5
    assert np.max(np.abs(out[3] / 1e30 - 1.0)) <= 1e-5
    for g in (2, 5):                                            # finite inputs: decode parity over the kernel's survivors
        m2 = mask[g:g + 1].copy()
        m2[0, adv[g]] = 0
        ref_g, _ = orc.decode(Y[g:g + 1], m2, alpha, beta, None, 1)
        assert group_err(out[g:g + 1], ref_g).max() <= TOL


# --------------------------------------------------------------------------------------
# Algorithm 1 (Q_0 free, null vector of the homogeneous system) as the per-class locator
# --------------------------------------------------------------------------------------
def _hom_both(gpu, Y, mask, alpha, beta, S, A, mode=0):
    torch, binding, dev = gpu
    out, adv, st = binding.approxifer_decode_byzantine_homogeneous(torch.from_numpy(Y).to(dev),
                                                                   torch.from_numpy(mask).to(dev), alpha, beta, S, A, mode)
    ref, adv_ref, st_ref = orc.decode_byzantine(Y, mask, alpha, beta, S, A, mode, locator=orc.LOCATOR_ALGORITHM_1)
    return out.cpu().numpy(), adv.cpu().numpy(), st.cpu().numpy(), ref, adv_ref, st_ref


def _decisive(Y, mask, beta, K, A, locator):
    """Groups whose oracle vote separates the A-th from the (A+1)-th most voted worker by two or more."""
    ok = np.zeros(Y.shape[0], bool)
    for g in range(Y.shape[0]):
        _, _, counts = orc.locate(Y[g], np.nonzero(mask[g])[0], beta, K, A, locator)
        top = np.sort(counts)[::-1]
        ok[g] = top[A - 1] - top[A] >= 2
    return ok


def test_homogeneous_locator_byzantine_workload(gpu):
    w = syn.scaled(syn.WORKLOADS["byzantine"], G=256)
    alpha, beta, Y, mask, adv_true = _byzantine_inputs(w)
    out, adv, st, ref, adv_ref, st_ref = _hom_both(gpu, Y, mask, alpha, beta, w.S, w.A)
    assert np.all(st == 0) and np.array_equal(st, st_ref)
    assert np.array_equal(adv, adv_ref) and np.array_equal(adv, adv_true)
    assert group_err(out, ref).max() <= TOL


@pytest.mark.parametrize("K,A,S,N,C,G", [
    (2, 1, 0, 6, 3, 16), (3, 2, 2, 12, 10, 16), (12, 2, 0, 28, 10, 4), (8, 2, 4, 24, 40, 4), (8, 2, 0, 64, 6, 2),
    (4, 1, 3, 13, 17, 8), (1, 1, 0, 48, 2, 4), (3, 1, 1, 9, 6, 600), (13, 3, 1, 33, 3, 3), (5, 2, 2, 23, 4, 8),
])
def test_homogeneous_locator_exactly_rational_predictions(gpu, K, A, S, N, C, G):
    # Theorem 1's setting: the null vector is the error locator times the denominator, the planted workers come back.
    # Here a worker on the node 0 can be an adversary too: Q_0 is free.
    rng = np.random.default_rng(K * 100 + A * 10 + S + 5)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, 96))
    Mf = rng.standard_normal((96, C)) / 10
    clean = (orc.encode(X, alpha, beta) @ Mf).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    adv_true = np.zeros((G, A), np.int32)
    Y = clean.copy()
    for g in range(G):
        avail = np.sort(rng.permutation(N)[: N - S])
        mask[g, avail] = 1
        adv_true[g] = np.sort(rng.permutation(avail)[:A])
        Y[g, adv_true[g]] += (10 * clean.std() * rng.standard_normal((A, C))).astype(np.float32)
    out, adv, st, ref, adv_ref, st_ref = _hom_both(gpu, Y, mask, alpha, beta, S, A)
    assert np.all(st == 0)
    assert np.array_equal(adv, adv_ref) and np.array_equal(adv, adv_true)
    assert group_err(out, ref).max() <= TOL


def test_homogeneous_locator_exactly_singular_systems(gpu):
    # K = 1 is replication: every honest worker returns the same float, the homogeneous system is singular to the
    # last bit (smallest singular value 0 or 1e-17) and its null vector is exact.  The factorisation then leaves a
    # zero, or rounding noise, on the diagonal of R: the planted workers must still come back, as from the oracle.
    K, N, C, G = 1, 10, 2, 400
    rng = np.random.default_rng(108)
    alpha, beta = orc.chebyshev_nodes(K, N)
    for A, S in ((2, 2), (1, 0), (3, 2)):
        X = rng.uniform(0, 1, (G, K, 48))
        clean = (orc.encode(X, alpha, beta) @ (rng.standard_normal((48, C)) / 7)).astype(np.float32)
        assert np.all(clean == clean[:, :1, :])
        mask = np.zeros((G, N), np.uint8)
        adv_true = np.zeros((G, A), np.int32)
        Y = clean.copy()
        for g in range(G):
            avail = np.sort(rng.permutation(N)[: N - S])
            mask[g, avail] = 1
            adv_true[g] = np.sort(rng.permutation(avail)[:A])
            Y[g, adv_true[g]] += (10 * (clean.std() + 1e-3) * rng.standard_normal((A, C))).astype(np.float32)
        out, adv, st, ref, adv_ref, st_ref = _hom_both(gpu, Y, mask, alpha, beta, S, A)
        assert np.all(st == 0)
        assert np.array_equal(adv, adv_true) and np.array_equal(adv_ref, adv_true)
        assert group_err(out, ref).max() <= TOL


def test_homogeneous_locator_finds_the_worker_on_node_zero(gpu):
    # an odd number of workers puts the middle worker on the node 0, where Algorithm 2's Q equals 1 by construction
    # (it can only be picked there if |Q| happens to exceed 1 on every other node); Algorithm 1's Q vanishes on it
    torch, binding, dev = gpu
    K, A, S, N, C, G = 3, 1, 0, 9, 6, 32
    rng = np.random.default_rng(3)
    alpha, beta = orc.chebyshev_nodes(K, N)
    assert abs(beta[4]) < 1e-15
    X = rng.uniform(0, 1, (G, K, 64))
    Mf = rng.standard_normal((64, C)) / 8
    Y = (orc.encode(X, alpha, beta) @ Mf).astype(np.float32)
    mask = np.ones((G, N), np.uint8)
    Y[:, 4] += (10 * Y.std() * rng.standard_normal((G, C))).astype(np.float32)
    out, adv, st, ref, adv_ref, _ = _hom_both(gpu, Y, mask, alpha, beta, S, A)
    assert np.all(st == 0) and np.all(adv == 4) and np.array_equal(adv, adv_ref)
    assert group_err(out, ref).max() <= TOL
    for g in range(4):                                      # per class, Algorithm 1 is unanimous
        _, I, _ = orc.locate(Y[g], np.arange(N), beta, K, A, orc.LOCATOR_ALGORITHM_1)
        assert np.all(I == 4)


def test_homogeneous_locator_on_data_that_is_not_rational(gpu):
    # softmax outputs and plain noise: no null vector, the smallest singular vector is a genuine fit and its
    # singular value need not be well separated.  The kernel's Jacobi iteration and the oracle's SVD must still
    # agree on every group whose vote is not a near tie.
    K, A, S, N, C, G = 4, 1, 2, 12, 10, 128
    rng = np.random.default_rng(78)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, 48))
    z = orc.encode(X, alpha, beta) @ rng.standard_normal((48, C))
    Y = (np.exp(z) / np.exp(z).sum(-1, keepdims=True)).astype(np.float32)
    Y[G // 2:] = rng.standard_normal((G - G // 2, N, C)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        avail = np.sort(rng.permutation(N)[: N - S])
        mask[g, avail] = 1
        Y[g, rng.permutation(avail)[:A]] += rng.standard_normal((A, C)).astype(np.float32)
    out, adv, st, ref, adv_ref, _ = _hom_both(gpu, Y, mask, alpha, beta, S, A)
    clear = _decisive(Y, mask, beta, K, A, orc.LOCATOR_ALGORITHM_1)
    assert clear.sum() >= G // 4
    assert np.array_equal(adv[clear], adv_ref[clear])
    same = np.all(adv == adv_ref, axis=1)
    assert same.mean() >= 0.95
    assert_rounding_ties(Y, mask, beta, K, A, adv, adv_ref, orc.LOCATOR_ALGORITHM_1)
    assert group_err(out[same], ref[same]).max() <= TOL


def test_homogeneous_locator_bad_and_ragged_masks(gpu):
    torch, binding, dev = gpu
    K, A, N, C, G = 4, 1, 16, 7, 48
    rng = np.random.default_rng(12)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, 64))
    clean = (orc.encode(X, alpha, beta) @ (rng.standard_normal((64, C)) / 8)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    Y = clean.copy()
    adv_true = np.full((G, A), -1, np.int32)
    for g in range(G):
        n = int(rng.integers(8, N + 1))                     # 8, 9: fewer than 2(K+A) = 10 available -> bad mask
        avail = np.sort(rng.permutation(N)[:n])
        mask[g, avail] = 1
        adv_true[g] = np.sort(rng.permutation(avail)[:A])
        Y[g, adv_true[g]] += (10 * clean.std() * rng.standard_normal((A, C))).astype(np.float32)
    out0 = torch.full((G, K, C), -3.0, dtype=torch.float32, device=dev)
    adv0 = torch.full((G, A), -7, dtype=torch.int32, device=dev)
    out, adv, st = binding.approxifer_decode_byzantine_homogeneous(torch.from_numpy(Y).to(dev),
                                                                   torch.from_numpy(mask).to(dev), alpha, beta,
                                                                   binding.S_FROM_MASK, A, 1, out=out0, adv=adv0)
    ref, adv_ref, st_ref = orc.decode_byzantine(Y, mask, alpha, beta, None, A, 1, locator=orc.LOCATOR_ALGORITHM_1)
    out, adv, st = out.cpu().numpy(), adv.cpu().numpy(), st.cpu().numpy()
    assert np.array_equal(st, st_ref) and 0 < st.sum() < G
    bad = st != 0
    assert np.all(out[bad] == -3.0) and np.all(adv[bad] == -7)
    assert np.array_equal(adv[~bad], adv_ref[~bad]) and np.array_equal(adv[~bad], adv_true[~bad])
    assert group_err(out[~bad], ref[~bad]).max() <= TOL


# --------------------------------------------------------------------------------------
# Algorithm 3 (Appendix A): the decoder by rational reconstruction, P(alpha_j) / Q(alpha_j)
# --------------------------------------------------------------------------------------
def _rational_case(seed, K, A, S, N, C, G, ragged=False):
    rng = np.random.default_rng(seed)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, 48))
    clean = (orc.encode(X, alpha, beta) @ (rng.standard_normal((48, C)) / 7)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    Y = clean.copy()
    for g in range(G):
        cnt = int(rng.integers(2 * (K + A), N + 1)) if ragged else N - S
        avail = np.sort(rng.permutation(N)[:cnt])
        mask[g, avail] = 1
        bad = rng.permutation(avail)[:A]
        Y[g, bad] += (10 * (clean.std() + 1e-3) * rng.standard_normal((A, C))).astype(np.float32)
    Y[mask == 0] = np.nan                                   # rows of missing workers must never be read
    return alpha, beta, Y, mask


@pytest.mark.parametrize("K,A,S,N,C,G", [(1, 1, 0, 8, 2, 8), (2, 1, 0, 6, 3, 16), (3, 1, 1, 9, 6, 40), (2, 2, 2, 12, 70, 9),
                                         (4, 1, 3, 13, 17, 8), (3, 1, 0, 64, 5, 3), (2, 1, 0, 20, 300, 2)])
def test_decode_rational_well_conditioned_shapes(gpu, K, A, S, N, C, G):
    # small K + A: the fit is well conditioned even on float32 data, and the plain 1e-5 bar holds for every group
    torch, binding, dev = gpu
    alpha, beta, Y, mask = _rational_case(K * 10 + A + N, K, A, S, N, C, G)
    out, st = binding.approxifer_decode_rational(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta, S, A)
    ref, st_ref = orc.decode_rational(Y, mask, alpha, beta, S, A)
    assert np.array_equal(st.cpu().numpy(), st_ref) and np.all(st_ref == 0)
    assert group_err(out.cpu().numpy(), ref).max() <= TOL


def test_decode_rational_ragged_and_bad_masks(gpu):
    torch, binding, dev = gpu
    K, A, N, C, G = 3, 1, 14, 9, 40
    alpha, beta, Y, mask = _rational_case(5, K, A, 0, N, C, G, ragged=True)
    mask[4] = 0
    mask[4, :2 * (K + A) - 1] = 1                            # one available worker too few
    Y[4] = 1.0
    out = torch.full((G, K, C), -3.0, dtype=torch.float32, device=dev)
    out, st = binding.approxifer_decode_rational(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta,
                                                 binding.S_FROM_MASK, A, out=out)
    ref, st_ref = orc.decode_rational(np.nan_to_num(Y), mask, alpha, beta, None, A)
    o, s = out.cpu().numpy(), st.cpu().numpy()
    assert np.array_equal(s, st_ref) and s[4] == 1 and s.sum() == 1
    assert np.all(o[4] == -3.0) and np.all(np.isfinite(o))
    good = s == 0
    assert group_err(o[good], ref[good]).max() <= TOL


@pytest.mark.parametrize("K,A,S,N,C,G", [(8, 2, 4, 24, 10, 64), (12, 2, 0, 28, 10, 16), (6, 2, 0, 40, 4, 8)])
def test_decode_rational_at_the_paper_sizes_within_the_conditioning_bound(gpu, K, A, S, N, C, G):
    # K + A = 10 .. 14 on float32 data: the fit's condition number is 1e8 and more, and this decoder is as fragile as
    # Appendix A says.  Every element must stay within the first-order bound of its own class's fit
    # (rational_tolerance), never less than the 1e-5 bar; and the typical group meets the plain bar.
    torch, binding, dev = gpu
    alpha, beta, Y, mask = _rational_case(K + A, K, A, S, N, C, G)
    out, st = binding.approxifer_decode_rational(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta, S, A)
    ref, st_ref = orc.decode_rational(Y, mask, alpha, beta, S, A)
    o = out.cpu().numpy().astype(np.float64)
    assert np.array_equal(st.cpu().numpy(), st_ref) and np.all(st_ref == 0)
    for g in range(G):
        avail = np.nonzero(mask[g])[0]
        scale = np.abs(ref[g]).max()
        for c in range(C):
            tol = np.maximum(rational_tolerance(beta[avail], Y[g, avail, c].astype(np.float64), K, A, alpha), TOL * scale)
            assert np.all(np.abs(o[g, :, c] - ref[g, :, c]) <= tol), (g, c)
    assert np.median(group_err(o, ref)) <= TOL


# --------------------------------------------------------------------------------------
# the paper's own operating points (Section 4.2; Appendix B), on synthetic stand-in data
# --------------------------------------------------------------------------------------
@pytest.mark.parametrize("K", [8, 10, 12])
@pytest.mark.parametrize("S", [1, 2, 3])
@pytest.mark.parametrize("shape", [(1, 28, 28), (3, 32, 32)])
def test_straggler_operating_points(gpu, K, S, shape):
    # K = 8, 10, 12 queries with S = 1, 2, 3 stragglers (N = K + S workers), 10 classes, MNIST- and
    # CIFAR-sized queries: encode, a non-linear stand-in model, every single mask decoded in both modes
    torch, binding, dev = gpu
    N, C, G = K + S, 10, 24
    D = int(np.prod(shape))
    rng = np.random.default_rng(K * 10 + S + D)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, D)).astype(np.float32)
    coded = binding.approxifer_encode(torch.from_numpy(X).to(dev), alpha, beta).cpu().numpy()
    ref_coded = orc.encode(X, alpha, beta)
    assert group_err(coded, ref_coded).max() <= TOL
    Mf = rng.standard_normal((D, C)) * (4.0 / np.sqrt(D))
    z = ref_coded @ Mf
    Y = (np.exp(z - z.max(-1, keepdims=True)) / np.exp(z - z.max(-1, keepdims=True)).sum(-1, keepdims=True)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        mask[g, rng.permutation(N)[:K]] = 1
    for mode in (0, 1):
        out, st, ref, st_ref = _decode_both(gpu, Y, mask, alpha, beta, S, mode)
        assert np.all(st == 0) and np.array_equal(st, st_ref)
        assert group_err(out, ref).max() <= TOL
        # top-1 decisions, the paper's accuracy metric, agree wherever the oracle's margin is not a rounding tie
        top2 = np.sort(ref, axis=-1)[..., -2:]
        clear = (top2[..., 1] - top2[..., 0]) > 1e-4 * np.abs(ref).max()
        assert np.array_equal(out.argmax(-1)[clear], ref.argmax(-1)[clear])


@pytest.mark.parametrize("E", [1, 2, 3])
@pytest.mark.parametrize("sigma", [1.0, 10.0, 100.0])
def test_byzantine_operating_points(gpu, E, sigma):
    # K = 12, S = 0, E = 1, 2, 3 adversaries adding zero-mean Gaussian noise of scale sigma = 1, 10, 100
    # (Section 4.2 "Byzantine-Robustness", Appendix B); N = 2(K + E) workers, 10 classes, linear stand-in model
    K, S, C, G = 12, 0, 10, 32
    N = 2 * (K + E)
    rng = np.random.default_rng(1000 * E + int(sigma))
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, 784))
    Mf = rng.standard_normal((784, C)) / 28.0
    clean = (orc.encode(X, alpha, beta) @ Mf).astype(np.float32)
    mask = np.ones((G, N), np.uint8)
    adv_true = np.zeros((G, E), np.int32)
    Y = clean.copy()
    for g in range(G):
        adv_true[g] = np.sort(rng.permutation(N)[:E])
        Y[g, adv_true[g]] += (sigma * rng.standard_normal((E, C))).astype(np.float32)
    out, adv, st, ref, adv_ref, st_ref = _byz_both(gpu, Y, mask, alpha, beta, S, E)
    assert np.all(st == 0)
    assert np.array_equal(adv, adv_ref)
    assert np.array_equal(adv, adv_true)
    assert group_err(out, ref).max() <= TOL


@pytest.mark.timeout(900)
def test_paper_operating_point_workloads_full_size(gpu):
    # the two MNIST-shaped workloads the benchmark times, at full size and in its launch configuration:
    # K = 8, one straggler (packed decoder, fused top-1) and K = 12, E = 2, 28 workers (projected Byzantine kernel)
    torch, binding, dev = gpu
    w = syn.WORKLOADS["mnist_k8"]
    alpha, beta = orc.chebyshev_nodes(w.K, w.W)
    X = syn.queries(w, threads=16)
    coded = binding.approxifer_encode(torch.from_numpy(X).to(dev), alpha, beta).cpu().numpy()
    worst = 0.0
    for g0 in range(0, w.G, 2048):
        worst = max(worst, group_err(coded[g0:g0 + 2048], orc.encode(X[g0:g0 + 2048], alpha, beta)).max())
    assert worst <= TOL, worst
    Y = syn.model_apply(w, syn.model_params(w), coded.astype(np.float64))
    mask = syn.masks(w)
    out, st, ref, st_ref = _decode_both(gpu, Y, mask, alpha, beta, w.S, 0)
    assert np.all(st == 0) and np.array_equal(st, st_ref)
    assert group_err(out, ref).max() <= TOL
    top1, score, st1 = binding.approxifer_decode_top1(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev),
                                                      alpha, beta, w.S, 0)
    srt = np.sort(ref, axis=-1)
    clear = (srt[..., -1] - srt[..., -2]) > 1e-9 * np.abs(ref).max(axis=-1)
    assert clear.mean() > 0.99 and np.array_equal(top1.cpu().numpy()[clear], ref.argmax(-1)[clear])

    wb = syn.WORKLOADS["mnist_byz_k12"]
    alpha, beta, Yb, maskb, adv_true = _byzantine_inputs(wb)
    outb, advb, stb = binding.approxifer_decode_byzantine(torch.from_numpy(Yb).to(dev), torch.from_numpy(maskb).to(dev),
                                                          alpha, beta, wb.S, wb.A)
    outb, advb, stb = outb.cpu().numpy(), advb.cpu().numpy(), stb.cpu().numpy()
    assert np.all(stb == 0) and np.array_equal(advb, adv_true)          # every planted set, bit for bit
    sample = np.arange(0, wb.G, 16)                                      # the oracle on every 16th group
    refb, adv_ref, _ = orc.decode_byzantine(Yb[sample], maskb[sample], alpha, beta, wb.S, wb.A)
    assert np.array_equal(advb[sample], adv_ref)
    assert group_err(outb[sample], refb).max() <= TOL


# --------------------------------------------------------------------------------------
# decoders on the float64 matrix cores
# --------------------------------------------------------------------------------------
@pytest.mark.parametrize("K,N,S", [
    (9, 11, 1), (12, 20, 8), (13, 16, 0), (16, 17, 1), (16, 40, 4), (17, 17, 0), (20, 26, 2), (32, 33, 0), (28, 50, 20), (33, 40, 3),
    (48, 64, 16), (64, 64, 0), (20, 50, -1), (16, 33, -1),
])
def test_decode_top1_on_the_matrix_cores(gpu, K, N, S):
    # k-steps and rounds as in the test below; one stripe of 64 classes, remainders of a stripe and of a vector, a stripe more than the
    # waves take at once, a workgroup of one wave (G >= 1024) and of many; a rejected mask; workers without an answer are NaN
    torch, binding, dev = gpu
    rng = np.random.default_rng(100 * K + N)
    alpha, beta = orc.chebyshev_nodes(K, N)
    for C, G in [(17, 3), (64, 1030), (66, 3), (101, 1030), (255, 3), (257, 300), (1001, 3), (1030, 256)]:
        n = N - S if S >= 0 else N - 2
        mask = (rng.random((G, N)).argsort(1).argsort(1) < n).astype(np.uint8)
        Y = rng.standard_normal((G, N, C)).astype(np.float32)
        Y[0, :, 5] = Y[0, :, 11] = 50.0                       # two classes tie: the smaller
        mask[1] = 0
        sent = np.where(mask[:, :, None] != 0, Y, np.float32("nan"))
        t, s, st = binding.approxifer_decode_top1(torch.from_numpy(sent).to(dev), torch.from_numpy(mask).to(dev), alpha, beta,
                                                  binding.S_FROM_MASK if S < 0 else S, 1)
        t, s, st = t.cpu().numpy(), s.cpu().numpy(), st.cpu().numpy()
        some = [0, 2, G - 1]
        ref, _ = orc.decode(Y[some], mask[some], alpha, beta, None if S < 0 else S, 1)
        assert st[1] != 0 and np.all(st[[0] + list(range(2, G))] == 0)
        assert np.all(t[1] == -1) and np.all(s[1] == 0.0)
        assert np.array_equal(t[0], np.full(K, 5))
        for k, g in enumerate(some):
            top = ref[k].max(axis=1)
            # one rounding of the winner's value; float64 sums before it as in the decoder
            assert np.all(np.abs(s[g] - top) <= 2.0 ** -24 * np.abs(top) + 1e-12 * 50.0)
            assert np.all(ref[k][np.arange(K), t[g]] >= top - 1e-12 * 50.0)


@pytest.mark.parametrize("K,N,S", [
    (9, 9, 0), (9, 12, 2), (12, 20, 8), (13, 16, 0), (16, 20, 4), (16, 17, 1), (17, 17, 0), (17, 40, 3), (20, 26, 2), (31, 36, 3),
    (32, 33, 0), (33, 40, 3), (48, 48, 0), (48, 64, 16), (64, 64, 0), (20, 50, -1), (16, 33, -1), (64, 64, -1),
])
def test_decode_on_the_matrix_cores(gpu, K, N, S):
    # few tiles, so that all but the shortest ragged rows of up to 24 queries come here: 4, 6, 9, 12 and 16 k-steps and remainders, one to four rounds of sixteen
    # queries, tiles of whole and of ragged sectors (one up to 63 vectors, 60 a tile less one), row ends of every remainder,
    # output rows of every phase, a rejected mask; predictions of workers that did not answer are NaN
    torch, binding, dev = gpu
    rng = np.random.default_rng(100 * K + N)
    alpha, beta = orc.chebyshev_nodes(K, N)
    for C, off_in, off_out in [(17, 0, 0), (18, 1, 3), (96, 0, 0), (97, 0, 5), (240, 2, 0), (251, 0, 0), (252, 0, 2), (253, 3, 1),
                               (256, 0, 0), (272, 0, 0), (476, 0, 0), (477, 1, 0), (1000, 0, 0), (1003, 0, 0)]:
        G = 4
        cnt = rng.integers(max(1, N // 2), N + 1, G) if S < 0 else np.full(G, N - S)
        mask = np.zeros((G, N), np.uint8)
        for g in range(G):
            mask[g, rng.choice(N, cnt[g], replace=False)] = 1
        Y = rng.standard_normal((G, N, C)).astype(np.float32)
        ref, _ = orc.decode(Y, mask, alpha, beta, None if S < 0 else S, 1)
        bad = mask.copy()
        if S < 0:
            bad[2] = 0
        elif S > 0:
            bad[2] = 1
        else:
            bad[2, 0] = 0
        Yn = np.where(bad[:, :, None] != 0, Y, np.float32("nan"))
        flat_in = torch.full((G * N * C + off_in + 3,), float("nan"), dtype=torch.float32, device=dev)
        flat_in[off_in:off_in + G * N * C] = torch.from_numpy(Yn).to(dev).reshape(-1)
        flat_out = torch.full((G * K * C + off_out + 40,), 7.5, dtype=torch.float32, device=dev)
        out = flat_out[off_out:off_out + G * K * C].view(G, K, C)
        _, st = binding.approxifer_decode(flat_in[off_in:off_in + G * N * C].view(G, N, C), torch.from_numpy(bad).to(dev), alpha, beta,
                                          binding.S_FROM_MASK if S < 0 else S, 1, out=out)
        assert st.cpu().tolist() == [0, 0, st.cpu().tolist()[2], 0] and st.cpu().tolist()[2] != 0
        got = out.cpu().numpy()
        good = [0, 1, 3]
        # one rounding to float32; the float64 sums before it (weights of either sign, Lebesgue constant below 10) leave 1e-12
        assert np.all(np.abs(got[good] - ref[good]) <= 2.0 ** -24 * np.abs(ref[good]) + 1e-12 * np.abs(Y).max()), C
        assert np.all(got[2] == 7.5)
        assert torch.all(flat_out[:off_out] == 7.5) and torch.all(flat_out[off_out + G * K * C:] == 7.5), C


# --------------------------------------------------------------------------------------
# per-group straggler counts (S = APPROXIFER_S_FROM_MASK): ragged masks
# --------------------------------------------------------------------------------------
@pytest.mark.parametrize("K,N,C,G", [(3, 9, 5, 12), (8, 12, 100, 40), (12, 20, 1000, 24), (16, 70, 36, 10), (5, 128, 3, 9),
                                     (10, 30, 10, 64), (16, 32, 16, 33)])
@pytest.mark.parametrize("mode", [0, 1])
def test_decode_ragged_masks(gpu, K, N, C, G, mode):
    torch, binding, dev = gpu
    alpha, beta, Y, mask = ragged_decode_case(K, N, C, G, mode)
    out = torch.full((G, K, C), -9.0, dtype=torch.float32, device=dev)
    out, st = binding.approxifer_decode(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta,
                                        binding.S_FROM_MASK, mode, out=out)
    with np.errstate(all="ignore"):
        ref, st_ref = orc.decode(Y, mask, alpha, beta, None, mode)
    out, st = out.cpu().numpy(), st.cpu().numpy()
    assert np.array_equal(st, st_ref) and st[2] == 1 and st.sum() == 1
    assert np.all(out[2] == -9.0)
    # every decoded group is compared, bar the ones the oracle-side conditioning test sets aside for this seed
    # (ILL_POSED_RAGGED, checked against the oracle by the CPU suite): none, or the one group whose mask puts a
    # pole of the printed sign rule on a query node
    finite = np.all(np.isfinite(ref.reshape(G, -1)), axis=1) & (st == 0) & well_posed(alpha, beta, mask, mode)
    assert G - 1 - finite.sum() == ILL_POSED_RAGGED.get((K, N, C, G, mode), 0)
    assert group_err(out[finite], ref[finite]).max() <= TOL
    assert np.array_equal(out[1], np.broadcast_to(Y[1, np.nonzero(mask[1])[0][0]], (K, C)))
    top1, score, st1 = binding.approxifer_decode_top1(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev),
                                                      alpha, beta, binding.S_FROM_MASK, mode)
    assert np.array_equal(st1.cpu().numpy(), st_ref)
    if C > 1:
        srt = np.sort(ref[finite], axis=-1)
        clear = (srt[..., -1] - srt[..., -2]) > 1e-9 * np.abs(ref[finite]).max(axis=-1)
        assert np.array_equal(top1.cpu().numpy()[finite][clear], ref[finite].argmax(-1)[clear])


def test_byzantine_ragged_masks(gpu):
    torch, binding, dev = gpu
    K, A, N, C, G = 4, 2, 20, 10, 48
    rng = np.random.default_rng(404)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.uniform(0, 1, (G, K, 64))
    Mf = rng.standard_normal((64, C)) / 8
    clean = (orc.encode(X, alpha, beta) @ Mf).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    Y = clean.copy()
    counts = rng.integers(2 * (K + A), N + 1, G)
    counts[0], counts[1], counts[2] = N, 2 * (K + A), 2 * (K + A) - 1   # all, the minimum of eq. (3), one too few
    adv_true = np.full((G, A), -1, np.int32)
    for g in range(G):
        avail = np.sort(rng.permutation(N)[: counts[g]])
        mask[g, avail] = 1
        adv_true[g] = np.sort(rng.permutation(avail)[:A])
        Y[g, adv_true[g]] += (10 * clean.std() * rng.standard_normal((A, C))).astype(np.float32)
    out = torch.full((G, K, C), -3.0, dtype=torch.float32, device=dev)
    adv = torch.full((G, A), -7, dtype=torch.int32, device=dev)
    out, adv, st = binding.approxifer_decode_byzantine(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev),
                                                       alpha, beta, binding.S_FROM_MASK, A, 1, out=out, adv=adv)
    ref, adv_ref, st_ref = orc.decode_byzantine(Y, mask, alpha, beta, None, A, 1)
    out, adv, st = out.cpu().numpy(), adv.cpu().numpy(), st.cpu().numpy()
    assert np.array_equal(st, st_ref) and st[2] == 1 and st.sum() == 1
    assert np.all(out[2] == -3.0) and np.all(adv[2] == -7)
    good = st == 0
    assert np.array_equal(adv[good], adv_ref[good]) and np.array_equal(adv[good], adv_true[good])
    assert group_err(out[good], ref[good]).max() <= TOL


# --------------------------------------------------------------------------------------
# wait rule: arrival times -> survivor mask
# --------------------------------------------------------------------------------------
@pytest.mark.parametrize("N,wait_for,G", [(1, 1, 3), (6, 4, 64), (12, 8, 1000), (24, 20, 257), (64, 1, 9), (65, 33, 9),
                                          (128, 128, 5), (128, 77, 130), (20, 12, 5000)])
def test_wait_mask(gpu, N, wait_for, G):
    torch, binding, dev = gpu
    rng = np.random.default_rng(N * 1000 + wait_for)
    arrival = rng.exponential(1.0, (G, N)).astype(np.float32)
    arrival[rng.random((G, N)) < 0.15] = np.float32(0.5)              # plenty of exact ties
    arrival[rng.random((G, N)) < 0.10] = np.inf                       # workers that never answer
    arrival[rng.random((G, N)) < 0.02] = np.nan
    arrival[rng.random((G, N)) < 0.02] = -np.inf
    arrival[0] = np.inf                                                # nobody answers
    if G > 1:
        arrival[1] = 1.0                                               # everybody at once
    mask = torch.full((G, N), 77, dtype=torch.uint8, device=dev)
    mask, count = binding.approxifer_wait_mask(torch.from_numpy(arrival).to(dev), wait_for, mask=mask)
    ref_mask, ref_count = orc.wait_mask(arrival, wait_for)
    assert np.array_equal(mask.cpu().numpy(), ref_mask)                # bit-exact
    assert np.array_equal(count.cpu().numpy(), ref_count)
    assert ref_count[0] == 0 and (G == 1 or ref_mask[1, :wait_for].all())


def test_wait_mask_feeds_the_decoder(gpu):
    # arrival times -> mask -> decode, all on the device, against the oracle's chain
    torch, binding, dev = gpu
    K, N, C, G = 8, 12, 10, 300
    rng = np.random.default_rng(99)
    alpha, beta = orc.chebyshev_nodes(K, N)
    arrival = rng.exponential(1.0, (G, N)).astype(np.float32)
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    mask, count = binding.approxifer_wait_mask(torch.from_numpy(arrival).to(dev), K)
    out, st = binding.approxifer_decode(torch.from_numpy(Y).to(dev), mask, alpha, beta, N - K, 1)
    ref_mask, _ = orc.wait_mask(arrival, K)
    ref, st_ref = orc.decode(Y, ref_mask, alpha, beta, N - K, 1)
    assert np.all(st.cpu().numpy() == 0) and np.all(st_ref == 0)
    assert group_err(out.cpu().numpy(), ref).max() <= TOL


# --------------------------------------------------------------------------------------
# HIP graph capture: the calls allocate nothing, keep no state and enqueue kernels only
# --------------------------------------------------------------------------------------
def test_calls_on_two_streams_keep_no_state_between_them(gpu):
    # The library keeps no state between calls: two chains (encode -> Byzantine decode with a workspace of its own,
    # few groups x many classes so that the workgroups of a group pool their votes there) enqueued alternately on two
    # streams of the default priority give, bit for bit, what each chain gives alone on the current stream.
    torch, binding, dev = gpu
    K, A, N, C, G, D = 8, 2, 24, 1000, 6, 512
    alpha, beta = orc.chebyshev_nodes(K, N)
    rng = np.random.default_rng(4242)
    chains = []
    for t in range(2):
        X = torch.from_numpy(rng.uniform(0, 1, (G, K, D)).astype(np.float32)).to(dev)
        Mf = torch.from_numpy((rng.standard_normal((D, C)) / 20).astype(np.float32)).to(dev)
        noise = torch.from_numpy((5 * rng.standard_normal((G, A, C))).astype(np.float32)).to(dev)
        bad = torch.from_numpy(np.stack([np.sort(rng.permutation(np.arange(1, N))[:A]) for _ in range(G)])).to(dev)
        mask = torch.ones((G, N), dtype=torch.uint8, device=dev)
        chains.append((X, Mf, noise, bad, mask))
    need = binding.approxifer_workspace_bytes(G, K, N, 0, A, C)
    assert need >= 4 * (N + 1) * G

    def run(chain, stream, ws):
        X, Mf, noise, bad, mask = chain
        with torch.cuda.stream(stream):
            coded = binding.approxifer_encode(X, alpha, beta, stream=stream)
            preds = (coded.reshape(G * N, D) @ Mf).reshape(G, N, C)
            preds.scatter_add_(1, bad[:, :, None].expand(-1, -1, C), noise)
            out, adv, st = binding.approxifer_decode_byzantine(preds, mask, alpha, beta, 0, A, 1, workspace=ws, stream=stream)
        return coded, out, adv, st, bad

    cur = torch.cuda.current_stream()
    alone = [run(c, cur, torch.zeros((need,), dtype=torch.uint8, device=dev)) for c in chains]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    spaces = [torch.zeros((need,), dtype=torch.uint8, device=dev) for _ in range(2)]
    both = [None, None]
    for rep in range(3):
        for t in range(2):
            both[t] = run(chains[t], streams[t], spaces[t])
    torch.cuda.synchronize()
    for t in range(2):
        coded, out, adv, st, bad = both[t]
        assert torch.all(st == 0) and torch.equal(adv.long(), bad)
        for got, want in zip(both[t][:4], alone[t][:4]):
            assert torch.equal(got, want)


def test_calls_can_be_captured_in_a_hip_graph_and_replayed(gpu):
    torch, binding, dev = gpu
    K, N, S, D, C, G = 8, 12, 4, 3072, 100, 32
    Kb, Ab, Sb, Nb, Cb = 8, 2, 4, 24, 300      # five class tiles: the Byzantine decoder's workgroups share groups
    rng = np.random.default_rng(123)
    alpha, beta = orc.chebyshev_nodes(K, N)
    alphab, betab = orc.chebyshev_nodes(Kb, Nb)
    q = torch.zeros((G, K, D), dtype=torch.float32, device=dev)
    coded = torch.zeros((G, N, D), dtype=torch.float32, device=dev)
    arrival = torch.zeros((G, N), dtype=torch.float32, device=dev)
    mask = torch.zeros((G, N), dtype=torch.uint8, device=dev)
    count = torch.zeros((G,), dtype=torch.int32, device=dev)
    preds = torch.zeros((G, N, C), dtype=torch.float32, device=dev)
    out = torch.zeros((G, K, C), dtype=torch.float32, device=dev)
    st = torch.zeros((G,), dtype=torch.int32, device=dev)
    top1 = torch.zeros((G, K), dtype=torch.int32, device=dev)
    predsb = torch.zeros((G, Nb, Cb), dtype=torch.float32, device=dev)
    maskb = torch.zeros((G, Nb), dtype=torch.uint8, device=dev)
    outb = torch.zeros((G, Kb, Cb), dtype=torch.float32, device=dev)
    advb = torch.zeros((G, Ab), dtype=torch.int32, device=dev)
    stb = torch.zeros((G,), dtype=torch.int32, device=dev)
    outh = torch.zeros((G, Kb, Cb), dtype=torch.float32, device=dev)
    advh = torch.zeros((G, Ab), dtype=torch.int32, device=dev)

    need = binding.approxifer_workspace_bytes(G, Kb, Nb, Sb, Ab, Cb)
    assert need > 0
    wsb = torch.empty((need,), dtype=torch.uint8, device=dev)    # the two Byzantine calls run one after the other

    def calls():
        binding.approxifer_encode(q, alpha, beta, coded=coded)
        binding.approxifer_wait_mask(arrival, N - S, mask=mask, count=count)
        binding.approxifer_decode(preds, mask, alpha, beta, S, 1, out=out, status=st)
        binding.approxifer_decode_top1(preds, mask, alpha, beta, S, 1, top1=top1, status=st, want_score=False)
        binding.approxifer_decode_byzantine(predsb, maskb, alphab, betab, Sb, Ab, 1, out=outb, adv=advb, status=stb,
                                            workspace=wsb)
        binding.approxifer_decode_byzantine_homogeneous(predsb, maskb, alphab, betab, Sb, Ab, 1, out=outh, adv=advh,
                                                        status=stb, workspace=wsb)

    def fresh_inputs(seed):
        r = np.random.default_rng(seed)
        X = r.uniform(0, 1, (G, K, D)).astype(np.float32)
        arr = r.exponential(1.0, (G, N)).astype(np.float32)
        Y = r.standard_normal((G, N, C)).astype(np.float32)
        Xb = r.uniform(0, 1, (G, Kb, 64))
        clean = (orc.encode(Xb, alphab, betab) @ (r.standard_normal((64, Cb)) / 8)).astype(np.float32)
        mb = np.zeros((G, Nb), np.uint8)
        Yb = clean.copy()
        for g in range(G):
            avail = np.sort(r.permutation(Nb)[: Nb - Sb])
            mb[g, avail] = 1
            bad = np.sort(r.permutation(avail)[:Ab])
            Yb[g, bad] += (10 * clean.std() * r.standard_normal((Ab, Cb))).astype(np.float32)
        return X, arr, Y, Yb, mb

    def upload(inp):
        X, arr, Y, Yb, mb = inp
        q.copy_(torch.from_numpy(X)); arrival.copy_(torch.from_numpy(arr)); preds.copy_(torch.from_numpy(Y))
        predsb.copy_(torch.from_numpy(Yb)); maskb.copy_(torch.from_numpy(mb))

    def check(inp):
        X, arr, Y, Yb, mb = inp
        assert group_err(coded.cpu().numpy(), orc.encode(X, alpha, beta)).max() <= TOL
        m_ref, c_ref = orc.wait_mask(arr, N - S)
        assert np.array_equal(mask.cpu().numpy(), m_ref) and np.array_equal(count.cpu().numpy(), c_ref)
        ref, _ = orc.decode(Y, m_ref, alpha, beta, S, 1)
        assert group_err(out.cpu().numpy(), ref).max() <= TOL
        srt = np.sort(ref, axis=-1)
        clear = (srt[..., -1] - srt[..., -2]) > 1e-9 * np.abs(ref).max(axis=-1)
        assert np.array_equal(top1.cpu().numpy()[clear], ref.argmax(-1)[clear])
        refb, adv_ref, _ = orc.decode_byzantine(Yb, mb, alphab, betab, Sb, Ab, 1)
        assert np.array_equal(advb.cpu().numpy(), adv_ref)
        assert group_err(outb.cpu().numpy(), refb).max() <= TOL
        refh, adv_refh, _ = orc.decode_byzantine(Yb, mb, alphab, betab, Sb, Ab, 1, orc.LOCATOR_ALGORITHM_1)
        assert np.array_equal(advh.cpu().numpy(), adv_refh)
        assert group_err(outh.cpu().numpy(), refh).max() <= TOL

    first = fresh_inputs(1)
    upload(first)
    calls()                                                 # eager, also loads every kernel before the capture
    torch.cuda.synchronize()
    check(first)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            calls()                                         # the binding passes torch's current stream: the capturing one
    torch.cuda.synchronize()
    for seed in (2, 3, 4):                                  # replays with new contents, eager work in between
        inp = fresh_inputs(seed)
        upload(inp)
        for t in (coded, out, outb, outh):
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        check(inp)


# --------------------------------------------------------------------------------------
# seeded random shapes: every entry point, every limit in play
# --------------------------------------------------------------------------------------
def test_random_shapes_all_entry_points(gpu):
    # APPROXIFER_FUZZ_SEED / APPROXIFER_FUZZ_TRIALS widen the sweep by hand; the defaults are what the suite runs
    import os
    from parity_cases import FUZZ_ALL_SEED, FUZZ_ALL_TRIALS
    torch, binding, dev = gpu
    seed = int(os.environ.get("APPROXIFER_FUZZ_SEED", FUZZ_ALL_SEED))
    trials = int(os.environ.get("APPROXIFER_FUZZ_TRIALS", FUZZ_ALL_TRIALS))
    set_aside = 0
    for t in fuzz_all_cases(seed, trials):
        K, N, S, C, G, mode, alpha, beta = t["K"], t["N"], t["S"], t["C"], t["G"], t["mode"], t["alpha"], t["beta"]
        print("trial", t["trial"], dict(K=K, N=N, S=S, D=t["D"], C=C, G=G, mode=mode), flush=True)
        X, Y, mask = t["X"], t["Y"], t["mask"]
        coded = binding.approxifer_encode(torch.from_numpy(X).to(dev), alpha, beta).cpu().numpy()
        assert group_err(coded, orc.encode(X, alpha, beta)).max() <= TOL
        with np.errstate(all="ignore"):
            ref, st_ref = orc.decode(Y, mask, alpha, beta, S, mode)
        finite = np.all(np.isfinite(ref.reshape(G, -1)), axis=1) & well_posed(alpha, beta, mask, mode)
        set_aside += int(G - finite.sum())
        out, st = binding.approxifer_decode(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta, S, mode)
        assert np.array_equal(st.cpu().numpy(), st_ref)
        if finite.any():
            assert group_err(out.cpu().numpy()[finite], ref[finite]).max() <= TOL
        top1, score, st = binding.approxifer_decode_top1(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev),
                                                         alpha, beta, S, mode)
        if finite.any() and C > 1:
            srt = np.sort(ref[finite], axis=-1)
            clear = (srt[..., -1] - srt[..., -2]) > 1e-9 * np.abs(ref[finite]).max(axis=-1)
            assert np.array_equal(top1.cpu().numpy()[finite][clear], ref[finite].argmax(-1)[clear])
        # Byzantine decoder on a shape that satisfies its counting rule
        A, Kb, Sb, alphab, betab, Yb, maskb = t["A"], t["Kb"], t["Sb"], t["alphab"], t["betab"], t["Yb"], t["maskb"]
        outb, advb, stb = binding.approxifer_decode_byzantine(torch.from_numpy(Yb).to(dev), torch.from_numpy(maskb).to(dev),
                                                              alphab, betab, Sb, A, 1)
        refb, adv_ref, st_refb = orc.decode_byzantine(Yb, maskb, alphab, betab, Sb, A, 1)
        assert np.array_equal(stb.cpu().numpy(), st_refb)
        advb = advb.cpu().numpy()
        same = np.all(advb == adv_ref, axis=1)
        # a located set may differ from the oracle's only where a class's pick is a float64 rounding tie (a single
        # class, or separations at the noise floor), and then only by as many votes as there are such classes
        assert_rounding_ties(Yb, maskb, betab, Kb, A, advb, adv_ref)
        if same.any():
            assert group_err(outb.cpu().numpy()[same], refb[same]).max() <= TOL
    if (seed, trials) == (FUZZ_ALL_SEED, FUZZ_ALL_TRIALS):
        assert set_aside == ILL_POSED_FUZZ_ALL              # no decoded group left out beyond the oracle-side count


def test_random_byzantine_shapes(gpu):
    # every register tile of the projected kernel and the general kernel behind it, and Algorithm 1's locator on the
    # same inputs: K + A up to 16, up to 64 available workers, odd and even counts, per-group counts, one to a few
    # hundred classes; exactly rational data (linear model), so the planted adversaries must come back wherever
    # float32 data still separate them
    import os
    from parity_cases import FUZZ_BYZ_SEED, FUZZ_BYZ_TRIALS
    torch, binding, dev = gpu
    seed = int(os.environ.get("APPROXIFER_FUZZ_SEED", FUZZ_BYZ_SEED))
    trials = int(os.environ.get("APPROXIFER_FUZZ_TRIALS", FUZZ_BYZ_TRIALS))
    set_aside = 0
    for t in fuzz_byzantine_cases(seed, trials):
        K, A, S, N, C, G, ragged, mode = t["K"], t["A"], t["S"], t["N"], t["C"], t["G"], t["ragged"], t["mode"]
        alpha, beta, Y, mask, adv_true = t["alpha"], t["beta"], t["Y"], t["mask"], t["adv_true"]
        M = K + A
        print("trial", t["trial"], dict(K=K, A=A, S=S, N=N, C=C, G=G, ragged=ragged, mode=mode), flush=True)
        S_arg = binding.S_FROM_MASK if ragged else S
        for locator, entry in ((orc.LOCATOR_ALGORITHM_2, binding.approxifer_decode_byzantine),
                               (orc.LOCATOR_ALGORITHM_1, binding.approxifer_decode_byzantine_homogeneous)):
            out, adv, st = entry(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta, S_arg, A, mode)
            ref, adv_ref, st_ref = orc.decode_byzantine(Y, mask, alpha, beta, None if ragged else S, A, mode, locator)
            out, adv, st = out.cpu().numpy(), adv.cpu().numpy(), st.cpu().numpy()
            assert np.array_equal(st, st_ref) and np.all(st == 0)
            same = np.all(adv == adv_ref, axis=1)
            assert_rounding_ties(Y, mask, beta, K, A, adv, adv_ref, locator)
            if M <= 12 and C >= 7:
                assert np.array_equal(adv[same], adv_true[same]), locator
            for g in range(G):                               # decode parity over the kernel's own survivor set
                m2 = mask[g:g + 1].copy()
                m2[0, adv[g]] = 0
                if not well_posed(alpha, beta, m2, mode)[0]:
                    set_aside += 1
                    continue
                ref_g, _ = orc.decode(Y[g:g + 1], m2, alpha, beta, None, mode)
                assert group_err(out[g:g + 1], ref_g).max() <= TOL
    if (seed, trials) == (FUZZ_BYZ_SEED, FUZZ_BYZ_TRIALS):
        assert set_aside == ILL_POSED_FUZZ_BYZANTINE
