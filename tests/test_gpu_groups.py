"""GPU parity for Group Quantization and Normalization (Eq. 13-15 of arXiv 2310.11453):
the grouped entry points of the C ABI against the grouped CPU oracle.

Bits, alpha_g and beta_g: exact.  Codes: bit-exact given the normalised input the GPU dumped;
x^ against the oracle's fp64 group LayerNorm.  Output: the oracle adds the K-group terms in
fp64, the GPU in fp32 in the order g = 0, 1, ...: relative Frobenius error <= 1e-5 (a few
fp32 roundings) given the normalised input the GPU dumped, far inside the 1e-3 of the plain
layer that also holds end to end; with groups_k = 1 it is exact.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu
f32 = np.float32


@pytest.fixture(scope="module")
def bl():
    import paper_2310_11453_amd as lib
    lib.load_library()
    assert torch.cuda.is_available()
    return lib


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.cpu().numpy()


def layer(M, K, N, seed):
    W = wl.make_weight(N, K, 0.02, seed=wl.seed_for(0, seed))
    W[: N // 2] += f32(0.01)          # row groups with different means
    W[:, K // 2:] *= f32(1.5)         # column groups with different scales
    X = wl.make_activation(M, K, seed=wl.seed_for(0, seed + 1), outlier_p=0.01, outlier_mul=8.0)
    X[:, : K // 4] += f32(2.0)        # K-slices of a token with different statistics
    return X, W


GROUPS = [(1, 1), (2, 1), (1, 2), (4, 4), (8, 8), (1, 8), (8, 1)]


@pytest.mark.parametrize("gn,gk", GROUPS)
def test_grouped_pack(bl, gn, gk):
    """Eq. 13: per-block alpha, beta and bits."""
    N, K = 512, 2048
    print(f"grouped pack N={N} K={K} gn={gn} gk={gk}", flush=True)
    _, W = layer(1, K, N, 100 + gn * 10 + gk)
    a, b = oracle.weight_stats_grouped(W, gn, gk)
    words = oracle.pack_canonical(oracle.binarize_grouped(W, a))
    packed, alpha, beta = bl.bitlinear_pack_weights_grouped(dev(W), gn, gk)
    assert np.array_equal(host(alpha), a) and np.array_equal(host(beta), b)
    canon = host(bl.bitlinear_packed_to_canonical_grouped(packed, N, K, gk)).view(np.uint32)
    assert np.array_equal(canon, words)


@pytest.mark.parametrize("per_tensor", [False, True])
@pytest.mark.parametrize("gk", [2, 4, 8])
def test_grouped_quant(bl, gk, per_tensor):
    """Eq. 14-15: group LayerNorm and gamma per slice of a token."""
    M, K = 37, 1024
    print(f"grouped quant M={M} K={K} gk={gk} per_tensor={per_tensor}", flush=True)
    X, _ = layer(M, K, 16, 200 + gk)
    codes, gamma, rowsum, xhat = bl.bitlinear_quant_act_grouped(dev(X), gk, per_tensor=per_tensor,
                                                                want_xhat=True)
    xh = host(xhat)
    ref_xh = oracle.layernorm(X, groups=gk)
    assert np.abs(xh - ref_xh).max() <= 2e-6
    g_ref = oracle.absmax(xh, per_tensor, groups=gk)
    q_ref = oracle.quantize(xh, g_ref, per_tensor, groups=gk)
    assert np.array_equal(host(gamma).reshape(-1), g_ref.reshape(-1))
    assert np.array_equal(host(codes), q_ref)
    rs_ref = q_ref.astype(np.int32).reshape(M, gk, K // gk).sum(axis=2)
    assert np.array_equal(host(rowsum), rs_ref)


def _check_forward(bl, M, K, N, gn, gk, per_tensor, seed):
    X, W = layer(M, K, N, seed)
    packed, alpha, beta = bl.bitlinear_pack_weights_grouped(dev(W), gn, gk)
    y = host(bl.bitlinear_forward_grouped(dev(X), packed, N, beta, gn, gk, per_tensor=per_tensor))
    ref = oracle.forward_grouped(X, W, gn, gk, per_tensor=per_tensor)
    assert np.array_equal(host(beta), ref["beta"])
    # end to end from raw X: the GPU's x^ may differ from the oracle's in the last bit of fp32
    # (fp64 statistics summed in another order), which moves a code only at an exact tie
    err = np.linalg.norm(y.astype(np.float64) - ref["y64"]) / np.linalg.norm(ref["y64"])
    assert err <= 1e-3, err
    # given the normalised input the GPU itself rounded: gamma_g, codes and row sums exactly, and
    # then the only difference left in Y is the fp32 order of the group sums (the oracle adds the
    # slices in fp64): 1e-5, and nothing at all with one K-group
    codes, gamma, rowsum, xhat = bl.bitlinear_quant_act_grouped(dev(X), gk, per_tensor=per_tensor,
                                                                want_xhat=True)
    given = oracle.forward_grouped(X, W, gn, gk, per_tensor=per_tensor, xhat=host(xhat))
    assert np.array_equal(host(codes), given["codes"])
    assert np.array_equal(host(gamma).reshape(-1), np.asarray(given["gamma"]).reshape(-1))
    err = np.linalg.norm(y.astype(np.float64) - given["y64"]) / np.linalg.norm(given["y64"])
    assert err <= 1e-5, err
    if gk == 1:
        assert np.array_equal(y, given["y"])
    return err


@pytest.mark.parametrize("gn,gk", GROUPS)
@pytest.mark.parametrize("M", [8, 24, 48, 100])
def test_grouped_forward(bl, M, gn, gk):
    """One batch size for each of the four ranges of the batch (up to 16, 17-32, 33-64 tokens and, above
    that, the small tiles, with K-groups as slices), per-token gamma.  The kernels for large layers have
    tests of their own below."""
    K, N = 2048, 512
    print(f"grouped forward M={M} K={K} N={N} gn={gn} gk={gk}", flush=True)
    _check_forward(bl, M, K, N, gn, gk, False, 300 + gn * 10 + gk)


@pytest.mark.parametrize("M", [4, 300])
def test_grouped_forward_per_tensor(bl, M):
    print(f"grouped forward per-tensor M={M}", flush=True)
    _check_forward(bl, M, 1024, 256, 4, 4, True, 400 + M)


def test_grouped_forward_ragged(bl):
    """Shapes that are not multiples of the kernels' tiles: N = 3 * 80, K = 4 * 96."""
    print("grouped forward ragged", flush=True)
    _check_forward(bl, 70, 384, 240, 3, 4, False, 500)
    _check_forward(bl, 5, 384, 240, 3, 4, False, 501)
    _check_forward(bl, 19, 384, 240, 3, 4, False, 502)
    _check_forward(bl, 33, 384, 240, 3, 4, False, 503)


@pytest.mark.parametrize("M,K,N,gn,gk", [(5, 16384, 256, 1, 8),   # 16 waves of two chunks
                                         (9, 6144, 256, 2, 4),    # 12 waves of one chunk
                                         (4, 4512, 8192, 1, 3),   # 9 waves, two tiles each, one round: codes parked
                                         (7, 4512, 8224, 2, 3),   # 9 waves, more than one round: codes read in place
                                         (16, 7104, 16416, 3, 2), # 14 waves, three rounds, K past a chunk's end
                                         (3, 32768, 128, 1, 8),   # too many chunks for one workgroup
                                         (40, 8192, 384, 1, 2),   # 33-64 tokens, long K-groups
                                         (64, 3072, 256, 2, 6)])  # 33-64 tokens, six groups in two items
def test_grouped_forward_group_placement(bl, tuning, M, K, N, gn, gk):
    """Up to 64 tokens the K-groups share workgroups where they fit (waves dealt to the groups in
    the small-batch kernel, one K-group of the workgroup per layer group in the mid-batch one) and
    are work items of their own otherwise; both placements give the same bits."""
    print(f"grouped placement M={M} K={K} N={N} gn={gn} gk={gk}", flush=True)
    _check_forward(bl, M, K, N, gn, gk, False, 600 + M)
    X, W = layer(M, K, N, 600 + M)
    packed, alpha, beta = bl.bitlinear_pack_weights_grouped(dev(W), gn, gk)
    y0 = host(bl.bitlinear_forward_grouped(dev(X), packed, N, beta, gn, gk))
    tuning("group_slices=1")
    y1 = host(bl.bitlinear_forward_grouped(dev(X), packed, N, beta, gn, gk))
    assert np.array_equal(y0, y1)


def force_group_stream(bl, tuning, op, M, K, N, gn, gk, grid, per_tensor):
    """Above 64 tokens: the kernel that walks a tile's K-groups, on `grid` workgroups, instead of the K-groups
    as slices.  Seen in the workspace: the call then asks for no slices."""
    tuning("prefill_tile=3")
    sliced = bl.workspace_bytes_grouped(op, M, N, K, gn, gk, per_tensor)
    tuning(f"prefill_tile=1,prefill_grid={grid}")
    assert bl.workspace_bytes_grouped(op, M, N, K, gn, gk, per_tensor) == sliced - gk * M * N * 4


# groups of one stage, two stages, one chunk, one stage past a chunk, an odd number of chunks and a K that
# ends inside a stage, on few enough workgroups that each walks several tiles
GROUP_STREAM_SHAPES = [(130, 32, 272, 1, 5, 2), (300, 64, 528, 3, 8, 2), (257, 96, 512, 1, 3, 1),
                       (300, 160, 272, 1, 4, 3), (129, 512, 288, 2, 2, 2), (200, 544, 520, 1, 4, 2),
                       (512, 576, 1024, 8, 2, 8), (150, 1120, 256, 1, 3, 1)]


@pytest.mark.parametrize("per_tensor", [False, True])
@pytest.mark.parametrize("M,Kg,N,gn,gk,grid", GROUP_STREAM_SHAPES)
def test_grouped_forward_large_batch_stream(bl, tuning, M, Kg, N, gn, gk, grid, per_tensor):
    """More than 64 tokens: the operand stream runs on across the ends of groups and tiles."""
    print(f"grouped stream M={M} Kg={Kg} N={N} gn={gn} gk={gk} grid={grid} per_tensor={per_tensor}", flush=True)
    force_group_stream(bl, tuning, bl.OP_FORWARD, M, Kg * gk, N, gn, gk, grid, per_tensor)
    _check_forward(bl, M, Kg * gk, N, gn, gk, per_tensor, 700 + M)


@pytest.mark.parametrize("per_tensor", [False, True])
@pytest.mark.parametrize("tile", [1, 2])
def test_grouped_forward_column_groups_large_tiles(bl, tuning, tile, per_tensor):
    """The large tiles with a beta per column group (one K-group), several tiles per workgroup."""
    M, K, N, gn = 300, 544, 528, 3
    print(f"column groups M={M} K={K} N={N} gn={gn} tile={tile} per_tensor={per_tensor}", flush=True)
    tuning(f"prefill_tile={tile},prefill_grid=2")
    _check_forward(bl, M, K, N, gn, 1, per_tensor, 750)


@pytest.mark.parametrize("M,Kg,N,gn,gk", [(65, 96, 272, 1, 5), (200, 544, 528, 3, 4), (130, 2080, 37, 1, 2)])
def test_grouped_forward_large_batch_slices(bl, tuning, M, Kg, N, gn, gk):
    """More than 64 tokens: every K-group an item of its own with its sums in a slice, on both tile
    heights, against the oracle and, bit for bit, against the kernel that walks a tile's groups."""
    print(f"grouped large-batch slices M={M} Kg={Kg} N={N} gn={gn} gk={gk}", flush=True)
    X, W = layer(M, Kg * gk, N, 800 + M)
    packed, alpha, beta = bl.bitlinear_pack_weights_grouped(dev(W), gn, gk)
    tuning("prefill_tile=1")
    y0 = host(bl.bitlinear_forward_grouped(dev(X), packed, N, beta, gn, gk))
    for tile in (3, 4):
        tuning(f"prefill_tile={tile}")
        assert np.array_equal(host(bl.bitlinear_forward_grouped(dev(X), packed, N, beta, gn, gk)), y0)
        _check_forward(bl, M, Kg * gk, N, gn, gk, False, 800 + M)


# The fold of the K-groups' sums: one column a thread below 2^18 outputs, four from there on where N is a multiple of
# four; one row, rows that end inside a workgroup, more groups than columns of scales in a line.
@pytest.mark.parametrize("per_tensor", [False, True])
@pytest.mark.parametrize("M,Kg,N,gn,gk", [(1, 64, 48, 3, 2), (16, 160, 16384, 4, 3), (64, 96, 4097, 1, 4),
                                          (63, 96, 4160, 4, 4), (64, 96, 4100, 1, 9), (130, 544, 2032, 1, 2)])
def test_fold_of_groups(bl, tuning, M, Kg, N, gn, gk, per_tensor):
    print(f"fold of groups M={M} Kg={Kg} N={N} gn={gn} gk={gk} per_tensor={per_tensor}", flush=True)
    K, Ng = Kg * gk, N // gn
    X, W = layer(M, K, N, 900 + M + gk)
    packed, _, beta = bl.bitlinear_pack_weights_grouped(dev(W), gn, gk)
    if M > 64:
        tuning("prefill_tile=4")
    y = bl.bitlinear_forward_grouped(dev(X), packed, N, beta, gn, gk, per_tensor=per_tensor)
    # each block by itself, its terms added in fp32 in the order of the groups: the same bits
    codes, gamma, rowsum, _ = bl.bitlinear_quant_act_grouped(dev(X), gk, per_tensor=per_tensor)
    ref = None
    for g in range(gk):
        sl = slice(g * Kg, (g + 1) * Kg)
        gam = gamma.reshape(-1, gk)[:, g].contiguous()
        cols = []
        for n in range(gn):
            p, _, b = bl.bitlinear_pack_weights(dev(W[n * Ng:(n + 1) * Ng, sl]))
            cols.append(bl.bitlinear_matmul(codes[:, sl].contiguous(), gam, rowsum.reshape(M, gk)[:, g].contiguous(),
                                            p, Ng, b, per_tensor=per_tensor))
        term = torch.cat(cols, 1)
        ref = term if ref is None else term + ref
    assert torch.equal(y, ref)


@pytest.mark.parametrize("M,Kg,N,gn,gk", [(130, 96, 272, 1, 2), (70, 544, 40, 1, 3)])
def test_grouped_forward_zero_keeps_its_sign(bl, tuning, M, Kg, N, gn, gk):
    """Weights of zero (beta_g = 0): every group's term is a zero with the sign of its integer sum, and the
    sum of the groups, added in the order 0, 1, ..., has the same sign bits from either kernel."""
    print(f"grouped zeros M={M} Kg={Kg} N={N} gn={gn} gk={gk}", flush=True)
    X, _ = layer(M, Kg * gk, N, 900 + M)
    packed, alpha, beta = bl.bitlinear_pack_weights_grouped(dev(np.zeros((N, Kg * gk), f32)), gn, gk)
    _, gamma, rowsum, _ = bl.bitlinear_quant_act_grouped(dev(X), gk)
    zeros = (-host(rowsum).reshape(M, gk)).astype(f32) * f32(0)  # all weights are -1: the integer sums are -rowsum
    ref = zeros[:, 0]
    for g in range(1, gk):
        ref = zeros[:, g] + ref
    assert np.signbit(ref).any() and not np.signbit(ref).all()
    for tile in (1, 3, 4):
        tuning(f"prefill_tile={tile}")
        y = host(bl.bitlinear_forward_grouped(dev(X), packed, N, beta, gn, gk))
        assert np.array_equal(y.view(np.uint32), np.repeat(ref[:, None], N, 1).view(np.uint32)), tile


def test_grouped_forward_full_size_30b(bl):
    """A 30B-shaped layer (7168 -> 28672) with eight groups on each axis, decode and prefill batch:
    alpha_g, beta_g and all bits; codes and gamma_g given the normalised input the GPU dumped;
    outputs on a stratified sample against the oracle's per-group sums."""
    K, N, G = 7168, 28672, 8
    W = wl.make_weight(N, K, 0.01, seed=wl.seed_for(3, 40))
    W[: N // 2] += f32(0.003)
    a, b = oracle.weight_stats_grouped(W, G, G)
    sign = oracle.binarize_grouped(W, a)
    packed, alpha, beta = bl.bitlinear_pack_weights_grouped(dev(W), G, G)
    del W
    assert np.array_equal(host(alpha), a) and np.array_equal(host(beta), b)
    canon = host(bl.bitlinear_packed_to_canonical_grouped(packed, N, K, G)).view(np.uint32)
    assert np.array_equal(canon, oracle.pack_canonical(sign))
    del canon
    Kg, Ng = K // G, N // G
    for M in (16, 300):
        print(f"grouped full size M={M}", flush=True)
        X = wl.make_activation(M, K, seed=wl.seed_for(3, 41 + M))
        X[:, : K // 4] += f32(1.0)
        y = host(bl.bitlinear_forward_grouped(dev(X), packed, N, beta, G, G))
        codes, gamma, rowsum, xhat = bl.bitlinear_quant_act_grouped(dev(X), G, want_xhat=True)
        xh = host(xhat)
        g_ref = oracle.absmax(xh, False, groups=G)
        q_ref = oracle.quantize(xh, g_ref, False, groups=G)
        assert np.array_equal(host(gamma).reshape(-1), g_ref) and np.array_equal(host(codes), q_ref)
        rng = np.random.default_rng(M)
        gm, gn = (M + 63) // 64, N // 64
        rows = np.minimum((np.arange(gm) * 64)[:, None] + rng.integers(0, 64, (gm, gn)), M - 1).ravel()
        cols = ((np.arange(gn) * 64)[None, :] + rng.integers(0, 64, (gm, gn))).ravel()
        gam = g_ref.reshape(M, G)
        ysum = np.zeros(rows.size)
        for g in range(G):  # each K-group dequantised with its own beta_g gamma_g, added in fp64
            acc = oracle.matmul_i32_sampled(np.ascontiguousarray(q_ref[:, g * Kg:(g + 1) * Kg]),
                                            np.ascontiguousarray(sign[:, g * Kg:(g + 1) * Kg]), rows, cols)
            sc = (b[cols // Ng, g] * gam[rows, g]) / f32(128.0)
            ysum += (acc.astype(f32) * sc).astype(np.float64)
        got = y[rows, cols].astype(np.float64)
        assert np.abs(got - ysum).max() <= 1e-5 * np.sqrt(np.mean(ysum ** 2))


def test_groups_of_one_match_the_plain_entry_points(bl):
    M, K, N = 50, 512, 256
    X, W = layer(M, K, N, 600)
    p0, a0, b0 = bl.bitlinear_pack_weights(dev(W))
    p1, a1, b1 = bl.bitlinear_pack_weights_grouped(dev(W), 1, 1)
    assert torch.equal(p0, p1) and torch.equal(a0, a1.reshape(-1)) and torch.equal(b0, b1.reshape(-1))
    y0 = bl.bitlinear_forward(dev(X), p0, N, b0)
    y1 = bl.bitlinear_forward_grouped(dev(X), p1, N, b1, 1, 1)
    assert torch.equal(y0, y1)


def test_grouped_argument_errors(bl):
    lib = bl.load_library()
    # groups that do not divide, or K-groups that are not multiples of 32: bad shape
    assert lib.bitlinear_packed_bytes_grouped(512, 2048, 3, 1) == 0
    assert lib.bitlinear_packed_bytes_grouped(512, 96, 1, 2) == 0
    # row groups that are not whole 16-row tiles: unsupported
    assert lib.bitlinear_packed_bytes_grouped(96, 64, 4, 1) == 0
    assert lib.bitlinear_packed_bytes_grouped(512, 2048, 8, 8) == 8 * (512 // 16) * 1024
    with pytest.raises(bl.BitLinearError):
        bl.bitlinear_pack_weights_grouped(dev(np.zeros((96, 64), f32)), 4, 1)
