"""GPU parity of the straight-through-estimator backward (Section 2.2 of arXiv 2310.11453)
against the CPU oracle: same bf16-rounded dY on both sides, fp32 accumulation on the GPU
against fp64 in the oracle.  Bar: relative Frobenius error <= 1e-3 (measured ~1e-6) and
max error <= 1e-3 of the rms."""
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


def close(a, ref):
    ref64 = ref.astype(np.float64)
    rms = np.sqrt(np.mean(ref64 ** 2)) + 1e-30
    assert np.linalg.norm(a - ref64) <= 1e-3 * np.linalg.norm(ref64) + 1e-30
    assert np.abs(a - ref64).max() <= 1e-3 * rms


# several tiles with ragged tails in every dimension, and both granularities of gamma
SHAPES = [(8, 512, 256), (12, 20, 64), (300, 200, 96), (64, 136, 1056), (257, 513, 544),
          (1024, 640, 512), (65, 3, 32), (1, 1, 96)]


# The library picks dW's tile from the shape (256 x 256, or 128 x 128 where that costs less); the bwd_ring
# switch forces either one so that both see the ragged shapes.
@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("per_tensor", [True, False])
@pytest.mark.parametrize("ring", ["2", "1"])
def test_backward_ste_matches_oracle(bl, tuning, M, N, K, per_tensor, ring):
    print(f"backward M={M} N={N} K={K} per_tensor={per_tensor} ring={ring}", flush=True)
    tuning(f"bwd_ring={ring}")
    sd = wl.seed_for(4, M + N + K)
    W = wl.make_weight(N, K, 0.02, sd)
    X = wl.make_activation(M, K, sd)
    dY = wl.make_grad(M, N, sd)
    packed, alpha, beta = bl.bitlinear_pack_weights(dev(W))
    codes, gamma, rowsum, _ = bl.bitlinear_quant_act(dev(X), per_tensor=per_tensor)
    dX, dW = bl.bitlinear_backward_ste(dev(dY), codes, gamma, packed, beta, per_tensor)
    sign = oracle.unpack_canonical(
        bl.bitlinear_packed_to_canonical(packed, N, K).cpu().numpy().view(np.uint32), K)
    dX_ref, dW_ref = oracle.backward_ste(dY, codes.cpu().numpy(), gamma.cpu().numpy(), sign,
                                         float(beta.cpu()[0]), per_tensor)
    close(dX.cpu().numpy(), dX_ref)
    close(dW.cpu().numpy(), dW_ref)
    # either output alone
    dX2, none = bl.bitlinear_backward_ste(dev(dY), codes, gamma, packed, beta, per_tensor,
                                          want_dw=False)
    assert none is None and torch.equal(dX2, dX)
    none, dW2 = bl.bitlinear_backward_ste(dev(dY), codes, gamma, None, beta, per_tensor,
                                          want_dx=False)
    assert none is None and torch.equal(dW2, dW)


# The copies of the operands come out of one launch, with four elements a load where rows and pointer allow it: the
# four combinations of that for dY and the codes give the same bits.
@pytest.mark.parametrize("M,N,K", [(70, 68, 96), (33, 1000, 544), (130, 66, 32), (129, 131, 64)])
@pytest.mark.parametrize("per_tensor", [True, False])
def test_backward_operands_at_any_alignment(bl, M, N, K, per_tensor):
    def moved(t):  # the same values one element behind an aligned address
        flat = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:]
        return flat.copy_(t.reshape(-1)).view(t.shape)

    packed, _, beta = bl.bitlinear_pack_weights(dev(wl.make_weight(N, K, 0.02, 5)))
    codes, gamma, _, _ = bl.bitlinear_quant_act(dev(wl.make_activation(M, K, 6)), per_tensor=per_tensor)
    dY = dev(wl.make_grad(M, N, 7))
    dX, dW = bl.bitlinear_backward_ste(dY, codes, gamma, packed, beta, per_tensor)
    for y, c in ((moved(dY), codes), (dY, moved(codes)), (moved(dY), moved(codes))):
        dX2, dW2 = bl.bitlinear_backward_ste(y, c, gamma, packed, beta, per_tensor)
        assert torch.equal(dX2, dX) and torch.equal(dW2, dW)


@pytest.mark.parametrize("spec,N", [("bwd_ring=1,bwd_grid=8", 520), ("bwd_ring=2,bwd_grid=4", 520),
                                    ("bwd_ring=2,bwd_grid=8", 1024)])
def test_backward_ring_kernel_walks_several_tiles(bl, tuning, spec, N):
    """The persistent kernels with fewer workgroups than tiles (the bwd_grid switch): dX has 16
    tiles on 8 workgroups, dW 12 of 256 x 256 on 8, then 40 of 128 x 128 on 8 and 64 on 16 (the tile order
    that groups tiles by L2)."""
    tuning(spec)
    M, K = 1024, 1024
    sd = wl.seed_for(4, 77)
    print(f"backward ring {spec} M={M} N={N} K={K}", flush=True)
    W = wl.make_weight(N, K, 0.02, sd)
    X = wl.make_activation(M, K, sd)
    dY = wl.make_grad(M, N, sd)
    packed, alpha, beta = bl.bitlinear_pack_weights(dev(W))
    codes, gamma, rowsum, _ = bl.bitlinear_quant_act(dev(X), per_tensor=False)
    dX, dW = bl.bitlinear_backward_ste(dev(dY), codes, gamma, packed, beta, False)
    sign = oracle.unpack_canonical(
        bl.bitlinear_packed_to_canonical(packed, N, K).cpu().numpy().view(np.uint32), K)
    dX_ref, dW_ref = oracle.backward_ste(dY, codes.cpu().numpy(), gamma.cpu().numpy(), sign,
                                         float(beta.cpu()[0]), False)
    close(dX.cpu().numpy(), dX_ref)
    close(dW.cpu().numpy(), dW_ref)


# dX in tiles of 256 and of 128 rows: one row, the rows around a tile's last, fewer stages than the ring and one more,
# columns of a second tile, slices, and several tiles a workgroup (with the tile order that groups tiles by L2).
# On integers, so exact.
@pytest.mark.parametrize("M,N,K", [(1, 32, 32), (127, 96, 256), (128, 130, 288), (129, 160, 544), (257, 520, 96),
                                   (1024, 136, 1024)])
@pytest.mark.parametrize("spec", ["", "bwd_splits=2", "bwd_grid=8"])
@pytest.mark.parametrize("rows", [1, 2])
def test_backward_dx_tiles_exact(bl, tuning, M, N, K, spec, rows):
    print(f"backward dX M={M} N={N} K={K} {spec} bwd_dx={rows}", flush=True)
    tuning(",".join(filter(None, [spec, f"bwd_dx={rows}"])))
    rng = np.random.default_rng(M + N)
    dY = rng.integers(-4, 5, (M, N)).astype(f32)
    packed, _, _ = bl.bitlinear_pack_weights(dev(wl.make_weight(N, K, 0.02, 5)))
    sign = oracle.unpack_canonical(
        bl.bitlinear_packed_to_canonical(packed, N, K).cpu().numpy().view(np.uint32), K)
    codes, one = torch.zeros(M, K, dtype=torch.int8, device="cuda"), torch.ones(1, device="cuda")
    dX, _ = bl.bitlinear_backward_ste(dev(dY), codes, one, packed, one, True, want_dw=False)
    assert np.array_equal(dX.cpu().numpy(), (dY.astype(np.int64) @ sign.astype(np.int64)).astype(f32))


@pytest.mark.parametrize("ring", ["2", "1"])
def test_backward_exact_when_dy_is_bf16_representable(bl, tuning, ring):
    """Small integers in dY, codes and signs: every product and partial sum is exact in fp32,
    so the GPU must reproduce the integer result bit for bit (catches layout mistakes that a
    tolerance would hide)."""
    tuning(f"bwd_ring={ring}")
    M, N, K = 96, 80, 160
    rng = np.random.default_rng(3)
    W = wl.make_weight(N, K, 0.02, 5)
    X = wl.make_activation(M, K, 5)
    dY = rng.integers(-4, 5, (M, N)).astype(f32)
    packed, alpha, beta = bl.bitlinear_pack_weights(dev(W))
    codes, gamma, rowsum, _ = bl.bitlinear_quant_act(dev(X), per_tensor=True)
    one = torch.ones(1, device="cuda")
    g128 = torch.full((1,), 128.0, device="cuda")
    dX, dW = bl.bitlinear_backward_ste(dev(dY), codes, g128, packed, one, True)
    sign = oracle.unpack_canonical(
        bl.bitlinear_packed_to_canonical(packed, N, K).cpu().numpy().view(np.uint32), K)
    q = codes.cpu().numpy().astype(np.int64)
    assert np.array_equal(dX.cpu().numpy(), (dY.astype(np.int64) @ sign.astype(np.int64)).astype(f32))
    assert np.array_equal(dW.cpu().numpy(), (dY.astype(np.int64).T @ q).astype(f32))


def test_backward_training_shape_sampled(bl):
    """Training-step shape (M=8192, 4096->16384, per-tensor gamma): sampled rows of dX and dW
    against the oracle."""
    M, K, N = 8192, 4096, 16384
    sd = wl.seed_for(4, 0)
    print(f"backward full M={M} N={N} K={K}", flush=True)
    W = wl.make_weight(N, K, 0.02, sd)
    X = wl.make_activation(M, K, sd)
    dY = wl.make_grad(M, N, sd)
    packed, alpha, beta = bl.bitlinear_pack_weights(dev(W))
    a, b = oracle.weight_stats(W)
    sign = oracle.binarize(W, a)
    del W
    codes, gamma, rowsum, _ = bl.bitlinear_quant_act(dev(X), per_tensor=True)
    del X
    dX, dW = bl.bitlinear_backward_ste(dev(dY), codes, gamma, packed, beta, True)
    rng = np.random.default_rng(11)
    rows_dx = np.concatenate([[0, 1, 4097, 8191], rng.integers(0, M, 12)])
    rows_dw = np.concatenate([[0, 255, 256, 16383], rng.integers(0, N, 12)])
    dX_ref, dW_ref = oracle.backward_ste(dY, codes.cpu().numpy(), gamma.cpu().numpy(), sign,
                                         float(b), True, rows_dx=rows_dx, rows_dw=rows_dw)
    close(dX.cpu().numpy()[rows_dx], dX_ref)
    close(dW.cpu().numpy()[rows_dw], dW_ref)


@pytest.mark.parametrize("M,N,K", [(8, 512, 256), (290, 520, 288), (96, 1056, 1024), (513, 2080, 544)])
@pytest.mark.parametrize("splits", [2, 3, 7])
def test_backward_slices_of_the_reduction_exact(bl, tuning, M, N, K, splits):
    """Both ring kernels with the reduction cut into slices (last slice shorter, slices of one stage,
    slices shorter than the ring) and folded, on integers: exact.  With a workspace that only holds
    the operand copies the product runs unsliced, with the same result."""
    print(f"backward slices M={M} N={N} K={K} splits={splits}", flush=True)
    tuning(f"bwd_splits={splits}")
    Np, Mp = (N + 31) // 32 * 32, (M + 31) // 32 * 32
    small = sum((b + 255) // 256 * 256 for b in (2 * M * Np, Np // 32 * K * 4, 2 * N * Mp, 2 * K * Mp)) + 256
    assert bl.workspace_bytes(bl.OP_BACKWARD, M, N, K, True) > small
    rng = np.random.default_rng(M + splits)
    W = wl.make_weight(N, K, 0.02, 5)
    dY = rng.integers(-4, 5, (M, N)).astype(f32)
    q = rng.integers(-128, 128, (M, K)).astype(np.int8)
    packed, _, _ = bl.bitlinear_pack_weights(dev(W))
    one = torch.ones(1, device="cuda")
    g128 = torch.full((1,), 128.0, device="cuda")
    sign = oracle.unpack_canonical(
        bl.bitlinear_packed_to_canonical(packed, N, K).cpu().numpy().view(np.uint32), K)
    dX_ref = (dY.astype(np.int64) @ sign.astype(np.int64)).astype(f32)
    dW_ref = (dY.astype(np.int64).T @ q.astype(np.int64)).astype(f32)
    for ws in (None, torch.empty(small, dtype=torch.uint8, device="cuda")):
        dX, dW = bl.bitlinear_backward_ste(dev(dY), dev(q), g128, packed, one, True, workspace=ws)
        assert np.array_equal(dX.cpu().numpy(), dX_ref)
        assert np.array_equal(dW.cpu().numpy(), dW_ref)


@pytest.mark.parametrize("per_tensor", [True, False])
def test_backward_without_tokens(bl, per_tensor):
    """A batch of zero tokens is a no-op through the binding too (which asks for the workspace first)."""
    N, K = 512, 256
    print(f"backward M=0 per_tensor={per_tensor}", flush=True)
    packed, _, beta = bl.bitlinear_pack_weights(dev(wl.make_weight(N, K, 0.02, 5)))
    dX, dW = bl.bitlinear_backward_ste(torch.empty((0, N), device="cuda"),
                                       torch.empty((0, K), dtype=torch.int8, device="cuda"),
                                       torch.ones(1, device="cuda"), packed, beta, per_tensor)
    assert dX.shape == (0, K) and dW.shape == (N, K)


@pytest.mark.parametrize("M,N,K", [(290, 520, 288), (513, 2080, 544)])
@pytest.mark.parametrize("per_tensor", [True, False])
def test_backward_slices_are_within_tolerance_of_uncut(bl, tuning, M, N, K, per_tensor):
    """Real values: slices change the order of the fp32 sums, so dX and dW may differ from the uncut ones in
    the last bits; both are as close to the oracle.  A rounding is at most 2^-24 of the running sum; R of them, of
    either sign, come to about sqrt(R) 2^-24 of the result's rms, 2.7e-6 at R = 2080, on each side: 1e-5."""
    print(f"backward slices, real values M={M} N={N} K={K} per_tensor={per_tensor}", flush=True)
    sd = wl.seed_for(4, M + N + K)
    W, X, dY = wl.make_weight(N, K, 0.02, sd), wl.make_activation(M, K, sd), wl.make_grad(M, N, sd)
    packed, alpha, beta = bl.bitlinear_pack_weights(dev(W))
    codes, gamma, rowsum, _ = bl.bitlinear_quant_act(dev(X), per_tensor=per_tensor)
    sign = oracle.unpack_canonical(
        bl.bitlinear_packed_to_canonical(packed, N, K).cpu().numpy().view(np.uint32), K)
    ref = oracle.backward_ste(dY, codes.cpu().numpy(), gamma.cpu().numpy(), sign, float(beta.cpu()[0]), per_tensor)
    uncut = None
    for splits in (1, 3):
        tuning(f"bwd_splits={splits}")
        got = [t.cpu().numpy().astype(np.float64)
               for t in bl.bitlinear_backward_ste(dev(dY), codes, gamma, packed, beta, per_tensor)]
        for g, r in zip(got, ref):
            close(g, r)
        for g, u in zip(got, uncut or got):
            assert np.linalg.norm(g - u) <= 1e-5 * np.linalg.norm(u)
        uncut = got
