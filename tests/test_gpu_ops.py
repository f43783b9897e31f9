"""GPU parity of the single operations exported by the C ABI against the oracle's steps."""
import numpy as np
import pytest
import torch

import oracle
from paper_2504_14775_amd import binding as B
from paper_2504_14775_amd import synth
from gpu_util import DEV, bits_of, tiled_bits, to_dev_bits, to_dev_weight

pytestmark = pytest.mark.gpu


def rand_bits(seed, stream, shape, sigma):
    n = int(np.prod(shape))
    return synth.bf16_bits(synth.normal_bf16(seed, stream, 0, n, sigma)).reshape(shape)


def padded_rows(bits, rows):
    out = np.zeros((rows, bits.shape[1]), dtype=np.uint16)
    out[: bits.shape[0]] = bits
    return out


@pytest.mark.parametrize("tile", [-1, 0, 1, 3, 6, 7])
@pytest.mark.parametrize("M,N,K", [(1, 256, 64), (52, 512, 256), (300, 768, 192), (257, 1280, 704), (1024, 256, 2048)])
def test_gemm_store_and_add(M, N, K, tile):
    print(f"gemm store/add M={M} N={N} K={K} tile={tile}", flush=True)
    a = rand_bits(1, 1, (M, K), 1.0)
    w = rand_bits(1, 2, (N, K), 0.05)
    ref = oracle.linear(oracle.bf16_to_f64(a), w)
    Mp = (M + 255) // 256 * 256
    da, dw = to_dev_bits(padded_rows(a, Mp)), to_dev_weight(w)
    out = torch.full((M, N), 7.0, dtype=torch.float32, device=DEV)
    B.gllm_op_gemm_bf16(da, dw, out, M, N, K, B.GEMM_STORE_F32, tile)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    scale = np.abs(ref).max()
    assert np.abs(got - ref).max() <= 2e-5 * scale + 1e-6
    B.gllm_op_gemm_bf16(da, dw, out, M, N, K, B.GEMM_ADD_F32, tile)
    torch.cuda.synchronize()
    got2 = out.cpu().numpy().astype(np.float64)
    assert np.abs(got2 - 2 * ref).max() <= 4e-5 * scale + 1e-6


@pytest.mark.parametrize("tile", [-1, 0, 1, 3, 6, 7])
@pytest.mark.parametrize("M,I,K", [(52, 768, 256), (130, 128, 128), (300, 1408, 320)])
def test_gemm_swiglu(M, I, K, tile):
    print(f"gemm swiglu M={M} I={I} K={K} tile={tile}", flush=True)
    a = rand_bits(2, 1, (M, K), 1.0)
    wg = rand_bits(2, 2, (I, K), 0.08)
    wu = rand_bits(2, 3, (I, K), 0.08)
    x = oracle.bf16_to_f64(a)
    ref = oracle.swiglu(oracle.linear(x, wg), oracle.linear(x, wu))
    # interleave as the ABI states: groups of 64 rows = 32 gate rows then the 32 matching up rows
    assert I % 128 == 0
    packed = np.zeros((2 * I, K), dtype=np.uint16)
    for blk in range(I // 32):
        packed[64 * blk: 64 * blk + 32] = wg[32 * blk: 32 * blk + 32]
        packed[64 * blk + 32: 64 * blk + 64] = wu[32 * blk: 32 * blk + 32]
    Mp = (M + 255) // 256 * 256
    out = torch.zeros((M, I), dtype=torch.bfloat16, device=DEV)
    B.gllm_op_gemm_bf16(to_dev_bits(padded_rows(a, Mp)), to_dev_weight(packed), out, M, 2 * I, K, B.GEMM_SWIGLU_BF16, tile)
    torch.cuda.synchronize()
    got = oracle.bf16_to_f64(bits_of(out))
    err = np.abs(got - ref)
    assert np.all(err <= np.abs(ref) * 2.0 ** -7 + 1e-4), float(err.max())


@pytest.mark.parametrize("T,H", [(3, 256), (52, 4096), (17, 5120)])
def test_rmsnorm(T, H):
    print(f"rmsnorm T={T} H={H}", flush=True)
    x = synth.normal_bf16(3, 1, 0, T * H, 2.0).to(torch.float32).reshape(T, H) * 1.37
    gamma = rand_bits(3, 2, (H,), 0.5)
    ref = oracle.rmsnorm(x.numpy().astype(np.float64), gamma, 1e-6)
    h = torch.empty((T, H), dtype=torch.bfloat16, device=DEV)
    B.gllm_op_rmsnorm(x.to(DEV), to_dev_bits(gamma), h, 1e-6)
    torch.cuda.synchronize()
    got = oracle.bf16_to_f64(bits_of(h))
    assert np.all(np.abs(got - ref) <= np.abs(ref) * 2.0 ** -8 * 1.01 + 1e-6)


@pytest.mark.parametrize("T,H", [(1, 1024), (1, 1028), (200, 4100), (256, 8192), (257, 8192), (256, 16384), (257, 16384)])
def test_rmsnorm_rows_and_widths_at_the_edges_of_its_forms(T, H):
    """Up to 256 rows a row has 1024 threads, more rows or at most 1024 columns 256: both sides of each edge, same bound as
    above (one rounding to bf16, plus 1 % of it for the fp32 sum)."""
    test_rmsnorm(T, H)


@pytest.mark.parametrize("M,N,K", [(300, 768, 192), (2, 192, 64), (513, 1536, 128)])
def test_gemm_256x192_tile(M, N, K):
    print(f"gemm 256x192 tile M={M} N={N} K={K}", flush=True)
    a = rand_bits(6, 1, (M, K), 1.0)
    w = rand_bits(6, 2, (N, K), 0.05)
    ref = oracle.linear(oracle.bf16_to_f64(a), w)
    Mp = (M + 255) // 256 * 256
    out = torch.full((M, N), 3.0, dtype=torch.float32, device=DEV)
    wpad = np.zeros(((N + 255) // 256 * 256, K), dtype=np.uint16); wpad[:N] = w
    B.gllm_op_gemm_bf16(to_dev_bits(padded_rows(a, Mp)), to_dev_weight(wpad), out, M, N, K, B.GEMM_STORE_F32, 5)
    B.gllm_op_gemm_bf16(to_dev_bits(padded_rows(a, Mp)), to_dev_weight(wpad), out, M, N, K, B.GEMM_ADD_F32, 5)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    assert np.abs(got - 2 * ref).max() <= 4e-5 * np.abs(ref).max() + 1e-6


@pytest.mark.parametrize("M", [257, 300, 320, 384, 600, 832])
def test_gemm_row_mixed_launch(M, rowmix=8):
    """Whole bands of 256 rows as 256x256 tiles plus a last band of 64 (up to 64 rows left) or 128 rows: store, add,
    SwiGLU and split-K planes."""
    N, K = 768, 384
    print(f"gemm row-mixed launch M={M}", flush=True)
    a = rand_bits(9, 1, (M, K), 1.0)
    w = rand_bits(9, 2, (N, K), 0.05)
    ref = oracle.linear(oracle.bf16_to_f64(a), w)
    Mp = (M + 255) // 256 * 256
    da, dw = to_dev_bits(padded_rows(a, Mp)), to_dev_weight(w)
    out = torch.full((M, N), 7.0, dtype=torch.float32, device=DEV)
    B.gllm_op_gemm_bf16(da, dw, out, M, N, K, B.GEMM_STORE_F32, rowmix)
    B.gllm_op_gemm_bf16(da, dw, out, M, N, K, B.GEMM_ADD_F32, rowmix)
    planes = torch.full((2, M, N), 9.0, dtype=torch.float32, device=DEV)
    B.gllm_op_gemm_bf16_splitk(da, dw, planes, M, N, K, rowmix, 2)
    torch.cuda.synchronize()
    scale = np.abs(ref).max()
    assert np.abs(out.cpu().numpy().astype(np.float64) - 2 * ref).max() <= 4e-5 * scale + 1e-6
    assert np.abs(planes.cpu().numpy().astype(np.float64).sum(axis=0) - ref).max() <= 2e-5 * scale + 1e-6
    # SwiGLU: the same matrix read as 384 gate/up pairs
    I = N // 2
    wg, wu = rand_bits(9, 3, (I, K), 0.08), rand_bits(9, 4, (I, K), 0.08)
    packed = np.zeros((2 * I, K), dtype=np.uint16)
    for blk in range(I // 32):
        packed[64 * blk: 64 * blk + 32] = wg[32 * blk: 32 * blk + 32]
        packed[64 * blk + 32: 64 * blk + 64] = wu[32 * blk: 32 * blk + 32]
    x = oracle.bf16_to_f64(a)
    ref_s = oracle.swiglu(oracle.linear(x, wg), oracle.linear(x, wu))
    act = torch.zeros((M, I), dtype=torch.bfloat16, device=DEV)
    B.gllm_op_gemm_bf16(da, to_dev_weight(packed), act, M, 2 * I, K, B.GEMM_SWIGLU_BF16, rowmix)
    torch.cuda.synchronize()
    err = np.abs(oracle.bf16_to_f64(bits_of(act)) - ref_s)
    assert np.all(err <= np.abs(ref_s) * 2.0 ** -7 + 1e-4), float(err.max())


@pytest.mark.parametrize("N", [576, 768])
@pytest.mark.parametrize("M", [257, 270, 288])
def test_gemm_288_row_tile(M, N):
    """All of 257..288 rows in one band, 288x192 tiles for 576 columns, 288x128 for 768 (to add 288x192): store, add
    and split-K planes; refused outside that row range, for other column counts and for SwiGLU."""
    K = 384
    print(f"gemm 288-row tile M={M} N={N}", flush=True)
    a = rand_bits(10, 1, (M, K), 1.0)
    w = rand_bits(10, 2, (N, K), 0.05)
    ref = oracle.linear(oracle.bf16_to_f64(a), w)
    da, dw = to_dev_bits(padded_rows(a, 512)), to_dev_weight(w)
    out = torch.full((M, N), 7.0, dtype=torch.float32, device=DEV)
    B.gllm_op_gemm_bf16(da, dw, out, M, N, K, B.GEMM_STORE_F32, 9)
    B.gllm_op_gemm_bf16(da, dw, out, M, N, K, B.GEMM_ADD_F32, 9)
    planes = torch.full((2, M, N), 9.0, dtype=torch.float32, device=DEV)
    B.gllm_op_gemm_bf16_splitk(da, dw, planes, M, N, K, 9, 2)
    torch.cuda.synchronize()
    scale = np.abs(ref).max()
    assert np.abs(out.cpu().numpy().astype(np.float64) - 2 * ref).max() <= 4e-5 * scale + 1e-6
    assert np.abs(planes.cpu().numpy().astype(np.float64).sum(axis=0) - ref).max() <= 2e-5 * scale + 1e-6
    for m, n, mode in ((256, N, B.GEMM_STORE_F32), (289, N, B.GEMM_STORE_F32), (M, 512, B.GEMM_STORE_F32), (M, 768, B.GEMM_SWIGLU_BF16)):
        with pytest.raises(B.GllmError) as e:
            B.gllm_op_gemm_bf16(da, to_dev_weight(rand_bits(10, 3, (768, K), 0.05)), torch.empty(512, 768, device=DEV), m, n, K, mode, 9)
        assert e.value.status == -7          # GLLM_E_UNSUPPORTED


def test_gemm_288_row_tile_reads_the_weights_once():
    """24768 columns are 129 tiles of 288x192, one round of the compute units, and 258 of 256x192, two: 85 and 118 us measured."""
    M, N, K = 257, 24768, 4096
    a = torch.randn(M, K, device=DEV).to(torch.bfloat16)
    w = [(torch.randn(N, K, device=DEV) * 0.02).to(torch.bfloat16) for _ in range(3)]
    out = torch.empty(M, N, device=DEV)
    us = {9: [], 5: []}
    for _ in range(12):
        for tile in us:
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for i in range(9):
                B.gllm_op_gemm_bf16(a, w[i % 3], out, M, N, K, B.GEMM_STORE_F32, tile)
            e1.record()
            e1.synchronize()
            us[tile].append(e0.elapsed_time(e1) * 1e3 / 9)
    one, two = (float(np.median(us[t][2:])) for t in (9, 5))
    print(f"gemm 288-row tile: one band {one:.1f} us, two bands {two:.1f} us", flush=True)
    assert one < 0.9 * two


def test_gemm_row_mixed_launch_refuses_shapes_without_a_short_last_band():
    a = torch.zeros(1024, 128, dtype=torch.bfloat16, device=DEV)
    w = torch.zeros(256, 128, dtype=torch.bfloat16, device=DEV)
    for M in (100, 256, 512, 400, 700):                      # no whole band, nothing left over, more than 128 rows left over
        with pytest.raises(B.GllmError) as e:
            B.gllm_op_gemm_bf16(a, w, torch.empty(M, 256, device=DEV), M, 256, 128, B.GEMM_STORE_F32, 8)
        assert e.value.status == -7          # GLLM_E_UNSUPPORTED


@pytest.mark.parametrize("tile", [-1, 4])
@pytest.mark.parametrize("mode", ["store", "swiglu"])
def test_gemm_mixed_tile_launch(mode, tile):
    """A grid whose last round of 256x256 tiles would be partial: 320 tiles -> 256 big + 128 half-width tiles."""
    M, N, K = 500, 40960, 128
    print(f"gemm mixed launch mode={mode} tile={tile}", flush=True)
    a = rand_bits(5, 1, (M, K), 1.0)
    x = oracle.bf16_to_f64(a)
    Mp = (M + 255) // 256 * 256
    if mode == "store":
        w = rand_bits(5, 2, (N, K), 0.05)
        ref = oracle.linear(x, w)
        out = torch.zeros((M, N), dtype=torch.float32, device=DEV)
        B.gllm_op_gemm_bf16(to_dev_bits(padded_rows(a, Mp)), to_dev_weight(w), out, M, N, K, B.GEMM_STORE_F32, tile)
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        assert np.abs(got - ref).max() <= 2e-5 * np.abs(ref).max() + 1e-6
    else:
        I = N // 2
        wg = rand_bits(5, 3, (I, K), 0.08)
        wu = rand_bits(5, 4, (I, K), 0.08)
        ref = oracle.swiglu(oracle.linear(x, wg), oracle.linear(x, wu))
        packed = np.zeros((N, K), dtype=np.uint16)
        pk = packed.reshape(I // 32, 2, 32, K)
        pk[:, 0] = wg.reshape(I // 32, 32, K)
        pk[:, 1] = wu.reshape(I // 32, 32, K)
        out = torch.zeros((M, I), dtype=torch.bfloat16, device=DEV)
        B.gllm_op_gemm_bf16(to_dev_bits(padded_rows(a, Mp)), to_dev_weight(packed), out, M, N, K, B.GEMM_SWIGLU_BF16, tile)
        torch.cuda.synchronize()
        got = oracle.bf16_to_f64(bits_of(out))
        assert np.all(np.abs(got - ref) <= np.abs(ref) * 2.0 ** -7 + 1e-4)


@pytest.mark.parametrize("tile,splits", [(0, 2), (3, 2), (3, 4), (3, 8), (-1, 2), (6, 2), (7, 4)])
def test_gemm_split_k_planes_sum_to_the_product(tile, splits):
    M, N, K = 300, 512, 1024
    print(f"gemm split-K tile={tile} splits={splits}", flush=True)
    a = rand_bits(7, 1, (M, K), 1.0)
    w = rand_bits(7, 2, (N, K), 0.05)
    ref = oracle.linear(oracle.bf16_to_f64(a), w)
    Mp = (M + 255) // 256 * 256
    planes = torch.full((splits, M, N), 9.0, dtype=torch.float32, device=DEV)
    B.gllm_op_gemm_bf16_splitk(to_dev_bits(padded_rows(a, Mp)), to_dev_weight(w), planes, M, N, K, tile, splits)
    torch.cuda.synchronize()
    got = planes.cpu().numpy().astype(np.float64)
    assert np.abs(got.sum(axis=0) - ref).max() <= 2e-5 * np.abs(ref).max() + 1e-6
    # each plane is the product over its own share of k
    x = oracle.bf16_to_f64(a)
    ks = K // splits
    part0 = oracle.linear(x[:, :ks], np.ascontiguousarray(w[:, :ks]))
    assert np.abs(got[0] - part0).max() <= 2e-5 * np.abs(part0).max() + 1e-6


def test_gemm_tile_ids_of_one_launch_and_few_k_steps():
    """Tiles 2 and 10 are tile 3, 11 is 4 and 12 is 8: callers may use either id.  The 256-column forms hold three LDS stages
    of W: shares of one, two and more k-steps, against the oracle (K roundings of 2^-24 of the sum of magnitudes)."""
    for M, N, K, ids, splits in ((700, 1024, 64, (3, 2, 10), 1), (700, 1024, 128, (3, 10), 1), (520, 768, 1152, (3, 10), 3),
                                 (520, 768, 192, (3, 10), 3), (300, 768, 640, (8, 12), 2), (500, 40960, 192, (4, 11), 1)):
        a, w = rand_bits(11, 1, (M, K), 1.0), rand_bits(11, 2, (N, K), 0.05)
        da, dw = to_dev_bits(padded_rows(a, (M + 255) // 256 * 256)), to_dev_weight(w)
        outs = []
        for tile in ids:
            planes = torch.full((splits, M, N), 5.0, dtype=torch.float32, device=DEV)
            B.gllm_op_gemm_bf16_splitk(da, dw, planes, M, N, K, tile, splits)
            outs.append(planes)
        torch.cuda.synchronize()
        assert all(torch.equal(outs[0], o) for o in outs[1:]), (M, N, K, ids, splits)
        x, y = oracle.bf16_to_f64(a), oracle.bf16_to_f64(w)
        err = np.abs(outs[0].cpu().numpy().astype(np.float64).sum(axis=0) - x @ y.T)
        assert np.all(err <= (np.abs(x) @ np.abs(y).T) * K * 2.0 ** -24), (M, N, K, ids, splits)


@pytest.mark.parametrize("N,K,splits", [(128, 64, 1), (640, 1152, 3), (4096, 256, 4), (4096, 384, 6), (8192, 128, 2), (16512, 128, 1), (33024, 128, 1), (65664, 128, 1)])
def test_gemm_up_to_128_rows(N, K, splits):
    """Tile 7 (up to 64 rows) takes 128 or 64 columns and three to six LDS stages by the number of tiles, tile 6 (up to 128 rows) 128
    or 64 columns and 96 or 128 rows: from two tiles to more than 512, shares of one k-step and more, both sides of 32, 64 and 96
    rows.  The rows behind the last one hold NaN and canaries; K roundings of 2^-24 of the sum of magnitudes bound the error."""
    w = rand_bits(13, 2, (N, K), 0.05)
    dw, y = to_dev_weight(w), oracle.bf16_to_f64(w)
    for M, tile in ((1, 7), (32, 7), (33, 7), (64, 7), (65, 6), (96, 6), (97, 6), (128, 6)):
        print(f"gemm up to 128 rows M={M} tile={tile} N={N} K={K} splits={splits}", flush=True)
        a = rand_bits(13, M, (M, K), 1.0)
        ap = np.full((256, K + 64), 0x7FC0, dtype=np.uint16)
        ap[:M, :K] = a
        planes = torch.full((splits, M + 8, N), 7.0, dtype=torch.float32, device=DEV)
        B.gllm_op_gemm_bf16_splitk(to_dev_bits(ap), dw, planes[:, :M], M, N, K, tile, splits)
        torch.cuda.synchronize()
        x = oracle.bf16_to_f64(a)
        got = planes.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got[:, :M].sum(axis=0) - x @ y.T) <= (np.abs(x) @ np.abs(y).T) * K * 2.0 ** -24), M
        assert np.all(got[:, M:] == 7.0)


@pytest.mark.parametrize("tile", [0, 1, 3, 5, 6, 7, 8])
@pytest.mark.parametrize("K", [64, 128, 448])
def test_gemm_tiles_at_their_edges(tile, K):
    """Row counts on both sides of every tile height, as few k-steps as LDS stages and fewer.  The rows behind the last
    one hold NaN (a tile must not use them) and the result has canaries behind its last row.  fp32 sums of K products of
    bf16 values: K roundings of 2^-24 of the sum of magnitudes bound the error."""
    N = 768
    for M in (1, 33, 64, 129, 192, 193, 256, 257, 300, 384, 385, 449, 577):
        if tile == 8 and not (M > 256 and 0 < M % 256 <= 128):
            continue
        print(f"gemm edges tile={tile} K={K} M={M}", flush=True)
        a, w = rand_bits(12, M, (M, K), 1.0), rand_bits(12, 2, (N, K), 0.05)
        ap = np.full(((M + 511) // 256 * 256, K + 64), 0x7FC0, dtype=np.uint16)      # row stride larger than k
        ap[:M, :K] = a
        out = torch.full((M + 40, N), 7.0, dtype=torch.float32, device=DEV)
        B.gllm_op_gemm_bf16(to_dev_bits(ap), to_dev_weight(w), out, M, N, K, B.GEMM_STORE_F32, tile)
        torch.cuda.synchronize()
        x, y = oracle.bf16_to_f64(a), oracle.bf16_to_f64(w)
        bound = (np.abs(x) @ np.abs(y).T) * K * 2.0 ** -24
        got = out.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got[:M] - x @ y.T) <= bound), (tile, K, M)
        assert np.all(got[M:] == 7.0)


@pytest.mark.parametrize("mode", ["store", "add", "swiglu", "split"])
def test_gemm_rows_off_a_sixteen_byte_boundary(mode):
    """An odd row stride and an operand that starts two bytes behind a boundary: the tiles cannot load these rows.  Rows that
    start 4, 8 or 12 bytes behind a 16-byte boundary, by their stride or by the operand's start: the tiles load them."""
    M, N, K = 37, 256, 128
    a, w = rand_bits(14, 1, (M, K), 1.0), rand_bits(14, 2, (N, K), 0.05)
    x, y = oracle.bf16_to_f64(a), oracle.bf16_to_f64(w)
    bound = (np.abs(x) @ np.abs(y).T) * K * 2.0 ** -24
    for ld, start in ((K + 1, 0), (K + 2, 1), (K + 2, 0), (K + 4, 2), (K + 8, 6), (K + 6, 8)):
        print(f"gemm unaligned rows mode={mode} ld={ld} start={start}", flush=True)
        da = torch.zeros(M * ld + 8, dtype=torch.bfloat16, device=DEV)[start:].as_strided((M, K), (ld, 1))
        da.copy_(to_dev_bits(a).view(torch.bfloat16))
        dw = to_dev_weight(w)
        out = torch.full((M, N), 2.0, dtype=torch.float32, device=DEV)
        if mode == "split":
            planes = torch.zeros((2, M, N), dtype=torch.float32, device=DEV)
            B.gllm_op_gemm_bf16_splitk(da, dw, planes, M, N, K, -1, 2)
            out = planes.sum(dim=0)
        elif mode == "swiglu":
            out = torch.zeros((M, N // 2), dtype=torch.bfloat16, device=DEV)
            B.gllm_op_gemm_bf16(da, dw, out, M, N, K, B.GEMM_SWIGLU_BF16)
        else:
            B.gllm_op_gemm_bf16(da, dw, out, M, N, K, B.GEMM_STORE_F32 if mode == "store" else B.GEMM_ADD_F32)
        torch.cuda.synchronize()
        if mode == "swiglu":
            gate, up = (np.concatenate([y[64 * b + o:64 * b + o + 32] for b in range(N // 64)]) for o in (0, 32))
            ref = oracle.swiglu(x @ gate.T, x @ up.T)
            assert np.all(np.abs(oracle.bf16_to_f64(bits_of(out)) - ref) <= np.abs(ref) * 2.0 ** -7 + 1e-4)
        else:
            got = out.cpu().numpy().astype(np.float64) - (2.0 if mode == "add" else 0.0)
            assert np.all(np.abs(got - x @ y.T) <= bound + 2.0 ** -22)


def test_gemm_forced_tile_is_checked_on_every_path():
    """A forced tile that does not fit the product is refused wherever the rows lie -- aligned, off a 4-byte boundary, too far
    apart for a tile -- and one that fits is accepted, also the 192-column one where n is no multiple of 128."""
    M, N, K = 37, 192, 128
    a, w = rand_bits(16, 1, (M, K), 1.0), rand_bits(16, 2, (N, K), 0.05)
    x, y = oracle.bf16_to_f64(a), oracle.bf16_to_f64(w)
    dw = to_dev_weight(w)
    for ld in (K, K + 1, 1 << 26):
        print(f"gemm forced tiles ld={ld}", flush=True)
        da = torch.empty((M - 1) * ld + K, dtype=torch.bfloat16, device=DEV).as_strided((M, K), (ld, 1))
        da.copy_(to_dev_bits(a).view(torch.bfloat16))
        for tile in (0, 1, 2, 3, 4, 6, 7, 8, 9, 10, 11, 12, 13):
            with pytest.raises(B.GllmError) as e:
                B.gllm_op_gemm_bf16(da, dw, torch.empty(M, N, device=DEV), M, N, K, B.GEMM_STORE_F32, tile)
            assert e.value.status == -7, tile          # GLLM_E_UNSUPPORTED
        for tile in (5, -1):
            out = torch.zeros((M, N), dtype=torch.float32, device=DEV)
            B.gllm_op_gemm_bf16(da, dw, out, M, N, K, B.GEMM_STORE_F32, tile)
            torch.cuda.synchronize()
            assert np.all(np.abs(out.cpu().numpy() - x @ y.T) <= (np.abs(x) @ np.abs(y).T) * K * 2.0 ** -24), (ld, tile)


def test_gemm_rows_farther_apart_than_32_bit_offsets_reach():
    """A row stride of 2^23 elements: 300 rows span more than 4 GiB, which the launch cuts into bands."""
    M, N, K, ld = 300, 256, 128, 1 << 23
    a, w = rand_bits(13, 1, (M, K), 1.0), rand_bits(13, 2, (N, K), 0.05)
    far = torch.empty(M * ld, dtype=torch.bfloat16, device=DEV).as_strided((M, K), (ld, 1))
    far.copy_(to_dev_bits(a).view(torch.bfloat16))
    out = torch.zeros((M, N), dtype=torch.float32, device=DEV)
    B.gllm_op_gemm_bf16(far, to_dev_weight(w), out, M, N, K, B.GEMM_STORE_F32)
    torch.cuda.synchronize()
    x, y = oracle.bf16_to_f64(a), oracle.bf16_to_f64(w)
    assert np.all(np.abs(out.cpu().numpy() - x @ y.T) <= (np.abs(x) @ np.abs(y).T) * K * 2.0 ** -24)


@pytest.mark.parametrize("M,ld", [(329, 6520000), (330, 6520000), (384, 5592404), (384, 5592406)])
def test_gemm_far_rows_under_the_tallest_tile(M, ld):
    """One band of 257..384 rows whose rows lie so far apart that just all of them, or not all, are within 32-bit offsets."""
    N, K = 256, 64
    print(f"gemm far rows M={M} ld={ld}", flush=True)
    a, w = rand_bits(15, 1, (M, K), 1.0), rand_bits(15, 2, (N, K), 0.05)
    far = torch.empty((M - 1) * ld + K, dtype=torch.bfloat16, device=DEV).as_strided((M, K), (ld, 1))
    far.copy_(to_dev_bits(a).view(torch.bfloat16))
    out = torch.zeros((M, N), dtype=torch.float32, device=DEV)
    B.gllm_op_gemm_bf16(far, to_dev_weight(w), out, M, N, K, B.GEMM_STORE_F32, 13)
    torch.cuda.synchronize()
    x, y = oracle.bf16_to_f64(a), oracle.bf16_to_f64(w)
    assert np.all(np.abs(out.cpu().numpy() - x @ y.T) <= (np.abs(x) @ np.abs(y).T) * K * 2.0 ** -24)


@pytest.mark.parametrize("ldw,N,whole", [(1 << 23, 128, False), (1 << 23, 192, False), (1 << 25, 128, False), (1 << 25, 128, True)])
def test_gemm_weights_with_a_k_extent_beyond_32_bit_offsets(ldw, N, whole):
    """Row blocks of W that lie 1 and 4 GiB apart: the product over a leading part of k, and over all of it with values in the
    first and the last 64 columns only (so that K = 128 in the error bound), in every mode and with a k-split."""
    M, K = 3 if whole else 150, ldw if whole else 192
    cols = np.concatenate([np.arange(64), np.arange(K - 64, K)]) if whole else np.arange(K)
    print(f"gemm far weights ldw={ldw} N={N} K={K}", flush=True)
    a, w = rand_bits(17, 1, (M, len(cols)), 1.0), rand_bits(17, 2, (N, len(cols)), 0.05)
    x, y = oracle.bf16_to_f64(a), oracle.bf16_to_f64(w)
    far = torch.zeros(N // 64, ldw // 64, 64, 64, dtype=torch.bfloat16, device=DEV)          # the tiled layout, block by block
    for i, c in enumerate(cols[::64]):
        far[:, int(c) // 64] = to_dev_bits(w[:, 64 * i:64 * i + 64]).view(N // 64, 64, 64)
    da = torch.zeros(M, K, dtype=torch.bfloat16, device=DEV)
    da[:, torch.from_numpy(cols).to(DEV)] = to_dev_bits(a)
    bound = (np.abs(x) @ np.abs(y).T) * len(cols) * 2.0 ** -24
    out = torch.zeros((M, N), dtype=torch.float32, device=DEV)
    B.gllm_op_gemm_bf16(da, far, out, M, N, K, B.GEMM_STORE_F32, -1, ldw=ldw)
    torch.cuda.synchronize()
    assert np.all(np.abs(out.cpu().numpy() - x @ y.T) <= bound)
    B.gllm_op_gemm_bf16(da, far, out, M, N, K, B.GEMM_ADD_F32, -1, ldw=ldw)
    torch.cuda.synchronize()
    assert np.all(np.abs(out.cpu().numpy() - 2 * (x @ y.T)) <= 2 * bound + 2.0 ** -23 * np.abs(2 * (x @ y.T)))
    s = 2 if whole else 3
    planes = torch.zeros((s, M, N), dtype=torch.float32, device=DEV)
    B.gllm_op_gemm_bf16_splitk(da, far.view(N, ldw), planes, M, N, K, -1, s)
    torch.cuda.synchronize()
    assert np.all(np.abs(planes.cpu().numpy().astype(np.float64).sum(axis=0) - x @ y.T) <= bound)
    if N % 128 == 0:
        act = torch.zeros((M, N // 2), dtype=torch.bfloat16, device=DEV)
        B.gllm_op_gemm_bf16(da, far, act, M, N, K, B.GEMM_SWIGLU_BF16, -1, ldw=ldw)
        torch.cuda.synchronize()
        gate, up = (np.concatenate([y[64 * b + o:64 * b + o + 32] for b in range(N // 64)]) for o in (0, 32))
        ref = oracle.swiglu(x @ gate.T, x @ up.T)
        assert np.all(np.abs(oracle.bf16_to_f64(bits_of(act)) - ref) <= np.abs(ref) * 2.0 ** -7 + 1e-4)


def test_pack_weight_writes_the_documented_tiled_layout():
    """gllm_op_pack_weight against the layout as the header states it (gpu_util.tiled_bits), bit for bit: a whole matrix,
    and a part of a wider one (row stride above k); then the product on a leading part of the packed k range."""
    w = rand_bits(12, 1, (320, 448), 0.05)
    out = torch.zeros(320 * 448, dtype=torch.bfloat16, device=DEV)
    B.gllm_op_pack_weight(to_dev_bits(w), out)
    torch.cuda.synchronize()
    assert np.array_equal(bits_of(out).reshape(320, 448), tiled_bits(w))
    part = torch.zeros(128 * 192, dtype=torch.bfloat16, device=DEV)
    B.gllm_op_pack_weight(to_dev_bits(w)[64:192, :192], part)
    torch.cuda.synchronize()
    assert np.array_equal(bits_of(part).reshape(128, 192), tiled_bits(np.ascontiguousarray(w[64:192, :192])))
    for bad in (to_dev_bits(w)[:100], to_dev_bits(w)[:, :100]):          # rows / columns that are no multiple of 64
        with pytest.raises(B.GllmError) as e:
            B.gllm_op_pack_weight(bad, out)
        assert e.value.status == -7          # GLLM_E_UNSUPPORTED
    M, N, K, k = 70, 256, 448, 192
    a = rand_bits(12, 2, (M, K), 1.0)
    wn = rand_bits(12, 3, (N, K), 0.05)
    res = torch.zeros(M, N, dtype=torch.float32, device=DEV)
    B.gllm_op_gemm_bf16(to_dev_bits(padded_rows(a, 256)), to_dev_weight(wn), res, M, N, k, B.GEMM_STORE_F32, -1)
    torch.cuda.synchronize()
    ref = oracle.linear(oracle.bf16_to_f64(a)[:, :k], np.ascontiguousarray(wn[:, :k]))
    assert np.abs(res.cpu().numpy() - ref).max() <= 2e-5 * np.abs(ref).max() + 1e-6
    with pytest.raises(B.GllmError):          # a k extent that is no multiple of 64
        B.gllm_op_gemm_bf16(to_dev_bits(padded_rows(a, 256)), to_dev_weight(wn), res, M, N, k, B.GEMM_STORE_F32, -1, ldw=200)


def _gate_up(bits):
    """Rows of a [2*I, K] matrix (gate rows, then up rows) in the order the ABI states: 32 gate rows, the 32 matching up rows."""
    I = bits.shape[0] // 2
    return np.concatenate([bits[:I].reshape(I // 32, 1, 32, -1), bits[I:].reshape(I // 32, 1, 32, -1)], axis=1).reshape(bits.shape)


@pytest.mark.parametrize("tile,N,rows", [(7, 256, (1, 31, 32, 33)), (7, 131072, (32, 33)), (13, 256, (257, 288, 289, 320, 321, 352, 353, 384)),
                                         (14, 512, (1, 160, 161, 193, 224, 225, 257, 321, 449, 960)),
                                         (15, 384, (1, 160, 161, 193, 224, 225, 257, 321, 449, 960)),
                                         (4, 66048, (65, 161, 193, 225))])
@pytest.mark.parametrize("K", [64, 320])
def test_gemm_band_heights_at_their_edges(tile, N, rows, K):
    """Both sides of every band height, plain and SwiGLU; NaN behind the last row of a, canaries behind the last row of the
    result.  K roundings of 2^-24 of the sum of magnitudes bound an fp32 sum; SwiGLU rounds to bf16 (2^-8 and the hardware
    exponential's and reciprocal's ulps) and takes the error of both sums."""
    for M in rows:
        print(f"gemm heights tile={tile} K={K} M={M}", flush=True)
        a, w = rand_bits(14, M, (M, K), 1.0), rand_bits(14, 2, (N, K), 0.05)
        ap = np.full((M + 64, K), 0x7FC0, dtype=np.uint16)
        ap[:M] = a
        x, y = oracle.bf16_to_f64(a), oracle.bf16_to_f64(w)
        ref, bound = x @ y.T, (np.abs(x) @ np.abs(y).T) * K * 2.0 ** -24
        out = torch.full((M + 40, N), 7.0, dtype=torch.float32, device=DEV)
        B.gllm_op_gemm_bf16(to_dev_bits(ap), to_dev_weight(w), out, M, N, K, B.GEMM_STORE_F32, tile)
        act = torch.full((M + 40, N // 2), 7.0, dtype=torch.bfloat16, device=DEV)
        B.gllm_op_gemm_bf16(to_dev_bits(ap), to_dev_weight(_gate_up(w)), act, M, N, K, B.GEMM_SWIGLU_BF16, tile)
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got[:M] - ref) <= bound) and np.all(got[M:] == 7.0), (tile, K, M)
        g, u = ref[:, :N // 2], ref[:, N // 2:]
        want = g / (1 + np.exp(-g)) * u
        slack = np.abs(want) * 2.0 ** -8 * 1.01 + 1.1 * np.abs(u) * bound[:, :N // 2] + np.abs(g) * bound[:, N // 2:] + 1e-30
        got = act.float().cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got[:M] - want) <= slack) and np.all(got[M:] == 7.0), (tile, K, M)


@pytest.mark.parametrize("splits,K", [(3, 384), (5, 640), (6, 1152), (7, 448)])
def test_gemm_splits_that_are_no_powers_of_two(splits, K):
    """Every plane of a split product holds the product over its share of k, in bands of equal height, one band of 257..384 rows
    and the 128-row tiles: K/splits roundings of 2^-24 of the sum of magnitudes."""
    N, part = 512, K // splits
    w = rand_bits(16, 2, (N, K), 0.05)
    y, dw = oracle.bf16_to_f64(w), to_dev_weight(w)
    for M, tiles in ((193, (0, 6, 14, 15)), (289, (13, 14, 15)), (600, (8, 14, 15))):
        a = rand_bits(16, M, (M, K), 1.0)
        x, da = oracle.bf16_to_f64(a), to_dev_bits(padded_rows(a, M + 64))
        for tile in tiles:
            print(f"gemm splits={splits} M={M} tile={tile}", flush=True)
            out = torch.full((splits, M, N), 7.0, dtype=torch.float32, device=DEV)
            B.gllm_op_gemm_bf16_splitk(da, dw, out, M, N, K, tile, splits)
            torch.cuda.synchronize()
            for s in range(splits):
                xs, ys = x[:, s * part:(s + 1) * part], y[:, s * part:(s + 1) * part]
                assert np.all(np.abs(out[s].cpu().numpy() - xs @ ys.T) <= (np.abs(xs) @ np.abs(ys).T) * part * 2.0 ** -24), (splits, M, tile, s)


@pytest.mark.parametrize("M,N,ldc,tile", [(62, 49152, 49152, 5), (60, 49344, 49350, 5), (61, 49344, 49350, 5), (64, 128 * 512, 128 * 512, 7), (92, 32896, 32896, 6),
                                          (19, 152064, 152064, 7), (20, 152064, 152070, 7), (64, 152064, 152064, 7), (33, 131840, 131844, 7), (33, 131072, 131072, 7),
                                          (70, 65792, 65800, 4), (15, 192 * 1372, (1 << 26) - 4, 5), (15, 192 * 1372, 1 << 26, 5)])
def test_gemm_fp32_results_of_one_round_and_of_more(M, N, ldc, tile):
    """Results of one round of tiles and of more, of less than 12 MB and of more, which are stored in another way, packed and with
    rows as far apart as the 32-bit byte offsets of that way reach and one step farther; nothing between the rows changes.  Of tile 7
    128-column tiles: 1024 of two stages of A, 1030 and 1188 with a compute unit each (of 32 rows for M = 20, of 64 above 32)."""
    K = 64
    print(f"gemm results M={M} N={N} ldc={ldc} tile={tile}", flush=True)
    assert tile != 7 or B.gllm_op_gemm_tile_columns(M, N, K, B.GEMM_STORE_F32, tile) == 128
    a, w = rand_bits(31, 1, (M, K), 1.0), rand_bits(31, 2, (N, K), 0.05)
    ref = oracle.linear(oracle.bf16_to_f64(a), w)
    flat = torch.full(((M - 1) * ldc + N + 64,), 7.0, dtype=torch.float32, device=DEV)
    out = torch.as_strided(flat, (M, N), (ldc, 1))
    B.gllm_op_gemm_bf16(to_dev_bits(padded_rows(a, 256)), to_dev_weight(w), out, M, N, K, B.GEMM_STORE_F32, tile)
    torch.cuda.synchronize()
    got = out.contiguous().cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() <= 2e-5 * np.abs(ref).max() + 1e-6
    for r in range(M):
        assert bool((flat[r * ldc + N: min((r + 1) * ldc, flat.numel())] == 7.0).all()), r


@pytest.mark.parametrize("M,N,tile", [(64, 128 * 512, 7), (100, 192 * 257, 5), (257, 192 * 412, 13)])
def test_gemm_fp32_results_with_rows_in_descending_order(M, N, tile):
    """A negative row stride of the results, of sizes that are stored by 32-bit offsets from a row where the stride allows it: the
    same bits as upwards, nothing beside them."""
    K = 64
    print(f"gemm descending rows M={M} N={N} tile={tile}", flush=True)
    a, w = to_dev_bits(padded_rows(rand_bits(32, 1, (M, K), 1.0), 288)), to_dev_weight(rand_bits(32, 2, (N, K), 0.05))
    up = torch.full((M, N), 7.0, device=DEV)
    down = torch.full((M + 2, N), 7.0, device=DEV)
    B.gllm_op_gemm_bf16(a, w, up, M, N, K, B.GEMM_STORE_F32, tile)
    B.gllm_op_gemm_bf16(a, w, down[M], M, N, K, B.GEMM_STORE_F32, tile, ldc=-N)
    torch.cuda.synchronize()
    assert torch.equal(down[1:M + 1].flip(0), up)
    assert bool((down[0] == 7.0).all()) and bool((down[M + 1] == 7.0).all())


@pytest.mark.parametrize("M", [257, 288])
@pytest.mark.parametrize("N", [32896, 49152, 79104])
def test_gemm_one_band_of_288_rows_by_either_width(M, N):
    """128-column tiles (32896), one round of 192-column ones (49152), a round of those and one of 128 columns (79104); rows past
    the last one and the padding of a row stay as they are."""
    K = 4096
    print(f"gemm one band M={M} N={N}", flush=True)
    assert B.gllm_op_gemm_tile_columns(M, N, K, B.GEMM_STORE_F32, 13) == {32896: 128, 49152: 192, 79104: 0}[N]
    torch.manual_seed(5)
    a = torch.randn(M, K, device=DEV).to(torch.bfloat16)
    w = (torch.randn(N, K, device=DEV) * 0.02).to(torch.bfloat16)
    packed = torch.empty_like(w)
    B.gllm_op_pack_weight(w, packed)
    out = torch.full((M + 1, N + 8), 7.0, dtype=torch.float32, device=DEV)
    for tile in (13, -1):
        out.fill_(7.0)
        B.gllm_op_gemm_bf16(a, packed, out, M, N, K, B.GEMM_STORE_F32, tile)
        torch.cuda.synchronize()
        assert bool((out[M] == 7.0).all()) and bool((out[:, N:] == 7.0).all())
        for c in range(0, N, 8192):
            x, y = a.double(), w[c:c + 8192].double()
            err = (out[:M, c:min(c + 8192, N)].double() - x @ y.T).abs()
            assert bool((err <= (x.abs() @ y.abs().T) * K * 2.0 ** -24).all()), (tile, c)
