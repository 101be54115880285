"""The matrix-core kernels for 17 to 1536 rows of x (wavefronts that split K and unpack W in registers) at the edges of
their tiles: K of fewer column tiles than K groups, ragged rows, every choice of rows per workgroup, and zero points too
small for the one-step unpack."""
import numpy as np
import pytest

from oracle import rwkvq_oracle as orc
from paper_2505_03803_amd import binding as B
from paper_2505_03803_amd import synth

import gpu_util as G

pytestmark = pytest.mark.gpu


def make(fmt, N, K, seed):
    rng = np.random.default_rng(seed)
    return synth.gen_sq(rng, N, K) if fmt == "sq" else synth.gen_vq(rng, N, K, 6 if fmt == "vq6" else 8)


# M: one row and one past the 64-, 96- and 128-row workgroups, eight K groups (M <= 128) and four; K: 1, 3, 5 and 9 column tiles
@pytest.mark.parametrize("fmt", ["sq", "vq6", "vq8"])
@pytest.mark.parametrize("N,K,M", [(256, 256, 17), (256, 2304, 64), (512, 768, 65), (256, 1280, 128), (256, 256, 129), (768, 2304, 193),
                                   (256, 1280, 385), (512, 512, 1025), (256, 256, 1536)])
@pytest.mark.parametrize("xdt", ["bf16", "f16"])
def test_against_the_oracle(fmt, N, K, M, xdt, options):
    print(f"mid {fmt} N={N} K={K} M={M} x={xdt}", flush=True)
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_MATRIX_CORES)
    mat = make(fmt, N, K, 11)
    x = synth.gen_activations(np.random.default_rng(M), M, K, xdt)
    # against the weights as fed: what is left is binary32 sums of up to 2304 products in four or eight partial sums, about
    # sqrt(K) 2^-24 of the row's norms (the distance to the unrounded weights is a statistical figure, 1.1e-3 rms for bf16)
    asfed = orc.linear(mat, orc.widen(x, xdt), "f64", weight_round=xdt)
    assert G.err_g2(G.gpu_gemm(B.upload(mat, native=True), x, xdt), asfed) <= 2e-5


# rows of W x rows of x that make the launcher take 64, 96 and 128 rows of x per workgroup (and 8 K groups at M = 100)
@pytest.mark.parametrize("M,n_mats,N", [(100, 1, 1024), (100, 5, 4096), (333, 1, 4096), (333, 4, 4096), (300, 9, 4096)])
def test_calls_of_several_matrices(M, n_mats, N, options):
    """Mixed formats in one launch; every matrix alone gives the same bits beyond 128 rows (calls of these sizes all take the
    kernels that split K, in four groups)."""
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_MATRIX_CORES)
    K = 512
    mats = [make(("sq", "vq6", "vq8")[i % 3], N, K, 20 + i) for i in range(n_mats)]
    xs = [synth.gen_activations(np.random.default_rng(40 + i), M, K, "bf16") for i in range(n_mats)]
    torch = G.torch_()
    dms, dev = [B.upload(m, native=True) for m in mats], [G.to_dev_bits(x) for x in xs]
    ys = [torch.empty((M, N), dtype=torch.float32, device="cuda") for _ in mats]
    B.rwkvq_linear_dispatch(B.DispatchTable([d.desc() for d in dms], dev, ys), M, B.BF16, B.F32)
    torch.cuda.synchronize()
    for i in (0, n_mats - 1):
        got = ys[i].cpu().numpy()
        assert G.err_g2(got.astype(np.float64), orc.linear(mats[i], orc.widen(xs[i], "bf16"), "f64", weight_round="bf16")) <= 2e-5
        alone = B.gemm(dms[i], dev[i], M, B.BF16, B.F32)
        torch.cuda.synchronize()
        if M > 128:
            assert np.array_equal(got, alone.cpu().numpy())


@pytest.mark.parametrize("fmt", ["sq", "vq6", "vq8"])
@pytest.mark.parametrize("n_mats,tiles", [(4, False), (32, True)])
def test_calls_that_fill_the_device(fmt, n_mats, tiles, options):
    """128 < M <= 1536: a call that gives every compute unit several tiles of 256 x 256 takes the kernels for large batches, a
    smaller one those that split K; seen by the order of the sums (five column tiles in a row, or in four groups)."""
    torch = G.torch_()
    N, K, M = 2048, 1280, 512
    dm = B.upload(make(fmt, N, K, 17), native=True)
    x = G.to_dev_bits(synth.gen_activations(np.random.default_rng(3), M, K, "bf16"))
    def call(rows):
        options(B.OPT_PREFILL_TILE_ROWS, rows)
        ys = [torch.empty((M, N), dtype=torch.float32, device="cuda") for _ in range(n_mats)]
        B.rwkvq_linear_dispatch(B.DispatchTable([dm.desc()] * n_mats, [x] * n_mats, ys), M, B.BF16, B.F32)
        torch.cuda.synchronize()
        assert all(torch.equal(ys[0], y) for y in ys[1:])
        return ys[0]
    free, forced = call(0), call(256)
    assert torch.equal(free, forced) == tiles
    assert float((free - forced).abs().max()) <= 2e-5 * float(forced.abs().max())


@pytest.mark.parametrize("xdt", ["bf16", "f16"])
@pytest.mark.parametrize("small", [False, True, "zero"])
def test_one_hot_rows_return_the_rounded_weights(xdt, small, options):
    """Row m selects column k_m: the output is Deq(W) rounded once to the type of x, bit for bit.  With a zero point in
    (0, 2^-11) q - z itself rounds; one such group, subnormal ones among them, makes its workgroup take the two-step form (a
    zero point of zero, either sign, does not)."""
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_MATRIX_CORES)
    N, K = 512, 1280
    mat = make("sq", N, K, 31)
    if small == "zero":
        mat.zeros.reshape(-1)[:] = np.where(np.arange(mat.zeros.size) % 3 == 0, 0x8000, 0)
        mat.zeros.reshape(N, -1)[300:310] = 0x1000            # and the smallest that is not small
    elif small:
        rng = np.random.default_rng(5)
        z = mat.zeros.reshape(N, K // 128)
        for n in range(N):                                   # fp16 bits 1 .. 0x0FFF, either sign; and an exact zero
            z[n, n % (K // 128)] = rng.integers(1, 0x1000) | (0x8000 if n & 1 else 0)
        z[7, 3], z[300, 0] = 0, 0x8000
    dm = B.upload(mat, native=True)
    want = G.gpu_dequant(dm, B.DTYPES[xdt])
    want = orc.widen(want, xdt)
    for M in (100, 320):
        x = np.zeros((M, K), np.float32)
        cols = (np.arange(M) * 37 + 5 * M) % K
        x[np.arange(M), cols] = 1.0
        bits = synth.f32_to_bf16_bits(x) if xdt == "bf16" else synth.f32_to_f16_bits(x)
        assert np.array_equal(G.gpu_gemm(dm, bits, xdt), want[:, cols].T.astype(np.float64)), M


# 17 to 64 rows of x per workgroup and the first of the next, two workgroups of 48 and of 64; rows of W that end inside a
# workgroup's 64 (SQ); 1, 3, 9 and 10 column tiles on eight K groups
@pytest.mark.parametrize("fmt,N,K", [("sq", 176, 768), ("sq", 272, 2560), ("sq", 16, 256), ("vq6", 256, 2304), ("vq6", 512, 256), ("vq8", 256, 2560), ("vq8", 256, 768)])
@pytest.mark.parametrize("M", [17, 32, 33, 48, 49, 64, 65, 97, 128])
@pytest.mark.parametrize("xdt", ["bf16", "f16"])
def test_unrounded_weights(fmt, N, K, M, xdt, options):
    """The streaming path's contract (products of the unrounded weights) at 17 <= M <= 128."""
    print(f"mid exact {fmt} N={N} K={K} M={M} x={xdt}", flush=True)
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_STREAM)
    mat = make(fmt, N, K, 12)
    x = synth.gen_activations(np.random.default_rng(M), M, K, xdt)
    got = G.gpu_gemm(B.upload(mat, native=True), x, xdt)
    # binary32 sums of up to 2560 products, as for the streaming kernels
    assert G.err_g2(got, orc.linear(mat, orc.widen(x, xdt), "f64")) <= 2e-5


# Workgroups of 16, 32 and 64 rows of W: up to 128 of 32 rows, up to 256, more; scalar-quantized matrices with a last one partly past the end
@pytest.mark.parametrize("fmt,N", [("sq", 4096), ("sq", 4112), ("sq", 4144), ("sq", 8192), ("sq", 8208), ("vq6", 4096), ("vq6", 4352), ("vq6", 8448),
                                   ("vq8", 4096), ("vq8", 4352), ("vq8", 8448)])
@pytest.mark.parametrize("M", [18, 47, 64])
@pytest.mark.parametrize("xdt", ["bf16", "f16"])
def test_unrounded_weights_by_rows_of_a_workgroup(fmt, N, M, xdt, options):
    K = 2304
    print(f"unrounded {fmt} N={N} M={M} x={xdt}", flush=True)
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_STREAM)
    rng = np.random.default_rng(N)
    m = synth.gen_sq(rng, N, K) if fmt == "sq" else synth.gen_vq(rng, N, K, int(fmt[2:]))
    x = synth.gen_activations(rng, M, K, xdt)
    y = G.gpu_gemm(B.upload(m, native=True), x, xdt)
    # 2304 products in binary32 partial sums
    assert G.err_g2(y, orc.linear(m, orc.widen(x, xdt), "f64")) <= 2e-5


@pytest.mark.parametrize("fmt", ["sq", "vq6", "vq8"])
@pytest.mark.parametrize("scale", [1e-20, 1e30, 1.5e38])
def test_unrounded_weights_at_the_ends_of_bf16(fmt, scale, options):
    """Rows of bf16 activations far from one: their group sums stay finite and as exact as at one."""
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_STREAM)
    N, K, M = 256, 512, 20
    mat = make(fmt, N, K, 13)
    x = np.random.default_rng(3).uniform(-1, 1, (M, K)).astype(np.float32) * np.float32(scale)
    if fmt != "sq":
        x *= np.float32(2.0 ** -4)                           # entries of 0.02: no output beyond binary32
    bits = synth.f32_to_bf16_bits(x)
    got = G.gpu_gemm(B.upload(mat, native=True), bits, "bf16")
    assert np.all(np.isfinite(got))
    assert G.err_g2(got, orc.linear(mat, orc.widen(bits, "bf16"), "f64")) <= 2e-5


@pytest.mark.parametrize("fmt", ["sq", "vq6", "vq8"])
def test_line_between_the_forms_of_the_streaming_path(fmt, options):
    """RWKVQ_OPT_STREAM_SPLIT_MAX_WORK at 17 <= M <= 128: 1 never takes the kernels that split K, 1000000 always does, a value in
    between moves the line at M <= 32 and leaves M > 32 alone, where a third pass of few rows is cheaper than a second tile
    of the others from some 2000 workgroups on; seen by the order of the sums."""
    torch = G.torch_()
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_STREAM)
    N, K = 4096, 1280
    dm = B.upload(make(fmt, N, K, 19), native=True)
    def call(M, n_mats, value):
        options(B.OPT_STREAM_SPLIT_MAX_WORK, value)
        x = G.to_dev_bits(synth.gen_activations(np.random.default_rng(M), M, K, "bf16"))
        ys = [torch.empty((M, N), dtype=torch.float32, device="cuda") for _ in range(n_mats)]
        B.rwkvq_linear_dispatch(B.DispatchTable([dm.desc()] * n_mats, [x] * n_mats, ys), M, B.BF16, B.F32)
        torch.cuda.synchronize()
        assert all(torch.equal(ys[0], y) for y in ys[1:])
        return ys[0]
    for M in (20, 48):
        stream, split = call(M, 2, 1), call(M, 2, 1000000)
        assert not torch.equal(stream, split)
        assert float((stream - split).abs().max()) <= 2e-5 * float(split.abs().max())
        # 64 rows of W in a workgroup: 128 workgroups, 1856 (29 matrices) over the line at M <= 32
        for value, few, many in ((0, split, stream if M <= 32 else split), (32768, split, stream if M <= 32 else split),
                                 (4096, stream if M <= 32 else split, None), (80000, split, split)):
            assert torch.equal(call(M, 2, value), few), (M, value)
            if many is not None:
                assert torch.equal(call(M, 29, value), many), (M, value)
    for M, few, many in ((66, True, False), (80, True, False), (48, True, True), (100, True, True)):
        stream, split = call(M, 2, 1), call(M, 2, 1000000)
        assert torch.equal(call(M, 2, 0), split if few else stream), M
        assert torch.equal(call(M, 40, 0), split if many else stream), M


@pytest.mark.parametrize("kbits", [6, 8])
@pytest.mark.parametrize("N,with_sq", [(16640, 0), (24576, 0), (256, 16800)])
@pytest.mark.parametrize("M", [17, 32, 48])
def test_small_activations_beside_large_ones(N, with_sq, kbits, M, options):
    """bf16 activations that lie 2^40 apart in a group of columns, the large ones at codebook entries of zero: the small ones decide
    the result.  Calls of 257 to 384 workgroups of 64 rows of W, where fp16 activations take a kernel of their own; with and without a
    scalar-quantized matrix beside."""
    print(f"2^40 apart N={N} with={with_sq} kbits={kbits} M={M}", flush=True)
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_STREAM)
    rng = np.random.default_rng(N + M + kbits)
    K = 768
    m = synth.gen_vq(rng, N, K, kbits)
    m.codes[:, ::4 * kbits] &= ~np.uint32((1 << kbits) - 1)                       # columns 0, 256, ..: entry 0, which is zero
    m.codebooks[:, :, 0] = 0
    x = orc.widen(synth.gen_activations(rng, M, K, "bf16"), "bf16")
    x[:, ::256] *= 2.0 ** 40
    mats, xs = [m], [synth.f32_to_bf16_bits(x)]
    if with_sq:
        mats.append(synth.gen_sq(rng, with_sq, K))
        xs.append(synth.gen_activations(rng, M, K, "bf16"))
    ys = [G.torch_().empty((M, q.N), dtype=G.torch_().float32, device="cuda") for q in mats]
    dms, dev = [B.upload(q, native=True) for q in mats], [G.to_dev_bits(v) for v in xs]
    B.rwkvq_linear_dispatch(B.DispatchTable([q.desc() for q in dms], dev, ys), M, B.BF16, B.F32)
    G.torch_().cuda.synchronize()
    for q, v, y in zip(mats, xs, ys):
        # binary32 sums of 768 products, as in test_against_the_oracle
        assert G.err_g2(y.cpu().numpy().astype(np.float64), orc.linear(q, orc.widen(v, "bf16"), "f64")) <= 2e-5
