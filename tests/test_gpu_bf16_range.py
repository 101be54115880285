"""bf16 activations at both ends of their range: every finite x is allowed, and a sum that would leave binary32 on the way to a y that
does not is no exception.  All kernels that multiply bf16 as it is, rows of very different magnitude in one call."""
import numpy as np
import pytest

from oracle import rwkvq_oracle as orc
from paper_2505_03803_amd import binding as B
from paper_2505_03803_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# rows of W, column tiles, rows of x, work up to which a small launch splits its columns (0: by rule, 1: never, 1000000: always):
# operands straight from memory with one, two and three row tiles per workgroup; the streaming kernels at batch 4, 16 and 32;
# activations copied into LDS, 16 and 32 rows of W; 17 to 48 rows in one round; 17 to 128 rows, 16, 32 and 64 rows of W
ROUTES = [(512, 3, 5, 0), (4352, 3, 5, 0), (4352, 5, 5, 0), (8448, 3, 5, 0), (512, 3, 3, 1), (512, 3, 15, 1), (512, 3, 20, 1), (256, 17, 16, 0), (4352, 17, 15, 0),
          (16640, 1, 17, 1000000), (16640, 2, 33, 1000000), (512, 3, 47, 0), (4352, 3, 100, 0), (8448, 2, 64, 0)]


def rows_match(y, mat, x, tol):
    ref = orc.linear(mat, orc.widen(x, "bf16"), "f64")
    for m in range(x.shape[0]):
        rms = np.sqrt(np.mean((ref[m] / np.abs(ref[m]).max()) ** 2)) * np.abs(ref[m]).max()
        err = (np.abs(y[m] - ref[m]) / np.maximum(np.abs(ref[m]), rms)).max()
        assert err <= tol, f"row {m}: {err}, largest {np.abs(ref[m]).max()}"


def route(options, split):
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_STREAM)
    options(B.OPT_STREAM_SPLIT_MAX_WORK, split)


# (8 + z) times a group's sum beyond 2^128 where s (sum of (q - z) x) is not
@pytest.mark.parametrize("N,columns,M,split", ROUTES)
@pytest.mark.parametrize("zero", [200.0, -200.0, 60000.0])
def test_sq_zero_points_far_from_the_codes(N, columns, M, split, zero, options):
    print(f"zero points N={N} columns={columns} M={M} split={split} zero={zero}", flush=True)
    route(options, split)
    rng, K = np.random.default_rng(N + M), 256 * columns
    mat = synth.gen_sq(rng, N, K)
    mat.zeros = synth.f32_to_f16_bits(zero * rng.uniform(0.9, 1.0, mat.zeros.shape))
    s = max(1.0 / (abs(zero) * K), 2.0 ** -23)
    mat.scales = synth.f32_to_f16_bits(s * rng.uniform(0.5, 1.5, mat.scales.shape))
    top = min(1.0, 1.0 / (s * abs(zero) * K)) * 1e38
    scale = np.array([top, 1.0, top / 16, 1e-30])[np.arange(M) % 4]
    x = synth.f32_to_bf16_bits((scale[:, None] * (1.0 + 0.2 * rng.standard_normal((M, K)))).astype(np.float32))
    y = G.gpu_gemm(B.upload(mat, native=True), x, "bf16")
    # a group's sum and the difference are binary32 sums of 128 numbers of one sign, every rounding 2^-24 of a partial sum
    rows_match(y, mat, x, 2e-5)


# Down to the smallest bf16 numbers, y a normal binary32 number: nothing on the way is less exact than binary32
@pytest.mark.parametrize("N,columns,M,split", ROUTES)
def test_sq_smallest_activations(N, columns, M, split, options):
    print(f"smallest activations N={N} columns={columns} M={M} split={split}", flush=True)
    route(options, split)
    rng, K = np.random.default_rng(N + M), 256 * columns
    mat = synth.gen_sq(rng, N, K)
    mat.scales = synth.f32_to_f16_bits(orc.widen(mat.scales, "f16") * 2000.0)
    scale = np.array([1e-36, 1e-38, 3e-39, 1.0])[np.arange(M) % 4]
    x = synth.f32_to_bf16_bits((scale[:, None] * rng.standard_normal((M, K))).astype(np.float32))
    y = G.gpu_gemm(B.upload(mat, native=True), x, "bf16")
    # as above; 3e-39 is 2^21 times the smallest binary32 number, and 768 to 4352 products have weights of about 60
    rows_match(y, mat, x, 2e-5)


VQ_ROUTES = [(N if N % 256 == 0 else 16640, c, M, s) for N, c, M, s in ROUTES]


# Products of a row of x that cancel, beyond 2^128 on the way: a tile's first 128 columns of one sign, the others of the other
@pytest.mark.parametrize("N,columns,M,split", VQ_ROUTES)
@pytest.mark.parametrize("kbits", [6, 8])
def test_vq_sums_that_come_back(N, columns, M, split, kbits, options):
    print(f"sums that come back N={N} columns={columns} M={M} split={split} kbits={kbits}", flush=True)
    route(options, split)
    rng, K = np.random.default_rng(N + M), 256 * columns
    mat = synth.gen_vq(rng, N, K, kbits)
    mat.codebooks = synth.f32_to_f16_bits(rng.uniform(8.0, 9.0, mat.codebooks.shape))
    scale = np.array([2e36 / np.sqrt(columns), 1.0, 1e35, 1e-30])[np.arange(M) % 4]
    sign = np.where(np.arange(K) % 256 < 128, 1.0, -1.0)
    x = synth.f32_to_bf16_bits((scale[:, None] * sign * rng.uniform(0.8, 1.2, (M, K))).astype(np.float32))
    y = G.gpu_gemm(B.upload(mat, native=True), x, "bf16")
    # eight roundings in a tile of partial sums up to 128 * 8.5 scale, 8 * 2^-24 * 1088 scale at most, next to a y that differs from
    # row to row of W by 0.29 scale sqrt(256) per tile (0.29: the deviation of the entries): 1.1e-4
    rows_match(y, mat, x, 2e-4)


# An entry that is infinite makes the sums it is in infinite, as with fp16 activations and at one row of x, and no other
@pytest.mark.parametrize("N,columns,M,split", VQ_ROUTES)
@pytest.mark.parametrize("kbits", [6, 8])
def test_vq_infinite_entry(N, columns, M, split, kbits, options):
    print(f"infinite entry N={N} columns={columns} M={M} split={split} kbits={kbits}", flush=True)
    route(options, split)
    rng, K = np.random.default_rng(N + M), 256 * columns
    mat = synth.gen_vq(rng, N, K, kbits)
    mat.codebooks[0, 0, 5, 1] = 0x7C00
    x = synth.f32_to_bf16_bits(rng.uniform(0.5, 1.5, (M, K)).astype(np.float32))
    y = G.gpu_gemm(B.upload(mat, native=True), x, "bf16")
    with np.errstate(invalid="ignore"):
        ref = orc.linear(mat, orc.widen(x, "bf16"), "f64")
    assert np.isposinf(ref).any() and not np.isnan(ref).any()
    assert np.array_equal(np.isposinf(y), np.isposinf(ref)) and not np.isnan(y).any()
    assert G.err_g2(np.where(np.isinf(y), 0.0, y), np.where(np.isinf(ref), 0.0, ref)) <= 2e-5
