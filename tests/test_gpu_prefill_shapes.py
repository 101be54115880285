"""The workgroup shapes of the kernels for large batches: tiles of 128 rows of W, and launches of whole rounds followed by the rest in
such tiles, give the bits of 256 x 256 tiles (which the oracle checks): every shape sums over K in one order."""
import numpy as np
import pytest

from paper_2505_03803_amd import binding as B
from paper_2505_03803_amd import synth

import gpu_util as G

pytestmark = pytest.mark.gpu


def make(fmt, N, K, seed):
    rng = np.random.default_rng(seed)
    return synth.gen_sq(rng, N, K) if fmt == "sq" else synth.gen_vq(rng, N, K, 6 if fmt == "vq6" else 8)


# rows of W of the call's matrices: one and two tiles of 256 in few workgroups; 33 and 36 tiles, the rest of a whole round within one
# matrix; and over the end of one into the next
@pytest.mark.parametrize("fmt", ["sq", "vq6", "vq8"])
@pytest.mark.parametrize("Ns", [(256,), (512,), (33 * 256,), (3 * 256, 33 * 256), (31 * 256, 5 * 256, 256)])
@pytest.mark.parametrize("M,K,xdt", [(1537, 512, "bf16"), (2048, 256, "f16"), (1999, 768, "bf16")])
def test_shapes_give_the_same_bits(fmt, Ns, M, K, xdt, options):
    print(f"prefill shapes {fmt} Ns={Ns} K={K} M={M} x={xdt}", flush=True)
    torch = G.torch_()
    dms = [B.upload(make(fmt, N, K, N), native=True) for N in Ns]
    xs = [torch.randn((M, K), device="cuda").to(torch.bfloat16 if xdt == "bf16" else torch.float16) for _ in Ns]
    out = []
    for rows in (256, 0):
        options(B.OPT_PREFILL_TILE_ROWS, rows)
        ys = [torch.full((M + 1, N), 7.0, dtype=torch.float32, device="cuda") for N in Ns]
        B.rwkvq_linear_dispatch(B.DispatchTable([d.desc() for d in dms], xs, ys), M, B.DTYPES[xdt], B.F32)
        torch.cuda.synchronize()
        out.append(ys)
    for a, b in zip(*out):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
        assert (a[M] == 7.0).all()


@pytest.mark.parametrize("xdt", ["bf16", "f16"])
def test_line_below_1536_rows_knows_the_rest(xdt, options):
    """336 tiles of 256 x 256: one whole round and a rest in tiles of half the rows of W, which is estimated at less than the kernels
    that split K (and those at less than any one shape): the bits of the large tiles."""
    print(f"line x={xdt}", flush=True)
    torch, rng = G.torch_(), np.random.default_rng(5)
    M, N, K = 1536, 14336, 1024
    m, x = synth.gen_sq(rng, N, K), G.to_dev_bits(synth.gen_activations(rng, M, K, xdt))
    dm, ys = B.upload(m, native=True), []
    for rows in (0, 256):
        options(B.OPT_PREFILL_TILE_ROWS, rows)
        ys.append(B.gemm(dm, x, M, B.DTYPES[xdt], B.F32))
        torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1])
