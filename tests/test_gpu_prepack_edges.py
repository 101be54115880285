"""Prepack at its smallest and at tile counts that are not a multiple of a workgroup's four: native and canonical layout
decode to the same binary32 weights."""
import numpy as np
import pytest

from oracle import rwkvq_oracle as orc
from paper_2505_03803_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt,N,K", [("sq", 16, 256), ("sq", 32, 256), ("sq", 16, 1280), ("sq", 80, 512),
                                     ("vq6", 256, 256), ("vq6", 768, 1280), ("vq8", 256, 256), ("vq8", 768, 1280)])
def test_prepack_edges(fmt, N, K):
    from paper_2505_03803_amd import binding as B
    import gpu_util as G
    rng = np.random.default_rng(5)
    mat = synth.gen_sq(rng, N, K) if fmt == "sq" else synth.gen_vq(rng, N, K, int(fmt[2]))
    got = G.gpu_dequant(B.upload(mat, native=True))
    assert np.array_equal(got.view(np.uint32), orc.dequant(mat).view(np.uint32))
