"""Edges of the calibration kernels: batch sizes on both sides of each instance of the order-statistic selection, samples with
ties, zeros of both signs and the largest finite values; a codebook whose vectors all fall to a few entries."""
import numpy as np
import pytest

from oracle import mu_oracle as MO
from oracle import rwkvq_oracle as orc
from paper_2505_03803_amd import binding as B
from paper_2505_03803_amd import synth

import gpu_util as G

pytestmark = pytest.mark.gpu


def dev(a):
    a = np.ascontiguousarray(a)
    return G.torch_().from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).cuda()


@pytest.mark.parametrize("Bn", [1, 2, 16, 17, 32, 33, 64, 65, 128, 129, 256, 257, 1016, 1017, 1024, 1025])
@pytest.mark.parametrize("dt", ["bf16", "f16", "f32"])
def test_clip_mean_instances(Bn, dt):
    torch = G.torch_()
    rng = np.random.default_rng(Bn)
    n = 33                                                    # two workgroups of positions and one more
    x = synth.gen_calibration(rng, Bn, n, dt)
    big = {"f16": 0x7BFF, "bf16": 0x7F7F}.get(dt)
    if dt == "f32":
        x[:, 0] = np.float32(0.25)                            # constant
        x[:, 1] = np.where(np.arange(Bn) % 3 == 0, np.float32(-0.0), np.float32(0.0))
        x[:, 2] = np.where(np.arange(Bn) % 2 == 0, np.finfo(np.float32).max / 2048, -np.finfo(np.float32).max / 2048)
        x[:, 3] = np.round(x[:, 3])                           # many ties
    else:
        x[:, 0] = x[0, 0]
        x[:, 1] = np.where(np.arange(Bn) % 3 == 0, 0x8000, 0)
        x[:, 2] = np.where(np.arange(Bn) % 2 == 0, big, big | 0x8000) if dt == "f16" else np.where(np.arange(Bn) % 2 == 0, 0x7900, 0xF900)
        x[:, 3] = x[rng.integers(0, min(Bn, 4), Bn), 3]
    out = torch.empty(n, dtype=torch.float32, device="cuda")
    for p in (0.0, 1.0, 33.0, 50.0):
        B.rwkvq_clip_mean(dev(x), B.DTYPES[dt], Bn, n, p, out)
        torch.cuda.synchronize()
        want = MO.clip_mean(x if dt == "f32" else orc.widen(x, dt), p)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), p


# 33 to 256 samples: percentiles on both sides of the line between the selection from the ends (ranks up to 4 and from B - 6 on) and
# the one by bits, at which the rank is whole and the interpolation weight zero, and with more positions than a multiple of eight
# workgroups; ties that end the selection early, and signed infinities as extremes
@pytest.mark.parametrize("Bn,n", [(33, 16), (64, 130), (101, 300), (128, 33), (200, 128), (256, 77)])
@pytest.mark.parametrize("dt", ["bf16", "f16", "f32"])
def test_clip_mean_from_the_ends(Bn, n, dt):
    torch, rng = G.torch_(), np.random.default_rng(Bn)
    x = synth.gen_calibration(rng, Bn, n, dt)
    x[:, 5] = x[rng.integers(0, 3, Bn), 5]
    x[1:, 6] = x[1, 6]
    x[3, 7], x[9, 7] = (np.inf, -np.inf) if dt == "f32" else {"bf16": (0x7F80, 0xFF80), "f16": (0x7C00, 0xFC00)}[dt]
    out = torch.empty(n, dtype=torch.float32, device="cuda")
    for rank in (0.0, 1.0, 3.5, 4.0, 4.99, 5.0, 6.0):
        p = 100.0 * rank / (Bn - 1)
        B.rwkvq_clip_mean(dev(x), B.DTYPES[dt], Bn, n, p, out)
        torch.cuda.synchronize()
        with np.errstate(invalid="ignore"):
            want = MO.clip_mean(x if dt == "f32" else orc.widen(x, dt), p)
        known = ~np.isnan(want)                               # (infinities minus themselves: the definition gives no number)
        assert np.array_equal(out.cpu().numpy().view(np.uint32)[known], want.view(np.uint32)[known]), p


# vectors that stay in LDS over the iterations (up to 4096, in chunks of 2048) and those that are read again
@pytest.mark.parametrize("n", [2, 2046, 2050, 4094, 6000, 8192, 8194])
@pytest.mark.parametrize("kbits", [6, 8])
def test_codebook_sizes(n, kbits):
    torch, rng = G.torch_(), np.random.default_rng(n)
    mu, xbar, cb = synth.gen_mu(rng, n, "bf16"), rng.standard_normal(n).astype(np.float32), synth.gen_codebook(rng, 1 << kbits)
    book, idx = dev(cb.copy()), torch.empty(n // 2, dtype=torch.uint8, device="cuda")
    B.rwkvq_mu_codebook([dev(mu)], [dev(xbar)], [n], B.BF16, kbits, 3, [book], [idx])
    torch.cuda.synchronize()
    want, want_idx, _ = MO.mu_codebook(orc.widen(mu, "bf16"), xbar, orc.widen(cb, "f16"), 3)
    assert np.array_equal(orc.widen(book.cpu().numpy().view(np.uint16), "f16"), want)
    assert np.array_equal(idx.cpu().numpy(), want_idx)


def test_clip_mean_of_1024_samples_takes_the_tile():
    """1024 samples are the most that the kernel with its samples in LDS takes; the one behind it reads them again for every rank
    (16 positions: 0.07 and 180 ms), so a line drawn too low shows as time."""
    torch = G.torch_()
    x, out = torch.randn((1024, 64), device="cuda"), torch.empty(64, device="cuda")
    B.rwkvq_clip_mean(x, B.F32, 1024, 64, 1.0, out)
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    B.rwkvq_clip_mean(x, B.F32, 1024, 64, 1.0, out)
    end.record()
    torch.cuda.synchronize()
    assert start.elapsed_time(end) < 10.0


@pytest.mark.parametrize("kbits", [6, 8])
def test_codebook_with_crowded_entries(kbits):
    """Constant weights (every vector to one entry), two values, and sizes around a share (256 or 1024 vectors) and a chunk (2048)."""
    torch = G.torch_()
    rng = np.random.default_rng(kbits)
    E = 1 << kbits
    for n in (2, 510, 514, 2050, 4094, 4098, 8192):
        for kind in range(2):
            m = np.full(n, 0.37, np.float32) if kind == 0 else np.where(rng.random(n) < 0.9, np.float32(0.2), np.float32(0.8))
            x = rng.standard_normal(n).astype(np.float32)
            cb0 = synth.gen_codebook(rng, E).reshape(E, 2)
            cb, idx = dev(cb0.copy()), torch.zeros(n // 2 + 15, dtype=torch.uint8, device="cuda")
            B.rwkvq_mu_codebook([dev(m)], [dev(x)], [n], B.F32, kbits, 4, [cb], [idx])
            torch.cuda.synchronize()
            wcb, widx, _ = MO.mu_codebook(m, x, orc.widen(cb0, "f16"), 4)
            assert np.array_equal(cb.cpu().numpy().view(np.uint16).reshape(-1), synth.f32_to_f16_bits(wcb).reshape(-1)), (n, kind)
            assert np.array_equal(idx.cpu().numpy()[:n // 2], widx.astype(np.uint8)), (n, kind)
