"""The nearest-entry assignment by cells (pairs compared only with the entries listed for their cell) against the definition."""
import numpy as np
import pytest

from oracle import encode_oracle as E

pytestmark = pytest.mark.gpu


def dev(a, dtype):
    import torch
    a = np.ascontiguousarray(a)
    return torch.from_numpy(a if dtype == "f32" else a.view(np.int16)).cuda()


def test_vq_assign_cells():
    """Where the listed entries could go wrong: entries in a tight cluster with one far out (cells with more entries than a list
    holds), all entries equal, entries on a lattice with pairs exactly between them, pairs far outside the cells, on entries,
    and one representable step off a tie; codebooks far from the origin; every pair outside (a full queue)."""
    from paper_2505_03803_amd import binding as B
    rng = np.random.default_rng(99)
    for kbits in (6, 8):
        En = 1 << kbits
        books = []
        books.append(np.concatenate([rng.normal(0, 1e-3, (En - 1, 2)), [[5.0, -7.0]]]))
        books.append(np.full((En, 2), 0.125))
        side = int(np.sqrt(En))
        books.append(np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(En, 2) / 8.0)
        books.append(rng.normal(0, 0.02, (En, 2)) + [30.0, -11.0])
        books.append(rng.normal(0, 0.02, (En, 2)))
        books.append(rng.normal(0, 0.02, (En, 2)))
        books.append(np.stack([np.linspace(-1, 1, En), np.zeros(En)], -1))      # on a line
        books.append(rng.integers(0, 3, (En, 2)) / 4.0)                         # many duplicates
        n_blocks = len(books)
        cb = np.stack(books).astype(np.float16)
        wide = np.empty((256, 256 * n_blocks), np.float32)
        for i in range(n_blocks):
            b = rng.normal(0, 0.02, (256, 128, 2)).astype(np.float32)
            e = cb[i].astype(np.float32)
            b[:64] = e[rng.integers(0, En, (64, 128))]                          # on entries
            mid = (e[rng.integers(0, En, (64, 128))] + e[rng.integers(0, En, (64, 128))]) / 2
            b[64:128] = mid                                                     # between two entries
            b[128:160] = np.nextafter(mid[:32], np.float32(1e9))
            b[160:168] *= 1e6
            b[168:172] *= 1e-30
            if i == 4: b[:] = rng.normal(0, 1, b.shape)                          # nearly all outside
            if i == 5: b[200:] = np.float32(3e4) * rng.normal(0, 1, b[200:].shape).astype(np.float32)
            wide[:, 256 * i: 256 * (i + 1)] = b.reshape(256, 256)
        bits = cb.view(np.uint16)[None]
        dm = B.vq_assign(dev(wide, "f32"), B.F32, dev(bits, "f16"), kbits)
        want = E.vq_assign_packed(wide, bits, kbits)
        assert np.array_equal(dm.codes.cpu().numpy().view(np.uint32), want), kbits
        for rows in (9, 17):                    # enough blocks that each is taken in two parts, and whole
            dm = B.vq_assign(dev(np.tile(wide, (rows, 1)), "f32"), B.F32, dev(np.tile(bits, (rows, 1, 1, 1)), "f16"), kbits)
            assert np.array_equal(dm.codes.cpu().numpy().view(np.uint32), np.tile(want, (rows, 1))), (kbits, rows)


@pytest.mark.parametrize("kbits", [6, 8])
@pytest.mark.parametrize("wdt", ["f32", "bf16"])
@pytest.mark.parametrize("rows", [1, 9, 17])                # blocks taken in quarters, halves and whole
def test_vq_assign_many_pairs_beside_the_cells(kbits, wdt, rows):
    """Every way that pairs without a list take: a few (sixteen lanes each), some hundreds (a thread each), more than the queue holds
    behind a first unit without any (whole units done over), a quarter and more of the first unit (every unit with every entry, for
    pairs outside the cells and for cells of crowded entries); with every distance infinite, entry 0."""
    from paper_2505_03803_amd import binding as B
    from paper_2505_03803_amd import synth
    rng = np.random.default_rng(7 + kbits)
    En = 1 << kbits
    shares = [0.003, 0.02, 0.24, 0.26, "last rows", "first rows", "crowded", "equal", "infinite"]
    cb = (rng.normal(0, 0.02, (len(shares), En, 2))).astype(np.float16)
    wide = rng.normal(0, 0.015, (256, 256 * len(shares))).astype(np.float32)
    for i, share in enumerate(shares):
        b = wide[:, 256 * i: 256 * (i + 1)]
        if isinstance(share, float):
            b[np.repeat(rng.random((256, 128)) < share, 2, axis=1)] *= 1e3
        elif share == "last rows":                          # (the first thread of each part sees rows 0 .. 63 of 256, 128 or 64)
            b[np.arange(256) % 64 > 20] *= 1e3
            b[:64] = rng.normal(0, 0.015, (64, 256))
        elif share == "first rows":
            b[:40] *= 1e3
        elif share == "crowded":                            # nine places, many entries on each
            cb[i] = rng.integers(-1, 2, (En, 2)) * 0.02
            b[:] = rng.integers(-1, 2, (256, 256)) * 0.02 + rng.normal(0, 1e-3, (256, 256))
        elif share == "equal":
            cb[i] = 0.01
        else:
            b[::3] = 3e38
    if wdt == "bf16":
        bits = synth.f32_to_bf16_bits(wide)
        wide = (bits.astype(np.uint32) << 16).view(np.float32)
    books = cb.view(np.uint16)[None]
    want = np.tile(E.vq_assign_packed(wide, books, kbits), (rows, 1))
    src = np.tile(wide if wdt == "f32" else bits, (rows, 1))
    dm = B.vq_assign(dev(src, wdt), B.DTYPES[wdt], dev(np.tile(books, (rows, 1, 1, 1)), "f16"), kbits)
    got = dm.codes.cpu().numpy().view(np.uint32)
    words = want.shape[1] // len(shares)
    for i, share in enumerate(shares):
        assert np.array_equal(got[:, words * i: words * (i + 1)], want[:, words * i: words * (i + 1)]), share


@pytest.mark.parametrize("kbits", [6, 8])
def test_vq_assign_lists_that_just_fit(kbits):
    """As many entries in one place as a list holds and one more: eight of a fine cell, sixteen of a cell, 32 of a cell on its way to finer ones;
    pairs on the place, around it and everywhere else."""
    from paper_2505_03803_amd import binding as B
    rng = np.random.default_rng(11)
    En = 1 << kbits
    counts = [7, 8, 9, 15, 16, 17, 31, 32, 33]
    cb = rng.normal(0, 0.02, (len(counts), En, 2)).astype(np.float16)
    wide = rng.normal(0, 0.02, (256, 256 * len(counts))).astype(np.float32)
    for i, n in enumerate(counts):
        at = rng.uniform(-0.02, 0.02, 2)
        cb[i, rng.permutation(En)[:n]] = at + rng.uniform(-2e-4, 2e-4, (n, 2))
        b = wide[:, 256 * i: 256 * (i + 1)].reshape(256, 128, 2)
        b[::2] = at + rng.normal(0, 3e-4, b[::2].shape)
        b[1::4] = at + rng.normal(0, 3e-3, b[1::4].shape)
    bits = cb.view(np.uint16)[None]
    got = B.vq_assign(dev(wide, "f32"), B.F32, dev(bits, "f16"), kbits).codes.cpu().numpy().view(np.uint32)
    assert np.array_equal(got, E.vq_assign_packed(wide, bits, kbits))


@pytest.mark.parametrize("kbits", [6, 8])
@pytest.mark.parametrize("rows", [1, 17])                   # quarters of blocks and whole ones
def test_vq_assign_equal_and_crowded_entries(kbits, rows):
    """Entries equal to one of a lower index (never nearest, on no list): half of them zero of either sign, pairs of equal ones, a few copies of
    one, none; and crowds of different entries around one place, on both sides of what a list is made for; more marked units than none."""
    from paper_2505_03803_amd import binding as B
    rng = np.random.default_rng(23)
    En = 1 << kbits
    kinds = ["half zero", "zeros of both signs", "pairs", "some", "crowd", "crowd just fits", "nine crowds", "half, rows apart", "infinite"]
    cb = rng.normal(0, 0.02, (len(kinds), En, 2)).astype(np.float16)
    wide = rng.normal(0, 0.02, (256, 256 * len(kinds))).astype(np.float32)
    for i, kind in enumerate(kinds):
        b = wide[:, 256 * i: 256 * (i + 1)]
        if kind == "half zero":
            cb[i, ::2] = 0
        elif kind == "zeros of both signs":
            cb[i, 1::2] = rng.choice(np.float16([0.0, -0.0]), (En // 2, 2))
        elif kind == "pairs":
            cb[i, 1::2] = cb[i, ::2]
        elif kind == "some":
            cb[i, rng.permutation(En)[:En // 8]] = cb[i, 3]
        elif kind.startswith("crowd"):                      # 32 and 96 entries near a cell, and more
            n = (90 if kbits == 8 else 28) if kind.endswith("fits") else En - En // 8
            cb[i, rng.permutation(En)[:n]] = [0.004, -0.003] + rng.normal(0, 2e-5, (n, 2))
        elif kind == "nine crowds":
            cb[i] = (rng.integers(-1, 2, (En, 2)) * 0.02) * (1 + 1e-3 * rng.standard_normal((En, 2)))
        elif kind == "half, rows apart":                    # pairs near the crowd in rows that follow the first unit of every thread
            cb[i, ::2] = rng.normal(0, 2e-5, (En // 2, 2))
            b[np.arange(256) % 64 > 20] *= 0.1
        else:
            cb[i, 5:12] = [np.inf, 0.01]
            cb[i, 20:24] = -np.inf
    books = cb.view(np.uint16)[None]
    with np.errstate(invalid="ignore", over="ignore"):
        want = np.tile(E.vq_assign_packed(wide, books, kbits), (rows, 1))
    dm = B.vq_assign(dev(np.tile(wide, (rows, 1)), "f32"), B.F32, dev(np.tile(books, (rows, 1, 1, 1)), "f16"), kbits)
    got = dm.codes.cpu().numpy().view(np.uint32)
    words = want.shape[1] // len(kinds)
    for i, kind in enumerate(kinds):
        assert np.array_equal(got[:, words * i: words * (i + 1)], want[:, words * i: words * (i + 1)]), kind


@pytest.mark.parametrize("kbits", [6, 8])
@pytest.mark.parametrize("rows", [13, 26])                  # blocks taken in halves and whole
def test_vq_assign_more_than_the_queue(kbits, rows):
    """About as many pairs outside the cells as the queue holds, as it and the room of the lists hold together, and nearly all behind the
    first units, none of them where the sample of 128 looks, so that the block is not given up before."""
    from paper_2505_03803_amd import binding as B
    rng = np.random.default_rng(23)
    En = 1 << kbits
    queue, room = (8192, 8192) if kbits == 6 else (4096, 16384)
    counts = [queue - 8, queue + 8, queue + room - 8, queue + room + 8, 24000]
    cb = rng.normal(0, 0.02, (len(counts), En, 2)).astype(np.float16)
    cb = np.clip(cb, -0.05, 0.05)
    wide = np.clip(rng.normal(0, 0.012, (256, 256 * len(counts))), -0.03, 0.03).astype(np.float32)
    parts = 2 if rows == 13 else 1
    t = np.arange(128)
    for i, n in enumerate(counts):
        b = wide[:, 256 * i: 256 * (i + 1)].reshape(256, 128, 2)
        free = np.ones((256, 128), bool)
        for part in range(parts):
            free[part * 256 // parts + t * 2 // parts, t * 37 & 127] = False
            free[part * 256 // parts: part * 256 // parts + 64] = False
        at = np.flatnonzero(free)
        at = rng.permutation(at)[:min(n, at.size)]
        b.reshape(-1, 2)[at] = rng.choice([-1, 1], (at.size, 2)) * rng.uniform(0.5, 0.7, (at.size, 2))
    bits = cb.view(np.uint16)[None]
    want = np.tile(E.vq_assign_packed(wide, bits, kbits), (rows, 1))
    got = B.vq_assign(dev(np.tile(wide, (rows, 1)), "f32"), B.F32, dev(np.tile(bits, (rows, 1, 1, 1)), "f16"), kbits).codes.cpu().numpy().view(np.uint32)
    words = want.shape[1] // len(counts)
    for i, n in enumerate(counts):
        assert np.array_equal(got[:, words * i: words * (i + 1)], want[:, words * i: words * (i + 1)]), n


@pytest.mark.parametrize("spread", [2e-4, 2e-3, 6e-3])
def test_vq_assign_crowds(spread):
    """256 entries of which n, all different, are crowded at one place or at two: fewer and more than what a cell of 16 x 16 lists before
    whole wavefronts list the cells within it, of which some keep eight or fewer; pairs on the crowd, around it and everywhere."""
    from paper_2505_03803_amd import binding as B
    rng = np.random.default_rng(31)
    counts = [44, 52, 60, 64, 68, 96, 128, 200, 250]
    cb = rng.normal(0, 0.02, (len(counts), 256, 2)).astype(np.float16)
    wide = rng.normal(0, 0.02, (256, 256 * len(counts))).astype(np.float32)
    for i, n in enumerate(counts):
        at = rng.uniform(-0.025, 0.025, (2, 2))[rng.integers(0, 1 + i % 2, n)]
        cb[i, rng.permutation(256)[:n]] = at + rng.uniform(-spread, spread, (n, 2))
        b = wide[:, 256 * i: 256 * (i + 1)].reshape(256, 128, 2)
        b[::4] = at[0] + rng.normal(0, spread, b[::4].shape)
        b[1::8] = at[-1] + rng.normal(0, 4 * spread, b[1::8].shape)
    bits = cb.view(np.uint16)[None]
    want = E.vq_assign_packed(wide, bits, 8)
    for rows in (1, 15):                        # blocks in quarters and whole
        got = B.vq_assign(dev(np.tile(wide, (rows, 1)), "f32"), B.F32, dev(np.tile(bits, (rows, 1, 1, 1)), "f16"), 8).codes.cpu().numpy().view(np.uint32)
        assert np.array_equal(got, np.tile(want, (rows, 1))), rows
