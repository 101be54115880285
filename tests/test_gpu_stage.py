"""The column split of batch 2..16 (small launches): every number of row tiles per workgroup, row tiles past the end of W, one and
several column tiles per wavefront, matrices of different K and format in a launch, against the oracle."""
import numpy as np
import pytest

from oracle import rwkvq_oracle as orc
from paper_2505_03803_amd import binding as B
from paper_2505_03803_amd import synth

import gpu_util as G

pytestmark = pytest.mark.gpu


# R: the fewest row tiles per workgroup that make at most 256 workgroups; 7: none of 1..6 does.  16 and 17 column tiles: the most that
# wavefronts take one each, and the fewest that they take in turns (six wavefronts with R = 1, nine with R >= 3, the last ones with
# fewer); 25: four turns of seven.  At M = 3 and R >= 3 the rows are of mixed lengths, and a workgroup takes one or two row tiles.
@pytest.mark.parametrize("R,columns", [(1, 1), (1, 16), (1, 17), (1, 25), (2, 16), (2, 17), (3, 5), (3, 17), (4, 1), (4, 17), (5, 3), (5, 17),
                                       (6, 2), (6, 17), (7, 1), (7, 9)])
@pytest.mark.parametrize("M,xdt", [(3, "bf16"), (16, "f16")])
def test_column_split(R, columns, M, xdt, options):
    print(f"column split R={R} columns={columns} M={M} x={xdt}", flush=True)
    options(B.OPT_STREAM_SPLIT_MAX_WORK, 1000000)
    torch, rng = G.torch_(), np.random.default_rng(R)
    rows = 3 if R == 1 else 256 * (R - 1) + 1 - 32       # row tiles of the scalar-quantized matrix; the others have 16 each
    K = 256 * columns
    few = K if R < 3 or columns == 1 else 256 * max(1, columns // 3)   # another K in the same launch
    mats = [synth.gen_sq(rng, 16 * rows, few if M == 3 else K), synth.gen_vq(rng, 256, K, 6), synth.gen_vq(rng, 256, few, 8)]
    xs = [synth.gen_activations(rng, M, m.K, xdt) for m in mats]
    dms, dev = [B.upload(m, native=True) for m in mats], [G.to_dev_bits(x) for x in xs]
    ys = [torch.full((M + 1, m.N), 7.0, dtype=torch.float32, device="cuda") for m in mats]
    B.rwkvq_linear_dispatch(B.DispatchTable([d.desc() for d in dms], dev, ys), M, B.DTYPES[xdt], B.F32)
    torch.cuda.synchronize()
    for m, x, y in zip(mats, xs, ys):
        got = y.cpu().numpy().astype(np.float64)
        assert (got[M] == 7.0).all()                      # nothing behind the last row
        # up to 6400 products in binary32 partial sums: about sqrt(K) 2^-24 of the row's norms
        assert G.err_g2(got[:M], orc.linear(m, orc.widen(x, xdt), "f64")) <= 2e-5


# More matrices than the two-dimensional grid takes: one, two and four row tiles per workgroup, one column tile per wavefront and several
@pytest.mark.parametrize("rows,n", [(3, 11), (40, 12), (100, 10), (130, 14)])
@pytest.mark.parametrize("columns", [2, 3, 17])
@pytest.mark.parametrize("M,xdt", [(3, "bf16"), (16, "f16")])
def test_column_split_of_many_matrices(rows, n, columns, M, xdt, options):
    print(f"column split of {n} matrices of {rows} row tiles columns={columns} M={M} x={xdt}", flush=True)
    options(B.OPT_STREAM_SPLIT_MAX_WORK, 1000000)
    torch, rng = G.torch_(), np.random.default_rng(rows + columns)
    kinds = [synth.gen_sq(rng, 16 * rows, 256 * columns), synth.gen_vq(rng, 256 * max(1, rows // 16), 256, 6),
             synth.gen_vq(rng, 256 * max(1, rows // 16), 256 * columns, 8)]
    up, xs = [B.upload(m, native=True) for m in kinds], [synth.gen_activations(rng, M, m.K, xdt) for m in kinds]
    of = [i % 3 for i in range(n)]
    dev = [G.to_dev_bits(xs[k]) for k in of]
    ys = [torch.full((M + 1, kinds[k].N), 7.0, dtype=torch.float32, device="cuda") for k in of]
    B.rwkvq_linear_dispatch(B.DispatchTable([up[k].desc() for k in of], dev, ys), M, B.DTYPES[xdt], B.F32)
    torch.cuda.synchronize()
    want = [orc.linear(m, orc.widen(x, xdt), "f64") for m, x in zip(kinds, xs)]
    for k, y in zip(of, ys):
        got = y.cpu().numpy().astype(np.float64)
        assert (got[M] == 7.0).all()
        assert G.err_g2(got[:M], want[k]) <= 2e-5          # as above


# Rows of one length in one round: one to six row tiles per workgroup, one column tile per wavefront and several; from 20 column tiles
# on the wavefronts go by the type of x and M (20 and 21: eight and twelve in bf16; 25: five to eight in fp16)
@pytest.mark.parametrize("R,columns", [(1, 20), (1, 25), (2, 21), (2, 25), (3, 3), (3, 17), (3, 21), (4, 5), (4, 17), (4, 20), (5, 3), (5, 17),
                                       (6, 3), (6, 18), (6, 21)])
@pytest.mark.parametrize("M,xdt", [(4, "f16"), (7, "bf16"), (9, "bf16"), (16, "f16")])
def test_column_split_of_one_length(R, columns, M, xdt):
    print(f"column split of one length R={R} columns={columns} M={M} x={xdt}", flush=True)
    torch, rng = G.torch_(), np.random.default_rng(R + columns)
    rows = 3 if R == 1 else 256 * (R - 1) + 1 - 32
    mats = [synth.gen_sq(rng, 16 * rows, 256 * columns), synth.gen_vq(rng, 256, 256 * columns, 6), synth.gen_vq(rng, 256, 256 * columns, 8)]
    xs = [synth.gen_activations(rng, M, m.K, xdt) for m in mats]
    dms, dev = [B.upload(m, native=True) for m in mats], [G.to_dev_bits(x) for x in xs]
    ys = [torch.full((M + 1, m.N), 7.0, dtype=torch.float32, device="cuda") for m in mats]
    B.rwkvq_linear_dispatch(B.DispatchTable([d.desc() for d in dms], dev, ys), M, B.DTYPES[xdt], B.F32)
    torch.cuda.synchronize()
    for m, x, y in zip(mats, xs, ys):
        got = y.cpu().numpy().astype(np.float64)
        assert (got[M] == 7.0).all()
        assert G.err_g2(got[:M], orc.linear(m, orc.widen(x, xdt), "f64")) <= 2e-5          # as above


# One round with one or two row tiles per workgroup: both sides of the lines between operands straight from memory and activations copied
# into LDS, by columns, M and format; the last workgroup of 32 rows half empty (4112), two matrices in one launch
@pytest.mark.parametrize("N,columns,Ms", [(1024, 8, (16,)), (1024, 9, (9, 10, 11, 12, 14)), (1024, 10, (9, 10, 13, 14)), (4096, 16, (9, 10, 13, 14)), (256, 17, (2, 16)),
                                          (4096, 17, (2, 3)), (512, 28, (2, 6)), (512, 29, (6, 7)), (4112, 16, (16,)),
                                          (4112, 17, (5, 6, 13, 14, 15)), (8192, 18, (6, 14, 15))])
@pytest.mark.parametrize("kind", ["sq", "vq6", "vq8"])
@pytest.mark.parametrize("xdt", ["f16", "bf16"])
def test_activations_copied_or_not(N, columns, Ms, kind, xdt):
    print(f"copied or not N={N} columns={columns} {kind} x={xdt}", flush=True)
    torch, rng, K = G.torch_(), np.random.default_rng(N + columns), 256 * columns
    first = N if kind == "sq" else max(256, N // 256 * 256)
    mats = [synth.gen_sq(rng, first, K) if kind == "sq" else synth.gen_vq(rng, first, K, int(kind[2:]))]
    if N == 512: mats.append(synth.gen_sq(rng, 48, K))
    dms = [B.upload(m, native=True) for m in mats]
    for M in Ms:
        xs = [synth.gen_activations(rng, M, K, xdt) for _ in mats]
        dev = [G.to_dev_bits(x) for x in xs]
        ys = [torch.full((M + 1, m.N), 7.0, dtype=torch.float32, device="cuda") for m in mats]
        B.rwkvq_linear_dispatch(B.DispatchTable([d.desc() for d in dms], dev, ys), M, B.DTYPES[xdt], B.F32)
        torch.cuda.synchronize()
        for m, x, y in zip(mats, xs, ys):
            got = y.cpu().numpy().astype(np.float64)
            assert (got[M] == 7.0).all()
            assert G.err_g2(got[:M], orc.linear(m, orc.widen(x, xdt), "f64")) <= 2e-5          # up to 7424 products, as above


# An option of batch 1: batch 2 to 16 takes the same kernel with either value
@pytest.mark.parametrize("M,xdt", [(2, "f16"), (8, "bf16"), (16, "f16")])
@pytest.mark.parametrize("N,columns", [(1024, 4), (8192, 16), (4096, 30), (24576, 3)])
def test_grid_option_changes_nothing(N, columns, M, xdt, options):
    print(f"grid option N={N} columns={columns} M={M} x={xdt}", flush=True)
    torch, rng = G.torch_(), np.random.default_rng(N + columns)
    m = synth.gen_sq(rng, N, 256 * columns)
    dm, dev = B.upload(m, native=True), G.to_dev_bits(synth.gen_activations(rng, M, m.K, xdt))
    ys = [torch.full((M, N), 7.0, dtype=torch.float32, device="cuda") for _ in range(2)]
    for i, y in enumerate(ys):
        options(B.OPT_SPLIT_GRID_2D, 1 + i)
        B.rwkvq_linear_dispatch(B.DispatchTable([dm.desc()], [dev], [y]), M, B.DTYPES[xdt], B.F32)
    torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1])


# 17 to 48 rows of x, calls of 257 to 384 workgroups of 64 rows of W: five and six row tiles per workgroup, the last one partly past the
# end of W, one and several column tiles per wavefront, another K and format in the same launch
@pytest.mark.parametrize("row_tiles,columns", [(1025, 1), (1060, 9), (1248, 4), (1252, 3), (1500, 2), (1504, 17)])
@pytest.mark.parametrize("M,xdt", [(17, "bf16"), (32, "f16"), (33, "f16"), (48, "f16"), (32, "bf16")])
def test_column_split_of_more_rows(row_tiles, columns, M, xdt, options):
    print(f"column split row tiles={row_tiles} columns={columns} M={M} x={xdt}", flush=True)
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_STREAM)
    options(B.OPT_STREAM_SPLIT_MAX_WORK, 1000000)
    torch, rng = G.torch_(), np.random.default_rng(row_tiles)
    K, few = 256 * columns, 256 * max(1, columns // 2)
    mats = [synth.gen_sq(rng, 16 * (row_tiles - 32), K if columns < 9 else few), synth.gen_vq(rng, 256, K, 6), synth.gen_vq(rng, 256, few, 8)]
    xs = [synth.gen_activations(rng, M, m.K, xdt) for m in mats]
    dms, dev = [B.upload(m, native=True) for m in mats], [G.to_dev_bits(x) for x in xs]
    ys = [torch.full((M + 1, m.N), 7.0, dtype=torch.float32, device="cuda") for m in mats]
    B.rwkvq_linear_dispatch(B.DispatchTable([d.desc() for d in dms], dev, ys), M, B.DTYPES[xdt], B.F32)
    torch.cuda.synchronize()
    for m, x, y in zip(mats, xs, ys):
        got = y.cpu().numpy().astype(np.float64)
        assert (got[M] == 7.0).all()
        # as above; the same products
        assert G.err_g2(got[:M], orc.linear(m, orc.widen(x, xdt), "f64")) <= 2e-5


# bf16 activations multiplied as they are by scalar-quantized matrices at 17 to 48 rows
@pytest.mark.parametrize("row_tiles,columns", [(1025, 1), (1060, 9), (1252, 3), (1280, 17)])
@pytest.mark.parametrize("M", [17, 33, 48])
def test_column_split_of_more_rows_bf16(row_tiles, columns, M, options):
    print(f"column split bf16 row tiles={row_tiles} columns={columns} M={M}", flush=True)
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_STREAM)
    options(B.OPT_STREAM_SPLIT_MAX_WORK, 1000000)
    torch, rng = G.torch_(), np.random.default_rng(row_tiles + M)
    mats = [synth.gen_sq(rng, 16 * (row_tiles - 3), 256 * columns), synth.gen_sq(rng, 48, 256 * max(1, columns // 2))]
    xs = [synth.gen_activations(rng, M, m.K, "bf16") for m in mats]
    dms, dev = [B.upload(m, native=True) for m in mats], [G.to_dev_bits(x) for x in xs]
    ys = [torch.full((M + 1, m.N), 7.0, dtype=torch.float32, device="cuda") for m in mats]
    B.rwkvq_linear_dispatch(B.DispatchTable([d.desc() for d in dms], dev, ys), M, B.BF16, B.F32)
    torch.cuda.synchronize()
    for m, x, y in zip(mats, xs, ys):
        got = y.cpu().numpy().astype(np.float64)
        assert (got[M] == 7.0).all()
        assert G.err_g2(got[:M], orc.linear(m, orc.widen(x, "bf16"), "f64")) <= 2e-5   # as above


# bf16 activations far from one, every format with one row tile per workgroup (as they are), two (8-bit VQ: converted) and three (VQ:
# converted), through the column split and the streaming kernels (1: never the split)
@pytest.mark.parametrize("scale", [1e-30, 1e30])
@pytest.mark.parametrize("kind", ["sq", "vq6", "vq8"])
@pytest.mark.parametrize("N,split", [(512, 0), (4352, 0), (8448, 0), (512, 1)])
def test_bf16_far_from_one(N, split, kind, scale, options):
    print(f"bf16 far from one N={N} {kind} scale={scale} split={split}", flush=True)
    options(B.OPT_STREAM_SPLIT_MAX_WORK, split)
    torch, rng, M = G.torch_(), np.random.default_rng(N), 5
    m = synth.gen_sq(rng, N, 768) if kind == "sq" else synth.gen_vq(rng, N, 768, int(kind[2:]))
    x = synth.f32_to_bf16_bits((rng.standard_normal((M, m.K)) * scale).astype(np.float32))
    y = G.gpu_gemm(B.upload(m, native=True), x, "bf16")
    # 768 products in binary32 partial sums, as above
    assert G.err_g2(y / scale, orc.linear(m, orc.widen(x, "bf16"), "f64") / scale) <= 2e-5


# The rule's two sides, bit for bit the kernel it is to take, and against the oracle: one round, always the column split (1536 row tiles are
# the most that fit one); several rounds up to 3200 row tiles and M = 12, or 4 from nine column tiles on; rows of at most 512 columns
# up to 4200 row tiles, 1536 beyond M = 8
@pytest.mark.parametrize("N,columns,M,xdt,forced", [(1024, 4, 8, "f16", 1000000), (256, 3, 2, "bf16", 1000000), (1024, 8, 16, "bf16", 1000000),
                                                    (24576, 3, 16, "f16", 1000000), (24592, 3, 16, "bf16", 1), (24592, 3, 12, "bf16", 1000000),
                                                    (51216, 3, 8, "f16", 1), (24592, 9, 4, "f16", 1000000), (24592, 9, 5, "f16", 1),
                                                    (1024, 2, 8, "f16", 1000000), (67200, 2, 8, "f16", 1000000), (67216, 2, 8, "f16", 1),
                                                    (24576, 2, 9, "bf16", 1000000), (24592, 2, 9, "bf16", 1)])
def test_rule(N, columns, M, xdt, forced, options):
    print(f"rule N={N} columns={columns} M={M} x={xdt}", flush=True)
    torch, rng = G.torch_(), np.random.default_rng(N + columns)
    m = synth.gen_sq(rng, N, 256 * columns)
    x = synth.gen_activations(rng, M, m.K, xdt)
    dm, dev = B.upload(m, native=True), G.to_dev_bits(x)
    ys = [torch.full((M, N), 7.0, dtype=torch.float32, device="cuda") for _ in range(2)]
    for i, y in enumerate(ys):
        if i:
            options(B.OPT_STREAM_SPLIT_MAX_WORK, forced)
        B.rwkvq_linear_dispatch(B.DispatchTable([dm.desc()], [dev], [y]), M, B.DTYPES[xdt], B.F32)
    torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1])
    assert G.err_g2(ys[0].cpu().numpy().astype(np.float64), orc.linear(m, orc.widen(x, xdt), "f64")) <= 2e-5


# Both sides of the rule at 17 to 48 rows, five and six row tiles per workgroup.  Up to eight column tiles a wavefront takes one here and a
# K group one there, and the partial sums are added in the same order, so the rule changes no bits: a call as the rule takes it, with the
# column split wherever it fits, and its first 1024 rows alone (too small a call for it)
@pytest.mark.parametrize("N,columns,M,xdt", [(16656, 2, 32, "f16"), (16656, 2, 33, "f16"), (16656, 2, 32, "bf16"), (16656, 2, 33, "bf16"), (16656, 8, 48, "bf16"),
                                             (24560, 2, 22, "f16"), (24560, 2, 23, "f16"), (24560, 8, 32, "f16"), (16656, 8, 48, "f16")])
def test_rule_of_more_rows(N, columns, M, xdt, options):
    print(f"rule N={N} columns={columns} M={M} x={xdt}", flush=True)
    torch, rng = G.torch_(), np.random.default_rng(N + columns)
    m = synth.gen_sq(rng, N, 256 * columns)
    few = synth.QMatrix("few", "sq", 1024, m.K, 0, m.codes[:1024].copy(), scales=m.scales[:1024].copy(), zeros=m.zeros[:1024].copy())
    x = synth.gen_activations(rng, M, m.K, xdt)
    dev = G.to_dev_bits(x)
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_STREAM)
    ys = []
    for q, forced in ((m, 0), (m, 1000000), (few, 0)):
        options(B.OPT_STREAM_SPLIT_MAX_WORK, forced)
        ys.append(torch.full((M, q.N), 7.0, dtype=torch.float32, device="cuda"))
        B.rwkvq_linear_dispatch(B.DispatchTable([B.upload(q, native=True).desc()], [dev], [ys[-1]]), M, B.DTYPES[xdt], B.F32)
        torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1]) and torch.equal(ys[0][:, :1024], ys[2])
    assert G.err_g2(ys[0].cpu().numpy().astype(np.float64), orc.linear(m, orc.widen(x, xdt), "f64")) <= 2e-5


# Matrices of two lengths at 33 and 48 rows, on both sides of the line by the longest rows (the same bits up to eight column tiles, as above)
@pytest.mark.parametrize("lengths", [(4, 4), (4, 6), (4, 8), (2, 8)])
@pytest.mark.parametrize("M,xdt", [(33, "f16"), (33, "bf16"), (48, "bf16")])
def test_rule_of_more_rows_of_two_lengths(lengths, M, xdt, options):
    print(f"two lengths {lengths} M={M} x={xdt}", flush=True)
    torch, rng = G.torch_(), np.random.default_rng(M)
    mats = [synth.gen_sq(rng, 16128, 256 * lengths[0]), synth.gen_sq(rng, 528, 256 * lengths[1])]
    xs = [synth.gen_activations(rng, M, m.K, xdt) for m in mats]
    dms, dev = [B.upload(m, native=True) for m in mats], [G.to_dev_bits(x) for x in xs]
    options(B.OPT_SMALL_BATCH_PATH, B.SMALL_BATCH_STREAM)
    got = []
    for forced in (0, 1000000):
        options(B.OPT_STREAM_SPLIT_MAX_WORK, forced)
        ys = [torch.full((M + 1, m.N), 7.0, dtype=torch.float32, device="cuda") for m in mats]
        B.rwkvq_linear_dispatch(B.DispatchTable([d.desc() for d in dms], dev, ys), M, B.DTYPES[xdt], B.F32)
        torch.cuda.synchronize()
        got.append(ys)
    for m, x, y, z in zip(mats, xs, *got):
        assert torch.equal(y, z) and (y[M] == 7.0).all()
        assert G.err_g2(y[:M].cpu().numpy().astype(np.float64), orc.linear(m, orc.widen(x, xdt), "f64")) <= 2e-5


# Rows of mixed lengths, two row tiles: both sides of the line by what stands on the device at once (one column tile per wavefront: 248
# workgroups of ten wavefronts, 488 of ten; several: 552 of four in more matrices than the two-dimensional grid takes, 184 of six, 264 of
# seven, 424 of six, 440 of seven and of eight, and 1056 of four, which fp16 and bf16 take differently, as they do the 424)
@pytest.mark.parametrize("shapes", [[(768, 768)] * 6 + [(2560, 768), (768, 2560)], [(2048, 768)] * 6 + [(2560, 768), (768, 2560)],
                                    [(768, 768)] * 12 + [(7680, 768), (768, 2560)],
                                    [(4608, 1280), (1280, 4608)], [(6912, 1536), (1536, 6912)], [(1280, 1280)] * 6 + [(4608, 1280), (1280, 4608)],
                                    [(2816, 2560)] * 4 + [(2816, 5120)], [(1280, 1280)] * 6 + [(5120, 1280), (1280, 7424)],
                                    [(4096, 768)] * 7 + [(4096, 768), (1024, 5120)]])
@pytest.mark.parametrize("kind", ["sq", "vq6"])
@pytest.mark.parametrize("M,xdt", [(3, "f16"), (15, "bf16")])
def test_rows_of_mixed_lengths(shapes, kind, M, xdt):
    print(f"mixed lengths {len(shapes)} matrices {shapes[0]} .. {shapes[-1]} {kind} M={M} x={xdt}", flush=True)
    torch, rng = G.torch_(), np.random.default_rng(M)
    of = {s: (synth.gen_sq(rng, *s) if kind == "sq" else synth.gen_vq(rng, *s, int(kind[2:]))) for s in sorted(set(shapes))}
    xs = {s: synth.gen_activations(rng, M, s[1], xdt) for s in of}
    dms, dev = {s: B.upload(m, native=True) for s, m in of.items()}, {s: G.to_dev_bits(x) for s, x in xs.items()}
    ys = [torch.full((M + 1, s[0]), 7.0, dtype=torch.float32, device="cuda") for s in shapes]
    B.rwkvq_linear_dispatch(B.DispatchTable([dms[s].desc() for s in shapes], [dev[s] for s in shapes], ys), M, B.DTYPES[xdt], B.F32)
    torch.cuda.synchronize()
    want = {s: orc.linear(of[s], orc.widen(xs[s], xdt), "f64") for s in of}
    for s, y in zip(shapes, ys):
        got = y.cpu().numpy().astype(np.float64)
        assert (got[M] == 7.0).all()
        assert G.err_g2(got[:M], want[s]) <= 2e-5           # up to 6912 products, as above
