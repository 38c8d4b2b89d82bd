"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same seeded inputs.

Bar: packed bytes, unpacked levels/headers and dequantized fp16 weights bit-exact; matmul outputs within
2e-3 of the oracle's fp64 result, measured as |y - y_ref| / max(|y_ref|, rms(y_ref)) per activation row.
"""
import sys

import numpy as np
import pytest

from paper_2401_08294_amd import synth

pytestmark = pytest.mark.gpu

TOL = 2e-3
NAMES = ["Q3H_B64", "Q4_B64", "Q4_B32", "Q8_B64", "Q8_B32", "Q6_B64", "Q5_B64", "Q3_B32", "Q2_B32"]
NAMES_WITH_MIDDLE_KERNEL = NAMES


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2401_08294_amd import iflow
    assert torch.cuda.is_available(), "needs a GPU"
    iflow.lib()
    return torch, iflow


def rel_err(y, yref):
    yref = np.asarray(yref, np.float64)
    rms = np.sqrt(np.mean(yref ** 2, axis=-1, keepdims=True))
    den = np.maximum(np.abs(yref), np.maximum(rms, 1e-30))
    return float(np.max(np.abs(np.asarray(y, np.float64) - yref) / den))


def gpu_quantize(torch, iflow, fmt, w):
    rows, cols = w.shape
    wd = torch.from_numpy(w).cuda()
    n = iflow.packed_bytes(fmt, rows, cols)
    packed = torch.full((n + 64,), 0xA5, dtype=torch.uint8, device="cuda")     # canary tail
    iflow.quantize(fmt, wd, rows, cols, packed, n)
    torch.cuda.synchronize()
    host = packed.cpu().numpy()
    assert (host[n:] == 0xA5).all(), "quantizer wrote past the packed size"
    return packed, host[:n]


def gpu_dequant(torch, iflow, fmt, packed, rows, cols):
    out = torch.empty((rows, cols), dtype=torch.float16, device="cuda")
    iflow.dequant(fmt, packed, rows, cols, out)
    torch.cuda.synchronize()
    return out.cpu().numpy().view(np.uint16)


def gpu_unpack(torch, iflow, fmt, packed, rows, cols):
    nbk = cols // iflow.format_block(fmt)
    lv = torch.empty((rows, cols), dtype=torch.uint8, device="cuda")
    sc = torch.empty((rows, nbk), dtype=torch.int16, device="cuda")
    of = torch.empty((rows, nbk), dtype=torch.int16, device="cuda")
    iflow.unpack_logical(fmt, packed, rows, cols, lv, sc, of)
    torch.cuda.synchronize()
    return lv.cpu().numpy(), sc.cpu().numpy().view(np.uint16), of.cpu().numpy().view(np.uint16)


def gpu_gemm(torch, iflow, fmt, packed, rows, cols, x16):
    batch = x16.shape[0]
    xd = torch.from_numpy(x16.view(np.int16)).cuda()
    y = torch.full((batch, rows), float("nan"), dtype=torch.float16, device="cuda")
    if batch == 1:
        iflow.qgemv(fmt, packed, rows, cols, xd, y)
    else:
        iflow.qgemm(fmt, packed, rows, cols, xd, batch, y)
    torch.cuda.synchronize()
    return y.cpu().numpy().astype(np.float64)


def check_all(torch, iflow, orc, name, w, x16, tag):
    """quantize -> bytes, unpack, dequant bit-exact; gemm within tolerance."""
    fmt = iflow.FORMATS[name]
    rows, cols = w.shape
    say(f"[case] {tag} fmt={name} rows={rows} cols={cols} batch={x16.shape[0]}")
    q, s, o = orc.quantize(orc.FORMATS[name], w)
    ref_bytes = orc.pack_device(orc.FORMATS[name], q, s, o)
    packed, got_bytes = gpu_quantize(torch, iflow, fmt, w)
    assert got_bytes.size == ref_bytes.size
    nbad = int(np.count_nonzero(got_bytes != ref_bytes))
    assert nbad == 0, f"{nbad} packed bytes differ, first at {int(np.flatnonzero(got_bytes != ref_bytes)[0])}"
    lv, sc, of = gpu_unpack(torch, iflow, fmt, packed, rows, cols)
    assert np.array_equal(lv, q) and np.array_equal(sc, s) and np.array_equal(of, o)
    if name == "Q3H_B64":                                       # the stored pair codes themselves (Eq.4), via the oracle's encoder
        table = np.array([[orc.pair_encode(a_, b_) for b_ in range(11)] for a_ in range(11)], np.uint8)
        codes = torch.empty((rows, cols // 2), dtype=torch.uint8, device="cuda")
        iflow.unpack_pair_codes(fmt, packed, rows, cols, codes)
        torch.cuda.synchronize()
        assert np.array_equal(codes.cpu().numpy(), table[q[:, 0::2], q[:, 1::2]]), "pair codes differ"
    ref_deq = orc.dequant(orc.FORMATS[name], q, s, o)
    got_deq = gpu_dequant(torch, iflow, fmt, packed, rows, cols)
    assert np.array_equal(got_deq, ref_deq), "dequantized fp16 weights differ"
    yref = orc.gemm(ref_deq, x16.view(np.uint16), threads=8)
    y = gpu_gemm(torch, iflow, fmt, packed, rows, cols, x16)
    assert not np.isnan(y).any(), "an output was never written"
    e = rel_err(y, yref)
    say(f"        max rel err {e:.3e}")
    assert e <= TOL
    return e


# ---- config 1: 1024 x 1024, sigma 0.02, batch 1 - every format ---------------------------------------
@pytest.mark.parametrize("name", NAMES)
def test_config1_all_steps(gpu, orc, name):
    torch, iflow = gpu
    w = synth.weights(1024, 1024, 0.02, synth.BASE_SEED + 1)
    x = synth.activations(1, 1024, synth.BASE_SEED + 101)
    check_all(torch, iflow, orc, name, w, x, "config1")


# ---- ragged and tiny shapes: single block, partial strips, rows that do not fill a workgroup ------------
@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("rows,nblocks", [(1, 1), (3, 2), (5, 65), (67, 64), (130, 172), (9, 200)])
def test_ragged_shapes(gpu, orc, name, rows, nblocks):
    torch, iflow = gpu
    cols = nblocks * iflow.format_block(iflow.FORMATS[name])
    w = synth.weights(rows, cols, 0.02, synth.BASE_SEED + rows * 1000 + nblocks)
    x = synth.activations(1, cols, synth.BASE_SEED + 7)
    check_all(torch, iflow, orc, name, w, x, "ragged")


# ---- very long rows: the one-vector kernel stages a whole row of activations in LDS; beyond its limit (144 KiB: 32 strips
#      of 2048 columns, 57 strips of 1024 for 8-bit; half as many with two vectors) the launcher takes the older kernel.
#      Both sides of the limit. ------------
@pytest.mark.parametrize("name,cols,batch", [("Q4_B64", 65536, 1), ("Q4_B64", 65536 + 2048, 1), ("Q8_B32", 57 * 1024, 1),
                                             ("Q8_B32", 58 * 1024 + 32, 1), ("Q6_B64", 65536 + 64, 1), ("Q2_B32", 65536 - 32, 1),
                                             ("Q4_B64", 32768, 2), ("Q4_B64", 32768 + 64, 2), ("Q8_B64", 28 * 1024 + 64, 2),
                                             ("Q5_B64", 65536, 2)])
def test_rows_at_the_staging_limit(gpu, orc, name, cols, batch):
    torch, iflow = gpu
    w = synth.weights(5, cols, 0.02, synth.BASE_SEED + 77)
    x = synth.activations(batch, cols, synth.BASE_SEED + 78)
    check_all(torch, iflow, orc, name, w, x, "long-rows")


# ---- many short rows: one block per row, a quarter of a million rows (launch grids, row-group arithmetic) -------------------
@pytest.mark.parametrize("name", ["Q3H_B64", "Q4_B32", "Q6_B64", "Q8_B64", "Q2_B32"])
@pytest.mark.parametrize("batch", [1, 3])
def test_tall_and_thin(gpu, orc, name, batch):
    torch, iflow = gpu
    rows, cols = 262144 + 3, 64
    w = synth.weights(rows, cols, 0.02, synth.BASE_SEED + 88)
    x = synth.activations(batch, cols, synth.BASE_SEED + 89)
    check_all(torch, iflow, orc, name, w, x, "tall-thin")


# ---- a seeded sweep over shapes and batch sizes on both sides of every kernel-selection threshold (1 | 2, for 8-bit formats 2..4 | up to 16 |
#      17 and more; column counts that are and are not multiples of 64 for the 32-wide blocks) -----------------------------------
def _sweep_cases():
    rng = np.random.default_rng(synth.BASE_SEED + 4242)
    batches = [1, 2, 3, 4, 5, 11, 12, 16, 17, 31, 32, 33, 64, 65, 130]
    cases = []
    for name in NAMES:
        for _ in range(4):
            rows = int(rng.integers(1, 300))
            nblocks = int(rng.integers(1, 141))
            batch = int(rng.choice(batches))
            cases.append((name, rows, nblocks, batch))
    return cases


@pytest.mark.parametrize("name,rows,nblocks,batch", _sweep_cases())
def test_seeded_shape_sweep(gpu, orc, name, rows, nblocks, batch):
    torch, iflow = gpu
    cols = nblocks * iflow.format_block(iflow.FORMATS[name])
    w = synth.weights(rows, cols, 0.02, synth.BASE_SEED + 17 * rows + nblocks, outlier_prob=0.001)
    x = synth.activations(batch, cols, synth.BASE_SEED + batch)
    check_all(torch, iflow, orc, name, w, x, "sweep")


# ---- small batches (2, 3, 4 share a pass; 5 and 16 take several) ----------------------------------------
@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("batch", [2, 3, 4, 5, 8, 16, 21])
def test_small_batch(gpu, orc, name, batch):
    torch, iflow = gpu
    rows, cols = 300, 4096 + 64 * 3
    w = synth.weights(rows, cols, 0.02, synth.BASE_SEED + 31, outlier_prob=0.001)
    x = synth.activations(batch, cols, synth.BASE_SEED + 32)
    check_all(torch, iflow, orc, name, w, x, "batch")


# ---- small batches on tall matrices: a workgroup takes several groups of sixteen rows in turn (two or three here, so both
#      an even and an odd count), over one strip or two ragged ones; weights drawn on the device, every output against the
#      one-vector kernel on the same bytes, sampled rows against the oracle ---------------------------------------------
def small_batch_tall(torch, iflow, orc, name, rows, cols, batch, seed):
    fmt, ofmt = iflow.FORMATS[name], orc.FORMATS[name]
    say(f"[case] small batch, tall: fmt={name} rows={rows} cols={cols} batch={batch}")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    wd = torch.randn((rows, cols), generator=gen, device="cuda", dtype=torch.float32) * 0.02
    n = iflow.packed_bytes(fmt, rows, cols)
    packed = torch.empty(n, dtype=torch.uint8, device="cuda")
    iflow.quantize(fmt, wd, rows, cols, packed, n)
    idx = synth.sample_rows(rows, 48, seed + 1)
    idx[:3] = [0, rows - 1, rows - 17 if rows > 17 else 0]
    w_rows = wd[torch.from_numpy(idx).cuda()].cpu().numpy()
    del wd
    x = synth.activations(batch, cols, seed + 2)
    y = gpu_gemm(torch, iflow, fmt, packed, rows, cols, x)
    assert np.isfinite(y).all()
    q, s, o = orc.quantize(ofmt, w_rows)
    yref = orc.gemm(orc.dequant(ofmt, q, s, o), x.view(np.uint16))
    rms = np.sqrt(np.mean(y ** 2, axis=-1, keepdims=True))
    e = float(np.max(np.abs(y[:, idx] - yref) / np.maximum(np.abs(yref), rms)))
    say(f"        max rel err on {len(idx)} sampled rows {e:.3e}")
    assert e <= TOL
    for b in range(batch):                                     # all rows: the one-vector kernel, same packed bytes
        y1 = gpu_gemm(torch, iflow, fmt, packed, rows, cols, x[b:b + 1])
        e1 = float(np.max(np.abs(y[b] - y1[0]) / np.maximum(np.abs(y1[0]), rms[b])))
        assert e1 <= TOL, f"vector {b}: {e1}"          # two fp16 roundings of sums taken in different orders


@pytest.mark.parametrize("name", NAMES_WITH_MIDDLE_KERNEL)
@pytest.mark.parametrize("cols", [1024, 4096 + 64 * 3])
def test_small_batch_tall(gpu, orc, name, cols):
    torch, iflow = gpu
    small_batch_tall(torch, iflow, orc, name, 16 * 256 * 2 + 16 * 100 + 5, cols, 5 if "Q8" in name else 3, synth.BASE_SEED + 940)
    small_batch_tall(torch, iflow, orc, name, 16 * 256 + 7, cols, 16, synth.BASE_SEED + 950)


def test_small_batch_more_rounds_than_one_launch_holds(gpu, orc):
    """Rows spanning two strips and more than sixteen row groups per workgroup: the entry point splits the rows."""
    torch, iflow = gpu
    small_batch_tall(torch, iflow, orc, "Q3H_B64", 16 * 256 * 17 + 40, 4096 + 64, 4, synth.BASE_SEED + 960)


# ---- 32-wide blocks allow column counts that are not a multiple of 64: those stay on the vector kernel at any batch ----
@pytest.mark.parametrize("name", ["Q4_B32", "Q8_B32", "Q3_B32", "Q2_B32"])
@pytest.mark.parametrize("batch", [3, 7, 40])
def test_odd_block_count_batches(gpu, orc, name, batch):
    torch, iflow = gpu
    rows, cols = 70, 32 * 67
    w = synth.weights(rows, cols, 0.02, synth.BASE_SEED + 61, outlier_prob=0.001)
    x = synth.activations(batch, cols, synth.BASE_SEED + 62)
    check_all(torch, iflow, orc, name, w, x, "odd block count")


# ---- 17 and more vectors run in tiles on the matrix cores (64-column chunks): ragged in every dimension ----
@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("batch,rows,nchunks", [(32, 64, 1), (100, 200, 69), (512, 70, 3)])
def test_large_batch_mfma(gpu, orc, name, batch, rows, nchunks):
    torch, iflow = gpu
    cols = 64 * nchunks
    w = synth.weights(rows, cols, 0.02, synth.BASE_SEED + 71 + batch, outlier_prob=0.001)
    x = synth.activations(batch, cols, synth.BASE_SEED + 72)
    e = check_all(torch, iflow, orc, name, w, x, "mfma")
    assert e <= 6e-4        # exact fp16 weights, fp32 accumulation: only the fp16 rounding of the output is left


def test_batch512_full_size_sampled_rows(gpu, orc):
    """The prefill-like case of the benchmark configs: 4096 x 4096, batch 512, Q3H, checked on sampled weight rows."""
    torch, iflow = gpu
    rows, cols, batch = 4096, 4096, 512
    fmt, ofmt = iflow.Q3H_B64, orc.Q3H_B64
    say(f"[case] batch512 full-size rows={rows} cols={cols}")
    w = synth.weights(rows, cols, 0.02, synth.BASE_SEED + 81)
    x = synth.activations(batch, cols, synth.BASE_SEED + 82)
    packed, _ = gpu_quantize(torch, iflow, fmt, w)
    y = gpu_gemm(torch, iflow, fmt, packed, rows, cols, x)
    idx = synth.sample_rows(rows, 96, synth.BASE_SEED + 83)
    q, s, o = orc.quantize(ofmt, w[idx])
    yref = orc.gemm(orc.dequant(ofmt, q, s, o), x.view(np.uint16), threads=8)
    e = rel_err(y[:, idx], yref)
    say(f"        max rel err on {len(idx)} sampled rows x {batch} {e:.3e}")
    assert np.isfinite(y).all() and e <= 6e-4


# ---- several projections of one activation vector in one launch -----------------------------------------
@pytest.mark.parametrize("name", ["Q3H_B64", "Q4_B64", "Q8_B32", "Q6_B64", "Q3_B32", "Q2_B32"])
def test_qgemv_multi_matches_single_launches(gpu, orc, name):
    torch, iflow = gpu
    fmt, ofmt = iflow.FORMATS[name], orc.FORMATS[name]
    cols = 4096 + 64 * 5
    row_counts = [100, 37, 256, 1]
    say(f"[case] multi fmt={name} rows={row_counts} cols={cols}")
    x = synth.activations(1, cols, synth.BASE_SEED + 91)
    xd = torch.from_numpy(x.view(np.int16)).cuda()
    packs, ys, refs = [], [], []
    for i, rows in enumerate(row_counts):
        w = synth.weights(rows, cols, 0.02, synth.BASE_SEED + 92 + i)
        packed, _ = gpu_quantize(torch, iflow, fmt, w)
        packs.append(packed)
        ys.append(torch.full((rows,), float("nan"), dtype=torch.float16, device="cuda"))
        q, s, o = orc.quantize(ofmt, w)
        refs.append(orc.gemm(orc.dequant(ofmt, q, s, o), x.view(np.uint16))[0])
    iflow.qgemv_multi(fmt, packs, row_counts, cols, xd, ys)
    torch.cuda.synchronize()
    for packed, rows, y, ref in zip(packs, row_counts, ys, refs):
        single = torch.empty((rows,), dtype=torch.float16, device="cuda")
        iflow.qgemv(fmt, packed, rows, cols, xd, single)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        assert not np.isnan(got).any()
        assert rel_err(got.astype(np.float64)[None, :], ref[None, :]) <= TOL
        assert np.array_equal(got.view(np.uint16), single.cpu().numpy().view(np.uint16))   # same arithmetic per row
    with pytest.raises(iflow.IflowError) as ei:
        iflow.qgemv_multi(fmt, packs * 3, row_counts * 3, cols, xd, ys * 3)          # more than eight matrices
    assert ei.value.status == iflow.ERR_SHAPE


# ---- degenerate values ---------------------------------------------------------------------------------
@pytest.mark.parametrize("name", NAMES)
def test_degenerate_blocks(gpu, orc, name):
    torch, iflow = gpu
    rows, cols = 8, 512
    w = synth.weights(rows, cols, 0.02, synth.BASE_SEED + 41)
    w[0, :] = 0.0                      # all-zero row
    w[1, :64] = -0.0                   # negative zeros
    w[2, :] = 0.37                     # constant blocks
    w[3, :] = np.linspace(-1, 1, cols, dtype=np.float32)      # ramp: exact ties are likely
    w[4, :] *= 1e-6                    # scale in fp16's subnormal range
    w[5, :] *= 1e-9                    # range underflows fp16: scale 0
    w[6, :128] = np.float32(1e-40)     # fp32 subnormals
    w[7, :] = np.round(w[7, :] * 500) / 4   # many exact .5 ties after division
    x = synth.activations(1, cols, synth.BASE_SEED + 42)
    check_all(torch, iflow, orc, name, w, x, "degenerate")


def test_exact_ties_round_half_away(gpu, orc):
    """scale 1, offset 0: levels are the weights themselves, .5 cases must round away from zero."""
    torch, iflow = gpu
    base = np.array([0, 0.5, 1.5, 2.5, 3.49, 3.51, 4.5, 10] * 8, np.float32)
    w = np.tile(base, (4, 1))
    x = synth.activations(1, 64, synth.BASE_SEED + 43)
    check_all(torch, iflow, orc, "Q3H_B64", w, x, "ties")
    w15 = np.tile(np.array([0, 0.5, 1.5, 2.5, 7.5, 14.5, 15, 3] * 8, np.float32), (4, 1))
    check_all(torch, iflow, orc, "Q4_B64", w15, x, "ties")
    for name, L in (("Q6_B64", 63), ("Q5_B64", 31), ("Q3_B32", 7), ("Q2_B32", 3)):
        wl = np.tile(np.array([0, 0.5, 1.5, 2.5, L - 0.5, L / 2, L, 1] * 8, np.float32), (4, 1))
        check_all(torch, iflow, orc, name, wl, x, "ties")


def test_outliers_config3_shape_slice(gpu, orc):
    """Config 3's value recipe (0.1 % of entries scaled by 10) on a slice of a 7B-shaped layer, in the 8-bit, 4-bit and 3.5-bit
    formats at the configuration's batch sizes 1, 2, 4, 8 and 16."""
    torch, iflow = gpu
    w = synth.weights(256, 11008, 0.02, synth.BASE_SEED + 3, outlier_prob=0.001)
    for name in ("Q3H_B64", "Q4_B64", "Q8_B64"):
        for batch in (1, 2, 4, 8, 16):
            x = synth.activations(batch, 11008, synth.BASE_SEED + 33 + batch)
            check_all(torch, iflow, orc, name, w, x, "config3-slice")


# ---- full-size shapes in the benchmark's launch configuration, checked on sampled rows ------------------
@pytest.mark.parametrize("rows,cols,sigma", [(4096, 4096, 0.02), (11008, 4096, 0.02), (4096, 11008, 0.02), (8192, 8192, 0.015)])
def test_full_size_sampled_rows(gpu, orc, rows, cols, sigma):
    torch, iflow = gpu
    name, fmt = "Q3H_B64", iflow.FORMATS["Q3H_B64"]
    say(f"[case] full-size fmt={name} rows={rows} cols={cols}")
    w = synth.weights(rows, cols, sigma, synth.BASE_SEED + rows + cols)
    x = synth.activations(1, cols, synth.BASE_SEED + 55)
    packed, got_bytes = gpu_quantize(torch, iflow, fmt, w)
    y = gpu_gemm(torch, iflow, fmt, packed, rows, cols, x)
    deq = gpu_dequant(torch, iflow, fmt, packed, rows, cols)
    idx = synth.sample_rows(rows, 192, synth.BASE_SEED + 56)
    ofmt = orc.FORMATS[name]
    q, s, o = orc.quantize(ofmt, w[idx])                       # blocks never cross rows: rows can be checked alone
    row_bytes = orc.packed_bytes(ofmt, 1, cols)
    ref_rows = orc.pack_device(ofmt, q, s, o).reshape(len(idx), row_bytes)
    assert np.array_equal(got_bytes.reshape(rows, row_bytes)[idx], ref_rows)
    ref_deq = orc.dequant(ofmt, q, s, o)
    assert np.array_equal(deq[idx], ref_deq)
    yref = orc.gemm(ref_deq, x.view(np.uint16), threads=8)
    # the rms floor of the error metric comes from the sampled rows (same distribution as the rest)
    e = rel_err(y[:, idx], yref)
    say(f"        max rel err on {len(idx)} sampled rows {e:.3e}")
    assert e <= TOL
    # properties that hold at any size: every output written and finite, linear in x
    assert np.isfinite(y).all()
    y2 = gpu_gemm(torch, iflow, fmt, packed, rows, cols, (x * np.float16(2)).astype(np.float16))
    assert np.array_equal(y2, 2 * y)


# ---- config 3 at its full 7B shapes: 8-bit, 4-bit and one bit-plane format, one to sixteen vectors, outliers ----
@pytest.mark.parametrize("name", ["Q4_B64", "Q8_B64", "Q6_B64"])
@pytest.mark.parametrize("rows,cols", [(4096, 4096), (11008, 4096), (4096, 11008)])
def test_config3_full_size_sampled_rows(gpu, orc, name, rows, cols):
    """The launches the benchmark times for the formats other than 3.5-bit (thousands of rows and several strips at once:
    more than one row group per wavefront), checked on sampled rows: packed bytes and fp16 weights bit-exact, products at 1,
    2, 4, 8 and 16 vectors within tolerance, every output finite."""
    torch, iflow = gpu
    fmt, ofmt = iflow.FORMATS[name], orc.FORMATS[name]
    say(f"[case] config-3 full size fmt={name} rows={rows} cols={cols}, 0.1 % outliers x 10")
    w = synth.weights(rows, cols, 0.02, synth.BASE_SEED + 3000 + rows + cols, outlier_prob=0.001)
    packed, got_bytes = gpu_quantize(torch, iflow, fmt, w)
    idx = synth.sample_rows(rows, 96, synth.BASE_SEED + 3001)
    q, s, o = orc.quantize(ofmt, w[idx])
    lv, sc, of = gpu_unpack(torch, iflow, fmt, packed, rows, cols)     # layout-independent: levels and headers of the sampled rows
    assert np.array_equal(lv[idx], q) and np.array_equal(sc[idx], s) and np.array_equal(of[idx], o)
    del lv, sc, of
    if name == "Q3H_B64":                                              # (formats whose rows are contiguous in the packed buffer)
        row_bytes = orc.packed_bytes(ofmt, 1, cols)
        assert np.array_equal(got_bytes.reshape(rows, row_bytes)[idx], orc.pack_device(ofmt, q, s, o).reshape(len(idx), row_bytes))
    ref_deq = orc.dequant(ofmt, q, s, o)
    deq = gpu_dequant(torch, iflow, fmt, packed, rows, cols)
    assert np.array_equal(deq[idx], ref_deq)
    del deq
    for batch in (1, 2, 4, 8, 16):
        x = synth.activations(batch, cols, synth.BASE_SEED + 3002 + batch)
        y = gpu_gemm(torch, iflow, fmt, packed, rows, cols, x)
        yref = orc.gemm(ref_deq, x.view(np.uint16), threads=8)
        e = rel_err(y[:, idx], yref)
        say(f"        batch {batch}: max rel err on {len(idx)} sampled rows {e:.3e}")
        assert np.isfinite(y).all() and e <= TOL


@pytest.mark.parametrize("name", ["Q4_B64", "Q8_B64"])
def test_config3_formats_at_a_70b_shape(gpu, orc, name):
    """28672 x 8192, one vector, in the 4- and 8-bit formats: the launch geometry of the tallest matrix the benchmark times."""
    torch, iflow = gpu
    fmt, ofmt = iflow.FORMATS[name], orc.FORMATS[name]
    rows, cols = 28672, 8192
    say(f"[case] 70B-shape fmt={name} rows={rows} cols={cols}, 0.1 % outliers x 10")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(synth.BASE_SEED + 3100)
    wd = torch.randn((rows, cols), generator=gen, device="cuda", dtype=torch.float32) * 0.015
    wd = torch.where(torch.rand((rows, cols), generator=gen, device="cuda") < 0.001, wd * 10.0, wd)
    n = iflow.packed_bytes(fmt, rows, cols)
    packed = torch.empty(n, dtype=torch.uint8, device="cuda")
    iflow.quantize(fmt, wd, rows, cols, packed, n)
    idx = synth.sample_rows(rows, 64, synth.BASE_SEED + 3101)
    w_rows = wd[torch.from_numpy(idx).cuda()].cpu().numpy()
    del wd
    q, s, o = orc.quantize(ofmt, w_rows)
    lv, sc, of = gpu_unpack(torch, iflow, fmt, packed, rows, cols)
    assert np.array_equal(lv[idx], q) and np.array_equal(sc[idx], s) and np.array_equal(of[idx], o)
    del lv, sc, of
    ref_deq = orc.dequant(ofmt, q, s, o)
    x = synth.activations(1, cols, synth.BASE_SEED + 3102)
    y = gpu_gemm(torch, iflow, fmt, packed, rows, cols, x)
    e = rel_err(y[:, idx], orc.gemm(ref_deq, x.view(np.uint16), threads=8))
    say(f"        max rel err on {len(idx)} sampled rows {e:.3e}")
    assert np.isfinite(y).all() and e <= TOL


# ---- 70B-shaped layers (config 4): sampled rows, batch 1 and 8 ----------------------------------------------
@pytest.mark.parametrize("rows,cols", [(28672, 8192), (8192, 28672)])
def test_70b_shapes_sampled_rows(gpu, orc, rows, cols):
    torch, iflow = gpu
    fmt, ofmt = iflow.Q3H_B64, orc.Q3H_B64
    say(f"[case] 70B-shape rows={rows} cols={cols}")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(synth.BASE_SEED + rows)
    wd = torch.randn((rows, cols), generator=gen, device="cuda", dtype=torch.float32) * 0.015
    n = iflow.packed_bytes(fmt, rows, cols)
    packed = torch.empty(n, dtype=torch.uint8, device="cuda")
    iflow.quantize(fmt, wd, rows, cols, packed, n)
    idx = synth.sample_rows(rows, 64, synth.BASE_SEED + 57)
    w_rows = wd[torch.from_numpy(idx).cuda()].cpu().numpy()          # the oracle sees the same fp32 bits as the GPU quantizer
    del wd
    q, s, o = orc.quantize(ofmt, w_rows)
    row_bytes = orc.packed_bytes(ofmt, 1, cols)
    got = packed.cpu().numpy().reshape(rows, row_bytes)[idx]
    assert np.array_equal(got, orc.pack_device(ofmt, q, s, o).reshape(len(idx), row_bytes))
    ref_deq = orc.dequant(ofmt, q, s, o)
    for batch in (1, 8):
        x = synth.activations(batch, cols, synth.BASE_SEED + 58 + batch)
        y = gpu_gemm(torch, iflow, fmt, packed, rows, cols, x)
        yref = orc.gemm(ref_deq, x.view(np.uint16), threads=8)
        e = rel_err(y[:, idx], yref)
        say(f"        batch {batch}: max rel err on {len(idx)} sampled rows {e:.3e}")
        assert np.isfinite(y).all() and e <= TOL


# ---- a captured decode-step weight stream (config 5, two layers deep) replays to the eager result -------------
def test_hip_graph_replay_matches_eager(gpu, orc):
    torch, iflow = gpu
    fmt = iflow.Q3H_B64
    shapes = [(512, 1024), (512, 1024), (1408, 1024), (1024, 1408)]      # q/k, gate-like, down-like slices
    say("[case] graph replay of two layers x four linears")
    layers = []
    for layer in range(2):
        mats = []
        for i, (rows, cols) in enumerate(shapes):
            w = synth.weights(rows, cols, 0.02, synth.BASE_SEED + 200 + 10 * layer + i)
            packed, _ = gpu_quantize(torch, iflow, fmt, w)
            mats.append((rows, cols, packed))
        layers.append(mats)
    xs = {c: torch.from_numpy(synth.activations(1, c, synth.BASE_SEED + 300 + c).view(np.int16)).cuda() for c in (1024, 1408)}
    ys = [[torch.zeros((rows,), dtype=torch.float16, device="cuda") for rows, _, _ in mats] for mats in layers]

    stream = torch.cuda.Stream()

    def run_all():
        for mats, outs in zip(layers, ys):
            iflow.qgemv_multi(fmt, [mats[0][2], mats[1][2]], [mats[0][0], mats[1][0]], 1024, xs[1024], outs[:2], stream=stream.cuda_stream)
            for (rows, cols, packed), y in list(zip(mats, outs))[2:]:
                iflow.qgemv(fmt, packed, rows, cols, xs[cols], y, stream=stream.cuda_stream)

    with torch.cuda.stream(stream):
        run_all()
        stream.synchronize()
        eager = [[y.clone() for y in outs] for outs in ys]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            run_all()
        for rep in range(3):                                   # replays with eager work and synchronisation in between
            for outs in ys:
                for y in outs:
                    y.zero_()
            stream.synchronize()
            graph.replay()
            stream.synchronize()
            for outs, ref in zip(ys, eager):
                for y, r in zip(outs, ref):
                    assert torch.equal(y, r), f"replay {rep} differs from the eager result"
            run_all()
            stream.synchronize()


# ---- unit vectors tie the product to the dequantizer; argument errors come back as codes ----------------
def test_unit_vector_returns_column(gpu, orc):
    torch, iflow = gpu
    for name in NAMES:
        fmt = iflow.FORMATS[name]
        rows, cols = 70, 4096 + 128
        w = synth.weights(rows, cols, 0.02, synth.BASE_SEED + 61)
        packed, _ = gpu_quantize(torch, iflow, fmt, w)
        deq = gpu_dequant(torch, iflow, fmt, packed, rows, cols).view(np.float16).astype(np.float64)
        for k in (0, 1, 63, 64, 4095, 4096, cols - 1):
            e = np.zeros((1, cols), np.float16)
            e[0, k] = 1
            y = gpu_gemm(torch, iflow, fmt, packed, rows, cols, e)[0]
            # the kernel removes a conversion bias of up to 2037 * x: exact to fp32 rounding of that magnitude
            assert np.max(np.abs(y - deq[:, k])) <= 2e-3 * np.max(np.abs(deq[:, k])) + 1e-4, (name, k)


def test_argument_errors(gpu):
    torch, iflow = gpu
    w = torch.zeros((4, 128), dtype=torch.float32, device="cuda")
    buf = torch.zeros(4096, dtype=torch.uint8, device="cuda")
    with pytest.raises(iflow.IflowError) as ei:
        iflow.quantize(iflow.Q3H_B64, w, 4, 100, buf, 4096)
    assert ei.value.status == iflow.ERR_SHAPE
    with pytest.raises(iflow.IflowError) as ei:
        iflow.quantize(iflow.Q3H_B64, w, 4, 128, buf, 16)
    assert ei.value.status == iflow.ERR_SIZE
    with pytest.raises(iflow.IflowError) as ei:
        iflow.quantize(9, w, 4, 128, buf, 4096)
    assert ei.value.status == iflow.ERR_FORMAT
    with pytest.raises(iflow.IflowError) as ei:
        iflow.quantize(iflow.Q3H_B64, w.data_ptr() + 4, 4, 128, buf, 4096)
    assert ei.value.status == iflow.ERR_ALIGN
    with pytest.raises(iflow.IflowError) as ei:
        iflow.qgemm(iflow.Q3H_B64, buf, 4, 128, w, 0, buf)
    assert ei.value.status == iflow.ERR_SHAPE


# ---- the batched paths under HIP-graph replay: small-batch MFMA kernel (two launches for a split tall matrix included)
#      and the batch-512 kernel, replayed with new activations, against eager results ----------------------------------
@pytest.mark.parametrize("name", ["Q3H_B64", "Q8_B64"])
def test_hip_graph_replay_of_batched_products(gpu, orc, name):
    torch, iflow = gpu
    fmt = iflow.FORMATS[name]
    say(f"[case] graph replay of batched products, fmt={name}")
    cases = [(600, 4096 + 128, 16), (16 * 256 * 2 + 9, 1024, 7), (200, 1024, 512)]
    mats = []
    for i, (rows, cols, batch) in enumerate(cases):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(synth.BASE_SEED + 980 + i)
        wd = torch.randn((rows, cols), generator=gen, device="cuda", dtype=torch.float32) * 0.02
        n = iflow.packed_bytes(fmt, rows, cols)
        packed = torch.empty(n, dtype=torch.uint8, device="cuda")
        iflow.quantize(fmt, wd, rows, cols, packed, n)
        X = torch.zeros((batch, cols), dtype=torch.float16, device="cuda")
        Y = torch.zeros((batch, rows), dtype=torch.float16, device="cuda")
        mats.append((rows, cols, batch, packed, X, Y))
    stream = torch.cuda.Stream()

    def run_all():
        for rows, cols, batch, packed, X, Y in mats:
            iflow.qgemm(fmt, packed, rows, cols, X, batch, Y, stream=stream.cuda_stream)

    def fill(seed):
        for i, (rows, cols, batch, packed, X, Y) in enumerate(mats):
            X.copy_(torch.from_numpy(synth.activations(batch, cols, seed + i).view(np.int16)).cuda().view(torch.float16))
            Y.fill_(float("nan"))

    fill(synth.BASE_SEED + 985)
    with torch.cuda.stream(stream):
        run_all()
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            run_all()
    for rep in range(3):
        fill(synth.BASE_SEED + 990 + 10 * rep)
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            run_all()
        stream.synchronize()
        eager = [m[5].cpu().numpy().view(np.uint16).copy() for m in mats]
        for m in mats:
            m[5].fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for i, m in enumerate(mats):
            got = m[5].cpu().numpy().view(np.uint16)
            assert np.array_equal(got, eager[i]), f"replay {rep}, case {i}: {(got != eager[i]).sum()} outputs differ"
            assert np.isfinite(m[5].cpu().numpy().astype(np.float32)).all()
