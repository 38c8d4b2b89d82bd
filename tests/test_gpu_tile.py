"""GPU parity of the tiled matrix-core product (17 and more activation vectors): the launcher's choice over shapes of all sizes, and every tile
by number in every format, with ragged rows, vectors and column chunks (a run of chunks that ends inside a group, chunks missing for some of the
wavefronts that share K, enough runs that every buffer is filled again several times), rows whose outputs can and cannot be stored
sixteen bytes at a time.

Reference: plain fp64 matrix product (torch) of the activations with iflow_dequant's fp16 weights, which other tests hold bit-exact
to the oracle.  The kernel multiplies exactly those weights and accumulates in fp32, so what is left is one fp16 rounding of the output
(2^-11 = 4.9e-4 of the value) and the fp32 sums (below 1e-4 at 13000 columns): 6e-4 of max(|y|, rms)."""
import ctypes as C

import pytest

from paper_2401_08294_amd import synth
from test_gpu_parity import NAMES, gpu, say  # noqa: F401

pytestmark = pytest.mark.gpu



def with_tile(torch, iflow, fmt, tile, packed, rows, cols, x, batch, y):
    """The product through tile number `tile`, whichever the launcher would take."""
    p = C.c_void_p
    st = iflow.lib().iflow_internal_qgemm_with_tile(fmt, tile, p(packed.data_ptr()), C.c_int64(rows), C.c_int64(cols), p(x.data_ptr()), C.c_int64(batch),
                                                    p(y.data_ptr()), p(torch.cuda.current_stream().cuda_stream))
    assert st == iflow.OK, st


def tile_shapes(iflow, fmt):
    """Per tile: rows, vectors, wavefront groups that share K, chunks fetched at once, such runs in LDS, longest row."""
    shapes, v = [], (C.c_int64 * 6)()
    while iflow.lib().iflow_internal_qgemm_tile_shape(fmt, len(shapes), v):
        shapes.append(tuple(v))
    return shapes


# rows, 64-column chunks, vectors, which the launcher's prices spread over most tiles (the tests below hold every tile to its reference whatever they say)
SHAPES = [
    (16625, 5, 673), (8200, 31, 1025), (16412, 3, 686), (16441, 5, 481), (16473, 3, 582), (16470, 7, 129), (16537, 5, 389),
    (16385, 1, 400), (16859, 5, 194), (12290, 3, 511), (16593, 5, 97), (16629, 5, 97), (16566, 65, 196), (11010, 65, 500), (16389, 13, 99),
    (16413, 5, 17), (16429, 3, 65), (8235, 5, 66), (4100, 33, 513), (8270, 9, 131), (3001, 17, 500), (16474, 13, 17), (8315, 13, 65),
    (8198, 9, 33), (4099, 65, 97), (8650, 9, 17), (8367, 5, 31), (4179, 5, 33), (4099, 65, 64), (97, 3, 127), (64, 2, 129), (70, 200, 33),
    (1, 8, 32), (1031, 65, 200), (33, 18, 19),
]


@pytest.mark.parametrize("name", NAMES)
def test_every_tile(gpu, name):
    torch, iflow = gpu
    fmt = iflow.FORMATS[name]
    g = torch.Generator(device="cuda")
    for i, (rows, chunks, batch) in enumerate(SHAPES):
        say(f"[case] tile {name} rows={rows} cols={64 * chunks} batch={batch}")
        cols = 64 * chunks
        g.manual_seed(synth.BASE_SEED + 4000 + i)
        w = torch.empty((rows, cols), device="cuda").normal_(0.0, 0.02, generator=g)
        x = torch.empty((batch, cols), device="cuda").normal_(generator=g).half()
        n = iflow.packed_bytes(fmt, rows, cols)
        packed = torch.empty((n,), dtype=torch.uint8, device="cuda")
        iflow.quantize(fmt, w, rows, cols, packed, n)
        w16 = torch.empty((rows, cols), dtype=torch.float16, device="cuda")
        iflow.dequant(fmt, packed, rows, cols, w16)
        y = torch.full((batch * rows + 64,), float("nan"), dtype=torch.float16, device="cuda")
        iflow.qgemm(fmt, packed, rows, cols, x, batch, y)
        torch.cuda.synchronize()
        assert torch.isnan(y[batch * rows:]).all(), "wrote past the last output"
        got = y[:batch * rows].view(batch, rows).double()
        ref = x.double() @ w16.double().T.contiguous()
        err = ((got - ref).abs() / torch.maximum(ref.abs(), ref.square().mean(1, keepdim=True).sqrt())).max().item()
        assert err <= 6e-4, f"{rows} x {cols}, {batch} vectors: {err:.2e}"      # (a NaN, an output never written, fails too)


@pytest.mark.parametrize("name", NAMES)
def test_each_tile_by_number(gpu, name):
    """Each tile by its number: two and a half times its rows and a bit more than its vectors, K of one chunk, of enough runs that every buffer of packed weights is
    filled again and used twice more by every group of wavefronts, of a length that leaves some groups a run less and the last one short, and (the 3.5-bit
    format's strips of 64 chunks) of two strips and a short third one."""
    torch, iflow = gpu
    fmt = iflow.FORMATS[name]
    g = torch.Generator(device="cuda")
    for tile, (trows, vectors, groups, run, buffers, _) in enumerate(tile_shapes(iflow, fmt)):
        full = (buffers + 2) * groups * run
        for i, (rows, chunks, batch) in enumerate([(2 * trows + trows // 2 + 5, full + 1, vectors + 7), (trows + 8, full + (groups // 2) * run + run - 1, vectors),
                                                   (trows // 2 + 1, 131, 2 * vectors - 1), (3, 1, 1)]):
            say(f"[case] tile {tile} ({trows} x {vectors}, {groups} along K) {name} rows={rows} cols={64 * chunks} batch={batch}")
            cols = 64 * chunks
            g.manual_seed(synth.BASE_SEED + 4700 + 8 * tile + i)
            w = torch.empty((rows, cols), device="cuda").normal_(0.0, 0.02, generator=g)
            x = torch.empty((batch, cols), device="cuda").normal_(generator=g).half()
            n = iflow.packed_bytes(fmt, rows, cols)
            packed = torch.empty((n,), dtype=torch.uint8, device="cuda")
            iflow.quantize(fmt, w, rows, cols, packed, n)
            w16 = torch.empty((rows, cols), dtype=torch.float16, device="cuda")
            iflow.dequant(fmt, packed, rows, cols, w16)
            y = torch.full((batch * rows + 64,), float("nan"), dtype=torch.float16, device="cuda")
            with_tile(torch, iflow, fmt, tile, packed, rows, cols, x, batch, y)
            torch.cuda.synchronize()
            assert torch.isnan(y[batch * rows:]).all(), "wrote past the last output"
            got = y[:batch * rows].view(batch, rows).double()
            ref = x.double() @ w16.double().T.contiguous()
            # (the rms of all outputs: a vector's own, over three rows, can be as small as its smallest value)
            err = ((got - ref).abs() / torch.maximum(ref.abs(), ref.square().mean().sqrt())).max().item()
            assert err <= 6e-4, f"tile {tile}: {rows} x {cols}, {batch} vectors: {err:.2e}"


# row tiles x tiles of vectors: fewer than the dies, one more and one less than a multiple of them and a multiple (rows outermost for two to five tiles of vectors), one band of vectors, a
# whole second one and a short one
PLACES = [(1, 1), (3, 2), (7, 1), (1, 9), (5, 3), (9, 4), (11, 5), (8, 8), (3, 11), (17, 13), (8, 1), (8, 2), (16, 5), (8, 6)]


@pytest.mark.parametrize("ntr,ntb", PLACES)
def test_every_place(gpu, ntr, ntb):
    """Every tile of the product is some workgroup's, whatever the counts: each output is written, by the smallest tile, with the last row tile and the last vectors ragged.
    Bound: as above, one fp16 rounding and sums of 64 products."""
    torch, iflow = gpu
    fmt = iflow.FORMATS["Q4_B64"]
    shapes = tile_shapes(iflow, fmt)
    tile = min(range(len(shapes)), key=lambda i: shapes[i][0] * shapes[i][1])
    rows, batch, cols = (ntr - 1) * shapes[tile][0] + 5, (ntb - 1) * shapes[tile][1] + 3, 64
    say(f"[case] places {ntr} x {ntb}: rows={rows} batch={batch}")
    g = torch.Generator(device="cuda")
    g.manual_seed(synth.BASE_SEED + 4900 + 16 * ntr + ntb)
    w = torch.empty((rows, cols), device="cuda").normal_(0.0, 0.02, generator=g)
    x = torch.empty((batch, cols), device="cuda").normal_(generator=g).half()
    n = iflow.packed_bytes(fmt, rows, cols)
    packed = torch.empty((n,), dtype=torch.uint8, device="cuda")
    iflow.quantize(fmt, w, rows, cols, packed, n)
    w16 = torch.empty((rows, cols), dtype=torch.float16, device="cuda")
    iflow.dequant(fmt, packed, rows, cols, w16)
    y = torch.full((batch, rows), float("nan"), dtype=torch.float16, device="cuda")
    with_tile(torch, iflow, fmt, tile, packed, rows, cols, x, batch, y)
    torch.cuda.synchronize()
    ref = x.double() @ w16.double().T.contiguous()
    err = ((y.double() - ref).abs() / torch.maximum(ref.abs(), ref.square().mean().sqrt())).max().item()
    assert err <= 6e-4, f"{rows} x {cols}, {batch} vectors: {err:.2e}"


@pytest.mark.parametrize("name", NAMES)
def test_infinity_in_the_last_columns(gpu, name):
    """An infinite activation in the last 64 columns makes its vector's outputs infinite (NaN only against a weight of zero), whatever kernel
    the number of vectors selects, and however the chunks come out over the wavefronts that share K; the other vectors stay as they are."""
    torch, iflow = gpu
    fmt = iflow.FORMATS[name]
    g = torch.Generator(device="cuda")
    for i, (rows, chunks, batch) in enumerate([(70, 65, 16), (70, 65, 17), (70, 1, 17), (1031, 9, 33), (4099, 13, 65), (16566, 65, 196), (16441, 5, 481),
                                               (16470, 7, 129), (8270, 9, 131)]):
        cols = 64 * chunks
        say(f"[case] infinity {name} rows={rows} cols={cols} batch={batch}")
        g.manual_seed(synth.BASE_SEED + 4500 + i)
        w = torch.empty((rows, cols), device="cuda").normal_(0.0, 0.02, generator=g)
        x = torch.empty((batch, cols), device="cuda").normal_(generator=g).half()
        x[batch // 2, cols - 3] = float("inf")
        x[batch - 1, cols - 64] = float("-inf")
        n = iflow.packed_bytes(fmt, rows, cols)
        packed = torch.empty((n,), dtype=torch.uint8, device="cuda")
        iflow.quantize(fmt, w, rows, cols, packed, n)
        w16 = torch.empty((rows, cols), dtype=torch.float16, device="cuda")
        iflow.dequant(fmt, packed, rows, cols, w16)
        y = torch.full((batch, rows), float("nan"), dtype=torch.float16, device="cuda")
        iflow.qgemm(fmt, packed, rows, cols, x, batch, y)
        torch.cuda.synchronize()
        ref = x.double() @ w16.double().T.contiguous()
        finite = torch.isfinite(ref)
        got = y.double()
        same = torch.where(finite, torch.isfinite(got), (got == ref) | (torch.isnan(got) & torch.isnan(ref)))
        assert same.all(), f"{rows} x {cols}, {batch} vectors: {int((~same).sum())} outputs of {int((~finite).sum())} infinite ones differ"
        rms = torch.where(finite, ref, torch.zeros_like(ref)).square().mean(1, keepdim=True).sqrt()
        err = torch.where(finite, (got - ref).abs() / torch.maximum(ref.abs(), rms), torch.zeros_like(ref)).max().item()
        assert err <= 6e-4, f"{rows} x {cols}, {batch} vectors: {err:.2e}"


@pytest.mark.parametrize("name", ["Q3H_B64", "Q8_B64", "Q5_B64", "Q2_B32"])
def test_long_rows(gpu, name):
    """Rows around the lengths where 32-bit offsets end: every tile that differs in its limit at exactly that limit with all its vectors (the largest
    offsets there are), the launcher's choice beyond the shorter limits, and passes of sixteen beyond the longest.  fp32 sums in steps of
    sixteen columns: 2^-24 sqrt(2^26 / 16 / 2) = 9e-5 of the rms on top of the output's rounding, bound 1e-3."""
    torch, iflow = gpu
    fmt = iflow.FORMATS[name]
    g = torch.Generator(device="cuda")
    g.manual_seed(synth.BASE_SEED + 4600)
    shapes = tile_shapes(iflow, fmt)
    limits = {}
    for tile, (rows, vectors, _, _, _, max_cols) in enumerate(shapes):
        limits.setdefault((vectors, max_cols), (tile, rows))
    cases = [(min(rows, 33), max_cols // 64 * 64, vectors, tile) for (vectors, max_cols), (tile, rows) in sorted(limits.items()) if max_cols <= 1 << 24]
    cases += [(3, 1 << 22, 17, None), (3, (1 << 22) + 64, 17, None), (2, (1 << 24) + 64, 40, None), (1, 1 << 26, 33, None), (1, (1 << 26) + 64, 17, None)]
    for rows, cols, batch, tile in cases:
        say(f"[case] long rows {name} rows={rows} cols={cols} batch={batch} tile={tile}")
        w = torch.empty((rows, cols), device="cuda").normal_(0.0, 0.02, generator=g)
        x = torch.empty((batch, cols), dtype=torch.float16, device="cuda").normal_(generator=g)
        n = iflow.packed_bytes(fmt, rows, cols)
        packed = torch.empty((n,), dtype=torch.uint8, device="cuda")
        iflow.quantize(fmt, w, rows, cols, packed, n)
        del w
        w16 = torch.empty((rows, cols), dtype=torch.float16, device="cuda")
        iflow.dequant(fmt, packed, rows, cols, w16)
        y = torch.full((batch, rows), float("nan"), dtype=torch.float16, device="cuda")
        if tile is None:
            iflow.qgemm(fmt, packed, rows, cols, x, batch, y)
        else:
            with_tile(torch, iflow, fmt, tile, packed, rows, cols, x, batch, y)
        ref = torch.zeros((batch, rows), dtype=torch.float64, device="cuda")
        whole = cols // 4096 * 4096
        for k in range(0, whole, 1 << 20):                     # (a batch of short products: a plain one runs this long a sum in a workgroup or two)
            xs, ws = (t[:, k:min(k + (1 << 20), whole)].double().view(t.shape[0], -1, 4096).transpose(0, 1).contiguous() for t in (x, w16))
            ref += torch.bmm(xs, ws.transpose(1, 2).contiguous()).sum(0)
        if whole < cols:
            ref += x[:, whole:].double() @ w16[:, whole:].double().T.contiguous()
        # (the rms of all outputs: with a row or two a vector's own can be as small as its smallest value, and the sums' error does not shrink with it)
        err = ((y.double() - ref).abs() / torch.maximum(ref.abs(), ref.square().mean().sqrt())).max().item()
        assert err <= 1e-3, f"{rows} x {cols}, {batch} vectors, tile {tile}: {err:.2e}"
        del x, w16, packed, y, ref
