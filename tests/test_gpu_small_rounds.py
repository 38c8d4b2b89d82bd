"""2 to 16 vectors with so many rows that a workgroup sums its partial tiles more than once: one round per workgroup, exactly four (one sum), five and
nine (two and three sums), rows in one strip of 4096 columns and in two, eight vectors and more (the second half of the activations is only
read then), with and without the modules around the product.

Reference: plain fp64 product (torch) with iflow_dequant's fp16 weights, the normalization and residual in fp64; the bound is the one of the
products elsewhere in these tests (2e-3 of max(|y|, rms): the normalized input is rounded to fp16, 2^-11 per weighted term, and the output)."""
import pytest

from paper_2401_08294_amd import synth
from test_gpu_parity import NAMES, TOL, gpu, say  # noqa: F401

pytestmark = pytest.mark.gpu
EPS = 1e-5


@pytest.mark.parametrize("name", NAMES)
def test_rounds(gpu, name):
    torch, iflow = gpu
    fmt = iflow.FORMATS[name]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g = torch.Generator(device="cuda")
    for i, (rounds, cols, batch, op) in enumerate([(1, 4096 + 64, 5, "rms"), (4, 64, 16, "plain"), (4, 4096 + 192, 8, "rms"), (5, 128, 9, "rms"),
                                                   (5, 4096 + 64, 16, "silu"), (9, 64, 7, "rms"), (9, 4096 + 64, 11, "gemm")]):
        rows = 16 * cus * (rounds - 1) + 16 * 5 + 3            # some workgroups have one round less
        say(f"[case] small batch {name} rows={rows} cols={cols} batch={batch} {op}")
        g.manual_seed(synth.BASE_SEED + 6000 + i)
        w = torch.empty((rows, cols), device="cuda").normal_(0.0, 0.02, generator=g)
        half = lambda *s: torch.empty(s, device="cuda").normal_(generator=g).half()
        x, res = half(batch, cols), half(batch, rows)
        n = iflow.packed_bytes(fmt, rows, cols)
        packed = torch.empty((n,), dtype=torch.uint8, device="cuda")
        iflow.quantize(fmt, w, rows, cols, packed, n)
        w16 = torch.empty((rows, cols), dtype=torch.float16, device="cuda")
        iflow.dequant(fmt, packed, rows, cols, w16)
        y = torch.full((batch, rows), float("nan"), dtype=torch.float16, device="cuda")
        v = x.double()
        if op == "gemm":
            iflow.qgemm(fmt, packed, rows, cols, x, batch, y)
            res = torch.zeros_like(res)
        elif op == "plain":
            iflow.qgemm_fused(fmt, packed, rows, cols, x, batch, y, residual=res)
        elif op == "rms":
            aux = half(cols)
            iflow.qgemm_fused(fmt, packed, rows, cols, x, batch, y, iflow.X_RMS_GAIN, aux, EPS, res)
            v = v * aux.double() / torch.sqrt((v * v).mean(1, keepdim=True) + EPS)
        else:
            aux = half(batch, cols)
            iflow.qgemm_fused(fmt, packed, rows, cols, x, batch, y, iflow.X_SILU_MUL, aux, 0.0, res)
            v = v * torch.sigmoid(v) * aux.double()
        torch.cuda.synchronize()
        ref = v @ w16.double().T.contiguous() + res.double()
        err = ((y.double() - ref).abs() / torch.maximum(ref.abs(), ref.square().mean(1, keepdim=True).sqrt())).max().item()
        assert err <= TOL, f"{rounds} rounds x {cols}, {batch} vectors, {op}: {err:.2e}"


@pytest.mark.parametrize("name", ["Q8_B32", "Q8_B64"])
def test_long_and_short_rows_of_codes(gpu, name):
    """8-bit codes on both sides of 2048 columns, where the loads of a step change: a last row group of every remainder that a load of four rows can have, column groups that end inside
    a wavefront's four and leave whole wavefronts without any, a second strip.  Bound as above."""
    torch, iflow = gpu
    fmt = iflow.FORMATS[name]
    g = torch.Generator(device="cuda")
    for i, (rows, cols, batch) in enumerate([(16, 2048, 5), (1, 2112, 5), (3, 2176, 8), (17, 2240, 9), (20, 2304, 16), (37, 4032, 6), (46, 4096, 16), (31, 4160, 7), (4099, 6208, 11)]):
        say(f"[case] small batch codes {name} rows={rows} cols={cols} batch={batch}")
        g.manual_seed(synth.BASE_SEED + 6100 + i)
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
        assert err <= TOL, f"{rows} x {cols}, {batch} vectors: {err:.2e}"
