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
