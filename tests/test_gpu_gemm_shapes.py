"""The merge GEMMs over every tile shape that their dispatch can take, against
the same products in float64: contiguous rows and the first stage's output
through sm_merge_token_table (table = GELU(Linear(emb)) row by row), gathered
rows and fp32 output through sm_merge_spans."""
import pytest
import torch

from gpu_util import TOL, dev, say
from paper_2609_27233_amd import lib as sm
from paper_2609_27233_amd import workload as wl

pytestmark = pytest.mark.gpu

# width, rows, and the kernel that the plan takes ("a+b": cut in two by rows;
# "plain": 128x128, in fp32 the vector-ALU kernel), which test_gemm_plan.py
# checks.  At d = 256 K is shorter than the LDS rings, 2048 and more walk
# longer ones.
BF16 = [
    (256, 1, "skinny"), (256, 8, "skinny"), (256, 9, "32x32"), (256, 33, "32x32"), (256, 1041, "32x64"),
    (256, 2100, "64x64"), (256, 4200, "96x64"), (256, 6200, "128x64"), (256, 6300, "128x64"), (256, 8290, "160x64"),
    (256, 10300, "192x64"), (256, 10400, "192x64"), (256, 12001, "plain"), (256, 25100, "plain"),
    (256, 33060, "plain"), (256, 41100, "plain"), (256, 65800, "256x256+32x32"), (512, 16500, "256x128+32x32"),
    (768, 300, "32x32"), (1024, 3300, "256x128"), (1024, 8210, "256x128+32x32"), (1024, 10001, "256x256"),
    (1024, 16560, "256x256+32x32"), (1024, 17240, "256x256+64x64"), (2048, 131, "32x64"), (2048, 2055, "256x128"),
    (4096, 610, "160x64")]
F32 = [
    (256, 1, "32x32"), (256, 33, "32x32"), (256, 1041, "32x32"), (256, 2040, "32x64"), (256, 2100, "32x32"),
    (256, 3200, "64x64"), (256, 4200, "32x32"), (256, 5100, "96x64"), (256, 6200, "128x64"), (256, 6300, "128x64"),
    (256, 8290, "160x64"), (256, 10300, "192x64"), (256, 10400, "192x64"), (256, 29000, "plain"),
    (1024, 1500, "96x64"), (768, 77, "32x32")]
# spans of one row each: the same count of gathered rows in the first product
# and of spans in the second, whose output is fp32
SPANS = [
    (256, 5, "skinny"), (256, 40, "32x32"), (256, 1041, "32x64"), (256, 2100, "64x64"), (256, 4200, "96x64"),
    (256, 6300, "128x64"), (256, 8290, "160x64"), (256, 10400, "192x64"), (256, 12001, "plain"),
    (1024, 3300, "256x128"), (1024, 8210, "256x128+32x32"), (3584, 300, "96x64"), (4096, 609, "160x64"),
    (4096, 1700, "256x128"), (4096, 2100, "256x128+32x32"), (4096, 2440, "256x256"), (8192, 1777, "256x256")]


def _check(dtype, d, rows, shift):
    g = wl.generator(d + rows, "cuda")
    std = 0.05 if dtype == torch.bfloat16 else 0.3
    flat = lambda n, s: wl.randn((n + shift,), dtype, g, device="cuda", std=s)[shift:]    # noqa: E731
    emb = flat(rows * d, 1.0).view(rows, d)
    params = wl.make_merge_params(d, 4, dtype, g, device="cuda")
    params["W_kv"] = flat(d * d, std).view(d, d)
    table = torch.full((rows * d + shift,), float("nan"), dtype=dtype, device=dev())[shift:].view(rows, d)
    err = torch.zeros(1, dtype=torch.int32, device=dev())
    say("gemm", dtype, d, rows, "shift", shift)
    sm.merge_token_table(emb, params, 4, table, err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0
    ref = torch.nn.functional.gelu(emb.double() @ params["W_kv"].double().t().contiguous() + params["b_kv"].double())
    e = float(((table.double() - ref).norm(dim=1) / ref.norm(dim=1)).max())
    say("rel_l2_max", e)
    # bf16: the output's rounding (at most 2^-9 of each value) and fp32 sums
    assert e <= (2.0 ** -8 if dtype == torch.bfloat16 else TOL[dtype])


@pytest.mark.parametrize("d,rows,tile", BF16)
def test_gemm_bf16(d, rows, tile):
    _check(torch.bfloat16, d, rows, 0)


@pytest.mark.parametrize("d,rows,tile", F32)
def test_gemm_f32(d, rows, tile):
    _check(torch.float32, d, rows, 0)


@pytest.mark.parametrize("d,spans,tile", SPANS)
def test_gemm_gathered_rows_and_fp32_output(d, spans, tile):
    """Spans of one row: their pooled row is LN_kv of the first product's, so
    the whole call has a float64 reference in plain matrix products."""
    g = wl.generator(d + spans, "cuda")
    dt = torch.bfloat16
    emb = wl.randn((3000, d), dt, g, device="cuda")
    p = wl.make_merge_params(d, 4, dt, g, device="cuda", spread=True)
    for k in ("W_kv", "W_o"):
        p[k] = wl.randn((d, d), dt, g, device="cuda", std=d ** -0.5)
    rows = torch.randint(0, 3000, (spans,), dtype=torch.int32, device=dev(), generator=g)
    offs = torch.arange(spans + 1, dtype=torch.int32, device=dev())
    out = torch.full((spans, d), float("nan"), dtype=dt, device=dev())
    ws = torch.empty(sm.merge_workspace_bytes(spans, spans, d, dt), dtype=torch.uint8, device=dev())
    err = torch.zeros(1, dtype=torch.int32, device=dev())
    say("gathered rows, fp32 output", d, spans, tile)
    sm.merge_spans(emb, rows, offs, p, 4, out, ws, err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0
    w = {k: v.double() for k, v in p.items()}
    x = emb.double()[rows.long()]
    for n in ("kv", "o"):
        x = torch.nn.functional.gelu(x @ w["W_" + n].t().contiguous() + w["b_" + n])
        x = torch.nn.functional.layer_norm(x, (d,), w["g_" + n], w["beta_" + n], 1e-5)
    e = float(((out.double() - x).norm(dim=1) / x.norm(dim=1)).max())
    say("rel_l2_max", e)
    # three roundings to bf16 (first rows, pooled rows, output), each at most 2^-9 of a value
    assert e <= TOL[dt]


@pytest.mark.parametrize("dtype,d,rows", [(torch.bfloat16, 256, 300), (torch.float32, 256, 300)] + [
    (torch.bfloat16, d, m) for d, m in ((256, 1), (512, 17), (1024, 64), (3584, 48), (1024, 65))])
def test_gemm_operands_off_16_bytes(dtype, d, rows):
    """One element past a 16-byte boundary: the kernels with plain loads, for
    up to 64 rows in bf16 the one of 16 columns a workgroup (K by four waves,
    8, 4 or 2 steps at a time)."""
    _check(dtype, d, rows, 1)
