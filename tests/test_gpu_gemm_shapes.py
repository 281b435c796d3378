"""The first stage's GEMM over every tile shape that its dispatch can take,
through sm_merge_token_table (table = GELU(Linear(emb)) row by row), against
the same product in float64."""
import pytest
import torch

from gpu_util import TOL, dev, say
from paper_2609_27233_amd import lib as sm
from paper_2609_27233_amd import workload as wl

pytestmark = pytest.mark.gpu

# at d = 256 (K shorter than the LDS rings) the row counts run through the
# tiles 32x32, 32x64, 64x64, 96x64, 128x64, 160x64, 192x64, 256x128, 256x128
# and 32x32 for the rest, 256x256; at 1024 256x256 with the rest cut off;
# 2048 and 4096 walk longer Ks
BF16 = [(256, m) for m in (1, 33, 1041, 2100, 4200, 6200, 8290, 10300, 25100, 33060, 41100)] + [
    (1024, 16560), (1024, 17240), (768, 300), (2048, 131), (2048, 2055), (4096, 610)]
F32 = [(256, m) for m in (1, 33, 1041, 2100, 4200, 6200, 8290, 10300)] + [(1024, 1500), (768, 77)]


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


@pytest.mark.parametrize("d,rows", BF16)
def test_gemm_bf16(d, rows):
    _check(torch.bfloat16, d, rows, 0)


@pytest.mark.parametrize("d,rows", F32)
def test_gemm_f32(d, rows):
    _check(torch.float32, d, rows, 0)


@pytest.mark.parametrize("dtype,d,rows", [(torch.bfloat16, 256, 300), (torch.float32, 256, 300)] + [
    (torch.bfloat16, d, m) for d, m in ((256, 1), (512, 17), (1024, 64), (3584, 48), (1024, 65))])
def test_gemm_operands_off_16_bytes(dtype, d, rows):
    """One element past a 16-byte boundary: the kernels with plain loads, for
    up to 64 rows in bf16 the one of 16 columns a workgroup (K by four waves,
    8, 4 or 2 steps at a time)."""
    _check(dtype, d, rows, 1)
