"""fp32 -> bf16 where a kernel stores an operand: round to nearest even, as torch's conversion on the CPU.

Seen through the appended V rows of one layer.  Every token's embedding is 1024 in one column and zero
elsewhere, so its row mean square is 2^12, its normalised operand exactly 16 times that column's gain, and
its V row that times one column of Wv: a product of two 8-bit significands, exact in fp32, with every
kind of remainder -- ties to even and to odd, carries into the exponent, and overflow past the largest
bf16."""
import numpy as np
import pytest
import torch

from paper_2608_08721_amd import runtime
from synth import configs, gen
from tests.lsv_testing import GpuModel, note

pytestmark = pytest.mark.gpu


def _bf16(rng, shape, lo, hi):
    """Random bf16 bit patterns of either sign with exponents 2^lo .. 2^(hi - 1)."""
    e = rng.integers(lo, hi, shape) + 127
    return (rng.integers(0, 2, shape) << 15 | e << 7 | rng.integers(0, 128, shape)).astype(np.uint16)


@pytest.mark.parametrize("rows", [48, 256])  # the 64-row body's epilogue, the batched body's reduce
def test_stored_operands_round_to_nearest_even(rows):
    shape = configs.TINY_BF16.with_layers(1)
    rng = np.random.default_rng(66)
    d = shape.d_model
    w = gen.model_weights(shape, 66)
    w["embed"][:] = 0
    for t in range(d):
        w["embed"][t, t] = 0x4480  # 1024
    layer = w["layers"][0]
    layer["attn_norm"] = _bf16(rng, d, -60, 100)
    layer["wv"] = _bf16(rng, layer["wv"].shape, -40, 28)
    layer["wv"][5, :] = 0x7fc0  # NaN stays NaN
    gm = GpuModel(shape, w, 1, runtime.kv_capacity(d), max_rows=rows)
    as_float = lambda bits: torch.from_numpy(gen.bf16_to_f32(bits))
    for t0 in range(0, d, rows):
        n = min(rows, d - t0)
        gm.verify([t0], np.arange(t0, t0 + n, dtype=np.int32), [0, n], max_rows=rows)
    v = gm.kv.read(0, 0, 0, d)[1].cpu()  # [kv head][position][head_dim]
    got = v.transpose(0, 1).reshape(d, -1)
    exact = (16.0 * as_float(layer["attn_norm"]))[:, None] * as_float(layer["wv"]).T
    want = exact.to(torch.bfloat16)
    low = exact.view(torch.int32) & 0xffff
    ties, over = int((low == 0x8000).sum()), int((torch.isinf(want) & ~torch.isinf(exact)).sum())
    note(f"  {rows} rows: {got.numel()} values, {ties} ties, {over} finite sums past the largest bf16")
    assert ties > 100 and over > 0
    nan = torch.isnan(want)
    assert nan[:, 5].all() and torch.equal(torch.isnan(got), nan)
    assert torch.equal(got.view(torch.int16)[~nan], want.view(torch.int16)[~nan])
