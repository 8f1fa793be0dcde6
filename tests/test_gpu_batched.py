"""GPU verify at the batched shapes: more than 64 block rows, which take the GEMMs' batched body
and the attention's passes and groups of query tiles.

* small bf16 model (d 1024, 8/2 x 128 heads), 8 sequences x 33 rows = 264 rows over
  ragged contexts;
* Llama-3-8B width with 1 of its layers, 8 sequences x 33 rows, contexts drawn from
  [1024, 8192] (the batched gamma = 32 workload);
* Qwen2.5-32B width with 1 layer, 4 x 17 rows, context 4096, then speculative rejection
  sampling at T = 1 on the GPU's own logits, bit-exact against the oracle rule;
* Llama-3-70B width with 1 layer, 4 x 33 rows, context 8192, greedy and T = 0.7 sampling.

Logits bar: each row within 2e-2 of its largest |logit| (bf16 operands, fp32 accumulation);
greedy decisions equal wherever the oracle's top-2 margin clears twice the error."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import accept as OA
from paper_2608_08721_amd import lsv, runtime
from synth import configs, gen
from tests.lsv_testing import GpuModel, i32, note
from tests.test_gpu_accept import gpu_accept, unsettled
from tests.test_gpu_forward import _bf16_case

pytestmark = pytest.mark.gpu


def _sampling_matches(g_logits, off, toks, temperature, seed):
    """GPU sampling acceptance on the GPU's logits vs the oracle rule on the same logits."""
    B, M, V = len(off) - 1, int(off[-1]), g_logits.shape[1]
    q = gen.draft_probs(seed, M - B, V)
    logits = g_logits.astype(np.float32)
    width = int(np.diff(off).max())
    acc, out, st, _ = gpu_accept(lsv.LSV_ACC_SAMPLE, logits, off, toks, width, q, temperature, seed, 77)
    want = OA.accept_sample(logits, off, toks, q, temperature, seed, 77, out_width=width)
    assert np.array_equal(st, want["status"])
    settled = 0
    for b in range(B):
        if unsettled(want["diag"][b]):
            continue
        settled += 1
        assert acc[b] == want["accept_len"][b], b
        assert np.array_equal(out[b], want["out_tokens"][b]), b
    note(f"    sampling T={temperature}: {settled}/{B} sequences bit-exact (rest within rounding of a threshold)")
    assert settled >= B - 1


def test_small_bf16_264_rows():
    rng = np.random.default_rng(21)
    contexts = [int(c) for c in rng.integers(1, 300, size=8)]
    _bf16_case(configs.SMALL_BF16, 21, contexts, [33] * 8)


def test_llama8b_width_batched_264_rows():
    shape = configs.LLAMA3_8B.with_layers(1)
    wl = configs.WORKLOADS["llama3-8b-b8-ragged"]
    contexts = [int(c) for c in gen.contexts(wl)]
    note(f"llama3-8b width, 1 layer, contexts {contexts}")
    _bf16_case(shape, 3, contexts, [33] * 8)


def test_qwen32b_width_sampling():
    shape = configs.QWEN25_32B.with_layers(1)
    note("qwen2.5-32b width, 1 layer, 4 x 17 rows, context 4096")
    gm, g_logits, o_logits, toks, off = _bf16_case(shape, 4, [4096] * 4, [17] * 4)
    _sampling_matches(g_logits, off, toks, 1.0, 404)


def test_llama70b_width_greedy_and_sampling():
    shape = configs.LLAMA3_70B.with_layers(1)
    note("llama3-70b width, 1 layer, 4 x 33 rows, context 8192")
    gm, g_logits, o_logits, toks, off = _bf16_case(shape, 5, [8192] * 4, [33] * 4)
    _sampling_matches(g_logits, off, toks, 0.7, 505)


def test_short_blocks_under_a_batched_bound():
    """Blocks of at most 32 rows under a bound above 64 (the selected lengths of a batch whose
    worst case is large): the one GEMM launch runs the 64-row bodies on them, and the split-K reduces,
    launched too, return at once; Llama-3-70B width with 28 rows under a 132-row bound, the small model
    with 20 rows under 272."""
    _bf16_case(configs.LLAMA3_70B.with_layers(1), 24, [8192, 8100, 5000, 7000], [8, 8, 6, 6], bound=132)
    _bf16_case(configs.SMALL_BF16, 25, [300, 40, 129], [9, 5, 6], bound=272)


@pytest.mark.parametrize("rows", [65, 128, 129, 257, 320, 321, 512])
def test_batched_body_row_counts(rows):
    """Row counts around the batched body's tilings (two to five activation tiles per wave: few column
    tiles take two chunks above 320 rows) on the tiny model, whose SwiGLU width of 688 ends in a k-block
    of six fragments."""
    _bf16_case(configs.TINY_BF16, 26, [40, 7], [rows - 20, 20])


@pytest.mark.parametrize("rows", [336, 384, 385, 448, 449, 512])
@pytest.mark.parametrize("d_model", [320, 576])
def test_batched_body_many_activation_tiles(rows, d_model):
    """Six to eight activation tiles per wave: gate/up and the LM head of 65 column tiles keep more than
    320 rows in one chunk.  d_model 320 gives one k range of ten steps, 576 two of nine, which is an odd
    step before the loop; both end in a k-block of two fragments."""
    shape = dataclasses.replace(configs.TINY_BF16, d_model=d_model, d_ff=4112, vocab=8320, n_layers=1,
                                name=f"tiny-bf16-65-tiles-{d_model}")
    _bf16_case(shape, 31, [40, 7], [rows - 20, 20])


def test_batched_body_rows_below_the_bound():
    """A two-chunk plan (bound 512) with rows for one chunk and a part of the other, and for one only."""
    _bf16_case(configs.TINY_BF16, 27, [40, 7], [80, 20], bound=512)
    _bf16_case(configs.SMALL_BF16, 28, [40], [70], bound=512)


@pytest.mark.parametrize("contexts,rows", [([2500, 90], [4, 440]), ([60, 3000, 700], [100, 3, 300]),
                                           ([1500], [65]), ([40, 40, 40, 40], [128] * 4)])
def test_query_groups_beside_short_sequences(contexts, rows):
    """A bound of 512 rows leaves room for query groups; each sequence takes them, or the context
    splits of a short block, by its own rows: a decoding sequence beside a prefill chunk, one of few
    query tiles between two of many, a block of 65 rows, and four alike."""
    shape = dataclasses.replace(configs.SMALL_BF16, n_q_heads=32, n_kv_heads=8, n_layers=1, name="small-bf16-32-8")
    _bf16_case(shape, 30, contexts, rows, bound=lsv.LSV_MAX_ROWS)


def test_query_groups_lose_no_precision():
    """512 rows of one sequence behind 2,100 positions as one block, whose query tiles the attention
    takes in groups over one or two long splits, and as eight blocks of 64 rows over fourteen short
    ones.  The probabilities are rounded to bf16 either way, so the block may stand no further off
    the oracle's float64 than the short blocks do.  Row errors scatter by some 4%, so the norm over
    512 rows by 0.2%, and the two errors share most of their roundings: a bar of 0.5% (equal splits
    read 1.0001; a maximum kept over a group's whole split reads 1.0104)."""
    shape = dataclasses.replace(configs.SMALL_BF16, n_q_heads=32, n_kv_heads=8, n_layers=1, name="small-bf16-32-8")
    seed, C, R = 29, 2100, lsv.LSV_MAX_ROWS
    gm, whole, want, toks, off = _bf16_case(shape, seed, [C], [R], bound=R)
    short = []
    for pos in range(0, R, 64):
        lg, st = gm.verify([C + pos], toks[pos:pos + 64], [0, 64], max_rows=64)
        assert st[0] == 0
        short.append(lg)
    scale = np.linalg.norm(want)
    e_whole, e_short = np.linalg.norm(whole - want) / scale, np.linalg.norm(np.concatenate(short) - want) / scale
    note(f"  512 rows off float64: {e_whole:.3e} as one block, {e_short:.3e} as blocks of 64 ({e_whole / e_short:.4f})")
    assert e_whole <= 1.005 * e_short


def test_one_capture_serves_short_blocks_and_query_groups():
    """A verify call captured once under a bound of 512 rows finds its plan from the device rows of each
    replay: one of query groups, one of context splits, mixed batches, and again."""
    shape = dataclasses.replace(configs.SMALL_BF16, n_q_heads=32, n_kv_heads=8, n_layers=1, name="small-bf16-32-8")
    seed, C, B, R = 32, [700, 300], 2, lsv.LSV_MAX_ROWS
    cap = runtime.kv_capacity(max(C) + R)
    gm = GpuModel(shape, gen.model_weights(shape, seed), B, cap, max_rows=R)
    for b in range(B):
        k, v = gen.synthetic_kv(shape, seed + b, 0, 1, C[b])
        gm.kv.write(0, b, 0, runtime.to_device(k[0]), runtime.to_device(v[0]))
    toks, seq_len, off = i32(gen.randint(seed, 900, R, shape.vocab)), i32(C), i32([0, 0, 0])

    def call():
        lsv.lsv_verify_block(gm.cfg, gm.dm.buf, gm.kv.buf, cap, B, seq_len, toks, off, R, cap, gm.logits, gm.status,
                             gm.ws.buf, gm.ws.nbytes)

    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for rows in ([256, 256], [9, 3], [500, 4], [3, 200], [256, 256], [9, 3]):
        off.copy_(i32([0, rows[0], sum(rows)]))
        call()
        torch.cuda.synchronize()
        want = gm.logits[:sum(rows)].clone()
        gm.logits.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(gm.logits[:sum(rows)], want) and bool(torch.isfinite(want).all()), rows
        assert not gm.status.any()
