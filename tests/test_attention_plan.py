"""The attention's plan on the host: csrc/lsv_attn_plan.h is plain C++, built here with the host
compiler and compared over batches, head counts, row bounds and contexts.

* a block of up to 64 rows has the same splits under every row bound;
* the splits of a sequence cover its keys and never exceed the partial buffers';
* the packed grid has a workgroup for every (sequence, query group, kv head, split) of any rows
  under the bound."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "lsv_attn_plan.h"
using namespace lsv;
extern "C" void plan(int batch, int nkv, int group, int max_rows, int max_ctx, int* p) {
  const AttnPlan a = plan_attention(batch, nkv, group, max_rows, max_ctx);
  p[0] = a.n_splits, p[1] = a.chunks_per_split, p[2] = a.packed, p[3] = a.grouped, p[4] = a.n_wgs;
}
extern "C" void sequence(int batch, int nkv, int group, int max_rows, int max_ctx, int rows, int C, int M, int* q) {
  const SeqPlan s = seq_plan(plan_attention(batch, nkv, group, max_rows, max_ctx), batch, nkv, max_ctx,
                             rows, C, M);
  q[0] = s.splits, q[1] = s.chunks, q[2] = s.groups, q[3] = s.coarse;
}
"""
HEADS = [(8, 4), (8, 5), (8, 8), (2, 4), (2, 2), (1, 16), (8, 1)]
CONTEXTS = [64, 150, 700, 2112, 4096, 8192, 8256, 20000, 33000]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2608_08721_amd", "csrc"), str(d / "plan.cpp"), "-o", str(d / "plan.so")],
                   check=True)
    return ctypes.CDLL(str(d / "plan.so"))


def plan(lib, *args):
    p = (ctypes.c_int * 5)()
    lib.plan(*args, p)
    return list(p)


def sequence(lib, *args):
    q = (ctypes.c_int * 4)()
    lib.sequence(*args, q)
    return list(q)


def test_short_blocks_have_one_plan_under_every_row_bound(lib):
    for nkv, group in HEADS:
        for batch in (1, 2, 4, 13, 64):
            for ctx in CONTEXTS:
                base = plan(lib, batch, nkv, group, 64, ctx)
                for bound in (1, 16, 65, 68, 132, 196, 264, 512):
                    assert plan(lib, batch, nkv, group, bound, ctx)[:2] == base[:2], (nkv, group, batch, ctx, bound)
                    for rows in (1, 17, 64):
                        C = max(0, ctx - 70)
                        if rows <= bound:
                            splits, chunks, groups, coarse = sequence(lib, batch, nkv, group, bound, ctx, rows, C, 64)
                            assert splits == -(-min(-(-(C + rows) // 64), -(-ctx // 64)) // base[1])
                            assert chunks == base[1] and not coarse
                            assert groups == 1 or (groups <= -(-rows * group // 128) and
                                                   batch * nkv * base[0] * groups <= 256)


def test_grid_and_partials_hold_every_block_under_the_bound(lib):
    rng = random.Random(5)
    grouped = 0
    for nkv, group in HEADS:
        for batch in (1, 2, 3, 4, 8, 13):
            for ctx in CONTEXTS:
                for bound in (65, 97, 132, 200, 264, 320, 385, 512):
                    n_splits, _, packed, has_groups, n_wgs = plan(lib, batch, nkv, group, bound, ctx)
                    assert n_wgs >= n_splits * nkv * batch and (packed or not has_groups)
                    grouped += has_groups
                    first = 16 * 24 // group + 1  # rows of a sequence's 25th query tile
                    for kind in range(7):
                        rows = [0] * batch
                        left = bound
                        for b in range(batch):  # equal rows, all in one, as many groups as fit, or random ones
                            want = [bound // batch, bound, first, first + 128 // group, rng.randint(0, left),
                                    rng.choice((1, first)), rng.choice((first, first + 256 // group))][kind]
                            rows[b] = max(0, min(want, left, ctx))
                            left -= rows[b]
                        units = 0
                        for b in range(batch):
                            C = ctx - rows[b] if kind != 4 else rng.randint(0, ctx - rows[b])
                            s, chunks, groups, coarse = sequence(lib, batch, nkv, group, bound, ctx, rows[b], C, sum(rows))
                            assert s <= n_splits and (rows[b] == 0 or s * chunks * 64 >= C + rows[b])
                            assert rows[b] == 0 or (s - 1) * chunks * 64 < C + rows[b]
                            assert not coarse or groups * 8 * 16 >= rows[b] * group
                            units += s * groups * nkv
                        if packed:
                            assert units <= n_wgs, (nkv, group, batch, ctx, bound, rows)
    assert grouped > 500


def test_query_groups_walk_hardly_longer_than_passes_would(lib):
    """What a compute unit walks: chunks per split times the rounds of the grid (256 units), against the
    same rows in passes over the context splits.  A group's loads serve one pass, so some more chunks
    cost no more time, but few long splits of groups that leave most of the chip idle (17 groups of
    eight kv heads) would walk up to 1.8 times as far."""
    for nkv, group in HEADS:
        for batch in (1, 2, 3, 4, 8):
            for ctx in CONTEXTS:
                for bound in (65, 97, 132, 200, 264, 320, 385, 512):
                    rows = bound // batch
                    if rows > ctx:
                        continue
                    n_splits, per_split = plan(lib, batch, nkv, group, bound, ctx)[:2]
                    s, chunks, groups, coarse = sequence(lib, batch, nkv, group, bound, ctx, rows, ctx - rows, rows * batch)
                    if not coarse:
                        continue
                    passes = -(-rows * group // 128)
                    walk = -(-batch * nkv * groups * s // 256) * chunks
                    assert walk <= 1.4 * passes * per_split * -(-n_splits * nkv * batch // 256), (nkv, group, batch, ctx, bound)
