// How the bf16 attention divides its work: the context into splits, a sequence's query tiles into
// groups, and the split kernel's grid.  Plain integer rules, the same on the host (which sizes the
// buffers and the grid) and on the device (which applies them to the block's own row counts).
#pragma once
#if defined(__HIPCC__)
#define LSV_PLAN __host__ __device__ inline
#else
#define LSV_PLAN inline
#endif

namespace lsv {

constexpr int kAttnChunk = 64;  // keys per LDS chunk in the bf16 split-context kernel
// Split plan: about kAttnWgs split workgroups, and no split longer than kMaxChunksPerSplit
// chunks (a split walks its chunks in sequence).  Fewer splits mean fewer partials to merge
// -- one batch of merge loads for up to 16 -- against longer chunk walks; 128 measured best
// for one sequence of 2K context (11 splits of 3 chunks).  The length cap keeps the
// workgroups of a batch with long contexts from running too long -- but never beyond one
// workgroup per compute unit: a grid larger than the chip runs its last workgroups in a
// second round, which costs more than longer splits (Llama-3-70B, four sequences of 8K
// context: 9 splits, 288 workgroups, 49 us; 8 splits, 256 workgroups, 34 us).
constexpr int kAttnWgs = 128;
constexpr int kMaxChunksPerSplit = 16;
constexpr int kAttnUnits = 256;  // compute units of gfx950 (MI350X, MI355X)
// Query groups: for sequences of more than kGroupTiles query tiles in a block of more than kGroupRows
// rows.  Above the line, passes against groups, two layers at Llama-3-8B width: 97 rows (25 tiles) behind
// 500 / 2,000 / 8,000 positions 361 / 386 / 439 us against 339 / 347 / 383, 128 rows 382 / 410 / 470
// against 353 / 365 / 405; one layer at Llama-3-70B width, 4 x 49 rows behind 8,000: 640 against 618.
// Below it, one sequence would gain as well (96 rows: 349 / 367 / 413 against 333 / 342 / 371), four of
// 33 rows at Llama-3-70B width would lose behind 8,000 positions (534 against 541) and gain behind 500
// (468 against 449).
constexpr int kGroupRows = 64;
constexpr int kGroupTiles = 24;
constexpr int kPassTiles = 8;  // query tiles of one pass (a group): one for each of the eight waves
constexpr int kLongGroupSplit = 64;

struct AttnPlan {
  int n_splits, chunks_per_split;  // splits of the context bound: partial buffers hold n_splits
  int packed;                      // the split kernel runs on a packed grid of n_wgs workgroups
  int grouped;                     // the grid has room for query groups
  int n_wgs;
  int group;                       // query heads per kv head
};

// Query tiles (16 query vectors each) of a sequence's rows.
LSV_PLAN int query_tiles(int rows, int group) { return (rows * group + 15) / 16; }

// Chunks per split of a sequence in `groups` query groups: as many splits as its groups leave compute
// units for in one round (every sequence of the batch taken to be like it, so that its rows do not
// depend on the others'), at most n_splits.  Where those are longer than kLongGroupSplit chunks, up to
// four rounds of shorter ones are taken if a unit then walks a fifth fewer (Llama-3-70B, 264 rows
// behind 32,000 positions, one layer: 17 groups leave room for one split in one round, 1333 us; seven
// splits in four rounds, 1145).
LSV_PLAN int group_chunks(int n_chunks, int units, int groups, int n_splits) {
  const int wgs = units * groups;  // of one split
  int want = kAttnUnits / wgs;
  if (want < 1) want = 1;
  if (want > n_splits) want = n_splits;
  int chunks = (n_chunks + want - 1) / want;
  if (chunks <= kLongGroupSplit) return chunks;
  int walk = (wgs * want + kAttnUnits - 1) / kAttnUnits * chunks;  // chunks that a compute unit walks
  for (int rounds = 2; rounds <= 4; ++rounds) {
    const int w = rounds * kAttnUnits / wgs;
    if (w < 1 || w > n_splits) continue;
    const int c = (n_chunks + w - 1) / w;
    if (rounds * c * 5 < walk * 4) {
      walk = rounds * c;
      chunks = c;
    }
  }
  return chunks;
}

// Query groups of a sequence in the plan's own splits (of which the batch has `wgs`): one per pass, as far
// as the compute units have room.
LSV_PLAN int short_groups(int wgs, int passes) {
  const int room = kAttnUnits / wgs;
  return room < 1 ? 1 : (room < passes ? room : passes);
}

// Long contexts over many (sequence, kv head) pairs -- when one round's splits would walk more
// than twice the length cap -- take a whole number of rounds' worth of splits instead, on a
// packed grid: the splits that hold keys come first, so in a batch of ragged contexts the
// empty splits of the short sequences no longer hold compute units while a long sequence walks
// its splits (Llama-3-8B, batch 8, contexts of 1.7K-8.2K: 4 splits of 33 chunks become 12 of
// 11).  With every context at the bound, three rounds of a third of the length cost what one
// round costs.  These split boundaries follow from the batch and the context bound alone, so a row's
// result does not depend on its block, its batch, the other sequences' lengths or the row bound.
//
// A sequence of many query tiles (a prefill chunk, a draft tree: more than kGroupTiles of them in a
// block of more than 64 rows) gives every pass of the eight waves a workgroup of its own instead:
// query groups, not context splits, then fill the chip, so a row has one or two partials instead of
// up to sixteen and a pass skips the chunks behind its last row.  Llama-3-8B, 512 rows behind 1.5K
// positions: 16 splits walked by 128 workgroups in 16 passes each become 2 splits x 16 groups x 8
// kv heads.  The device row counts decide this, sequence by sequence (seq_plan): under a large row
// bound a short block keeps the splits above, and with them its parallelism and its bits (Llama-3-8B,
// 9 rows behind 8,000 positions, two layers under a bound of 264 rows: 294 us in the splits that the
// bound's groups would leave, 235 in these, 229 under a bound of 64).  As far as the compute units
// have room, its passes get workgroups of their own over the same splits, with the same bits (64 rows
// behind 8,000 positions under a bound of 264: 376 us in one workgroup per split, 347 in two; 431 in the
// bound's).  The row bound only decides whether the grid has room for groups.
inline AttnPlan plan_attention(int batch, int nkv, int group, int max_rows, int max_ctx) {
  const int n_chunks = (max_ctx + kAttnChunk - 1) / kAttnChunk;
  const int units = batch * nkv;
  int want = (kAttnWgs + units - 1) / units;
  const int by_length = (n_chunks + kMaxChunksPerSplit - 1) / kMaxChunksPerSplit;
  if (want < by_length) want = by_length;
  const int fit = kAttnUnits / units;  // splits per (sequence, kv head) in one round
  AttnPlan p;
  p.group = group;
  p.packed = fit >= 1 && by_length > 2 * fit;
  if (p.packed)
    want = (by_length + fit - 1) / fit * fit;
  else if (want > fit)
    want = fit;
  if (want > n_chunks) want = n_chunks;
  if (want < 1) want = 1;
  p.chunks_per_split = (n_chunks + want - 1) / want;
  p.n_splits = (n_chunks + p.chunks_per_split - 1) / p.chunks_per_split;
  p.n_wgs = p.n_splits * units;
  const int mean_tiles = query_tiles((max_rows + batch - 1) / batch, group);
  p.grouped = max_rows > kGroupRows && mean_tiles > kGroupTiles;
  if (p.grouped) {
    // a packed grid for any rows under the bound: every sequence's splits, and what groups add to
    // them -- gain(g) for a sequence of g groups, which has at least r(g) rows, so over all sequences
    // at most max_rows times the largest gain(g) / r(g)
    p.packed = 1;
    int extra = 0, most = 0;
    for (int g = 2; (g - 1) * kPassTiles < query_tiles(max_rows, group); ++g) {
      int gain = nkv * p.n_splits * (short_groups(units * p.n_splits, g) - 1);
      if (g * kPassTiles > kGroupTiles) {
        const int cps = group_chunks(n_chunks, units, g, p.n_splits);
        const int coarse = nkv * (g * ((n_chunks + cps - 1) / cps) - p.n_splits);
        if (coarse > gain) gain = coarse;
      }
      const int r = 16 * (g - 1) * kPassTiles / group + 1;  // (g - 1) * kPassTiles + 1 tiles or more
      if (gain > most) most = gain;
      if (max_rows * gain / r > extra) extra = max_rows * gain / r;
    }
    p.n_wgs += extra < batch * most ? extra : batch * most;
  }
  return p;
}

// Splits of `chunks` chunks that hold keys of a sequence of `rows` rows behind C cached positions; none
// for a sequence without rows.
LSV_PLAN int splits_with_keys(int chunks, int ctx_limit, int rows, int C) {
  if (rows <= 0) return 0;
  const int L = C + rows < ctx_limit ? C + rows : ctx_limit;
  const int nch = L > 0 ? (L + kAttnChunk - 1) / kAttnChunk : 0;
  return (nch + chunks - 1) / chunks;
}

// How a sequence of `rows` rows behind C cached positions, in a block of M rows, is divided: `splits`
// runs of `chunks` chunks that hold keys (at most AttnPlan::n_splits, since positions past ctx_limit
// do not count) and `groups` of query tiles; coarse: in splits of its own, not the plan's.
struct SeqPlan {
  int splits, chunks, groups, coarse;
};
LSV_PLAN SeqPlan seq_plan(const AttnPlan& p, int batch, int nkv, int ctx_limit, int rows, int C, int M) {
  SeqPlan q = {0, p.chunks_per_split, 1, 0};
  const int tiles = query_tiles(rows, p.group), passes = (tiles + kPassTiles - 1) / kPassTiles;
  if (p.grouped && M > kGroupRows && tiles > kGroupTiles) {
    q.coarse = 1;
    q.groups = passes;
    q.chunks = group_chunks((ctx_limit + kAttnChunk - 1) / kAttnChunk, batch * nkv, passes, p.n_splits);
  } else if (p.grouped && rows > 0) {
    q.groups = short_groups(batch * nkv * p.n_splits, passes);
  }
  q.splits = splits_with_keys(q.chunks, ctx_limit, rows, C);
  return q;
}

}  // namespace lsv
