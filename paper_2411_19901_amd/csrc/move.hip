// lpaMove kernels for gfx950 (paper Algorithm 1, lpaMove; Algorithm 2,
// sketchAccumulate; Sections 4.1-4.5).
//
// Work decomposition (fixed once per graph by the degree binning):
//   * a "unit" is a run of at most S consecutive CSR entries of one vertex;
//     vertices of degree <= S are one unit, vertices above S ("hubs") are
//     split into ceil(deg / S) segment units;
//   * one lane owns one unit and feeds its entries into a register sketch in
//     CSR order, so no sketch merging is needed below S;
//   * a wavefront takes 64 units at a time (units are ordered by decreasing
//     length, so its lanes finish together) and stages T entries of each of
//     its 64 rows through LDS per step: the column, weight and gathered label
//     loads are issued row-contiguous by the whole wavefront, then every
//     lane consumes its own row from LDS;
//   * LPA_MODE_ASYNC: segment sketches are written out as partial sketches
//     and merged per hub by k_hub_merge (Section 4.3, partial sketches);
//     labels and flags are updated in place;
//   * LPA_MODE_DET: vertices above S are scanned by one wavefront each, which
//     stages 64 entries at a time and feeds them one by one into a sketch
//     held one slot per lane, so every sketch sees its row in CSR order;
//     labels are double-buffered (Jacobi).
//
// The CSR arrays are streamed once per iteration with non-temporal loads so
// that they do not evict the label lines that the gathers reuse.
//
// Sketch step (Section 4.1, with the decrement reading used throughout the
// library): a pair (c, w) adds w to the slot holding c; otherwise it fills a
// free slot (value 0); otherwise every slot loses d = min(w, smallest slot)
// and the residue w - d, if positive, fills a slot that became free.  Keys
// left behind in free slots may still match c: adding w to a free slot that
// holds c gives the same multiset of live (label, weight) pairs as placing
// (c, w) in any free slot, and keys stay unique because a key is only
// written when c is in no slot.  A weight of 0 leaves the sketch unchanged,
// which is how self-loops and padding are skipped without a branch.
#include "lpa_internal.h"
#include "wave.h"

#include <limits.h>
#include <math.h>

#include <type_traits>

namespace lpa {


// Row offset v of a graph as position type Pos: int reads the int32 offsets
// (graphs of fewer than 2^31 entries); long long reads either width.
template <class Pos>
__device__ __forceinline__ Pos row_at(const RowPtr &rp, int v) {
  if constexpr (sizeof(Pos) == 8)
    return rp[v];
  else
    return as_global(rp.p32)[v];
}

// First position and length of row v, both offsets in one load: in the 64-bit
// kernels the two widths lie in two branches, and a branch per offset put a wait
// between the two loads of int32 offsets (a ring of 6 10^8 vertices, unit weights,
// det, 5 iterations: 34.4 to 28.5 ms; in place 39.4 to 32.1).
template <class Pos>
__device__ __forceinline__ void row_of(const RowPtr &rp, int v, Pos &beg, int &len) {
  if constexpr (sizeof(Pos) == 8) {
    if (rp.p64) {
      const gptr<const int64_t> p = as_global(rp.p64) + v;
      const long long b = p[0], e = p[1];
      beg = b;
      len = (int)(e - b);
    } else {
      const gptr<const int32_t> p = as_global(rp.p32) + v;
      const int b = p[0], e = p[1];
      beg = (long long)(unsigned)b;
      len = e - b;
    }
  } else {
    beg = row_at<Pos>(rp, v);
    len = (int)(row_at<Pos>(rp, v + 1) - beg);
  }
}

// Element i of an array.  Narrow positions (Pos = int: graphs of fewer than 2^30
// entries and vertices) are byte offsets below 2^32, which loads add to a
// scalar base: one register per address, and none of the 64-bit sums.
template <class Pos, class T>
__device__ __forceinline__ gptr<T> element(gptr<T> base, Pos i) {
  if constexpr (sizeof(Pos) == 4) {
    using Byte = typename std::conditional<std::is_const<T>::value, const char, char>::type;
    return (gptr<T>)((gptr<Byte>)base + (unsigned)i * (unsigned)sizeof(T));
  } else {
    return base + i;
  }
}

// Index of the labels and flags of the vertex at degree-order position p
// (id v): its id, or its position when the graph keeps its state ranked.
// The same index is what `col` holds for the vertex, so a row entry equal to
// it is the vertex itself.
__device__ __forceinline__ int state_at(const MoveArgs &a, int p, int v) { return a.ranked ? p : v; }

// ---------------------------------------------------------------------------
// Register sketch: one lane owns all K slots.
// ---------------------------------------------------------------------------
template <int K>
struct LaneSketch {
  int key[K];
  float val[K];

  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int s = 0; s < K; ++s) {
      key[s] = -1;
      val[s] = 0.0f;
    }
  }

  __device__ __forceinline__ void add(int c, float w) {
    bool hit = false;
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const bool m = key[s] == c;
      hit = hit || m;
      val[s] = m ? val[s] + w : val[s];
    }
    if (!hit) {
      // With a free slot the minimum is 0: nothing is subtracted and the
      // whole weight is placed.  Otherwise the decrement step.
      float d = w;
#pragma unroll
      for (int s = 0; s < K; ++s) d = fminf(d, val[s]);
#pragma unroll
      for (int s = 0; s < K; ++s) val[s] = val[s] - d;
      const float r = w - d;
      bool placed = !(r > 0.0f);
#pragma unroll
      for (int s = 0; s < K; ++s) {
        const bool t = !placed && val[s] == 0.0f;
        key[s] = t ? c : key[s];
        val[s] = t ? r : val[s];
        placed = placed || t;
      }
    }
  }

  // Heaviest live slot, ties to the lowest label; keep when empty.
  __device__ __forceinline__ int max_key(int keep) const {
    int bk = keep;
    float bv = 0.0f;
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const bool better = val[s] > bv || (val[s] == bv && val[s] > 0.0f && key[s] < bk);
      bk = better ? key[s] : bk;
      bv = better ? val[s] : bv;
    }
    return bk;
  }

  // Feed another sketch's live slots (merge of partial sketches).
  __device__ __forceinline__ void merge_from(const int *pk, const float *pv) {
#pragma unroll
    for (int s = 0; s < K; ++s) add(pk[s], pv[s] > 0.0f ? pv[s] : 0.0f);
  }
};

// ---------------------------------------------------------------------------
// The weighted Boyer-Moore vote of Algorithm 3 (nu-BM-LPA): one candidate
// (key, val).  A pair (c, w) adds w when c is the candidate, subtracts w when
// the candidate's weight is larger, and otherwise becomes the candidate.
// The paper starts the candidate at (C[i], 0); starting at (-1, 0) gives the
// same result: from weight 0 the first positive pair becomes (c, w) either
// way, a zero-weight pair leaves a weight-0 candidate empty in effect, and
// a positive weight never returns to 0 (val > w implies val - w > 0 with
// denormals kept).  So an empty vote keeps the current label.
// Selected by K = 0 in the kernels below.
// ---------------------------------------------------------------------------
struct BmSketch {
  int key[1];
  float val[1];

  __device__ __forceinline__ void clear() {
    key[0] = -1;
    val[0] = 0.0f;
  }

  __device__ __forceinline__ void add(int c, float w) {
    const bool same = key[0] == c;
    const bool down = !same && val[0] > w;
    val[0] = same ? val[0] + w : (down ? val[0] - w : w);
    key[0] = (same || down) ? key[0] : c;
  }

  __device__ __forceinline__ int max_key(int keep) const { return val[0] > 0.0f ? key[0] : keep; }

  // Partial votes of one hub combine by the largest weight (ties to the
  // lowest label), as the paper's pair-max block reduction does.
  __device__ __forceinline__ void merge_from(const int *pk, const float *pv) {
    const bool better = pv[0] > val[0] || (pv[0] == val[0] && pv[0] > 0.0f && pk[0] < key[0]);
    key[0] = better ? pk[0] : key[0];
    val[0] = better ? pv[0] : val[0];
  }
};

template <int K>
struct SketchOf {
  using type = LaneSketch<K>;
};
template <>
struct SketchOf<0> {
  using type = BmSketch;
};
// Slots stored per partial sketch.
constexpr int slots_of(int K) { return K == 0 ? 1 : K; }

// One staging step takes TW entries (TW <= T) of each of the 64 rows.  The
// wavefront's lanes take slots: slot i * 64 + lane holds entry t0 + j of row r,
// (r, j) = (slot / TW, slot % TW), so a row's slots are loaded by neighbouring
// lanes; it is stored at r * (TW + 1) + j (rows padded against bank conflicts).
// A step of TW <= T / 2 leaves label words 64 (TW + 1) onwards unused: with
// KEEP, slot s's column index is kept at kept_col<TW>(s) there, for the marking
// pass.
template <int TW>
__device__ __forceinline__ int kept_col(int slot) { return kWave * (TW + 1) + slot; }

template <int TW>
__device__ __forceinline__ int slot_word(int r, int j) { return r * (TW + 1) + j; }

// The step in four-slot batches of three phases (column indices, weights,
// labels), so that each phase's loads are in flight together; a slot past its
// row's end issues no load and is stored as padding (label -1, weight 0), as is
// an entry of the vertex itself.
constexpr int kLoadBatch = 4;

template <int TW, bool KEEP, int T, class Pos>
__device__ __forceinline__ void stage_load(const MoveArgs &a, Stage<T, Pos, false> &st, int lane,
                                           int t0) {
  constexpr int B = TW < kLoadBatch ? TW : kLoadBatch;
#pragma unroll
  for (int i0 = 0; i0 < TW; i0 += B) {
    bool ok[B];
    Pos e[B];
    int c[B], lab[B];
    float x[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int slot = (i0 + b) * kWave + lane, r = slot / TW, j = slot % TW;
      ok[b] = t0 + j < st.row[r].x;
      e[b] = st.beg[r] + (Pos)(t0 + j);
    }
#pragma unroll
    for (int b = 0; b < B; ++b) c[b] = ok[b] ? __builtin_nontemporal_load(element(a.col, e[b])) : -1;
#pragma unroll
    for (int b = 0; b < B; ++b)
      x[b] = !ok[b] ? 0.0f : (a.w ? __builtin_nontemporal_load(element(a.w, e[b])) : 1.0f);
#pragma unroll
    for (int b = 0; b < B; ++b) lab[b] = ok[b] ? *element<Pos>(a.C, c[b]) : -1;
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int slot = (i0 + b) * kWave + lane, r = slot / TW, j = slot % TW;
      st.lab[slot_word<TW>(r, j)] = lab[b];
      st.w[slot_word<TW>(r, j)] = c[b] == st.row[r].y ? 0.0f : x[b];
      if constexpr (KEEP && 2 * TW <= T) st.lab[kept_col<TW>(slot)] = c[b];
    }
  }
}

// UNIT: the columns of a step go into registers, all of a lane's slots in
// flight together, the next step's while this one is consumed; then the
// labels, eight slots at a time.  A slot past its row's end reads the row's last
// entry (without any, another row's: staged_position) and the label of vertex 0,
// lines that others of the step read too, so no branch stands between a step's
// loads: it waits for memory twice, or three times for 16 entries, instead of
// eight times in stage_load.  Such graphs have no weights to stream and rows of a
// few labels that hit the caches, so they wait more than they move: R-MAT-22 det k =
// 8, iterations 0 and 8, 2.7 and 2.1 to 1.9 and 1.3 ms; 512 SBM graphs det k = 8 55.4
// to 52.6 ms per solve (at four wavefronts per SIMD: kMoveMostWaves).
// (With weights and labels that miss, the batches of stage_load are faster: the
// order above cost 6% on R-MAT-24, whose columns and weights then miss L2 more
// often, 216 against 205 million line misses in the first iteration.)
template <int TW, class Pos, int T>
__device__ __forceinline__ void stage_cols(const MoveArgs &a, const Stage<T, Pos, true> &st,
                                           int lane, int t0, int (&c)[TW]) {
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    const int slot = i * kWave + lane, r = slot / TW, j = slot % TW;
    c[i] = __builtin_nontemporal_load(
        element(a.col, staged_position<Pos>(st.beg[r], st.row[r].x, t0 + j)));
  }
}

// Labels of the step's columns c into the stage; a slot past its row's end or
// naming the vertex itself gets label -1.
template <bool KEEP, int TW, class Pos, int T>
__device__ __forceinline__ void stage_labels(const MoveArgs &a, Stage<T, Pos, true> &st, int lane,
                                             int t0, const int (&c)[TW]) {
  constexpr int B = TW < 8 ? TW : 8;
#pragma unroll
  for (int i0 = 0; i0 < TW; i0 += B) {
    int lab[B];
    unsigned on = 0;
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int slot = (i0 + b) * kWave + lane, r = slot / TW, j = slot % TW;
      const int2 row = st.row[r];
      const bool in = t0 + j < row.x;
      on |= in && c[i0 + b] != row.y ? 1u << b : 0u;
      lab[b] = *element<Pos>(a.C, in ? c[i0 + b] : 0);
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int slot = (i0 + b) * kWave + lane;
      st.lab[slot_word<TW>(slot / TW, slot % TW)] = (on >> b) & 1u ? lab[b] : -1;
      if constexpr (KEEP && 2 * TW <= T) st.lab[kept_col<TW>(slot)] = c[i0 + b];
    }
  }
}

// Feed entries [beg, beg + len) of row `self` to feed(label, weight) in CSR
// order (len = 0: nothing); entries of the vertex itself and past the row's
// end come with weight 0.  All lanes of the wavefront must call it together.
// Each step takes 4, 8 or T entries per row, the narrowest that covers what
// the wavefront's longest row has left: with short rows a wide step would
// leave most load slots idle.  With KEEP, returns the step width when every
// row fit one step of width 4 or 8 (the rows' column indices are then kept in
// the stage); otherwise 0.  Keeping them costs registers: only kernels that
// stay within their register budget with it pass KEEP.
template <bool KEEP, int T, class Pos, bool UNIT, class Feed>
__device__ __forceinline__ int staged_rows(const MoveArgs &a, Stage<T, Pos, UNIT> &st, int lane,
                                           Pos beg, int len, int self, Feed &&feed) {
  static_assert(T == 16, "step widths 4, 8 and 16");
  if constexpr (!UNIT) st.beg[lane] = beg;
  st.row[lane] = make_int2(len, self);
  const int maxlen = wave_max(len);
  if (maxlen == 0) return 0;
  if constexpr (UNIT)
    st.beg[lane] = staged_begin(beg, len, rl_as(beg, __ffsll((long long)__ballot(len > 0)) - 1));
  wave_lds_sync();
  int t0 = 0;
  // this lane's row: its first entries of a step of tw staged ones (later
  // columns of the step are past the end of every row)
  const auto consume = [&](int tw) {
    wave_lds_sync();
    const int tn = min(tw, maxlen - t0);
    const int row = lane * (tw + 1);
    for (int j = 0; j < tn; ++j) {
      const int lab = st.lab[row + j];
      if constexpr (UNIT)
        feed(lab, lab >= 0 ? 1.0f : 0.0f);
      else
        feed(lab, st.w[row + j]);
    }
    wave_lds_sync();
    t0 += tw;
  };
  if constexpr (UNIT) {
    if (maxlen > 8) {
      int c[T];
      stage_cols(a, st, lane, 0, c);
      for (;;) {
        stage_labels<KEEP>(a, st, lane, t0, c);
        const bool more = maxlen - (t0 + T) > 8;
        if (more) stage_cols(a, st, lane, t0 + T, c);
        consume(T);
        if (!more) break;
      }
    }
    if (t0 < maxlen) {
      if (maxlen - t0 <= 4) {
        int c[4];
        stage_cols(a, st, lane, t0, c);
        stage_labels<KEEP>(a, st, lane, t0, c);
        consume(4);
      } else {
        int c[8];
        stage_cols(a, st, lane, t0, c);
        stage_labels<KEEP>(a, st, lane, t0, c);
        consume(8);
      }
    }
  } else {
    while (t0 < maxlen) {
      const int rem = maxlen - t0;
      const int tw = rem <= 4 ? 4 : (rem <= 8 ? 8 : T);
      if (tw == 4)
        stage_load<4, KEEP>(a, st, lane, t0);
      else if (tw == 8)
        stage_load<8, KEEP>(a, st, lane, t0);
      else
        stage_load<T, KEEP>(a, st, lane, t0);
      consume(tw);
    }
  }
  return KEEP && maxlen <= 8 ? (maxlen <= 4 ? 4 : 8) : 0;
}

// Double scan (Section 4.4, Algorithm 4 rescan): the live slots of the
// single scan's sketch are the candidates; a second pass in CSR order sums
// each candidate's exact weight, and the heaviest wins (ties to the lowest
// label; no candidate keeps `keep`).
template <int K>
struct Rescan {
  int key[K];  // candidate labels, -1 for slots that were empty
  float acc[K];

  __device__ __forceinline__ void from(const LaneSketch<K> &S) {
#pragma unroll
    for (int s = 0; s < K; ++s) {
      key[s] = S.val[s] > 0.0f ? S.key[s] : -1;
      acc[s] = 0.0f;
    }
  }
  __device__ __forceinline__ void add(int c, float x) {
#pragma unroll
    for (int s = 0; s < K; ++s) acc[s] = (c >= 0 && key[s] == c) ? acc[s] + x : acc[s];
  }
  __device__ __forceinline__ int best(int keep) const {
    int bk = keep;
    float bv = 0.0f;
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const bool better = acc[s] > bv || (acc[s] == bv && acc[s] > 0.0f && key[s] < bk);
      bk = better ? key[s] : bk;
      bv = better ? acc[s] : bv;
    }
    return bk;
  }
};

// Flag a neighbour of a changed vertex as unprocessed (plain byte store:
// reading the flag first to skip repeated marks measured slower).
__device__ __forceinline__ void mark(const MoveArgs &a, int j) { a.act_next[j] = 1; }

// Mark the neighbours of every lane whose `moved` is set (entries [beg, beg +
// len) of its row), with row-contiguous column loads by the whole wavefront:
// all of a step's column loads are issued before its flag stores.
template <int TW, class Pos, class St>
__device__ __forceinline__ void mark_step(const MoveArgs &a, const St &st, int lane, int t0) {
  bool ok[TW];
  int c[TW];
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    const int slot = i * kWave + lane;
    const int r = slot / TW, j = slot % TW;
    ok[i] = t0 + j < st.row[r].x;
    c[i] = ok[i] ? __builtin_nontemporal_load(element(a.col, st.beg[r] + (Pos)(t0 + j))) : 0;
  }
#pragma unroll
  for (int i = 0; i < TW; ++i)
    if (ok[i]) mark(a, c[i]);
}

// Mark the neighbours of entries [beg, end) of one row, the whole wavefront
// taking 64 x U entries at a time (loads first, then stores).  The move
// kernels use kMarkUnroll; k_hub_mark, which only marks, takes a whole hub
// segment per step so that one load latency is waited for per segment.
constexpr int kMarkUnroll = 4;

template <int U = kMarkUnroll, class Pos>
__device__ __forceinline__ void mark_row(const MoveArgs &a, Pos beg, Pos end, int lane) {
  const unsigned len = (unsigned)(end - beg);  // a row has fewer than 2^31 entries
  for (unsigned q0 = 0; q0 < len; q0 += U * kWave) {
    int c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const unsigned q = q0 + u * kWave + lane;
      c[u] = q < len ? __builtin_nontemporal_load(a.col + (beg + (Pos)q)) : -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c[u] >= 0) mark(a, c[u]);
  }
}

// Mark from the columns that a single staging step of width TW kept in the
// stage: each lane takes the slots it loaded (st.row already holds no entries
// for rows that did not move).
template <int TW, class St>
__device__ __forceinline__ void mark_kept(const MoveArgs &a, const St &st, int lane) {
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    const int slot = i * kWave + lane, r = slot / TW, j = slot % TW;
    if (j < st.row[r].x) mark(a, st.lab[kept_col<TW>(slot)]);
  }
}

// Mark the neighbours of every lane whose `moved` is set (entries [beg, beg +
// len) of its row), with row-contiguous column loads by the whole wavefront
// and the same step widths as staged_rows.  kept = the width staged_rows
// returned for these rows (the stage then still holds their columns and
// nothing is read from the CSR), or 0.
template <int T, class Pos, bool UNIT>
__device__ __forceinline__ void staged_mark(const MoveArgs &a, Stage<T, Pos, UNIT> &st, int lane,
                                            Pos beg, int len, bool moved, int kept) {
  if (__ballot(moved) == 0ull) return;
  st.beg[lane] = beg;
  st.row[lane].x = moved ? len : 0;
  const int maxlen = wave_max(moved ? len : 0);
  wave_lds_sync();
  if (kept != 0) {
    if (kept == 4)
      mark_kept<4>(a, st, lane);
    else
      mark_kept<8>(a, st, lane);
    wave_lds_sync();
    return;
  }
  for (int t0 = 0; t0 < maxlen;) {
    const int rem = maxlen - t0;
    if (rem <= 4) {
      mark_step<4, Pos>(a, st, lane, t0);
      t0 += 4;
    } else if (rem <= 8) {
      mark_step<8, Pos>(a, st, lane, t0);
      t0 += 8;
    } else {
      mark_step<T, Pos>(a, st, lane, t0);
      t0 += T;
    }
  }
  wave_lds_sync();
}

// ---------------------------------------------------------------------------
// LPA_MODE_DET hub path: one wavefront per vertex, CSR order.
//
// The row is read in super-chunks of kHubDepth x 64 entries (lane t of
// chunk d holds entry base + 64 d + t): the next super-chunk's column,
// weight and label loads are in flight while the current one is consumed,
// so the serial sketch chain is not paced by the gather latency.
// ---------------------------------------------------------------------------
constexpr int kHubDepth = 8;

template <int D>
struct HubChunks {
  int lab[D];
  float x[D];  // 0 for padding and self-loops

  // self: the vertex's own index as its row entries name it.  Column
  // indices, then weights, then labels: no load waits for another of its
  // phase, so each phase's D loads are in flight together (a weight load
  // conditioned on its column index would wait for that index first).
  template <class Pos>
  __device__ __forceinline__ void load(const MoveArgs &a, int self, Pos sb, Pos end, int lane) {
    int c[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const Pos e = sb + d * kWave + lane;
      c[d] = e < end ? __builtin_nontemporal_load(a.col + e) : -1;
    }
    if (a.w) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const Pos e = sb + d * kWave + lane;
        x[d] = e < end ? __builtin_nontemporal_load(a.w + e) : 0.0f;
      }
    } else {
#pragma unroll
      for (int d = 0; d < D; ++d) x[d] = 1.0f;
    }
#pragma unroll
    for (int d = 0; d < D; ++d) lab[d] = c[d] >= 0 ? a.C[c[d]] : 0;
#pragma unroll
    for (int d = 0; d < D; ++d) x[d] = (c[d] < 0 || c[d] == self) ? 0.0f : x[d];
  }
};

// Call consume(lab, x, cnt) for every 64-entry chunk of [beg, end) in order
// (cnt = entries of the chunk; lanes >= cnt hold padding).
template <class Pos, class Consume>
__device__ __forceinline__ void hub_feed(const MoveArgs &a, int self, Pos beg, Pos end, int lane,
                                         Consume &&consume) {
  // The chain of one hub bounds the whole iteration while the other
  // wavefronts of its SIMD stream short rows: let it issue first.
  __builtin_amdgcn_s_setprio(3);
  HubChunks<kHubDepth> cur, nxt;
  cur.load(a, self, beg, end, lane);
  for (Pos sb = beg; sb < end; sb += kHubDepth * kWave) {
    const Pos nb = sb + kHubDepth * kWave;
    if (nb < end) nxt.load(a, self, nb, end, lane);
#pragma unroll 1
    for (int d = 0; d < kHubDepth; ++d) {
      const Pos base = sb + d * kWave;
      if (base >= end) break;
      consume(cur.lab[0], cur.x[0], (int)min((Pos)kWave, (Pos)(end - base)));
#pragma unroll
      for (int q = 0; q + 1 < kHubDepth; ++q) {
        cur.lab[q] = cur.lab[q + 1];
        cur.x[q] = cur.x[q + 1];
      }
    }
    cur = nxt;
  }
  __builtin_amdgcn_s_setprio(0);
}

// The det hub chains: one wavefront feeds one row, entry by entry, into a
// sketch held one slot per lane.  The chain is serial, so its time is the
// instructions issued per entry.  One wavefront issues a dependent vector
// instruction every 4.4 cycles, but a value that passes from a vector compare
// through a scalar register to a branch or back to the vector unit costs 28
// to 36 (measured), so the common step is straight vector code, and what would
// need a branch is looked for in groups of kHubGroup entries.
//
// The row is read kHubChunk entries at a time, two chunks ahead (HubReader):
// a chunk's columns are in flight while the chunk before it waits for its
// labels, which arrive while the one before that is consumed.  A chunk's
// entries that count (not the vertex itself) are appended to a queue in LDS,
// from which every lane reads the same entry, so there is no cross-lane read
// and no wait for memory inside the chain; the chain takes the queue kWave
// entries at a time.
constexpr int kHubChunk = 256;
constexpr int kHubGroup = 8;
constexpr int kHubParts = kHubChunk / kWave;
constexpr int kHubQueue = kHubChunk + kWave;  // a chunk and what the chain has not taken yet
constexpr int kNoLabel = -2;  // no vertex's label

// The queue in kHubWords words of this wavefront's LDS, 16-byte aligned: labels
// (2 * kHubGroup words of no label lie before the first) and weights.
constexpr int kHubWords = 2 * kHubGroup + 2 * kHubQueue;
static_assert(kHubWords <= kWave * (kStageT + 1), "the queue lies in the row stage");
struct HubQueue {
  int *lab;
  float *wt;
  __device__ __forceinline__ HubQueue(int *buf, int lane)
      : lab(buf + 2 * kHubGroup), wt(reinterpret_cast<float *>(buf + 2 * kHubGroup + kHubQueue)) {
    if (lane < 2 * kHubGroup) buf[lane] = kNoLabel;
  }
};

// Offsets are from the row's first entry: a row has fewer than 2^31 entries, so
// they and the chunks beyond its end fit 32 bits whatever the width of Pos.
// Lanes past the end read the last entry again: without a branch around the
// loads no register is copied, and none is waited for before it is used.
template <bool UNIT, class Pos>
struct HubReader {
  int col[kHubParts], lab[kHubParts];
  float x[kHubParts];
  unsigned skip;  // bit d: part d's entry of this lane counts for nothing

  __device__ __forceinline__ void cols(const MoveArgs &a, Pos beg, unsigned len, int lane,
                                       unsigned o) {
#pragma unroll
    for (int d = 0; d < kHubParts; ++d) {
      const unsigned e = min(o + d * kWave + lane, len - 1);
      col[d] = __builtin_nontemporal_load(a.col + (beg + (Pos)e));
    }
  }
  // of the columns held in col, at o
  __device__ __forceinline__ void labels(const MoveArgs &a, int self, Pos beg, unsigned len,
                                         int lane, unsigned o) {
    skip = 0;
#pragma unroll
    for (int d = 0; d < kHubParts; ++d) {
      lab[d] = a.C[col[d]];
      skip |= (o + d * kWave + lane >= len || col[d] == self) ? 1u << d : 0u;
    }
    if constexpr (!UNIT) {
      if (a.w) {
#pragma unroll
        for (int d = 0; d < kHubParts; ++d) {
          const unsigned e = min(o + d * kWave + lane, len - 1);
          x[d] = __builtin_nontemporal_load(a.w + (beg + (Pos)e));
        }
      }
    }
  }
};

// Queues the entries of [beg, end) that count and for which drop(lab, on) does
// not hold (it is called by all lanes, on: the lane's entry counts), and calls
// block(q) for queue entries q .. q + 63 as they fill up; returns the number
// of entries then left in the queue, fewer than 64, from its start.
template <bool UNIT, class Pos, class Drop, class Block>
__device__ __forceinline__ int hub_rows(const MoveArgs &a, const HubQueue &Q, int self, Pos beg,
                                        Pos end, int lane, Drop &&drop, Block &&block) {
  const unsigned len = (unsigned)(end - beg);
  if (len == 0) return 0;
  // The chain of one hub bounds the whole iteration while the other
  // wavefronts of its SIMD stream short rows: let it issue first.
  __builtin_amdgcn_s_setprio(3);
  HubReader<UNIT, Pos> R;
#pragma unroll
  for (int d = 0; d < kHubParts; ++d) R.x[d] = 1.0f;
  R.cols(a, beg, len, lane, 0);
  R.labels(a, self, beg, len, lane, 0);
  R.cols(a, beg, len, lane, kHubChunk);
  int n = 0;
  for (unsigned o = 0; o < len; o += kHubChunk) {
    const unsigned long long below = (1ull << lane) - 1ull;
    drop.chunk();
#pragma unroll
    for (int d = 0; d < kHubParts; ++d) {
      const bool counts = !((R.skip >> d) & 1u);
      const bool dropped = drop(R.lab[d], counts);
      const bool on = counts && !dropped;
      const unsigned long long m = __ballot(on);
      const int at = n + (int)__popcll(m & below);
      if (on) {
        Q.lab[at] = R.lab[d];
        if constexpr (!UNIT) Q.wt[at] = R.x[d];
      }
      n += (int)__popcll(m);
    }
    wave_lds_sync();
    R.labels(a, self, beg, len, lane, o + kHubChunk);
    R.cols(a, beg, len, lane, o + 2 * kHubChunk);
    int q = 0;
    for (; q + kWave <= n; q += kWave) block(q);
    if (q > 0) {  // what is left moves to the front
      const int l = Q.lab[q + lane];
      float w = 1.0f;
      if constexpr (!UNIT) w = Q.wt[q + lane];
      wave_lds_sync();
      Q.lab[lane] = l;
      if constexpr (!UNIT) Q.wt[lane] = w;
      wave_lds_sync();
      n -= q;
    }
  }
  __builtin_amdgcn_s_setprio(0);
  return n;
}

struct DropNone {
  __device__ __forceinline__ void chunk() {}
  __device__ __forceinline__ bool operator()(int, bool) { return false; }
};

// Keeps the reads of the next group's entries where they are written: before
// this group is consumed.
__device__ __forceinline__ void reads_start_here() { asm volatile("" ::: "memory"); }

// Calls step(label, weight) for queue entries [q, q + 64) in order, all lanes
// with the same entry.
template <class Step>
__device__ __forceinline__ void hub_each(const HubQueue &Q, int q, Step &&step) {
  const int4 *l4 = reinterpret_cast<const int4 *>(Q.lab + q);
  const float4 *w4 = reinterpret_cast<const float4 *>(Q.wt + q);
  int4 nl = l4[0];
  float4 nw = w4[0];
#pragma unroll 2
  for (int i = 0; i < kWave / 4; ++i) {
    const int4 l = nl;
    const float4 w = nw;
    const int ni = (i + 1) & (kWave / 4 - 1);
    nl = l4[ni];
    nw = w4[ni];
    reads_start_here();
    step(l.x, w.x);
    step(l.y, w.y);
    step(l.z, w.z);
    step(l.w, w.w);
  }
}

// Calls step(label, weight) for every entry of [beg, end) that counts, in CSR
// order, all lanes with the same entry.
template <class Pos, class Step>
__device__ __forceinline__ void hub_stream(const MoveArgs &a, int *buf, int self, Pos beg, Pos end,
                                           int lane, Step &&step) {
  const HubQueue Q(buf, lane);
  const int n = hub_rows<false>(a, Q, self, beg, end, lane, DropNone(),
                                [&](int q) { hub_each(Q, q, step); });
#pragma unroll 1
  for (int q = 0; q < n; ++q) step(Q.lab[q], Q.wt[q]);
  wave_lds_sync();
}

// Slots across lanes: for K <= 16 each 16-lane row holds a copy of the sketch
// (its lanes 0 .. K - 1; a group's entries are looked up one per row), for
// K = 32 lanes 0 .. 31 do.  Slots are kept in increasing order of value, free
// slots first (the slots' positions do not change the choice); the other lanes
// hold a value above every slot's.
template <int K>
constexpr unsigned kSlotMask = K >= 32 ? ~0u : (1u << (K & 31)) - 1u;

template <int K>
__device__ __forceinline__ int slot_of(int lane) {
  return K <= 16 ? lane & 15 : lane;
}

// The value of slot 0.
template <int K>
__device__ __forceinline__ unsigned first_slot(unsigned v) {
  if constexpr (K <= 16)
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x150, 0xF, 0xF, true);  // row_newbcast
  else
    return (unsigned)rfl((int)v);
}

// The value of the next slot; TOP above the last slot.
template <int K, unsigned TOP>
__device__ __forceinline__ unsigned next_slot(unsigned v) {
  if constexpr (K == 16)  // no spare lane: a row shift whose last lane keeps TOP
    return (unsigned)__builtin_amdgcn_update_dpp((int)TOP, (int)v, 0x101, 0xF, 0xF, false);
  else
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x134, 0xF, 0xF, true);  // wave_rol:1
}

// A slot's value grew to x: it moves up to its place.  p: the slot; c: its key.
template <int K, unsigned TOP>
__device__ __forceinline__ void slot_grew(int lane, int p, int c, unsigned x, int &key,
                                          unsigned &v) {
  const unsigned up = next_slot<K, TOP>(v);
  const int kup = (int)next_slot<K, 0>((unsigned)key);
  const unsigned nv = max(v, min(up, x));
  const int nk = x > up ? kup : (x > v ? c : key);
  const bool from = slot_of<K>(lane) >= p;
  v = from ? nv : v;
  key = from ? nk : key;
}

// Runs queue entries [q, q + 64) in groups of kHubGroup.  fast(c, w) is the
// step of an entry whose label is in no slot, slow(c, w) looks the label up
// first; an entry takes the fast step when its label is in no slot and repeats
// none of the 15 entries before it, and most groups hold no other.  A group's
// labels are looked up (two compares: row r of the lanes takes entries r and
// r + 4) before the group ahead of it runs, so that nothing waits for the
// answer; the keys which that group adds are among those 15 labels.
// key: the slots' keys, K <= 16.
template <int K, bool UNIT, class Fast, class Slow>
__device__ __forceinline__ void hub_groups(const HubQueue &Q, int q, int lane, const int &key,
                                           Fast &&fast, Slow &&slow) {
  static_assert(kHubGroup == 8, "two lookups of four entries");
  struct Group {
    int4 l[2];
    float4 w[2];
  };
  auto fetch = [&](Group &g, int i) {
    const int4 *l4 = reinterpret_cast<const int4 *>(Q.lab + i);
    g.l[0] = l4[0];
    g.l[1] = l4[1];
    if constexpr (!UNIT) {
      const float4 *w4 = reinterpret_cast<const float4 *>(Q.wt + i);
      g.w[0] = w4[0];
      g.w[1] = w4[1];
    }
  };
  const int *look = Q.lab + q + (lane >> 4);
  unsigned long long rep;
  {
    const int *mine = Q.lab + q + lane;
    const int e = mine[0];
    unsigned least = ~0u;
#pragma unroll
    for (int t = 1; t < 2 * kHubGroup; ++t) least = min(least, (unsigned)(mine[-t] ^ e));
    rep = __ballot(least == 0u);
  }
  Group A, B;
  fetch(A, q);
  unsigned long long h0 = __ballot(key == look[0]), h1 = __ballot(key == look[4]);
  int la = look[8], lb = look[12];
  auto run = [&](const Group &g, Group &nxt, int i) {  // i: offset of g in the 64 entries
    const unsigned long long hits[2] = {h0, h1};
    const unsigned rp = (unsigned)rep;
    h0 = __ballot(key == la);
    h1 = __ballot(key == lb);
    rep >>= kHubGroup;
    const int far = (i + 2 * kHubGroup) & (kWave - 1);
    fetch(nxt, q + ((i + kHubGroup) & (kWave - 1)));
    la = look[far];
    lb = look[far + 4];
    reads_start_here();
    const int c[8] = {g.l[0].x, g.l[0].y, g.l[0].z, g.l[0].w, g.l[1].x, g.l[1].y, g.l[1].z, g.l[1].w};
    float w[8];
    if constexpr (UNIT) {
#pragma unroll
      for (int j = 0; j < 8; ++j) w[j] = 1.0f;
    } else {
      const float u[8] = {g.w[0].x, g.w[0].y, g.w[0].z, g.w[0].w,
                          g.w[1].x, g.w[1].y, g.w[1].z, g.w[1].w};
#pragma unroll
      for (int j = 0; j < 8; ++j) w[j] = u[j];
    }
    if (hits[0] | hits[1] | (rp & 0xFF)) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const unsigned in = (unsigned)(hits[j >> 2] >> (16 * (j & 3))) & kSlotMask<K>;
        if (in | ((rp >> j) & 1u))
          slow(c[j], w[j]);
        else
          fast(c[j], w[j]);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) fast(c[j], w[j]);
    }
  };
#pragma unroll 1
  for (int i = 0; i < kWave; i += 2 * kHubGroup) {
    run(A, B, i);
    run(B, A, i + kHubGroup);
  }
}

// The sketch with weights.  Values are handled as bit patterns where they are
// compared (non-negative floats order like unsigned integers).  With v0 the
// smallest value, a pair (c, w) that no key holds does the same to every state:
// every slot loses m = min(v0, w), and x = |v0 - w| takes the place of the
// lowest slot's value: w - v0 under the key c if w > v0 (with a free slot
// v0 = 0, so nothing is lost and w is placed), else v0 - w under its own key.
// Subtraction of one m keeps the order, so x only moves up to its place, one
// minimum and one maximum with the next slot's value: eleven vector
// instructions, no branch, no search for the smallest or for a free slot.
// A pair of weight 0 changes nothing.
template <int K>
__device__ __forceinline__ void weighted_miss(int c, float w, int &key, unsigned &v) {
  const unsigned v0 = first_slot<K>(v), wb = __float_as_uint(w);
  const float m = __uint_as_float(min(v0, wb));
  const unsigned x = __float_as_uint(__uint_as_float(max(v0, wb)) - m);
  const unsigned d = __float_as_uint(__uint_as_float(v) - m);
  const unsigned up = next_slot<K, 0x7f800000u>(d);
  const int kup = (int)next_slot<K, 0>((unsigned)key);
  v = max(d, min(up, x));
  key = x > up ? kup : (x > d ? c : key);
}

template <int K>
__device__ __forceinline__ void weighted_entry(int lane, int c, float w, int &key, unsigned &v) {
  const unsigned hm = (unsigned)__ballot(key == c) & kSlotMask<K>;
  if (hm) {
    const int p = __ffs((int)hm) - 1;
    const unsigned x = __float_as_uint(rl_f(__uint_as_float(v), p) + w);
    slot_grew<K, 0x7f800000u>(lane, p, c, x, key, v);
  } else {
    weighted_miss<K>(c, w, key, v);
  }
}

// One row with weights.  FRESH: every label differs from every key
// (MoveArgs::fresh_hubs).  Measured on a row of 163,428 entries, k = 8: 30 ns
// per entry FRESH, 35 to 43 with 0 to 5% of hits (one vote and one decision per
// entry took 95 and 140 to 200).  R-MAT-21, k = 4, whose largest row has some
// 100,000: 22 to 4.1 ms per iteration.
template <int K, bool FRESH, class Pos>
__device__ __forceinline__ void det_weighted(const MoveArgs &a, int *buf, int x0, Pos beg, Pos end,
                                             int lane, int &key, float &val) {
  unsigned v = slot_of<K>(lane) < K ? 0u : 0x7f800000u;
  if constexpr (FRESH) {
    hub_stream(a, buf, x0, beg, end, lane,
               [&](int c, float w) { weighted_miss<K>(c, w, key, v); });
  } else if constexpr (K > 16) {
    hub_stream(a, buf, x0, beg, end, lane,
               [&](int c, float w) { weighted_entry<K>(lane, c, w, key, v); });
  } else {
    const HubQueue Q(buf, lane);
    const auto entry = [&](int c, float w) { weighted_entry<K>(lane, c, w, key, v); };
    const int n = hub_rows<false>(a, Q, x0, beg, end, lane, DropNone(), [&](int q) {
      hub_groups<K, false>(
          Q, q, lane, key, [&](int c, float w) { weighted_miss<K>(c, w, key, v); }, entry);
    });
#pragma unroll 1
    for (int q = 0; q < n; ++q) entry(Q.lab[q], Q.wt[q]);
    wave_lds_sync();
  }
  val = slot_of<K>(lane) < K ? __uint_as_float(v) : 0.0f;
}

// The sketch with unit weights on a row of fewer than 2^24 entries: slot
// values are whole numbers, exact in fp32, and are counted as integers.  An
// entry that no key holds takes 1 from every slot and is used up when all are
// live; otherwise it takes the last free slot, whose next slot is live: seven
// vector instructions, and the slots stay in order.
constexpr unsigned kUnitTop = 1u << 30;

// 1 in a register whose value the compiler does not know: it would otherwise
// turn a minimum with 1 into a comparison with 0, whose result goes through
// scalar registers.
__device__ __forceinline__ unsigned opaque_one() {
  unsigned one = 1u;
  asm("" : "+v"(one));
  return one;
}

// one: 1, from opaque_one.
template <int K>
__device__ __forceinline__ void unit_miss(unsigned one, int c, int &key, unsigned &v) {
  const unsigned m = min(first_slot<K>(v), one), t = min(next_slot<K, kUnitTop>(v), one);
  const unsigned here = __builtin_elementwise_sub_sat(t, v);  // 1: v is 0 and the next is not
  v = v - m + here;
  key = here ? c : key;
}

template <int K>
__device__ __forceinline__ void unit_entry(unsigned one, int lane, int c, int &key, unsigned &v) {
  const unsigned hm = (unsigned)__ballot(key == c) & kSlotMask<K>;
  if (hm) {
    const int p = __ffs((int)hm) - 1;
    slot_grew<K, kUnitTop>(lane, p, c, (unsigned)rl((int)v, p) + 1u, key, v);
  } else {
    unit_miss<K>(one, c, key, v);
  }
}

// Leaves out of the chain the entries of the top slot's label, and counts them:
// while the top slot holds more than the entries ahead could take from it, it
// stays live whatever they are, so entries of its label only add to it, in
// any order (on R-MAT graphs one label soon holds a tenth, later nearly all of
// a hub's row).  Each time all slots lose 1, the other slots and the entry
// that is used up lose K together, out of what these slots hold and the entries
// add: at most (kHubQueue + (K - 1) * the second value) / K times.
template <int K>
struct DropTop {
  int lane;
  const int &key;
  unsigned &v;
  int top;
  bool safe;
  __device__ __forceinline__ DropTop(int l, const int &k, unsigned &x) : lane(l), key(k), v(x) {}
  __device__ __forceinline__ void chunk() {
    const long long others = K > 1 ? (long long)(K - 1) * rl((int)v, K > 1 ? K - 2 : 0) : 0;
    safe = (long long)(rl((int)v, K - 1) - 1) * K > kHubQueue + others;
    top = rl(key, K - 1);
  }
  __device__ __forceinline__ bool operator()(int lab, bool on) {
    const bool heavy = on && safe && lab == top;
    const unsigned tops = (unsigned)__popcll(__ballot(heavy));  // of the whole wavefront
    v += slot_of<K>(lane) == K - 1 ? tops : 0u;
    return heavy;
  }
};

// One row with unit weights: 27 to 35 ns per entry of the chain on a row of
// 163,428, k = 8 (140 with one vote and one decision per entry); R-MAT-22, k = 8,
// iterations 1 to 5: 23 to 5.5 ms.
template <int K, class Pos>
__device__ __forceinline__ void det_unit(const MoveArgs &a, int *buf, int x0, Pos beg, Pos end,
                                         int lane, int &key, float &val) {
  const HubQueue Q(buf, lane);
  const unsigned one = opaque_one();
  unsigned v = slot_of<K>(lane) < K ? 0u : kUnitTop;
  const auto entry = [&](int c, float) { unit_entry<K>(one, lane, c, key, v); };
  const int n = hub_rows<true>(a, Q, x0, beg, end, lane, DropTop<K>(lane, key, v), [&](int q) {
    if constexpr (K <= 16)
      hub_groups<K, true>(
          Q, q, lane, key, [&](int c, float) { unit_miss<K>(one, c, key, v); }, entry);
    else
#pragma unroll 1
      for (int i = 0; i < kWave; ++i) entry(Q.lab[q + i], 1.0f);
  });
#pragma unroll 1
  for (int q = 0; q < n; ++q) entry(Q.lab[q], 1.0f);
  wave_lds_sync();
  val = slot_of<K>(lane) < K ? (float)v : 0.0f;
}

// Unit weights at iteration 0 from the initial labels, no neighbour twice
// (MoveArgs::fresh_hubs): every entry is a label of its own, so K entries fill
// the slots and the next empties them all again.  What is left after L
// entries is the last L mod (K + 1) of them, one slot each with value 1; the
// row is only counted (the vertex itself is no entry).
template <int K, class Pos>
__device__ __forceinline__ void det_unit_fresh(const MoveArgs &a, int x0, Pos beg, Pos end,
                                               int lane, int &key, float &val) {
  constexpr int U = 16;
  int own = 0;  // entries that are the vertex itself (at most one)
  const unsigned len = (unsigned)(end - beg);
  for (unsigned q0 = 0; q0 < len; q0 += U * kWave) {
    int c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const unsigned q = q0 + u * kWave + lane;
      c[u] = q < len ? __builtin_nontemporal_load(a.col + (beg + (Pos)q)) : -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) own += c[u] == x0 ? 1 : 0;
  }
  const unsigned entries = len - (unsigned)__popcll(__ballot(own != 0));
  const int left = (int)(entries % (K + 1));
  // the last 64 entries hold the last K + 1 that count
  const int c = (unsigned)lane < len ? a.col[end - 1 - lane] : x0;
  const bool counts = c != x0;
  const int rank = (int)__popcll(__ballot(counts) & ((1ull << lane) - 1ull));
  const bool live = counts && rank < left;
  // lane s takes the rank-s entry
  const unsigned long long lm = __ballot(live);
  const int l = live ? a.C[c] : -1;
  unsigned long long rest = lm;
#pragma unroll
  for (int s = 0; s < K; ++s) {
    const bool on = rest != 0;
    const int ls = rl(l, on ? __ffsll((long long)rest) - 1 : 0);
    rest &= rest - 1;
    key = on && lane == s ? ls : key;
    val = on && lane == s ? 1.0f : val;
  }
}

// Double scan: the labels of key (-1: none) re-weighted exactly, each slot's
// entries added in CSR order by the slot's lane (val starts at 0), a run of
// entries with scalar lane indices and no cross-lane votes.
template <int K, class Pos>
__device__ __forceinline__ void det_rescan(const MoveArgs &a, int x0, Pos beg, Pos end, int lane,
                                           const int key, float &val) {
  hub_feed(a, x0, beg, end, lane, [&](int lab, float x, int cnt) {
    int slot = -1;
#pragma unroll
    for (int s = 0; s < K; ++s) slot = (lab == rl(key, s)) ? s : slot;
    unsigned long long run = __ballot(slot >= 0 && lane < cnt && x > 0.0f);
    while (run) {
      const int h = __ffsll((long long)run) - 1;
      run &= run - 1;
      const int sh = rl(slot, h);
      const float xh = rl_f(x, h);
      val = (lane == sh) ? val + xh : val;
    }
  });
}

// One hub in det mode.  p: the vertex's degree-order position; buf: LDS of
// this wavefront for hub_stream.
template <int K, bool RS, class Pos>
__device__ void hub_vertex_det(const MoveArgs &a, int *buf, int p, unsigned long long &scanned,
                               unsigned long long &changed) {
  const int lane = threadIdx.x & (kWave - 1);
  const int v = a.order[p], x0 = state_at(a, p, v);
  const int cv = a.C[x0];
  if (a.act_cur[x0] == 0) {
    if (lane == 0) a.Cn[x0] = cv;
    return;
  }
  if (lane == 0) a.act_cur[x0] = 0;
  const Pos beg = rfl_as(row_at<Pos>(a.row_ptr, v)), end = rfl_as(row_at<Pos>(a.row_ptr, v + 1));
  int key = -1;
  float val = 0.0f;
  if (!a.w && (long long)(end - beg) < (1ll << 24)) {
    if (a.fresh_hubs)
      det_unit_fresh<K>(a, x0, beg, end, lane, key, val);
    else
      det_unit<K>(a, buf, x0, beg, end, lane, key, val);
  } else if (a.fresh_hubs) {
    det_weighted<K, true>(a, buf, x0, beg, end, lane, key, val);
  } else {
    det_weighted<K, false>(a, buf, x0, beg, end, lane, key, val);
  }
  if constexpr (RS) {
    // double scan: the live slots' labels are re-weighted exactly, each
    // slot's entries added in CSR order by the slot's lane
    key = val > 0.0f ? key : -1;
    val = 0.0f;
    det_rescan<K>(a, x0, beg, end, lane, key, val);
  }
  // heaviest live slot, ties to the lowest label; keep when empty
  int bk = cv;
  float bv = 0.0f;
#pragma unroll
  for (int s = 0; s < K; ++s) {
    const float vs = rl_f(val, s);
    const int ks = rl(key, s);
    if (vs > bv || (vs == bv && vs > 0.0f && ks < bk)) {
      bk = ks;
      bv = vs;
    }
  }
  const int c = bk;
  const bool moved = c != cv && (!a.pickless || c < cv);
  if (lane == 0) a.Cn[x0] = moved ? c : cv;
  if (moved) {
    changed += 1;
    mark_row<16>(a, beg, end, lane);
  }
  scanned += (unsigned long long)(end - beg);
}

// LPA_SHARED_VARS: the same slot-per-lane sketch and CSR order as
// hub_vertex_det, with the lanes communicating through shared variables in
// LDS instead of wavefront votes (the shared-variable protocol of Algorithm
// 5 and Section 4.1): per entry, the lane whose slot holds the label
// announces its slot index; if none does, the lanes of empty slots take the
// lowest index with an LDS atomic minimum; if none is empty, the smallest
// slot value is found the same way (non-negative floats order like their
// bit patterns) and every slot is decremented.  Same results as
// hub_vertex_det; one entry at a time, with LDS round trips instead of
// register votes.
template <int K, class Pos>
__device__ void hub_vertex_det_sv(const MoveArgs &a, int p, unsigned long long &scanned,
                                  unsigned long long &changed) {
  __shared__ int sv[kBlock / kWave][2];  // per wavefront: [0] slot index, [1] minimum (bits)
  const int lane = threadIdx.x & (kWave - 1);
  int *has = sv[threadIdx.x / kWave];
  const int v = a.order[p], x0 = state_at(a, p, v);
  const int cv = a.C[x0];
  if (a.act_cur[x0] == 0) {
    if (lane == 0) a.Cn[x0] = cv;
    return;
  }
  if (lane == 0) a.act_cur[x0] = 0;
  const Pos beg = rfl_as(row_at<Pos>(a.row_ptr, v)), end = rfl_as(row_at<Pos>(a.row_ptr, v + 1));
  int key = -1;
  float val = 0.0f;
  auto first_free = [&]() {  // lowest empty slot, K if none
    if (lane == 0) has[0] = K;
    wave_lds_sync();
    if (lane < K && val == 0.0f) atomicMin(&has[0], lane);
    wave_lds_sync();
    const int s = rfl(has[0]);
    wave_lds_sync();
    return s;
  };
  hub_feed(a, x0, beg, end, lane, [&](int lab, float x, int cnt) {
    for (int t = 0; t < cnt; ++t) {
      const int c = rl(lab, t);
      const float w = rl_f(x, t);
      if (!(w > 0.0f)) continue;  // zero weight: no-op (self-loops, padding)
      if (lane == 0) has[0] = -1;
      wave_lds_sync();
      if (lane < K && key == c) has[0] = lane;  // keys are unique: one writer at most
      wave_lds_sync();
      const int hs = rfl(has[0]);
      wave_lds_sync();
      if (hs >= 0) {
        if (lane == hs) val += w;
        continue;
      }
      float r = w;
      int s = first_free();
      if (s == K) {  // every slot live: decrement by d = min(w, smallest slot)
        if (lane == 0) has[1] = __float_as_int(w);
        wave_lds_sync();
        if (lane < K) atomicMin(&has[1], __float_as_int(val));
        wave_lds_sync();
        const float m = __int_as_float(rfl(has[1]));
        wave_lds_sync();
        if (lane < K) val = val - m;
        r = w - m;
        s = r > 0.0f ? first_free() : K;
      }
      if (lane == s) {  // the (residue of the) pair takes the free slot
        key = c;
        val = r;
      }
    }
  });
  // heaviest live slot, ties to the lowest label; keep when empty
  int bk = cv;
  float bv = 0.0f;
#pragma unroll
  for (int s = 0; s < K; ++s) {
    const float vs = rl_f(val, s);
    const int ks = rl(key, s);
    if (vs > bv || (vs == bv && vs > 0.0f && ks < bk)) {
      bk = ks;
      bv = vs;
    }
  }
  const bool moved = bk != cv && (!a.pickless || bk < cv);
  if (lane == 0) a.Cn[x0] = moved ? bk : cv;
  if (moved) {
    changed += 1;
    mark_row<16>(a, beg, end, lane);
  }
  scanned += (unsigned long long)(end - beg);
}

// LPA_MODE_DET hub path for the vote of Algorithm 3: every lane holds the
// same candidate and takes the row's entries in CSR order (an entry of weight
// 0 changes nothing that a later entry or the choice could tell).
template <class Pos>
__device__ void hub_vertex_det_bm(const MoveArgs &a, int *buf, int p, unsigned long long &scanned,
                                  unsigned long long &changed) {
  const int lane = threadIdx.x & (kWave - 1);
  const int v = a.order[p], x0 = state_at(a, p, v);
  const int cv = a.C[x0];
  if (a.act_cur[x0] == 0) {
    if (lane == 0) a.Cn[x0] = cv;
    return;
  }
  if (lane == 0) a.act_cur[x0] = 0;
  const Pos beg = rfl_as(row_at<Pos>(a.row_ptr, v)), end = rfl_as(row_at<Pos>(a.row_ptr, v + 1));
  BmSketch S;
  S.clear();
  hub_stream(a, buf, x0, beg, end, lane, [&](int c, float w) { S.add(c, w); });
  const int c = S.max_key(cv);
  const bool moved = c != cv && (!a.pickless || c < cv);
  if (lane == 0) a.Cn[x0] = moved ? c : cv;
  if (moved) {
    changed += 1;
    mark_row<16>(a, beg, end, lane);
  }
  scanned += (unsigned long long)(end - beg);
}

// ---------------------------------------------------------------------------
// Lane units (both modes).  Unit u < n_seg is segment u - hub_pbase[h] of
// hub h = seg_hub[u] (async only); otherwise whole vertex order[n_hubs + u -
// n_seg].
// ---------------------------------------------------------------------------
// The stage keeps a step's columns for marking in the kernels whose registers hold
// them: not in the async one of k = 16 (31 spilled: 1000^2 grid with weights 564 to
// 434 us per solve, planted partitions of 10^6 vertices 1139 to 1035; R-MAT-22, bound
// by its long rows, 8.87 to 8.90 ms), nor in the unit-weight ones of k = 8 (9 to 19
// spilled: 2000^2 grid in place 1045 to 998 us, planted partitions of 10^5 vertices
// 366 to 317; 512 SBM graphs 52.8 to 52.6 ms).
template <int K, bool ASYNC, bool RS, class Pos, bool SV, bool UNIT>
constexpr bool kKeepCols =
    !RS && !SV && sizeof(Pos) == 4 && !(K == 16 && ASYNC) && !(K == 8 && UNIT);

template <int K, bool ASYNC, bool RS, class Pos, bool SV, bool UNIT>
__device__ __forceinline__ void lane_units(const MoveArgs &a, Stage<kStageT, Pos, UNIT> &st, int u,
                                           unsigned long long &scanned,
                                           unsigned long long &changed) {
  const int lane = threadIdx.x & (kWave - 1);
  int v = -1, sx = -1, len = 0, cv = 0, pslot = -1;  // sx: state index of v
  Pos beg = 0;
  bool whole = false, active = false;
  if (ASYNC && u < a.n_seg) {
    const int h = a.seg_hub[u];
    v = a.order[h];
    sx = state_at(a, h, v);
    active = a.hub_act[h] != 0;
    const int q = u - a.hub_pbase[h];
    const Pos rb = row_at<Pos>(a.row_ptr, v), re = row_at<Pos>(a.row_ptr, v + 1);
    beg = rb + (Pos)q * a.seg_len;
    len = (int)min((Pos)a.seg_len, (Pos)(re - beg));
    pslot = u;
  } else if (u < a.n_seg + a.n_lane - a.n_short) {
    const int p = a.n_hubs + (u - a.n_seg);
    v = a.order[p];
    sx = state_at(a, p, v);
    whole = true;
    active = a.act_cur[sx] != 0;
    cv = a.C[sx];
    if (active) {
      a.act_cur[sx] = 0;
      row_of<Pos>(a.row_ptr, v, beg, len);
    }
  }
  if (!active) len = 0;
  typename SketchOf<K>::type S;
  S.clear();
  constexpr bool KEEP = kKeepCols<K, ASYNC, RS, Pos, SV, UNIT>;
  int kept = staged_rows<KEEP>(a, st, lane, beg, len, sx,
                               [&](int lab, float x) { S.add(lab, x); });
  scanned += (unsigned long long)len;
  int c = cv;
  if constexpr (RS) {
    // second pass over whole rows only: hub segments are re-weighted after
    // their sketches are merged (k_hub_rescan)
    Rescan<K> R;
    R.from(S);
    kept = staged_rows<KEEP>(a, st, lane, beg, whole ? len : 0, sx,
                             [&](int lab, float x) { R.add(lab, x); });
    if (whole) c = R.best(cv);
  } else {
    if (whole) c = S.max_key(cv);
  }
  bool moved = false;
  if (pslot >= 0) {
    if (active) {  // partial sketch of one hub segment
      constexpr int P = slots_of(K);
#pragma unroll
      for (int s = 0; s < P; ++s) {
        a.part_key[(size_t)pslot * P + s] = S.key[s];
        a.part_val[(size_t)pslot * P + s] = S.val[s];
      }
    }
  } else if (whole) {
    moved = active && c != cv && (!a.pickless || c < cv);
    if (ASYNC) {
      if (moved) a.C[sx] = c;
    } else {
      a.Cn[sx] = moved ? c : cv;
    }
  }
  // every lane reaches here: the marking pass is wavefront-cooperative
  changed += (unsigned long long)__popcll(__ballot(moved));
  staged_mark(a, st, lane, beg, len, moved, kept);
}

// ---------------------------------------------------------------------------
// Short units (both modes, single scan): the last n_short lane vertices,
// whose rows have at most kShortDeg entries.  A wavefront takes kShortRows x
// 64 of them and every lane reads its own kShortRows rows, with no LDS stage:
// the rows' offsets, then all their column indices, weights and labels are
// loaded phase by phase before any sketch step.  Such rows cost little
// bandwidth but four dependent loads each (vertex id, row offsets, columns,
// labels), so a wavefront that waits for two rows per lane at a time keeps
// twice the loads of a staged lane unit in flight.  Each row's entries feed
// its sketch in CSR order with the same weights as in lane_units (the stage's
// padding entries after a row's end are no-ops there), so det results are
// the same.
// q0: index of the unit's first vertex among the short vertices.
// ---------------------------------------------------------------------------
template <int K, bool ASYNC, class Pos>
__device__ __forceinline__ void short_units(const MoveArgs &a, int q0, unsigned long long &scanned,
                                            unsigned long long &changed) {
  constexpr int R = kShortRows, D = kShortDeg;
  const int lane = threadIdx.x & (kWave - 1);
  const int p0 = a.n_hubs + a.n_lane - a.n_short;  // degree-order position of the first one
  int v[R], sx[R], cv[R], len[R];
  bool act[R];
  Pos beg[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int q = q0 + r * kWave + lane;
    v[r] = q < a.n_short ? a.order[p0 + q] : -1;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int q = q0 + r * kWave + lane;
    sx[r] = v[r] >= 0 ? state_at(a, p0 + q, v[r]) : -1;
    act[r] = sx[r] >= 0 && a.act_cur[sx[r]] != 0;
    cv[r] = sx[r] >= 0 ? a.C[sx[r]] : 0;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    beg[r] = 0;
    len[r] = 0;
    if (act[r]) {
      a.act_cur[sx[r]] = 0;
      row_of<Pos>(a.row_ptr, v[r], beg[r], len[r]);
    }
  }
  int c[R][D], lab[R][D];
  float x[R][D];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < D; ++j)
      c[r][j] = j < len[r] ? __builtin_nontemporal_load(a.col + (beg[r] + j)) : -1;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < D; ++j)
      x[r][j] = j < len[r] ? (a.w ? __builtin_nontemporal_load(a.w + (beg[r] + j)) : 1.0f) : 0.0f;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < D; ++j) lab[r][j] = c[r][j] >= 0 ? a.C[c[r][j]] : -1;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    typename SketchOf<K>::type S;
    S.clear();
#pragma unroll
    for (int j = 0; j < D; ++j)
      if (j < len[r]) S.add(lab[r][j], c[r][j] == sx[r] ? 0.0f : x[r][j]);
    const int ch = S.max_key(cv[r]);
    const bool moved = act[r] && ch != cv[r] && (!a.pickless || ch < cv[r]);
    if (sx[r] >= 0) {
      if (ASYNC) {
        if (moved) a.C[sx[r]] = ch;
      } else {
        a.Cn[sx[r]] = moved ? ch : cv[r];
      }
    }
    changed += (unsigned long long)__popcll(__ballot(moved));
    scanned += (unsigned long long)len[r];
    if (moved) {
#pragma unroll
      for (int j = 0; j < D; ++j)
        if (j < len[r]) mark(a, c[r][j]);
    }
  }
}

// ---------------------------------------------------------------------------
// Multi-graph launches.  Work items of all graphs of a launch are numbered
// consecutively; prefix[g] is the first item of graph g.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int find_graph(const int32_t *prefix_, int G, int item) {
  const kptr<int32_t> prefix = as_const(prefix_);
  int lo = 0, hi = G;  // prefix[lo] <= item < prefix[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (prefix[mid] <= item)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// Status of graph g for all but the stop test, through the scalar cache: the
// stop test, its only writer, runs when every workgroup has read it (finish_last)
// or in a launch of its own (k_finish).
__device__ __forceinline__ kptr<GraphStatus> status_of(const Launch &L, int g) {
  return as_const(as_const(L.d)[g].st);
}

// Descriptor of graph g, through the scalar cache (the table is written
// only by the host, before the launches).
using DescRef = const GraphDesc LPA_CONST &;
__device__ __forceinline__ DescRef desc_of(const Launch &L, int g) { return as_const(L.d)[g]; }

__device__ __forceinline__ MoveArgs make_args(DescRef d, int iter) {
  MoveArgs a;
  a.n = d.n;
  a.row_ptr.p32 = d.row_ptr.p32;
  a.row_ptr.p64 = d.row_ptr.p64;
  a.col = as_global(d.col);
  a.w = as_global(d.w);
  a.C = as_global(d.C[iter & 1]);
  a.Cn = as_global(d.C[(iter + 1) & 1]);
  a.act_cur = as_global(d.act[iter & 1]);
  a.act_next = as_global(d.act[(iter + 1) & 1]);
  a.order = as_global(d.order);
  a.ranked = d.ranked;
  a.n_hubs = d.n_hubs;
  a.n_lane = d.n_lane;
  a.n_short = d.n_short;
  a.seg_len = d.seg_len;
  a.n_seg = d.hub_shared ? 0 : d.n_seg;  // shared hubs: no segment units in k_move
  a.seg_hub = as_global(d.seg_hub);
  a.hub_pbase = as_global(d.hub_pbase);
  a.hub_act = as_global(d.hub_act);
  a.part_key = as_global(d.part_key);
  a.part_val = as_global(d.part_val);
  a.iter = iter;
  a.pickless = (d.rho > 0 && iter % d.rho == 0) ? 1 : 0;
  a.fresh_hubs = (iter == 0 && d.hub_rows_distinct && as_const(d.st)->fresh) ? 1 : 0;
  return a;
}

// Add a wavefront's per-graph totals to the graph's counters (all lanes
// call it together).
__device__ __forceinline__ void flush_counts(unsigned long long *dN, unsigned long long *sc,
                                             unsigned long long &scanned_lane,
                                             unsigned long long &scanned_w,
                                             unsigned long long &changed_w) {
#pragma unroll
  for (int off = kWave / 2; off >= 1; off >>= 1) scanned_lane += __shfl_xor(scanned_lane, off);
  if ((threadIdx.x & (kWave - 1)) == 0 && dN) {
    const unsigned long long t = scanned_lane + scanned_w;
    if (t) atomicAdd(sc, t);
    if (changed_w) atomicAdd(dN, changed_w);
  }
  scanned_lane = scanned_w = changed_w = 0;
}

// The last flush of a launch: every wavefront ends at once, and atomics on
// one counter serialise, so the workgroup's wavefronts combine their counts
// per counter (those that ended on the same graph) and one lane adds each
// sum.  Every thread of the workgroup must call it.
__device__ __forceinline__ void flush_last_counts(unsigned long long *dN, unsigned long long *sc,
                                                  unsigned long long &scanned_lane,
                                                  unsigned long long &scanned_w,
                                                  unsigned long long &changed_w, int wib) {
  constexpr int NW = kBlock / kWave;
  __shared__ unsigned long long *f_dN[NW], *f_sc[NW];
  __shared__ unsigned long long f_changed[NW], f_scanned[NW];
#pragma unroll
  for (int off = kWave / 2; off >= 1; off >>= 1) scanned_lane += __shfl_xor(scanned_lane, off);
  if ((threadIdx.x & (kWave - 1)) == 0) {
    f_dN[wib] = dN;
    f_sc[wib] = sc;
    f_changed[wib] = changed_w;
    f_scanned[wib] = scanned_lane + scanned_w;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 0; w < NW; ++w) {
      if (!f_dN[w]) continue;
      unsigned long long c = f_changed[w], t = f_scanned[w];
      for (int u = w + 1; u < NW; ++u)
        if (f_dN[u] == f_dN[w]) {  // the same graph and iteration: the same two counters
          c += f_changed[u];
          t += f_scanned[u];
          f_dN[u] = nullptr;
        }
      if (t) atomicAdd(f_sc[w], t);
      if (c) atomicAdd(f_dN[w], c);
    }
  }
  scanned_lane = scanned_w = changed_w = 0;
}

// Convergence test of Algorithm 1 for graph g of the launch: after iteration
// l, stop when l is not a pick-less iteration and dN / N < tol, or when
// max_iter iterations have run.
__device__ __forceinline__ void finish_graph(const Launch &L, int g) {
  const GraphDesc &d = L.d[g];
  GraphStatus *st = d.st;
  int iter = st->iter, done = st->done;
  int changed = 0;  // dN of the iteration this launch ran (0: none ran)
  if (!done) {
    const int l = iter;
    // the atomics of this launch's other workgroups lie behind the caches
    const unsigned long long dN =
        __hip_atomic_load(d.dN + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool pl = d.rho > 0 && l % d.rho == 0;
    const double frac = (double)dN / (double)d.n;
    changed = (int)dN;  // at most n < 2^31
    st->iter = iter = l + 1;
    if ((!pl && frac < d.tol) || l + 1 >= d.max_iter) {
      st->done = done = 1;
      atomicAdd(L.finished, 1);
    }
  }
  L.status_out[3 * g] = iter;
  L.status_out[3 * g + 1] = done;
  L.status_out[3 * g + 2] = changed;
}

// The stop test at the end of a move kernel that is its iteration's only one
// (Launch::fuse_finish): the workgroup that takes the last ticket runs it, when
// every other one has read the statuses and added its counts.  All it needs
// from the others are those atomics, so each workgroup waits for its own to
// complete before it takes its ticket; a fence would write its XCD's L2 back,
// once per workgroup (the 4096^2 grid's iterations: 0.39 against 0.34 ms).  A
// launch of its own takes 4 us and the gap before it, whatever the size; the
// tickets are atomics on one address, one per workgroup, in launches after
// convergence too.  So small launches run the test here (kFuseBlocks).  Every
// thread of the workgroup must call it, after its counts are flushed.
__device__ __forceinline__ void finish_last(const Launch &L) {
  __shared__ int last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();  // every wavefront's counts are added
  if (threadIdx.x == 0)
    last = __hip_atomic_fetch_add(L.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                   gridDim.x - 1
               ? 1
               : 0;
  __syncthreads();
  if (!last) return;
  for (int g = threadIdx.x; g < L.G; g += blockDim.x) finish_graph(L, g);
  if (threadIdx.x == 0) *L.ticket = 0;  // for the next launch
}

// Work item `local` of one graph: a hub, or 64 lane units, or 64 short units.
template <int K, bool ASYNC, bool RS, class Pos, bool HUBS, bool UNIT, bool SV>
__device__ __forceinline__ void move_item(const MoveArgs &a, Stage<kStageT, Pos, UNIT> &stage,
                                          int local, int lane, unsigned long long &scanned_lane,
                                          unsigned long long &scanned_w,
                                          unsigned long long &changed_w) {
  // det mode: one wavefront per hub first; async mode has none (its hubs
  // are cut into segments, which are lane units), and neither have det
  // launches over graphs without hubs, so their kernels carry no hub-chain
  // code
  int hub_items = 0;
  if constexpr (!ASYNC && HUBS) {
    hub_items = a.n_hubs;
    if (local < hub_items) {
      if constexpr (K == 0)
        hub_vertex_det_bm<Pos>(a, stage.lab, local, scanned_w, changed_w);
      else if constexpr (SV)
        hub_vertex_det_sv<K, Pos>(a, local, scanned_w, changed_w);
      else
        hub_vertex_det<K, RS, Pos>(a, stage.lab, local, scanned_w, changed_w);
      return;
    }
  }
  // lane units (hub segments first in async mode, then whole vertices),
  // then the short units
  const int lane_local = local - hub_items;
  const int units = a.n_seg + a.n_lane - a.n_short;
  const int unit_items = (int)(((unsigned)units + kWave - 1) / kWave);
  if constexpr (!RS) {
    if (lane_local >= unit_items) {
      short_units<K, ASYNC, Pos>(a, (lane_local - unit_items) * (kWave * kShortRows),
                                 scanned_lane, changed_w);
      return;
    }
  }
  lane_units<K, ASYNC, RS, Pos, SV, UNIT>(a, stage, lane_local * kWave + lane, scanned_lane,
                                          changed_w);
}

// HUBS: the launch has hubs that take one wavefront each (det mode).  UNIT: no
// graph of the launch has weights.
template <int K, bool ASYNC, bool RS, class Pos, bool HUBS, bool UNIT, bool SV = false>
__device__ __forceinline__ void move_body(const Launch &L) {
  __shared__ Stage<kStageT, Pos, UNIT> stage[kBlock / kWave];
  const int lane = threadIdx.x & (kWave - 1);
  const int wib = rfl(threadIdx.x / kWave);
  const int wave = rfl(blockIdx.x * (kBlock / kWave) + wib);
  const int nwaves = gridDim.x * (kBlock / kWave);
  unsigned long long scanned_lane = 0, changed_w = 0, scanned_w = 0;
  int cur = -1;
  unsigned long long *cdN = nullptr, *csc = nullptr;
  for (int item = wave; item < L.total_items; item += nwaves) {
    const int g = rfl(find_graph(L.prefix_items, L.G, item));
    const kptr<GraphStatus> st = status_of(L, g);
    if (st->done) continue;
    const int iter = st->iter;
    DescRef d = desc_of(L, g);
    if (g != cur) {
      flush_counts(cdN, csc, scanned_lane, scanned_w, changed_w);
      cur = g;
      cdN = d.dN + iter;
      csc = d.scanned + iter;
    }
    MoveArgs a = make_args(d, iter);
    if constexpr (UNIT) a.w = nullptr;
    move_item<K, ASYNC, RS, Pos, HUBS, UNIT, SV>(
        a, stage[wib], item - as_const(L.prefix_items)[g], lane, scanned_lane, scanned_w,
        changed_w);
  }
  flush_last_counts(cdN, csc, scanned_lane, scanned_w, changed_w, wib);
  if (L.fuse_finish) finish_last(L);
}

// CSR positions are int for graphs of int32 offsets and fewer than 2^30 entries
// and vertices (W = false), long long otherwise (W = true, which also reads
// int32 offsets): positions whose byte offsets fit 32 bits keep one register
// per load address (element).
template <bool W>
using PosOf = typename std::conditional<W, long long, int>::type;

// One iteration's label moves (single scan) ...  With 32-bit positions the
// kernel is held to 128 registers up to k = 16, which keeps four wavefronts
// per SIMD for the gathers (async k = 16 runs 8% faster on R-MAT-24 than with
// three), and to 168 for k = 32 in det mode (three).  So are the kernels of 64-bit positions up to k =
// 8: det, the 4096^2 grid with int64 offsets, 6.76 to 6.46 ms per solve; async with
// unit weights, which take 130 registers otherwise, a ring of 2^26 vertices 9.16 to
// 7.29 ms per 10 iterations and a 3000^2 grid 1.86 to 1.71, though R-MAT-22, whose
// long rows gain less from the fourth wavefront than the spills cost, goes from
// 8.6 to 9.0.  The other instantiations are left to the compiler.
template <int K, bool ASYNC, bool W>
constexpr int kMoveWaves = W                     ? (K <= 8 ? 4 : 1)
                           : (K <= 16)           ? 4
                           : (K == 32 && !ASYNC) ? 3
                                                 : 1;

// No more than four for unit weights at k = 8: the det kernel would take 96
// registers and five, which the 4096^2 grid likes (6.11 to 5.80 ms per solve), but not
// batches of graphs (512 SBM graphs 52.6 to 54.4 ms).
template <int K, bool W, bool UNIT>
constexpr int kMoveMostWaves = !W && UNIT && K == 8 ? 4 : 8;

template <int K, bool ASYNC, bool W, bool HUBS, bool UNIT>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(kMoveWaves<K, ASYNC, W>, kMoveMostWaves<K, W, UNIT>)))
void k_move(Launch L) {
  move_body<K, ASYNC, false, PosOf<W>, HUBS, UNIT>(L);
}

// ... and with the double scan (LPA_RESCAN; sketch rule only).  The det kernels are
// held to four wavefronts where the hub chains' registers would leave three
// (135 at k = 8), k = 8, us per solve: 1000^2 grid 1366 to 1113, with weights 859 to
// 723, planted partitions of 10^6 vertices 2147 to 1827, R-MAT-19 12,090 to 11,950.
template <int K, bool ASYNC, bool W>
constexpr int kRescanWaves = !ASYNC && (K <= 8 || (K == 16 && !W)) ? 4 : 1;

template <int K, bool ASYNC, bool W>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(kRescanWaves<K, ASYNC, W>))) void k_move_rescan(Launch L) {
  move_body<K, ASYNC, true, PosOf<W>, !ASYNC, false>(L);
}

// ... and with shared variables instead of votes in the hub path
// (LPA_SHARED_VARS; LPA_MODE_DET, sketch rule, single scan).
template <int K, bool W>
__global__ __launch_bounds__(kBlock) void k_move_sv(Launch L) {
  move_body<K, false, false, PosOf<W>, true, false, true>(L);
}

// ---------------------------------------------------------------------------
// LPA_MODE_ASYNC hub epilogue.
// ---------------------------------------------------------------------------
// Snapshot and clear the unprocessed flags of the hubs before the move
// kernel, so that marks made while their segments are scanned are kept for
// the next iteration.
__global__ void k_hub_snapshot(Launch L) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < L.total_hubs;
       t += gridDim.x * blockDim.x) {
    const int g = find_graph(L.prefix_hubs, L.G, t);
    const GraphDesc &d = L.d[g];
    if (d.st->done) continue;
    const int h = t - L.prefix_hubs[g];
    const int x = d.ranked ? h : d.order[h];
    d.hub_act[h] = d.act[0][x];
    d.act[0][x] = 0;
  }
}

// A hub's decision is recorded in hub_act (its flag snapshot is no longer
// needed once the hub is decided): 1 if its label moved.  k_hub_mark then
// flags the neighbours of moved hubs, one wavefront per hub segment.
__device__ __forceinline__ void record_moved_hub(const MoveArgs &a, int h, bool moved) {
  if (h < a.n_hubs) a.hub_act[h] = moved ? 1 : 0;
}

// Flat feed for k = 8 and 16 with the sketch spread over a hub's four-lane
// group: lane q of the group holds slots P q .. P q + P - 1 (P = k / 4), and
// the group's lanes exchange values with quad permutes (DPP), so one sketch
// update is a few instructions per lane instead of a pass over all k slots.
// Same arithmetic and the same slot rules as LaneSketch<k>: a matching key
// adds the weight; otherwise every slot drops by d = min(w, smallest slot)
// and a positive residue takes the lowest free slot; heaviest slot wins,
// ties to the lowest label.
template <int CTRL>
__device__ __forceinline__ int quad_dpp(int x) {
  return dpp<CTRL>(x);
}
template <int CTRL>
__device__ __forceinline__ float quad_dpp_f(float x) {
  return dpp_f<CTRL>(x);
}
constexpr int kQuadX1 = 0xB1;  // lanes (1, 0, 3, 2) of the quad
constexpr int kQuadX2 = 0x4E;  // lanes (2, 3, 0, 1)

template <int P>
struct QuadSketch {
  int k[P];
  float v[P];
  int s0;  // index of this lane's first slot

  __device__ __forceinline__ void clear(int sub) {
#pragma unroll
    for (int q = 0; q < P; ++q) {
      k[q] = -1;
      v[q] = 0.0f;
    }
    s0 = P * sub;
  }

  __device__ __forceinline__ void add(int c, float w) {
    bool m = false;
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const bool mq = k[q] == c;
      v[q] = mq ? v[q] + w : v[q];
      m = m || mq;
    }
    int hit = m ? 1 : 0;
    hit |= quad_dpp<kQuadX1>(hit);
    hit |= quad_dpp<kQuadX2>(hit);
    if (!hit) {
      float d = w;
#pragma unroll
      for (int q = 0; q < P; ++q) d = fminf(d, v[q]);
      d = fminf(d, quad_dpp_f<kQuadX1>(d));
      d = fminf(d, quad_dpp_f<kQuadX2>(d));
#pragma unroll
      for (int q = 0; q < P; ++q) v[q] = v[q] - d;
      const float r = w - d;
      if (r > 0.0f) {
        int f = 4 * P;  // lowest free slot of the group
#pragma unroll
        for (int q = P - 1; q >= 0; --q) f = v[q] == 0.0f ? s0 + q : f;
        f = min(f, quad_dpp<kQuadX1>(f));
        f = min(f, quad_dpp<kQuadX2>(f));
#pragma unroll
        for (int q = 0; q < P; ++q) {
          if (f == s0 + q) {
            k[q] = c;
            v[q] = r;
          }
        }
      }
    }
  }

  __device__ __forceinline__ int max_key(int keep) const {
    int bk = keep;
    float bv = 0.0f;
#pragma unroll
    for (int q = 0; q < P; ++q) {
      if (v[q] > bv || (v[q] == bv && v[q] > 0.0f && k[q] < bk)) {
        bk = k[q];
        bv = v[q];
      }
    }
    int ok = quad_dpp<kQuadX1>(bk);
    float ov = quad_dpp_f<kQuadX1>(bv);
    if (ov > bv || (ov == bv && ov > 0.0f && ok < bk)) {
      bk = ok;
      bv = ov;
    }
    ok = quad_dpp<kQuadX2>(bk);
    ov = quad_dpp_f<kQuadX2>(bv);
    if (ov > bv || (ov == bv && ov > 0.0f && ok < bk)) {
      bk = ok;
      bv = ov;
    }
    return bk;
  }
};

// Feed the partial held by lane T of the quad (its live slots in slot order)
// into Q; a slot of weight 0 would change nothing and is skipped.
template <int T, int K>
__device__ __forceinline__ void quad_feed_partial(QuadSketch<K / 4> &Q, const int *ck,
                                                  const float *cw) {
#pragma unroll
  for (int s = 0; s < K; ++s) {
    const int kk = quad_dpp<T * 0x55>(ck[s]);
    const float vv = quad_dpp_f<T * 0x55>(cw[s]);
    if (vv > 0.0f) Q.add(kk, vv);
  }
}

// Flat feed of one hub's np <= 64 partials (k = 8 or 16) by its four-lane
// group, segment order; returns the merged sketch's heaviest label (keep cv).
template <int K>
__device__ __forceinline__ int hub_flat_merge(const MoveArgs &a, int p0, int np, int sub, int cv) {
  QuadSketch<K / 4> Q;
  Q.clear(sub);
  int ck[K], nk[K];
  float cw[K], nv[K];
#pragma unroll
  for (int s = 0; s < K; ++s) {
    ck[s] = nk[s] = -1;
    cw[s] = nv[s] = 0.0f;
  }
  if (sub < np) {
#pragma unroll
    for (int s = 0; s < K; ++s) {
      ck[s] = a.part_key[(size_t)(p0 + sub) * K + s];
      cw[s] = a.part_val[(size_t)(p0 + sub) * K + s];
    }
  }
  for (int b = 0; b < np; b += kHubLanes) {
    if (b + kHubLanes + sub < np) {
#pragma unroll
      for (int s = 0; s < K; ++s) {
        nk[s] = a.part_key[(size_t)(p0 + b + kHubLanes + sub) * K + s];
        nv[s] = a.part_val[(size_t)(p0 + b + kHubLanes + sub) * K + s];
      }
    }
    const int nt = min(kHubLanes, np - b);
    quad_feed_partial<0, K>(Q, ck, cw);
    if (nt > 1) quad_feed_partial<1, K>(Q, ck, cw);
    if (nt > 2) quad_feed_partial<2, K>(Q, ck, cw);
    if (nt > 3) quad_feed_partial<3, K>(Q, ck, cw);
#pragma unroll
    for (int s = 0; s < K; ++s) {
      ck[s] = nk[s];
      cw[s] = nv[s];
    }
  }
  return Q.max_key(cv);
}

// Hub taken by lane group `grp` of merge item `it` of a graph with `ni`
// merge items: hubs are dealt out across the items (group j of item i takes
// hub j * ni + i).  The largest hubs sit next to each other in the degree
// order; dealt out, each lands in a wavefront of its own instead of one
// wavefront merging them one after another.
__device__ __forceinline__ int merge_hub(int it, int grp, int ni) { return grp * ni + it; }

__device__ __forceinline__ int merge_items(const Launch &L, int g) {
  return as_const(L.prefix_merge)[g + 1] - as_const(L.prefix_merge)[g];
}

// Merge the partial sketches of every active hub (Section 4.3).  A wavefront
// takes kMergeHubs hubs of one graph (merge_hub), kHubLanes lanes each.  For
// a hub with at most 64 partials the partials are fed one by one, in segment
// order, into a single sketch, which every lane of the group computes alike: lane
// t of the group loads partials t, t + kHubLanes, ... (the next one's loads
// in flight) and hands each over by a lane exchange.  Feeding every partial
// into one sketch follows the paper's merge into the first group's sketch;
// combining already merged sketches pairwise instead measured lower
// modularity.  Larger hubs are merged by the whole wavefront (lane l merges
// partials l, l + 64, ..., then a pairwise exchange across lanes).
// RS = false: the hub takes the merged sketch's heaviest label.  RS = true
// (double scan): the merged sketch's live labels are stored as the hub's
// candidates for k_hub_rescan / k_hub_pick.
template <int K, bool RS>
__device__ __forceinline__ void hub_merge_body(const Launch &L) {
  const int lane = threadIdx.x & (kWave - 1);
  const int sub = lane & (kHubLanes - 1);
  const int wave = rfl((blockIdx.x * kBlock + threadIdx.x) / kWave);
  const int nwaves = gridDim.x * (kBlock / kWave);
  unsigned long long changed_w = 0, zero_lane = 0, zero_w = 0;
  int cur = -1;
  unsigned long long *cdN = nullptr;
  using SK = typename SketchOf<K>::type;
  constexpr int P = slots_of(K);
  for (int item = wave; item < L.total_merge; item += nwaves) {
    const int g = rfl(find_graph(L.prefix_merge, L.G, item));
    const kptr<GraphStatus> st = status_of(L, g);
    if (st->done) continue;
    const int iter = st->iter;
    DescRef gd = desc_of(L, g);
    if (g != cur) {
      flush_counts(cdN, cdN, zero_lane, zero_w, changed_w);
      cur = g;
      cdN = gd.dN + iter;
    }
    const MoveArgs a = make_args(gd, iter);
    const int it = item - as_const(L.prefix_merge)[g], ni = rfl(merge_items(L, g));
    const int h = merge_hub(it, lane / kHubLanes, ni);
    int x = -1, p0 = 0, np = 0, cv = 0;  // x: the hub's state index
    bool active = false;
    if (h < a.n_hubs) {
      x = state_at(a, h, a.order[h]);
      active = a.hub_act[h] != 0;
      p0 = a.hub_pbase[h];
      np = a.hub_pbase[h + 1] - p0;
      cv = a.C[x];
    }
    int c = cv;
    const bool small = active && np <= kWave;
    SK S;
    S.clear();
    if constexpr ((K == 8 || K == 16) && !RS) {
      if (small) c = hub_flat_merge<K>(a, p0, np, sub, cv);
    } else if (small) {  // np is the same on every lane of the group
      const int gbase = lane & ~(kHubLanes - 1);
      int ck[P], nk[P];
      float cw[P], nv[P];
#pragma unroll
      for (int s = 0; s < P; ++s) {
        ck[s] = -1;
        cw[s] = 0.0f;
        nk[s] = -1;
        nv[s] = 0.0f;
      }
      if (sub < np) {
#pragma unroll
        for (int s = 0; s < P; ++s) {
          ck[s] = a.part_key[(size_t)(p0 + sub) * P + s];
          cw[s] = a.part_val[(size_t)(p0 + sub) * P + s];
        }
      }
      for (int b = 0; b < np; b += kHubLanes) {
        if (b + kHubLanes + sub < np) {
#pragma unroll
          for (int s = 0; s < P; ++s) {
            nk[s] = a.part_key[(size_t)(p0 + b + kHubLanes + sub) * P + s];
            nv[s] = a.part_val[(size_t)(p0 + b + kHubLanes + sub) * P + s];
          }
        }
        const int nt = min(kHubLanes, np - b);
        for (int t = 0; t < nt; ++t) {
          int pk[P];
          float pv[P];
#pragma unroll
          for (int s = 0; s < P; ++s) {
            pk[s] = __shfl(ck[s], gbase + t);
            pv[s] = __shfl(cw[s], gbase + t);
          }
          S.merge_from(pk, pv);
        }
#pragma unroll
        for (int s = 0; s < P; ++s) {
          ck[s] = nk[s];
          cw[s] = nv[s];
        }
      }
    }
    if (small) {
      if constexpr (RS) {
        if (sub == 0) {
#pragma unroll
          for (int s = 0; s < P; ++s)
            gd.hub_cand[(size_t)h * P + s] = S.val[s] > 0.0f ? S.key[s] : -1;
        }
      } else if constexpr (K != 8 && K != 16) {
        c = S.max_key(cv);
      }
    }
    unsigned long long big = __ballot(active && !small && sub == 0);
    while (big) {
      const int src = __ffsll((long long)big) - 1;
      big &= big - 1;
      const int bp0 = __shfl(p0, src), bnp = __shfl(np, src), bcv = __shfl(cv, src);
      SK B;
      B.clear();
      for (int p = bp0 + lane; p < bp0 + bnp; p += kWave) {
        int pk[P];
        float pv[P];
#pragma unroll
        for (int s = 0; s < P; ++s) {
          pk[s] = a.part_key[(size_t)p * P + s];
          pv[s] = a.part_val[(size_t)p * P + s];
        }
        B.merge_from(pk, pv);
      }
#pragma unroll 1
      for (int off = kWave / 2; off >= 1; off >>= 1) {
        int pk[P];
        float pv[P];
#pragma unroll
        for (int s = 0; s < P; ++s) {  // snapshot the partner before merging
          pk[s] = __shfl_xor(B.key[s], off);
          pv[s] = __shfl_xor(B.val[s], off);
        }
        B.merge_from(pk, pv);
      }
      if constexpr (RS) {
        const int bh = merge_hub(it, src / kHubLanes, ni);
        if (lane == 0) {
#pragma unroll
          for (int s = 0; s < P; ++s)
            gd.hub_cand[(size_t)bh * P + s] = B.val[s] > 0.0f ? B.key[s] : -1;
        }
      } else {
        const int bc = rfl(B.max_key(bcv));
        if (lane / kHubLanes == src / kHubLanes) c = bc;
      }
    }
    if constexpr (!RS) {
      const bool moved = active && c != cv && (!a.pickless || c < cv);
      if (moved && sub == 0) a.C[x] = c;
      changed_w += (unsigned long long)__popcll(__ballot(moved && sub == 0));
      if (sub == 0) record_moved_hub(a, h, moved);
    }
  }
  flush_counts(cdN, cdN, zero_lane, zero_w, changed_w);
}

template <int K>
__global__ __launch_bounds__(kBlock) void k_hub_merge(Launch L) {
  hub_merge_body<K, false>(L);
}

// Double scan, hub candidates: merge the partial sketches into candidates.
template <int K>
__global__ __launch_bounds__(kBlock) void k_hub_cand(Launch L) {
  hub_merge_body<K, true>(L);
}

// Double scan, hub re-weighting: one wavefront per hub segment sums the
// exact weight of each of its hub's candidates over the segment's entries
// (any order: LPA_MODE_ASYNC only) into the segment's partial values.
template <int K>
__global__ __launch_bounds__(kBlock) void k_hub_rescan(Launch L) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = rfl((blockIdx.x * kBlock + threadIdx.x) / kWave);
  const int nwaves = gridDim.x * (kBlock / kWave);
  for (int item = wave; item < L.total_segs; item += nwaves) {
    const int g = rfl(find_graph(L.prefix_segs, L.G, item));
    const kptr<GraphStatus> st = status_of(L, g);
    if (st->done) continue;
    DescRef gd = desc_of(L, g);
    const MoveArgs a = make_args(gd, st->iter);
    const int u = item - as_const(L.prefix_segs)[g];
    const int h = a.seg_hub[u];
    if (a.hub_act[h] == 0) continue;
    const int v = a.order[h], self = state_at(a, h, v);
    const int q = u - a.hub_pbase[h];
    const long long rb = a.row_ptr[v], re = a.row_ptr[v + 1];
    const long long beg = rb + (long long)q * a.seg_len, end = min(beg + a.seg_len, re);
    int cand[K];
    float acc[K];
#pragma unroll
    for (int s = 0; s < K; ++s) {
      cand[s] = gd.hub_cand[(size_t)h * K + s];
      acc[s] = 0.0f;
    }
    constexpr int U = 4;
    for (long long e0 = beg; e0 < end; e0 += U * kWave) {
      int lab[U];
      float x[U];
#pragma unroll
      for (int t = 0; t < U; ++t) {
        const long long e = e0 + t * kWave + lane;
        lab[t] = -1;
        x[t] = 0.0f;
        if (e < end) {
          const int j = __builtin_nontemporal_load(a.col + e);
          x[t] = (j == self) ? 0.0f : (a.w ? __builtin_nontemporal_load(a.w + e) : 1.0f);
          lab[t] = a.C[j];
        }
      }
#pragma unroll
      for (int t = 0; t < U; ++t)
#pragma unroll
        for (int s = 0; s < K; ++s)
          acc[s] = (lab[t] >= 0 && lab[t] == cand[s]) ? acc[s] + x[t] : acc[s];
    }
#pragma unroll
    for (int s = 0; s < K; ++s) {
#pragma unroll
      for (int off = kWave / 2; off >= 1; off >>= 1) acc[s] += __shfl_xor(acc[s], off);
      if (lane == 0) a.part_val[(size_t)u * K + s] = acc[s];
    }
  }
}

// Double scan, hub decision: add up the segments' candidate weights, take
// the heaviest candidate (ties to the lowest label), update the label and
// flag the neighbours.  Same hub-to-lane layout as k_hub_merge (merge_hub).
template <int K>
__global__ __launch_bounds__(kBlock) void k_hub_pick(Launch L) {
  const int lane = threadIdx.x & (kWave - 1);
  const int sub = lane & (kHubLanes - 1);
  const int wave = rfl((blockIdx.x * kBlock + threadIdx.x) / kWave);
  const int nwaves = gridDim.x * (kBlock / kWave);
  unsigned long long changed_w = 0, zero_lane = 0, zero_w = 0;
  int cur = -1;
  unsigned long long *cdN = nullptr;
  for (int item = wave; item < L.total_merge; item += nwaves) {
    const int g = rfl(find_graph(L.prefix_merge, L.G, item));
    const kptr<GraphStatus> st = status_of(L, g);
    if (st->done) continue;
    const int iter = st->iter;
    DescRef gd = desc_of(L, g);
    if (g != cur) {
      flush_counts(cdN, cdN, zero_lane, zero_w, changed_w);
      cur = g;
      cdN = gd.dN + iter;
    }
    const MoveArgs a = make_args(gd, iter);
    const int it = item - as_const(L.prefix_merge)[g], ni = rfl(merge_items(L, g));
    const int h = merge_hub(it, lane / kHubLanes, ni);
    int x = -1, p0 = 0, np = 0, cv = 0;  // x: the hub's state index
    bool active = false;
    if (h < a.n_hubs) {
      x = state_at(a, h, a.order[h]);
      active = a.hub_act[h] != 0;
      p0 = a.hub_pbase[h];
      np = a.hub_pbase[h + 1] - p0;
      cv = a.C[x];
    }
    float tot[K];
#pragma unroll
    for (int s = 0; s < K; ++s) tot[s] = 0.0f;
    const bool small = active && np <= kWave;
    if (small)
      for (int p = p0 + sub; p < p0 + np; p += kHubLanes)
#pragma unroll
        for (int s = 0; s < K; ++s) tot[s] += a.part_val[(size_t)p * K + s];
#pragma unroll
    for (int s = 0; s < K; ++s)  // add up each lane group's sums
#pragma unroll
      for (int off = 1; off < kHubLanes; off <<= 1) tot[s] += __shfl_xor(tot[s], off);
    unsigned long long big = __ballot(active && !small && sub == 0);
    while (big) {
      const int src = __ffsll((long long)big) - 1;
      big &= big - 1;
      const int bp0 = __shfl(p0, src), bnp = __shfl(np, src);
      float t[K];
#pragma unroll
      for (int s = 0; s < K; ++s) t[s] = 0.0f;
      for (int p = bp0 + lane; p < bp0 + bnp; p += kWave)
#pragma unroll
        for (int s = 0; s < K; ++s) t[s] += a.part_val[(size_t)p * K + s];
#pragma unroll
      for (int s = 0; s < K; ++s) {
#pragma unroll
        for (int off = kWave / 2; off >= 1; off >>= 1) t[s] += __shfl_xor(t[s], off);
        tot[s] = (lane / kHubLanes == src / kHubLanes) ? t[s] : tot[s];
      }
    }
    int c = cv;
    if (active) {
      float bv = 0.0f;
#pragma unroll
      for (int s = 0; s < K; ++s) {
        const int ks = gd.hub_cand[(size_t)h * K + s];
        const bool better = ks >= 0 && (tot[s] > bv || (tot[s] == bv && tot[s] > 0.0f && ks < c));
        c = better ? ks : c;
        bv = better ? tot[s] : bv;
      }
    }
    const bool moved = active && c != cv && (!a.pickless || c < cv);
    if (moved && sub == 0) a.C[x] = c;
    changed_w += (unsigned long long)__popcll(__ballot(moved && sub == 0));
    if (sub == 0) record_moved_hub(a, h, moved);
  }
  flush_counts(cdN, cdN, zero_lane, zero_w, changed_w);
}

// Flag the neighbours of every hub that moved in this iteration: one
// wavefront per hub segment, coalesced column loads.
__global__ __launch_bounds__(kBlock) void k_hub_mark(Launch L) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = rfl((blockIdx.x * kBlock + threadIdx.x) / kWave);
  const int nwaves = gridDim.x * (kBlock / kWave);
  for (int item = wave; item < L.total_segs; item += nwaves) {
    const int g = rfl(find_graph(L.prefix_segs, L.G, item));
    const kptr<GraphStatus> st = status_of(L, g);
    if (st->done) continue;
    const MoveArgs a = make_args(desc_of(L, g), st->iter);
    const int u = item - as_const(L.prefix_segs)[g];
    const int h = a.seg_hub[u];
    if (a.hub_act[h] == 0) continue;
    const int v = a.order[h];
    const int q = u - a.hub_pbase[h];
    const long long rb = a.row_ptr[v], re = a.row_ptr[v + 1];
    const long long beg = rb + (long long)q * a.seg_len, end = min(beg + a.seg_len, re);
    mark_row<16>(a, beg, end, lane);
  }
}

// LPA_HUB_SHARED (ablation of Section 4.3's partial sketches): one workgroup
// per active hub feeds all of the hub's entries into a single sketch in
// LDS that its 256 threads update concurrently with LDS atomics, in the
// manner of the shared mode of Algorithm 5: add to a matching slot, else
// claim a free slot by compare-and-swap (retry if another thread took it),
// else subtract from every slot (by d = min(w, smallest slot), then place
// the residue).  Updates race, so the sketch is approximate; every retry
// loop is bounded.  The hub then takes the heaviest slot.
template <int K>
__device__ __forceinline__ void shared_add(int *key, float *val, int c, float w) {
  for (int attempt = 0; attempt < 2 * K + 2 && w > 0.0f; ++attempt) {
    int hit = -1, freeslot = -1;
    float seen = 0.0f, m = w;
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const float vs = __hip_atomic_load(&val[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      const int ks = __hip_atomic_load(&key[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (ks == c && vs > 0.0f && hit < 0) hit = s;
      if (!(vs > 0.0f) && freeslot < 0) {
        freeslot = s;
        seen = vs;
      }
      m = fminf(m, vs);
    }
    if (hit >= 0) {
      atomicAdd(&val[hit], w);
      return;
    }
    if (freeslot >= 0) {
      const unsigned want = __float_as_uint(seen);
      if (atomicCAS((unsigned *)&val[freeslot], want, __float_as_uint(w)) == want) {
        __hip_atomic_store(&key[freeslot], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return;
      }
      continue;  // another thread took the slot: look again
    }
    if (m > 0.0f) {
#pragma unroll
      for (int s = 0; s < K; ++s) atomicAdd(&val[s], -m);
    }
    w -= m;  // the residue, if any, looks for a slot that just emptied
  }
}

template <int K>
__global__ __launch_bounds__(256) void k_hub_shared(Launch L) {
  __shared__ int key[K];
  __shared__ float val[K];
  for (int item = blockIdx.x; item < L.total_hubs; item += gridDim.x) {
    const int g = find_graph(L.prefix_hubs, L.G, item);
    const kptr<GraphStatus> st = status_of(L, g);
    if (st->done) continue;
    DescRef gd = desc_of(L, g);
    const MoveArgs a = make_args(gd, st->iter);
    const int h = item - as_const(L.prefix_hubs)[g];
    if (a.hub_act[h] == 0) continue;
    const int v = a.order[h], self = state_at(a, h, v);
    if (threadIdx.x < K) {
      key[threadIdx.x] = -1;
      val[threadIdx.x] = 0.0f;
    }
    __syncthreads();
    const long long rb = a.row_ptr[v], re = a.row_ptr[v + 1];
    for (long long e = rb + threadIdx.x; e < re; e += blockDim.x) {
      const int j = __builtin_nontemporal_load(a.col + e);
      if (j == self) continue;
      const float w = a.w ? __builtin_nontemporal_load(a.w + e) : 1.0f;
      shared_add<K>(key, val, a.C[j], w);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const int cv = a.C[self];
      int c = cv;
      float bv = 0.0f;
      for (int s = 0; s < K; ++s)
        if (val[s] > bv || (val[s] == bv && val[s] > 0.0f && key[s] < c)) {
          c = key[s];
          bv = val[s];
        }
      const bool moved = c != cv && (!a.pickless || c < cv);
      if (moved) {
        a.C[self] = c;
        atomicAdd(gd.dN + st->iter, 1ull);
      }
      a.hub_act[h] = moved ? 1 : 0;  // k_hub_mark flags the neighbours
      atomicAdd(gd.scanned + st->iter, (unsigned long long)(re - rb));
    }
    __syncthreads();
  }
}

__global__ void k_finish(Launch L) {
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < L.G; g += gridDim.x * blockDim.x)
    finish_graph(L, g);
}

// All remaining iterations of small graphs in one launch, one workgroup per
// graph (det mode, single scan, no hubs, 32-bit positions; the host's solve_in_one
// says which).  A small graph's iteration is one chain of dependent loads and,
// as a launch of its own, its start and its stop test's atomics; here the arrays
// stay in the compute unit's cache, a barrier parts the iterations and the counts
// are summed in LDS.  What is left is the sketch updates of four wavefronts on
// each SIMD: 11 us per iteration of 16 items (1,009 vertices, unit weights, k = 8:
// 291 to 233 us per solve; 200 vertices: 191 to 118).  Every wavefront of a workgroup is
// on one compute unit and reads and writes through its one vector cache, so a
// barrier (which waits for the stores) is all the ordering that the next
// iteration's reads need; what scalar loads read (descriptors) is not written.
template <int K, bool UNIT>
__global__ __launch_bounds__(kSolveBlock) void k_solve(Launch L, int iters) {
  constexpr int NW = kSolveBlock / kWave;
  __shared__ Stage<kStageT, int, UNIT> stage[NW];
  __shared__ unsigned long long s_changed[2][NW], s_scanned[2][NW];
  const int lane = threadIdx.x & (kWave - 1);
  const int wib = rfl(threadIdx.x / kWave);
  for (int g = blockIdx.x; g < L.G; g += gridDim.x) {
    DescRef d = desc_of(L, g);
    GraphStatus *st = d.st;
    const int first = rfl(st->iter), was_done = rfl(st->done);
    __syncthreads();  // read by all, before thread 0 writes it
    int iter = first, done = was_done, changed = 0;
    for (int i = 0; i < iters && !done; ++i) {
      unsigned long long scanned_lane = 0, changed_w = 0, scanned_w = 0;
      MoveArgs a = make_args(d, iter);
      if constexpr (UNIT) a.w = nullptr;
      for (int item = wib; item < d.items; item += NW)
        move_item<K, false, false, int, false, UNIT, false>(a, stage[wib], item, lane,
                                                            scanned_lane, scanned_w, changed_w);
#pragma unroll
      for (int off = kWave / 2; off >= 1; off >>= 1) scanned_lane += __shfl_xor(scanned_lane, off);
      // two sets of sums, used in turn: one barrier per iteration
      if (lane == 0) {
        s_changed[i & 1][wib] = changed_w;
        s_scanned[i & 1][wib] = scanned_lane + scanned_w;
      }
      __syncthreads();
      unsigned long long c = 0, t = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        c += s_changed[i & 1][w];
        t += s_scanned[i & 1][w];
      }
      changed = rfl((int)c);  // at most n < 2^31
      if (threadIdx.x == 0) {
        d.dN[iter] = c;
        d.scanned[iter] = t;
      }
      // the stop test of finish_graph
      const bool pl = d.rho > 0 && iter % d.rho == 0;
      const double frac = (double)changed / (double)d.n;
      ++iter;
      done = rfl((!pl && frac < d.tol) || iter >= d.max_iter ? 1 : 0);
    }
    if (threadIdx.x == 0) {
      st->iter = iter;
      st->done = done;
      if (done && !was_done) atomicAdd(L.finished, 1);
      L.status_out[3 * g] = iter;
      L.status_out[3 * g + 1] = done;
      L.status_out[3 * g + 2] = changed;
    }
  }
}

template <bool UNIT>
static hipError_t launch_solve_u(int k, const Launch &L, int iters, hipStream_t s) {
  const dim3 grid(L.G), block(kSolveBlock);
  switch (k) {
    case 1: hipLaunchKernelGGL((k_solve<1, UNIT>), grid, block, 0, s, L, iters); break;
    case 2: hipLaunchKernelGGL((k_solve<2, UNIT>), grid, block, 0, s, L, iters); break;
    case 4: hipLaunchKernelGGL((k_solve<4, UNIT>), grid, block, 0, s, L, iters); break;
    case 8: hipLaunchKernelGGL((k_solve<8, UNIT>), grid, block, 0, s, L, iters); break;
    case 16: hipLaunchKernelGGL((k_solve<16, false>), grid, block, 0, s, L, iters); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_solve(int k, const Launch &L, int iters, hipStream_t s) {
  return L.unit ? launch_solve_u<true>(k, L, iters, s) : launch_solve_u<false>(k, L, iters, s);
}

// The single-scan move kernel of a launch (see move_body): its instances leave
// out what no graph of the launch needs.  With 16 or more slots the registers do
// not hold the wider loads of the unit-weight staging (k = 16 spilled 33 at
// four wavefronts per SIMD), so those take the general instance.
template <int K, bool ASYNC, bool W>
static auto move_kernel(bool hubs, bool unit) -> void (*)(Launch) {
  constexpr bool U = K <= 8;
  if (!ASYNC && hubs)
    return unit && U ? k_move<K, ASYNC, W, !ASYNC, U> : k_move<K, ASYNC, W, !ASYNC, false>;
  return unit && U ? k_move<K, ASYNC, W, false, U> : k_move<K, ASYNC, W, false, false>;
}

// The move kernel runs the stop test itself (finish_last) in launches of at most
// this many workgroups and graphs.  Solves with a launch of its own / in the move
// kernel, k = 8, us: planted partitions with weights, 78 workgroups (20,000
// vertices) 334 / 327, 156 357 / 375, 312 407 / 424, 1024 (500,000) 904 / 1001;
// grids with weights, 78 194 / 186, 176 203 / 203, 312 221 / 233, 1024 (1000^2)
// 428 / 524; unit-weight grids, which run all their iterations, 78 245 / 225, 312
// 311 / 290, 1024 630 / 634.  Batches of 100-vertex graphs: 128 graphs 333 / 312,
// 256 364 / 366, 512 465 / 504 (the last workgroup tests all graphs).
constexpr int kFuseBlocks = 128;
constexpr int kFuseGraphs = 256;

// ---------------------------------------------------------------------------
template <int K, bool ASYNC, bool RS, bool W, bool HS = false, bool SV = false>
static hipError_t launch_t(const Launch &launch, int grid, int merge_grid, hipStream_t s,
                           hipEvent_t ev_beg, hipEvent_t ev_end) {
  hipError_t e = hipSuccess;
  Launch L = launch;
  const bool hub_kernels = ASYNC && (L.total_hubs > 0 || L.total_merge > 0);
  L.fuse_finish = !L.no_finish && L.total_items > 0 && !hub_kernels && grid <= kFuseBlocks &&
                          L.G <= kFuseGraphs
                      ? 1
                      : 0;
  if (ASYNC && L.total_hubs > 0) {
    const int sg = (L.total_hubs + 255) / 256 < 1024 ? (L.total_hubs + 255) / 256 : 1024;
    hipLaunchKernelGGL(k_hub_snapshot, dim3(sg), dim3(256), 0, s, L);
  }
  if (ev_beg && (e = hipEventRecord(ev_beg, s)) != hipSuccess) return e;
  if (L.total_items > 0) {
    if constexpr (RS)
      hipLaunchKernelGGL((k_move_rescan<K, ASYNC, W>), dim3(grid), dim3(kBlock), 0, s, L);
    else if constexpr (SV)
      hipLaunchKernelGGL((k_move_sv<K, W>), dim3(grid), dim3(kBlock), 0, s, L);
    else
      hipLaunchKernelGGL((move_kernel<K, ASYNC, W>(L.det_hubs > 0, L.unit != 0)), dim3(grid),
                         dim3(kBlock), 0, s, L);
  }
  if (ev_end && (e = hipEventRecord(ev_end, s)) != hipSuccess) return e;
  if constexpr (HS) {  // shared hub sketches replace segments and merging
    if (L.total_hubs > 0) {
      const int hg = L.total_hubs < grid * 4 ? L.total_hubs : grid * 4;
      hipLaunchKernelGGL((k_hub_shared<K>), dim3(hg), dim3(256), 0, s, L);
      if (L.total_segs > 0) hipLaunchKernelGGL(k_hub_mark, dim3(grid), dim3(kBlock), 0, s, L);
    }
  } else if (ASYNC && L.total_merge > 0) {
    if constexpr (RS) {
      hipLaunchKernelGGL((k_hub_cand<K>), dim3(merge_grid), dim3(kBlock), 0, s, L);
      if (L.total_segs > 0)
        hipLaunchKernelGGL((k_hub_rescan<K>), dim3(grid), dim3(kBlock), 0, s, L);
      hipLaunchKernelGGL((k_hub_pick<K>), dim3(merge_grid), dim3(kBlock), 0, s, L);
    } else {
      hipLaunchKernelGGL((k_hub_merge<K>), dim3(merge_grid), dim3(kBlock), 0, s, L);
    }
    if (L.total_segs > 0) hipLaunchKernelGGL(k_hub_mark, dim3(grid), dim3(kBlock), 0, s, L);
  }
  if (!L.no_finish && !L.fuse_finish) {
    const int fg = (L.G + 255) / 256 < 64 ? (L.G + 255) / 256 : 64;
    hipLaunchKernelGGL(k_finish, dim3(fg > 0 ? fg : 1), dim3(256), 0, s, L);
  }
  return hipGetLastError();
}

template <int K, bool ASYNC, bool RS, bool W, bool SV = false>
static int occ_t(bool hubs, bool unit) {
  int nb = 0;
  const void *f;
  if constexpr (RS)
    f = (const void *)k_move_rescan<K, ASYNC, W>;
  else if constexpr (SV)
    f = (const void *)k_move_sv<K, W>;
  else
    f = (const void *)move_kernel<K, ASYNC, W>(hubs, unit);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, kBlock, 0) != hipSuccess) return 1;
  return nb > 0 ? nb : 1;
}

template <bool ASYNC, bool RS, bool W>
static hipError_t launch_mode(int k, const Launch &L, int grid, int merge_grid, hipStream_t s,
                              hipEvent_t b, hipEvent_t e) {
  switch (k) {
    case 1: return launch_t<1, ASYNC, RS, W>(L, grid, merge_grid, s, b, e);
    case 2: return launch_t<2, ASYNC, RS, W>(L, grid, merge_grid, s, b, e);
    case 4: return launch_t<4, ASYNC, RS, W>(L, grid, merge_grid, s, b, e);
    case 8: return launch_t<8, ASYNC, RS, W>(L, grid, merge_grid, s, b, e);
    case 16: return launch_t<16, ASYNC, RS, W>(L, grid, merge_grid, s, b, e);
    case 32: return launch_t<32, ASYNC, RS, W>(L, grid, merge_grid, s, b, e);
    default: return hipErrorInvalidValue;
  }
}

template <bool ASYNC, bool RS, bool W>
static int occ_mode(int k, bool hubs, bool unit) {
  switch (k) {
    case 1: return occ_t<1, ASYNC, RS, W>(hubs, unit);
    case 2: return occ_t<2, ASYNC, RS, W>(hubs, unit);
    case 4: return occ_t<4, ASYNC, RS, W>(hubs, unit);
    case 8: return occ_t<8, ASYNC, RS, W>(hubs, unit);
    case 16: return occ_t<16, ASYNC, RS, W>(hubs, unit);
    case 32: return occ_t<32, ASYNC, RS, W>(hubs, unit);
    default: return 1;
  }
}

template <bool HS, bool W>
static hipError_t launch_hs(int k, const Launch &L, int grid, int merge_grid, hipStream_t s,
                            hipEvent_t b, hipEvent_t e) {
  switch (k) {
    case 1: return launch_t<1, true, false, W, HS>(L, grid, merge_grid, s, b, e);
    case 2: return launch_t<2, true, false, W, HS>(L, grid, merge_grid, s, b, e);
    case 4: return launch_t<4, true, false, W, HS>(L, grid, merge_grid, s, b, e);
    case 8: return launch_t<8, true, false, W, HS>(L, grid, merge_grid, s, b, e);
    case 16: return launch_t<16, true, false, W, HS>(L, grid, merge_grid, s, b, e);
    case 32: return launch_t<32, true, false, W, HS>(L, grid, merge_grid, s, b, e);
    default: return hipErrorInvalidValue;
  }
}

template <bool W>
static hipError_t launch_sv(int k, const Launch &L, int grid, int merge_grid, hipStream_t s,
                            hipEvent_t b, hipEvent_t e) {
  switch (k) {
    case 1: return launch_t<1, false, false, W, false, true>(L, grid, merge_grid, s, b, e);
    case 2: return launch_t<2, false, false, W, false, true>(L, grid, merge_grid, s, b, e);
    case 4: return launch_t<4, false, false, W, false, true>(L, grid, merge_grid, s, b, e);
    case 8: return launch_t<8, false, false, W, false, true>(L, grid, merge_grid, s, b, e);
    case 16: return launch_t<16, false, false, W, false, true>(L, grid, merge_grid, s, b, e);
    case 32: return launch_t<32, false, false, W, false, true>(L, grid, merge_grid, s, b, e);
    default: return hipErrorInvalidValue;
  }
}

template <bool W>
static int occ_sv(int k) {
  switch (k) {
    case 1: return occ_t<1, false, false, W, true>(true, false);
    case 2: return occ_t<2, false, false, W, true>(true, false);
    case 4: return occ_t<4, false, false, W, true>(true, false);
    case 8: return occ_t<8, false, false, W, true>(true, false);
    case 16: return occ_t<16, false, false, W, true>(true, false);
    case 32: return occ_t<32, false, false, W, true>(true, false);
    default: return 1;
  }
}

template <bool W>
static hipError_t launch_iteration_w(int k, bool async_mode, bool rescan, bool hub_shared,
                                     bool shared_vars, const Launch &L, int grid, int merge_grid,
                                     hipStream_t s, hipEvent_t ev_beg, hipEvent_t ev_end) {
  if (shared_vars) {  // det sketch rule without double scan only
    if (async_mode || rescan || hub_shared || k == 0) return hipErrorInvalidValue;
    return launch_sv<W>(k, L, grid, merge_grid, s, ev_beg, ev_end);
  }
  if (hub_shared) {  // async sketch rule without double scan only
    if (!async_mode || rescan || k == 0) return hipErrorInvalidValue;
    return launch_hs<true, W>(k, L, grid, merge_grid, s, ev_beg, ev_end);
  }
  if (k == 0) {  // the vote of Algorithm 3 (no double scan)
    if (rescan) return hipErrorInvalidValue;
    return async_mode ? launch_t<0, true, false, W>(L, grid, merge_grid, s, ev_beg, ev_end)
                      : launch_t<0, false, false, W>(L, grid, merge_grid, s, ev_beg, ev_end);
  }
  if (rescan)
    return async_mode ? launch_mode<true, true, W>(k, L, grid, merge_grid, s, ev_beg, ev_end)
                      : launch_mode<false, true, W>(k, L, grid, merge_grid, s, ev_beg, ev_end);
  return async_mode ? launch_mode<true, false, W>(k, L, grid, merge_grid, s, ev_beg, ev_end)
                    : launch_mode<false, false, W>(k, L, grid, merge_grid, s, ev_beg, ev_end);
}

hipError_t launch_iteration(int k, bool async_mode, bool rescan, bool hub_shared,
                            bool shared_vars, bool wide, const Launch &L, int grid,
                            int merge_grid, hipStream_t s, hipEvent_t ev_beg, hipEvent_t ev_end) {
  return wide ? launch_iteration_w<true>(k, async_mode, rescan, hub_shared, shared_vars, L, grid,
                                         merge_grid, s, ev_beg, ev_end)
              : launch_iteration_w<false>(k, async_mode, rescan, hub_shared, shared_vars, L, grid,
                                          merge_grid, s, ev_beg, ev_end);
}

template <bool W>
static int move_blocks_w(int k, bool async_mode, bool rescan, bool shared_vars, bool hubs,
                         bool unit) {
  if (shared_vars && k > 0 && !async_mode && !rescan) return occ_sv<W>(k);
  if (k == 0)
    return async_mode ? occ_t<0, true, false, W>(hubs, unit) : occ_t<0, false, false, W>(hubs, unit);
  if (rescan)
    return async_mode ? occ_mode<true, true, W>(k, hubs, unit)
                      : occ_mode<false, true, W>(k, hubs, unit);
  return async_mode ? occ_mode<true, false, W>(k, hubs, unit)
                    : occ_mode<false, false, W>(k, hubs, unit);
}

hipError_t launch_finish(const Launch &L, hipStream_t s) {
  const int fg = (L.G + 255) / 256 < 64 ? (L.G + 255) / 256 : 64;
  hipLaunchKernelGGL(k_finish, dim3(fg > 0 ? fg : 1), dim3(256), 0, s, L);
  return hipGetLastError();
}

int move_blocks_per_cu(int k, bool async_mode, bool rescan, bool shared_vars, bool wide, bool hubs,
                       bool unit) {
  return wide ? move_blocks_w<true>(k, async_mode, rescan, shared_vars, hubs, unit)
              : move_blocks_w<false>(k, async_mode, rescan, shared_vars, hubs, unit);
}

}  // namespace lpa
