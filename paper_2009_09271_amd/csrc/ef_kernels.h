// HIP kernels of the efsparse hot path (gfx950).
//
// The plain streaming kernels give each thread one coalesced float4 group (64-thread workgroups,
// kRbTile elements each).  The selection kernels work on rows: a row is the part of one segment
// inside one data tile of kTile elements, so that every workgroup of the selection pipeline serves
// exactly one segment.
//
// Top-k and random-k (Section 3) share one pipeline; no kernel synchronises across workgroups:
//   k_sample_gather  top-k only: the keys of a sample per segment (the whole segment when it has
//   k_sample_select  at most kExactMax elements, else runs spread over it); per segment either
//                    the exact winner rule (small segments) or a candidate threshold set so that
//                    the candidates very likely number at least k_l.
//   k_stream_sel     per row: fused accumulate (acc = g + e, written to e), candidate test (top-k:
//                    the rule above; random-k: Philox key < tau_l, a binomial bound on k_l), the
//                    row's candidates in index order to its slot, and a histogram of them (top-k).
//                    Random-k on layouts whose rows and key window fit k_select's LDS: also the
//                    row's undecided candidates (key in [ulo_l, tau_l)) listed, so that
//                    k_collect_randk is not needed.
//   k_resolve        top-k, per segment: the histogram bin holding the k_l-th best candidate.
//   k_collect        top-k, per row: candidates above that bin are counted, the undecided ones are
//                    listed (random-k without direct lists: k_collect_randk).
//   k_select         per segment: the exact threshold among the listed candidates, then the
//                    message offset of every row.  Layouts with a very large k_l or very many
//                    rows instead add the list's winners to the rows' counts, which k_rowsum
//                    scans (a list too long for that: k_rowcount counts again, k_rowtie
//                    resolves ties at the threshold).
//   k_emit           per row: the winners in index order to the message and e = +0 there (where
//                    the pass already stored +0, at every candidate of random-k and at the
//                    keys from R_Z on of dense top-k segments, losers get their values back).
// A top-k segment with fewer than k_l candidates, or whose candidates do not fit the workspace, is
// collected again at a lower threshold (k_resolve sets it, k_collect re-reads the rows); only if
// that falls short too, or for random-k, is it resolved exactly over all of its elements by
// k_select.  Random-k's selection can also run without data, ahead of the step (the keys depend
// only on seed, step and position); the step is then one streaming pass (k_randk_apply).
// Block-random-k is one fused streaming pass (k_randblock_step).  The aggregates (Algorithm 1) sum
// each output element over the workers in worker order: in registers for block messages, in an
// LDS tile for sparse ones.
#pragma once

#include "ef_device.h"

namespace efs {

struct WSel {
  uint32_t* diag;      // [4]  diagnostics bits
  uint32_t* res;       // [L][kResWords] per-segment selection record
  uint32_t* hist;      // [L][kHCopies][kHBins] candidate histogram per segment, in copies that
                       // spread the atomics of concurrent rows
  uint32_t* samp;      // [nruns * kSampleRun] top-k sample keys
  uint32_t* counts;    // [nrows] candidates per row
  uint32_t* rcnt;      // [nrows] winners per row
  uint32_t* roff;      // [nrows] message position of each row's first winner
  uint32_t* rtie;      // [nrows] top-k: elements equal to the key A (counted, not stored)
  uint32_t* lcnt;      // [L][kSubLists][kLineWords] sizes of the sub-lists, one cache line each
  uint32_t* scnt;      // [L][kSubLists][kLineWords] random-k without direct lists: certain winners of the
                       //   segment's rows (row r adds to counter r % 16)
  uint32_t* bsum;      // [kRowBlocks] many-row layouts: winners of each block of rows
  uint32_t* coff;      // [nrows] first entry of each row's candidates in the pool (kDropped: not
                       //   stored); one segment: written only for rows beyond their static slot
  uint32_t* pcnt;      // [kPools][kLineWords] fill counters of the overflow pool's parts
  uint16_t* cand_loc;  // [pool0 + capB] candidate pool: each row's static slot (soff, S), then the overflow
  float* cand_val;     //   pool for rows with more candidates (index order per row): a candidate's element
                       //   within the row's data tile (random-k: kCertain added when its key is below
                       //   ulo) and its value.  Top-k's key' is the value's magnitude
  uint32_t* cand_key;  //   random-k: key' of the candidates without kCertain
  uint32_t* list_idx;  // sub-lists of undecided candidates, per segment (see SubLists)
  uint32_t* list_key;
  uint2* pairs;        // random-k, direct layouts: each row's undecided (key', index) pairs at its
                       //   pool entries (the list arrays' memory)
  const uint32_t* soff;  // [nrows+1] first entry of each row's static slot (several segments)
  uint32_t S;          // one segment: static slot entries per row (row r's slot starts at r * S and
                       //   holds min(S, the row's elements))
  uint32_t pool0;      // first entry of the overflow pool (the static slots end there)
  uint32_t capB;       // overflow pool entries, kPools equal parts (row r reserves in part r % kPools)
};

constexpr uint32_t kDropped = 0xFFFFFFFFu;  // coff of a row whose candidates did not fit
constexpr uint32_t kAccRow = 0x80000000u;   // counts flag of a top-k row emitted from acc (winning
                                            //   ties); the count is then the row's length
constexpr uint32_t kCertain = 0x8000u;      // cand_loc flag
constexpr int kPools = 16;                  // parts of the overflow pool, one counter each
constexpr uint32_t kRowBlocks = 256;        // many-row layouts: blocks of rows (at most) whose winners are
                                            //   scanned by themselves

__device__ __forceinline__ uint32_t* res_of(const WSel& w, int l) { return w.res + (size_t)l * kResWords; }

// Several workers' steps in one launch of a selection kernel: worker blockIdx.y's buffers.  The
// gradient and residual of each worker are separate allocations (pointer tables); workspaces and
// messages lie at fixed strides from worker 0's.
constexpr int kBatchMax = 64;  // workers per launch of the selection kernels
struct Batch {
  uint64_t ws;                   // bytes between the workers' workspaces
  uint32_t msg;                  // entries between the workers' messages
  const void* g[kBatchMax];      // each worker's gradient (null: compress only)
  const float* src[kBatchMax];   // each worker's input: the residual e (fused steps) or acc
  float* e[kBatchMax];           // each worker's residual to update (null: compress only)
  uint32_t seed_lo[kBatchMax], seed_hi[kBatchMax];  // random-k: each worker's seed
};

template <typename P>
__device__ __forceinline__ P* shifted(P* p, uint64_t bytes) {
  return p ? reinterpret_cast<P*>(reinterpret_cast<uint8_t*>(const_cast<void*>(static_cast<const void*>(p))) + bytes)
           : p;
}

__device__ __forceinline__ WSel ws_at(WSel w, uint64_t off) {
  if (off == 0) return w;
  w.diag = shifted(w.diag, off);
  w.res = shifted(w.res, off);
  w.hist = shifted(w.hist, off);
  w.samp = shifted(w.samp, off);
  w.counts = shifted(w.counts, off);
  w.rcnt = shifted(w.rcnt, off);
  w.roff = shifted(w.roff, off);
  w.rtie = shifted(w.rtie, off);
  w.lcnt = shifted(w.lcnt, off);
  w.scnt = shifted(w.scnt, off);
  w.bsum = shifted(w.bsum, off);
  w.coff = shifted(w.coff, off);
  w.pcnt = shifted(w.pcnt, off);
  w.cand_loc = shifted(w.cand_loc, off);
  w.cand_val = shifted(w.cand_val, off);
  w.cand_key = shifted(w.cand_key, off);
  w.list_idx = shifted(w.list_idx, off);
  w.list_key = shifted(w.list_key, off);
  w.pairs = shifted(w.pairs, off);
  return w;  // (soff is a layout table: not shifted)
}

constexpr int kLineWords = 32;  // 128-byte L2 line: counters hit by many atomics get a line each
__device__ __forceinline__ uint32_t* lcnt_of(const WSel& w, int l, uint32_t c) {
  return w.lcnt + ((size_t)l * kSubLists + c) * kLineWords;
}
__device__ __forceinline__ uint32_t* scnt_of(const WSel& w, int l, uint32_t c) {
  return w.scnt + ((size_t)l * kSubLists + c) * kLineWords;
}
// The first element of a row's data tile.
__device__ __forceinline__ uint32_t row_tile(const Tables& T, uint32_t row) {
  return T.L == 1 ? row * kTile : T.row_rec[4u * (size_t)row + 3u];
}
__device__ __forceinline__ uint32_t* pcnt_of(const WSel& w, uint32_t part) { return w.pcnt + (size_t)part * kLineWords; }

// Reserves n pool entries for row `row` (more than its static slot holds) in part row % kPools of
// the overflow pool; kDropped if the part is full.  One thread.
__device__ __forceinline__ uint32_t pool_reserve(const WSel& w, uint32_t row, uint32_t n) {
  const uint32_t part = row % kPools, q = w.capB / kPools;
  const uint32_t at = atomicAdd(pcnt_of(w, part), n);
  if (at > q || n > q - at) return kDropped;
  return w.pool0 + part * q + at;
}

// The first pool entry of a row holding cnt candidates, given its coff word co: one segment: its
// static slot unless they did not fit there.
__device__ __forceinline__ uint32_t row_entry(const Tables& T, const WSel& w, uint32_t row, uint32_t cnt,
                                              uint32_t co) {
  if (T.L > 1) return co;
  return cnt > min(w.S, (uint32_t)T.d - row * kTile) ? co : row * w.S;
}

// The static slot of a row: first entry and capacity.
__device__ __forceinline__ void static_slot(const Tables& T, const WSel& w, uint32_t row, uint32_t& at, uint32_t& cap) {
  if (T.L == 1) {  // every row but the last is a whole tile
    at = row * w.S;
    cap = min(w.S, (uint32_t)T.d - row * kTile);
  } else {
    at = w.soff[row];
    cap = w.soff[row + 1] - at;
  }
}

// First entry of sub-list c of segment l: sub-list c owns seg_lq[l] entries of the segment's region
// (loaded once per row, ahead of the row's loop).
__device__ __forceinline__ size_t sublist_base(const Tables& T, int l, uint32_t c) {
  return (size_t)T.seg_lbase[l] + (size_t)c * (uint32_t)T.seg_lq[l];
}

// The sub-lists of one segment read as one array of M[kSubLists] entries (any order).
struct SubLists {
  const uint32_t* arr;
  size_t base;  // the segment's list region
  uint32_t q;   // entries per sub-list
  uint32_t M[kSubLists + 1];  // M[c]: entries in sub-lists before c
  __device__ __forceinline__ uint32_t operator[](uint32_t f) const {
    uint32_t c = 0, b = 0;
#pragma unroll
    for (int x = 1; x < kSubLists; ++x) {
      if (f >= M[x]) {
        c = (uint32_t)x;
        b = M[x];
      }
    }
    return arr[base + (size_t)c * q + (f - b)];
  }
};

// ---------------------------------------------------------------------------------------------
// Utility kernels
// ---------------------------------------------------------------------------------------------
// The plain streaming kernels take one float4 group per thread in 64-thread workgroups (kRbTile
// elements each): short-lived workgroups keep the end of the grid short, where a streaming pass
// otherwise loses bandwidth.  Measured for the fused block-random-k step on ResNet-50 flat: 64
// threads 47.2 us per step, 128: 48.2, 256: 48.6; four float4 groups per thread: about 50.5.
constexpr int kRbNT = 64;
constexpr uint32_t kRbTile = 4u * kRbNT;

__device__ __forceinline__ int group_extent(uint32_t i0, uint32_t hi) {
  return i0 < hi ? (int)min(4u, hi - i0) : 0;
}

// Algorithm 1 accumulate step: acc = g + e.
template <int GDT>
__global__ __launch_bounds__(kRbNT) void k_accumulate(int32_t d, const void* g, const float* e, float* acc) {
  const uint32_t lo = blockIdx.x * kRbTile, hi = min((uint32_t)d, lo + kRbTile);
  const uint32_t i0 = lo + threadIdx.x * 4u;
  const int nv = group_extent(i0, hi);
  float gv[4], ev[4], a[4];
  if (hi - lo == kRbTile) {  // whole group (every workgroup but the last)
    load4gf<GDT>(g, i0, gv);
    load4f(e, i0, ev);
  } else {
    load4g<GDT>(g, i0, nv, gv);
    load4(e, i0, nv, ev);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) a[q] = gv[q] + ev[q];
  store4(acc, i0, nv, a);
}

__global__ __launch_bounds__(kRbNT) void k_copy(int32_t d, const float* src, float* dst) {
  const uint32_t lo = blockIdx.x * kRbTile, hi = min((uint32_t)d, lo + kRbTile);
  const uint32_t i0 = lo + threadIdx.x * 4u;
  const int nv = group_extent(i0, hi);
  float v[4];
  if (hi - lo == kRbTile) load4f(src, i0, v);
  else load4(src, i0, nv, v);
  store4(dst, i0, nv, v);
}

// e[idx[j]] = +0 for every message entry (indices outside [0, d) are skipped).
__global__ __launch_bounds__(kNT) void k_sparse_zero(int32_t d, int32_t K, const uint32_t* idx, float* e) {
  const int j = blockIdx.x * kNT + threadIdx.x;
  if (j < K) {
    const uint32_t i = idx[j];
    if (i < (uint32_t)d) e[i] = 0.0f;
  }
}

// ---------------------------------------------------------------------------------------------
// Block-random-k (Section 3): one random start per segment, the run of k_l values after it.
// ---------------------------------------------------------------------------------------------
struct RunSeg {
  uint32_t o, n, k, P, s;
};

__device__ __forceinline__ RunSeg run_seg(const Tables& T, int l, uint32_t step, uint32_t s0, uint32_t s1) {
  RunSeg r;
  r.o = (uint32_t)T.seg_off[l];
  r.n = (uint32_t)T.seg_off[l + 1] - r.o;
  r.k = (uint32_t)T.seg_k[l];
  r.P = (uint32_t)T.seg_P[l];
  r.s = block_start((uint32_t)l, step, s0, s1, (uint32_t)T.seg_bl[l], (uint32_t)T.seg_nb[l]);
  return r;
}

// Position of element i within the run of its segment (>= k when not sent).
__device__ __forceinline__ uint32_t run_pos(const RunSeg& r, uint32_t i) {
  const uint32_t j = i - r.o;
  return j >= r.s ? j - r.s : j + r.n - r.s;
}

// The start of every segment that begins in [lo, hi) (segments sf..sl hold the data tile).  With
// one segment, its record rs is already loaded: no further load, which would make the
// workgroup's last wavefront wait for its stores before it ends (loads and stores share one
// counter).
__device__ __forceinline__ void write_starts(const Tables& T, int sf, int sl, const RunSeg& rs, uint32_t lo,
                                             uint32_t hi, uint32_t step, uint32_t s0, uint32_t s1,
                                             uint32_t* start) {
  if (sf == sl) {
    if (threadIdx.x == 0 && rs.o >= lo && rs.o < hi) start[sf] = rs.s;
    return;
  }
  for (int l = sf + (int)threadIdx.x; l <= sl; l += kRbNT) {
    const uint32_t ol = (uint32_t)T.seg_off[l];
    if (ol >= lo && ol < hi)
      start[l] = block_start((uint32_t)l, step, s0, s1, (uint32_t)T.seg_bl[l], (uint32_t)T.seg_nb[l]);
  }
}

// Fused worker step: acc = g + e; val[P_l + t] = acc on the run; e' = +0 on the run, acc elsewhere.
// One float4 group per thread for a float32 gradient (kRbTile elements per workgroup); two groups
// (kRbNT groups apart, each coalesced over the wavefront) for bf16, whose groups are 8-byte loads.
template <int GDT>
constexpr uint32_t rb_groups() { return GDT == 1 ? 2u : 1u; }
template <int GDT>
constexpr uint32_t rb_tile() { return kRbTile * rb_groups<GDT>(); }

template <int GDT>
__global__ __launch_bounds__(kRbNT) void k_randblock_step(Tables T, const void* g, float* e, uint32_t s0,
                                                        uint32_t s1, uint32_t step, uint32_t* start,
                                                        float* val) {
  if constexpr (GDT == 0) {
    const uint32_t lo = blockIdx.x * kRbTile, hi = min((uint32_t)T.d, lo + kRbTile);
    const uint32_t c = lo / kTile;  // the data tile holding this group: its first and last segment
    const int sf = T.chunk_sf[c], sl = T.chunk_sl[c];
    const uint32_t i0 = lo + threadIdx.x * 4u;
    const int nv = i0 < hi ? (int)min(4u, hi - i0) : 0;
    float gv[4], ev[4];
    if (hi - lo == kRbTile) {  // whole group (every workgroup but the last)
      load4gf<GDT>(g, i0, gv);
      load4f(e, i0, ev);
    } else {
      load4g<GDT>(g, i0, nv, gv);
      load4(e, i0, nv, ev);
    }
    RunSeg rs = run_seg(T, sf, step, s0, s1);
    int cur = sf;
    float out[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float a = gv[q] + ev[q];
      out[q] = a;
      if (q < nv) {
        const uint32_t i = i0 + q;
        if (sf != sl) {
          const int l = seg_of(i, sf, sl, T.seg_off);
          if (l != cur) {
            rs = run_seg(T, l, step, s0, s1);
            cur = l;
          }
        }
        const uint32_t t = run_pos(rs, i);
        if (t < rs.k) {
          val[rs.P + t] = a;
          out[q] = 0.0f;
        }
      }
    }
    store4(e, i0, nv, out);
    write_starts(T, sf, sl, rs, lo, hi, step, s0, s1, start);
  } else {
    constexpr uint32_t NG = rb_groups<GDT>(), TILE = rb_tile<GDT>();
    const uint32_t lo = blockIdx.x * TILE, hi = min((uint32_t)T.d, lo + TILE);
    const uint32_t c = lo / kTile;  // the data tile holding these groups: its first and last segment
    const int sf = T.chunk_sf[c], sl = T.chunk_sl[c];
    uint32_t i0[NG];
    int nv[NG];
#pragma unroll
    for (uint32_t r = 0; r < NG; ++r) {
      i0[r] = lo + (r * kRbNT + threadIdx.x) * 4u;
      nv[r] = i0[r] < hi ? (int)min(4u, hi - i0[r]) : 0;
    }
    float gv[NG][4], ev[NG][4];
    if (hi - lo == TILE) {  // whole tile (every workgroup but the last)
#pragma unroll
      for (uint32_t r = 0; r < NG; ++r) {
        load4gf<GDT>(g, i0[r], gv[r]);
        load4f(e, i0[r], ev[r]);
      }
    } else {
#pragma unroll
      for (uint32_t r = 0; r < NG; ++r) {
        load4g<GDT>(g, i0[r], nv[r], gv[r]);
        load4(e, i0[r], nv[r], ev[r]);
      }
    }
    RunSeg rs = run_seg(T, sf, step, s0, s1);
    int cur = sf;
#pragma unroll
    for (uint32_t r = 0; r < NG; ++r) {
      float out[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float a = gv[r][q] + ev[r][q];
        out[q] = a;
        if (q < nv[r]) {
          const uint32_t i = i0[r] + q;
          if (sf != sl) {
            const int l = seg_of(i, sf, sl, T.seg_off);
            if (l != cur) {
              rs = run_seg(T, l, step, s0, s1);
              cur = l;
            }
          }
          const uint32_t t = run_pos(rs, i);
          if (t < rs.k) {
            val[rs.P + t] = a;
            out[q] = 0.0f;
          }
        }
      }
      store4(e, i0[r], nv[r], out);
    }
    write_starts(T, sf, sl, rs, lo, hi, step, s0, s1, start);
  }
}

// Message position p -> segment (binary search over P).
__device__ __forceinline__ int seg_of_msg(uint32_t p, int L, const int32_t* P) { return seg_of(p, 0, L - 1, P); }

// compress_randblock: val[p] = acc at run position p; start[l] from the t = 0 entry.
__global__ __launch_bounds__(kNT) void k_randblock_gather(Tables T, int32_t K, const float* acc, uint32_t s0,
                                                          uint32_t s1, uint32_t step, uint32_t* start,
                                                          float* val) {
  const uint32_t p = blockIdx.x * kNT + threadIdx.x;
  if (p >= (uint32_t)K) return;
  const int l = seg_of_msg(p, T.L, T.seg_P);
  const RunSeg rs = run_seg(T, l, step, s0, s1);
  const uint32_t t = p - rs.P;
  uint32_t j = rs.s + t;
  if (j >= rs.n) j -= rs.n;
  val[p] = acc[rs.o + j];
  if (t == 0) start[l] = rs.s;
}

// In-place residual update for a block message: e[o_l + (s_l + t) mod d_l] = +0.
__global__ __launch_bounds__(kNT) void k_block_zero(Tables T, int32_t K, const uint32_t* start, float* e) {
  const uint32_t p = blockIdx.x * kNT + threadIdx.x;
  if (p >= (uint32_t)K) return;
  const int l = seg_of_msg(p, T.L, T.seg_P);
  const uint32_t o = T.seg_off[l], n = T.seg_off[l + 1] - o, t = p - T.seg_P[l];
  const uint32_t s = start[l] % n;
  uint32_t j = s + t;
  if (j >= n) j -= n;
  e[o + j] = 0.0f;
}

// Out-of-place residual update for a block message: e = +0 on the runs, acc elsewhere.  One float4
// group per thread (kRbTile elements per workgroup).
__global__ __launch_bounds__(kRbNT) void k_block_update(Tables T, const float* acc, const uint32_t* start, float* e) {
  const uint32_t lo = blockIdx.x * kRbTile, hi = min((uint32_t)T.d, lo + kRbTile);
  const uint32_t c = lo / kTile;  // the data tile holding this group: its first and last segment
  const int sf = T.chunk_sf[c], sl = T.chunk_sl[c];
  const uint32_t i0 = lo + threadIdx.x * 4u;
  const int nv = group_extent(i0, hi);
  float v[4];
  if (hi - lo == kRbTile) load4f(acc, i0, v);
  else load4(acc, i0, nv, v);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (q < nv) {
      const uint32_t i = i0 + q;
      const int l = sf == sl ? sf : seg_of(i, sf, sl, T.seg_off);
      const uint32_t o = T.seg_off[l], n = T.seg_off[l + 1] - o;
      const uint32_t s = start[l] % n, j = i - o;
      const uint32_t t = j >= s ? j - s : j + n - s;
      if (t < (uint32_t)T.seg_k[l]) v[q] = 0.0f;
    }
  }
  store4(e, i0, nv, v);
}

// ---------------------------------------------------------------------------------------------
// Aggregate (Algorithm 1): out = (sum over workers in order, from +0) / W, each output tile
// written once.
// ---------------------------------------------------------------------------------------------
// Output tiles of the sparse aggregate: kAggTile elements, summed by one wavefront (kAggRounds
// float4 groups per lane).
constexpr uint32_t kAggTile = 1024;  // 1024: 20.6 us on random-k messages; 2048: 23.8; 4096: 31.2
constexpr int kAggRounds = (int)kAggTile / (4 * 64);

// Column sum over W rows of K values (shared coordinates): sum_u v[u K + j] in row order from +0.0,
// loads of kSumBatch rows in flight together.
constexpr int kSumBatch = 8;
__device__ __forceinline__ float column_sum(const float* v, int32_t W, int32_t K, uint32_t j) {
  float s = 0.0f;
  for (int u0 = 0; u0 < W; u0 += kSumBatch) {
    float t[kSumBatch];
#pragma unroll
    for (int u = 0; u < kSumBatch; ++u) t[u] = u0 + u < W ? v[(size_t)(u0 + u) * K + j] : 0.0f;
#pragma unroll
    for (int u = 0; u < kSumBatch; ++u)
      if (u0 + u < W) s += t[u];
  }
  return s;
}

// tile_start[w * ts_stride + tau] = first entry of message w whose index lies in an aggregate tile
// >= tau (tau = 0..nt; an index >= d counts as tile nt).  Grid: (gx, W); each thread takes U
// entries at a time (coalesced, all loads in flight together) and the workgroups stride over the
// message: U = 1 with a thread per entry for short messages (the quickest form: one round), U = 8
// and a capped grid for long ones, so that 3.2e9 entries (32 messages of 1e8) do not need as many
// threads (1e9 elements at 1 %: 692 -> 450 us; at 10 %: 6.8 -> 3.8 ms).
// With `sums` (shared coordinates: W = 1 message whose values are vW workers' rows `vals`), entry
// j's thread also writes sums[j], the column sum of the rows in worker order.
// Entry j starts the tiles after its predecessor's tile, up to its own (past the last entry the
// tiles up to nt start at K).  A short run of tiles is written by its entry's thread; a longer one
// (a gap in a message crowded into a few layers) as one coalesced run, after each round (a thread
// writes its long run itself if the workgroup's list of them is full).  Runs of up to kRunWave
// tiles are taken in turn by the workgroup's four wavefronts: 16 messages over 1.1e8 elements with
// gaps of 40 / 600 / 2000 tiles take 12.0 / 10.9 / 11.2 us, by the whole workgroup one run after
// another 17.0 / 13.2 / 13.4.  Longer ones, of which a workgroup seldom has four, are written by the
// whole workgroup: 4 messages over 1e9 elements with gaps of 40,000 tiles 66 us (all the entries in
// the first hundredth of 1.1e8 elements: 9 us, by one wavefront 31).
// For ascending messages the entries' runs partition 0..nt.
constexpr uint32_t kRunOwn = 32;        // runs of at most this many tiles are written by their own thread
                                        // (ResNet-50 top-k messages: 8.2 us with 128, 5.0 with 16-64)
constexpr int kRangeUBig = 8;           // entries per thread per round for long messages
constexpr int64_t kRangeBig = 1 << 22;  // total entries (W K) from which the long form is used
constexpr uint32_t kRangeStash = 512;   // long runs listed per workgroup and round
constexpr uint32_t kRunWave = 4096;     // long runs of up to this many tiles are written by one wavefront
                                        // (gaps of 4000 tiles, 4 messages over 1e9: 19.8 us, by four 23)

template <int kRangeU>
__global__ __launch_bounds__(kNT) void k_agg_ranges(int32_t d, int32_t K, int32_t nt, const uint32_t* idx,
                                                    uint32_t* tile_start, uint64_t ts_stride, const float* vals,
                                                    int32_t vW, float* sums) {
  __shared__ uint32_t s_nlong;
  __shared__ uint32_t s_ta[kRangeStash], s_n[kRangeStash], s_j[kRangeStash], s_own[kRangeStash];
  const int w = blockIdx.y;
  const uint32_t* m = idx + (size_t)w * K;
  uint32_t* ts = tile_start + (size_t)w * ts_stride;
  const size_t tbase = (size_t)w * ts_stride;
  auto tile = [&](uint32_t i) -> uint32_t { return i < (uint32_t)d ? i / kAggTile : (uint32_t)nt; };
  // tile tau of entry e's run starts at e, except past the last entry's own tile (at K); the other
  // entries' runs end at their own tiles
  auto value = [&](uint32_t e, uint32_t tau, uint32_t e_own) -> uint32_t { return tau > e_own ? (uint32_t)K : e; };
  if (threadIdx.x == 0) s_nlong = 0;
  __syncthreads();
  const uint32_t round = gridDim.x * (uint32_t)kNT * (uint32_t)kRangeU;
  for (uint32_t j0 = blockIdx.x * (uint32_t)kNT * (uint32_t)kRangeU; j0 < (uint32_t)K; j0 += round) {
    // each entry and its predecessor: the predecessor is the previous lane's entry (a shuffle);
    // only a wavefront's first lane loads it (a second load of every entry doubled the requests
    // this pass makes of the caches: 1e8 elements, 16 messages at 10 %: 192 -> 146 us)
    uint32_t cur[kRangeU], prv[kRangeU];
    const uint32_t lane = threadIdx.x & 63u;
    const bool first = lane == 0u;
#pragma unroll
    for (int u = 0; u < kRangeU; ++u) {
      const uint32_t j = j0 + (uint32_t)u * kNT + threadIdx.x;
      cur[u] = j < (uint32_t)K ? m[j] : 0u;
      prv[u] = first && j < (uint32_t)K && j > 0 ? m[j - 1] : 0u;
    }
#pragma unroll
    for (int u = 0; u < kRangeU; ++u) {
      const uint32_t up = __shfl_up(cur[u], 1u, 64);
      if (!first) prv[u] = up;
    }
    // shared coordinates (one message for vW workers): also the column sums of their values
    if (sums && w == 0) {
#pragma unroll
      for (int u = 0; u < kRangeU; ++u) {
        const uint32_t j = j0 + (uint32_t)u * kNT + threadIdx.x;
        if (j < (uint32_t)K) sums[j] = column_sum(vals, vW, K, j);
      }
    }
#pragma unroll
    for (int u = 0; u < kRangeU; ++u) {
      const uint32_t j = j0 + (uint32_t)u * kNT + threadIdx.x;
      if (j >= (uint32_t)K) continue;
      const uint32_t own = tile(cur[u]);
      const uint32_t ta = j == 0 ? 0u : tile(prv[u]) + 1u;
      const uint32_t tb = j == (uint32_t)K - 1u ? (uint32_t)nt : own;
      const uint32_t n = tb + 1u > ta ? tb + 1u - ta : 0u;
      bool mine = n <= kRunOwn;
      if (!mine) {
        const uint32_t p = atomicAdd(&s_nlong, 1u);
        if (p < kRangeStash) {
          s_ta[p] = ta;
          s_n[p] = n;
          s_j[p] = j;
          s_own[p] = own;
        } else {
          mine = true;
        }
      }
      if (mine)
        for (uint32_t k = 0; k < n; ++k) ts[ta + k] = value(j, ta + k, own);
    }
    __syncthreads();
    const uint32_t nl = min(s_nlong, kRangeStash);
    // run q by the threads t of NT
    auto write = [&](uint32_t q, uint32_t t, auto nth) {
      constexpr uint32_t NT = decltype(nth)::value;
      const uint32_t qa = s_ta[q], qe = qa + s_n[q], qj = s_j[q], qown = s_own[q];
      // 16-byte stores over the part of the run aligned in memory, single words at its two ends
      const uint32_t a4 = min(qe, qa + (uint32_t)((4u - (tbase + qa) % 4u) % 4u));
      const uint32_t b4 = a4 + (qe - a4) / 4u * 4u;
      if (t < a4 - qa) ts[qa + t] = value(qj, qa + t, qown);
      if (t < qe - b4) ts[b4 + t] = value(qj, b4 + t, qown);
      for (uint32_t o = a4 + 4u * t; o < b4; o += 4u * NT) {
        const uint4 v = make_uint4(value(qj, o, qown), value(qj, o + 1, qown), value(qj, o + 2, qown),
                                   value(qj, o + 3, qown));
        *reinterpret_cast<uint4*>(ts + o) = v;
      }
    };
    for (uint32_t q = 0; q < nl; ++q) {
      if (s_n[q] > kRunWave) write(q, threadIdx.x, std::integral_constant<uint32_t, kNT>{});
      else if (q % (kNT / 64u) == threadIdx.x / 64u) write(q, lane, std::integral_constant<uint32_t, 64>{});
    }
    __syncthreads();
    if (threadIdx.x == 0) s_nlong = 0;
    __syncthreads();
  }
}

// Workgroups of the range pass per message: one per kNT * U entries, capped for long messages so
// that all messages together fill the chip a few times over.
inline bool agg_ranges_big(int32_t K, int32_t W) { return (int64_t)K * W >= kRangeBig; }
inline uint32_t agg_ranges_gx(int32_t K, int32_t W) {
  if (!agg_ranges_big(K, W)) return (uint32_t)(((int64_t)K + kNT - 1) / kNT);
  const uint32_t need = (uint32_t)(((int64_t)K + kNT * kRangeUBig - 1) / (kNT * kRangeUBig));
  const uint32_t cap = (uint32_t)std::max<int32_t>(1, 8192 / std::max<int32_t>(W, 1));
  return std::max<uint32_t>(1u, std::min(need, cap));
}

// out = sum / W in IEEE float32.  For W a power of two the quotient is the exact scaling
// sum * (1 / W), which rounds identically (both are the one correctly rounded result of the same
// real number), and a multiply costs one instruction instead of a division sequence.
__device__ __forceinline__ float agg_scale(float sum, int32_t W, bool pow2, float inv) {
  return pow2 ? sum * inv : __fdiv_rn(sum, (float)W);
}

// Output stage of the aggregates.  q = the worker sum, divided by wdiv when averaging.  q goes to
// `out` when given; when `x` is given, Algorithm 1's parameter update is applied in the same pass:
// d = q (+ wd x when wd != 0); with a momentum buffer m: m = beta m + d, d = m; then x = x - d
// (each float32 operation rounded on its own).
struct AggOut {
  float* out;     // the aggregate, or nullptr
  float* x;       // parameters to update, or nullptr
  float* m;       // momentum buffer, or nullptr
  float beta, wd;
  int32_t wdiv;   // divisor of the average: the number of workers
  int32_t average;
};

__device__ __forceinline__ void agg_mean4(const AggOut& O, const float sum[4], float q[4]) {
  const bool pow2 = (O.wdiv & (O.wdiv - 1)) == 0;
  const float inv = 1.0f / (float)O.wdiv;  // exact when wdiv is a power of two
#pragma unroll
  for (int j = 0; j < 4; ++j) q[j] = O.average ? agg_scale(sum[j], O.wdiv, pow2, inv) : sum[j];
}

__device__ __forceinline__ void agg_step4(const AggOut& O, const float q[4], float x[4], float m[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float dj = q[j];
    if (O.wd != 0.0f) dj = dj + O.wd * x[j];
    if (O.m) {
      m[j] = O.beta * m[j] + dj;
      dj = m[j];
    }
    x[j] = x[j] - dj;
  }
}

__device__ __forceinline__ void agg_emit4(const AggOut& O, uint32_t i0, int nv, const float sum[4]) {
  float q[4];
  agg_mean4(O, sum, q);
  if (O.out) store4(O.out, i0, nv, q);
  if (O.x) {
    float x[4], m[4];
    load4(O.x, i0, nv, x);
    if (O.m) load4(O.m, i0, nv, m);
    agg_step4(O, q, x, m);
    store4(O.x, i0, nv, x);
    if (O.m) store4(O.m, i0, nv, m);
  }
}

// A whole group whose parameters and momentum are loaded already.
__device__ __forceinline__ void agg_update4(const AggOut& O, uint32_t i0, const float sum[4], f4 xv, f4 mv) {
  float q[4], x[4] = {xv.x, xv.y, xv.z, xv.w}, m[4] = {mv.x, mv.y, mv.z, mv.w};
  agg_mean4(O, sum, q);
  if (O.out) store4(O.out, i0, 4, q);
  agg_step4(O, q, x, m);
  store4(O.x, i0, 4, x);
  if (O.m) store4(O.m, i0, 4, m);
}

constexpr int kAggChunk = 4;        // sparse aggregate: entries per lane loaded together past the first 64
constexpr int kAggClaim = 256;      // sparse aggregate: claim slots (positions hash to x mod 256)

// Sparse aggregate: one wavefront per workgroup and one output tile of kAggTile elements per
// workgroup; many small workgroups resident per CU overlap each other's two load round trips
// (the tile's ranges, then its entries).  Lane j of a group of up to 64 workers holds worker
// j's entry range in the tile.  A tile no message enters is stored as zeros at once.  Otherwise
// its sums build up in an LDS tile: the tile's entries, in worker order, are added 64 at a time;
// lanes whose entries share a position add one after another in lane order (the lowest lane that
// still has to add claims the position's slot with an LDS atomic minimum; positions sharing a slot
// only wait for each other), which is worker order.  Entries past the first 64 are loaded
// kAggChunk per lane at a time.
struct AggLds {
  alignas(16) float acc[kAggTile];  // read and written as float4 groups
  uint32_t claim[kAggClaim];  // ~0 between adds
  uint32_t pre[65];           // entry prefix of each worker of the group
  uint32_t a[64];             // each worker's first entry in the tile
};

// Staged entry f of a worker group -> message entry: binary search of the prefixes.
__device__ __forceinline__ size_t agg_entry(const AggLds& S, int nw, int w0, int32_t K, uint32_t f) {
  int lo = 0, hi = nw - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (S.pre[mid] <= f) lo = mid; else hi = mid - 1;
  }
  return (size_t)(w0 + lo) * K + S.a[lo] + (f - S.pre[lo]);
}

// Prefixes of the worker group [w0, w0 + nw) whose ranges lane j holds (unclamped); returns the
// group's entry count.  Wave-uniform.
__device__ __forceinline__ uint32_t agg_group(AggLds& S, int nw, int32_t K, uint32_t ra, uint32_t rb) {
  const int lane = threadIdx.x;
  ra = min(ra, (uint32_t)K);
  rb = min(rb, (uint32_t)K);
  const uint32_t c = lane < nw && rb > ra ? rb - ra : 0u;
  const uint32_t inc = wave_incl_scan(c);
  S.pre[lane] = inc - c;
  S.a[lane] = ra;
  if (lane == 63) S.pre[64] = inc;
  __syncthreads();  // a one-wavefront workgroup: orders the LDS writes above before the reads
  return __shfl(inc, 63, 64);
}

// Adds one batch of up to 64 entries (lane order = worker order) into the LDS tile.
__device__ __forceinline__ void agg_add(AggLds& S, uint32_t lo, uint32_t hi, uint32_t i, float v, bool ok) {
  const uint32_t lane = threadIdx.x;
  bool pending = ok && i >= lo && i < hi;
  const uint32_t x = pending ? i - lo : 0u, c = x % kAggClaim;
  while (__ballot(pending)) {
    if (pending) atomicMin(&S.claim[c], lane);
    __syncthreads();
    if (pending && S.claim[c] == lane) {
      S.acc[x] += v;
      S.claim[c] = ~0u;
      pending = false;
    }
    __syncthreads();
  }
}

// Adds entries [f0, E) of the group set up by agg_group, kAggChunk per lane at a time.
__device__ __forceinline__ void agg_add_rest(AggLds& S, int nw, int w0, int32_t K, const uint32_t* idx,
                                             const float* val, uint32_t lo, uint32_t hi, uint32_t f0, uint32_t E) {
  for (; f0 < E; f0 += 64u * kAggChunk) {
    uint32_t ci[kAggChunk];
    float cv[kAggChunk];
#pragma unroll
    for (int u = 0; u < kAggChunk; ++u) {
      const uint32_t f = f0 + (uint32_t)u * 64u + threadIdx.x;
      const size_t j = f < E ? agg_entry(S, nw, w0, K, f) : 0;
      ci[u] = idx[j];
      cv[u] = val[j];
    }
#pragma unroll
    for (int u = 0; u < kAggChunk; ++u) agg_add(S, lo, hi, ci[u], cv[u], f0 + (uint32_t)u * 64u + threadIdx.x < E);
  }
}

// Tiles whose workers hold more than this many entries each on average add them worker by worker
// (agg_add_workers; BERT's d, 16 workers at 10 %: 310 us; at 1 %, about 10 entries per worker and
// tile, the loads of one worker at a time leave five lanes in six idle and the staged form is
// faster; 12, 16 and 24 in place of 48 measured the same within 1 % at 1, 3 and 10 %).
constexpr uint32_t kAggDense = 48;
// Dense tiles: chunks of 64 entries loaded together.  Sixteen hide the latency of the tiles that a
// sparse message crowds into (top-k messages of ResNet-50 at 1 %, 16 workers: 38 us, with four 42).
// Where every tile is so full, 16 in flight in each of a chip's wavefronts are more than the L2s hold,
// and lines that two chunks share are fetched twice: messages of over a quarter of the elements load
// four (BERT's d at 30 %, 16 workers: 859 us with sixteen, 803 with four; at 10 % 310 with either).
constexpr int kAggW = 16, kAggWFull = 4;

// Dense tiles: the group's workers one after another, in order.  A message holds each position at
// most once, so the adds of one worker never collide: a chunk of up to 64 of one worker's entries
// is added by its lanes at once, with no claims and no barriers (the one wavefront's LDS accesses
// take effect in program order, so a position's adds run in worker order).  The chunks (worker by
// worker, 64 entries each) are numbered through a prefix over the workers' chunk counts; AW chunks
// are loaded together (coalesced), then added in order.  A lane without an entry gets an index past
// the tile as its load's alternative (cleared by a second test after the loads, BERT's d at 10 %, 16
// workers: 387 us).  (Reading four chunks' sums together measured the same as one after another; LDS
// float atomics, which would return nothing to wait for, took 911 us there: they are processed a lane
// at a time.)
template <int AW>
__device__ __forceinline__ void agg_add_workers(AggLds& S, int nw, int w0, int32_t K, const uint32_t* idx,
                                                const float* val, uint32_t lo, uint32_t hi) {
  const uint32_t lane = threadIdx.x;
  const uint32_t n = lane < (uint32_t)nw ? S.pre[lane + 1] - S.pre[lane] : 0u;  // worker `lane`'s entries
  const uint32_t a = S.a[lane];
  const uint32_t ch = (n + 63u) / 64u, chi = wave_incl_scan(ch);
  const uint32_t cpre = chi - ch;  // first chunk of worker `lane`
  const uint32_t nch = __shfl(chi, 63, 64);
  for (uint32_t q0 = 0; q0 < nch; q0 += AW) {
    uint32_t ci[AW];
    float cv[AW];
#pragma unroll
    for (int u = 0; u < AW; ++u) {
      const uint32_t q = q0 + (uint32_t)u;
      // chunk q's worker: the last one whose chunks start at or before q (wave-uniform)
      const int w = (int)__popcll(__ballot(lane < (uint32_t)nw && cpre <= q)) - 1;
      const uint32_t f = (q - (uint32_t)__builtin_amdgcn_readlane((int)cpre, w)) * 64u + lane;
      const bool ok = q < nch && f < (uint32_t)__builtin_amdgcn_readlane((int)n, w);
      const size_t j = (size_t)(w0 + w) * K + (uint32_t)__builtin_amdgcn_readlane((int)a, w) + f;
      ci[u] = ok ? idx[j] : hi;  // hi: adds nothing below
      cv[u] = ok ? val[j] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < AW; ++u)
      if (ci[u] >= lo && ci[u] < hi) S.acc[ci[u] - lo] += cv[u];
  }
}

// Adds a worker group's E entries by the form that suits their number.
__device__ __forceinline__ void agg_add_group(AggLds& S, int nw, int w0, int32_t d, int32_t K, const uint32_t* idx,
                                              const float* val, uint32_t lo, uint32_t hi, uint32_t E) {
  if (E <= kAggDense * (uint32_t)nw) agg_add_rest(S, nw, w0, K, idx, val, lo, hi, 0u, E);
  else if ((uint32_t)K > (uint32_t)d / 4u) agg_add_workers<kAggWFull>(S, nw, w0, K, idx, val, lo, hi);
  else agg_add_workers<kAggW>(S, nw, w0, K, idx, val, lo, hi);
}

// Workgroup b -> tile: workgroups are dispatched to the 8 XCDs in turn (b mod 8), so XCD x is
// given chunks of kXcdChunk contiguous tiles in turn (chunks x, x + 8, ...), and the tiles past
// the last whole round of chunks in one contiguous part (a bijection for any n).  Neighbouring
// tiles share the cache lines of the range table and of the messages, and, within a chunk, an L2;
// the chunks spread a cluster of crowded tiles (top-k messages) over all the XCDs, where one
// contiguous eighth of the tiles per XCD left one XCD with most of the work.
constexpr uint32_t kXcds = 8;
constexpr uint32_t kXcdChunk = 32;
__device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t n) {
  const uint32_t x = b % kXcds, j = b / kXcds;
  const uint32_t full = n / (kXcds * kXcdChunk) * kXcdChunk;  // each XCD's workgroups in whole rounds
  if (j < full) return ((j / kXcdChunk) * kXcds + x) * kXcdChunk + j % kXcdChunk;
  const uint32_t base = full * kXcds, rn = n - base, q = rn / kXcds, r = rn % kXcds;
  return base + x * q + min(x, r) + (j - full);
}

// UPD: with the parameter update.  A whole tile's parameters and momentum are then loaded along with
// the ranges, so that the update waits for no third round trip at the end (8 workers at 1 % on
// ResNet-18's d with momentum: 42.7 -> 34.8 us; 187 MB at least, 29 us).  Where many workers' messages
// hold several entries per element the wait is short beside the adds and the registers cost up to 4 %
// (2.56e7 elements at 40 %, 16 workers: 402 us, loaded last 389; 2 workers 105 / 114, with momentum).
template <bool UPD>
__global__ __launch_bounds__(64) void k_agg_sparse(int32_t d, int32_t W, int32_t K, int32_t nt,
                                                   const uint32_t* idx, const float* val,
                                                   const uint32_t* tile_start, AggOut O) {
  __shared__ AggLds S;
  const int lane = threadIdx.x;
  const uint32_t t = xcd_tile(blockIdx.x, (uint32_t)nt);  // the grid has exactly nt workgroups
  const uint32_t lo = t * kAggTile, hi = min((uint32_t)d, lo + kAggTile);
  // ranges of the first worker group (lane j: worker j; lanes past W read worker W - 1's)
  const int nw0 = min(W, 64);
  const uint32_t* ts = tile_start + (size_t)min(lane, nw0 - 1) * (nt + 1) + t;
  const uint32_t ra = ts[0], rb = ts[1];
  const bool ahead = UPD && hi - lo == kAggTile;
  f4 xv[UPD ? kAggRounds : 1], mv[UPD ? kAggRounds : 1];
  if (ahead) {
#pragma unroll
    for (int r = 0; r < (UPD ? kAggRounds : 0); ++r) {
      const uint32_t i0 = lo + (uint32_t)(r * 64 + lane) * 4u;
      xv[r] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(O.x + i0));
      if (O.m) mv[r] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(O.m + i0));
    }
  }
  for (uint32_t x = lane; x < kAggClaim; x += 64) S.claim[x] = ~0u;
  const uint32_t E = agg_group(S, nw0, K, ra, rb);
  if (W <= 64 && E == 0 && !ahead) {
#pragma unroll
    for (int r = 0; r < kAggRounds; ++r) {
      const uint32_t i0 = lo + (uint32_t)(r * 64 + lane) * 4u;
      const int n = i0 < hi ? (int)min(4u, hi - i0) : 0;
      const float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      agg_emit4(O, i0, n, z);
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < kAggRounds; ++r) {
    const f4 z = {0.0f, 0.0f, 0.0f, 0.0f};
    *reinterpret_cast<f4*>(&S.acc[(r * 64 + lane) * 4]) = z;
  }
  __syncthreads();
  agg_add_group(S, nw0, 0, d, K, idx, val, lo, hi, E);
  for (int w0 = 64; w0 < W; w0 += 64) {  // further worker groups
    const int nw = min(64, W - w0);
    const uint32_t* tg = tile_start + (size_t)(w0 + min(lane, nw - 1)) * (nt + 1) + t;
    const uint32_t Eg = agg_group(S, nw, K, tg[0], tg[1]);
    agg_add_group(S, nw, w0, d, K, idx, val, lo, hi, Eg);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kAggRounds; ++r) {
    const uint32_t x = (uint32_t)(r * 64 + lane) * 4u;
    const uint32_t i0 = lo + x;
    const int n = i0 < hi ? (int)min(4u, hi - i0) : 0;
    const f4 s4 = *reinterpret_cast<const f4*>(&S.acc[x]);
    const float v[4] = {s4.x, s4.y, s4.z, s4.w};
    if (UPD && ahead) agg_update4(O, i0, v, xv[UPD ? r : 0], mv[UPD ? r : 0]);
    else agg_emit4(O, i0, n, v);
  }
}

// Single-segment layouts (flat scope): one workgroup per tile of R float4 groups per thread, no
// tables to look up and no barrier.  Each wavefront loads the starts of 64 workers at a time
// (lane j: worker wb + j), finds those whose run meets the tile with one ballot and visits them in
// ascending order.
template <int R>
__global__ __launch_bounds__(kNT) void k_agg_block1(int32_t d, int32_t W, int32_t K, const uint32_t* start,
                                                    const float* val, AggOut O) {
  constexpr uint32_t kT = (uint32_t)R * 4u * kNT;
  const uint32_t lo = blockIdx.x * kT, hi = min((uint32_t)d, lo + kT);
  const uint32_t n = (uint32_t)d, k = (uint32_t)K;
  const int lane = threadIdx.x & 63;
  float a[R][4];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) a[r][q] = 0.0f;
  for (int wb = 0; wb < W; wb += 64) {
    const int nw = min(64, W - wb);
    uint32_t s = 0;
    bool hit = false;
    if (lane < nw) {
      s = start[wb + lane] % n;
      const uint32_t e1 = min(s + k, n);
      // run piece 1: [s, e1); piece 2 (wrapped): [0, s + k - e1), empty unless the run wraps
      hit = max(lo, s) < min(hi, e1) || lo < min(hi, s + k - e1);
    }
    uint64_t todo = __ballot(hit);
    while (todo) {
      const int j = __ffsll((long long)todo) - 1;
      todo &= todo - 1;
      const uint32_t sw = __shfl(s, j, 64);
      const float* v = val + (size_t)(wb + j) * K;
      // piece 1 ends at e1 = min(s + k, n); piece 2 ([0, s + k - e1)) is empty unless the run wraps
      const uint32_t e1 = min(sw + k, n);
      const uint32_t a1 = max(lo, sw), b1 = min(hi, e1), b2 = min(hi, sw + k - e1);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint32_t i0 = lo + (uint32_t)(r * kNT + threadIdx.x) * 4u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t i = i0 + q;
          if (i >= a1 && i < b1) a[r][q] += v[i - sw];
          else if (i < b2) a[r][q] += v[i + n - sw];
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i0 = lo + (uint32_t)(r * kNT + threadIdx.x) * 4u;
    const int nv = i0 < hi ? (int)min(4u, hi - i0) : 0;
    agg_emit4(O, i0, nv, a[r]);
  }
}

// Output stage for the elements q of the group at i0 whose bit q is set in `mask` (any subset: a
// group that straddles a segment boundary is written in parts by the two segments' workgroups).
__device__ __forceinline__ void agg_emit4m(const AggOut& O, uint32_t i0, uint32_t mask, const float sum[4]) {
  if (mask == 0xFu) {
    agg_emit4(O, i0, 4, sum);
    return;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (!((mask >> q) & 1u)) continue;
    const float s1[4] = {sum[q], 0.0f, 0.0f, 0.0f};
    agg_emit4(O, i0 + (uint32_t)q, 1, s1);
  }
}

// Multi-segment layouts: one workgroup per (1024-element data tile, segment) pair with an element
// in common, listed by a table built with the layout; otherwise as k_agg_block1 within the
// segment: the segment's block starts of 64 workers at a time, the workers whose run meets the
// tile found with one ballot and visited in ascending order.  Each element gets at most one value
// per worker, and the tile's elements outside the segment belong to the other pairs of the tile.
constexpr uint32_t kAggBT = 4u * kNT;  // one float4 group per thread

__global__ __launch_bounds__(kNT) void k_agg_block(Tables T, int32_t W, int32_t K, const uint32_t* start,
                                                   const float* val, AggOut O) {
  static_assert(kBtWords == 8, "two 16-byte loads per record");
  const uint4* rec = reinterpret_cast<const uint4*>(T.btile) + 2u * blockIdx.x;
  const uint4 r0 = rec[0], r1 = rec[1];  // one round trip: no chain through the segment tables
  const int l = (int)r0.y;
  const uint32_t o = r0.z, n = r0.w, k = r1.x, P = r1.y;
  const uint32_t tlo = r0.x * kAggBT;
  const uint32_t lo = max(tlo, o), hi = min(tlo + kAggBT, o + n);
  const uint32_t i0 = tlo + threadIdx.x * 4u;
  const int lane = threadIdx.x & 63;
  float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int wb = 0; wb < W; wb += 64) {
    const int nw = min(64, W - wb);
    uint32_t s = 0;
    bool hit = false;
    if (lane < nw) {
      s = start[(size_t)(wb + lane) * T.L + l] % n;
      // run piece 1: [o + s, o + e1), e1 = min(s + k, n); piece 2 (wrapped): [o, o + s + k - e1),
      // empty unless the run wraps (written without a conditional, as in k_agg_block1)
      const uint32_t e1 = min(s + k, n);
      hit = max(lo, o + s) < min(hi, o + e1) || lo < min(hi, o + (s + k - e1));
    }
    uint64_t todo = __ballot(hit);
    while (todo) {
      const int j = __ffsll((long long)todo) - 1;
      todo &= todo - 1;
      const uint32_t sw = __shfl(s, j, 64);
      const float* v = val + (size_t)(wb + j) * K + P;
      const uint32_t e1 = min(sw + k, n);
      const uint32_t a1 = max(lo, o + sw), b1 = min(hi, o + e1), b2 = min(hi, o + (sw + k - e1));
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t i = i0 + (uint32_t)q;
        if (i >= a1 && i < b1) a[q] += v[i - o - sw];
        else if (i >= lo && i < b2) a[q] += v[i - o + n - sw];
      }
    }
  }
  uint32_t mask = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (i0 + (uint32_t)q >= lo && i0 + (uint32_t)q < hi) mask |= 1u << q;
  if (mask) agg_emit4m(O, i0, mask, a);
}

// ---------------------------------------------------------------------------------------------
// Random-k with the selection prepared ahead: the keys depend only on the seed, the step and the
// position (Section 3, random-k), so the message indices can be chosen before the gradient
// exists.  The step is then one streaming pass, one workgroup per kAggTile-element tile (one
// float4 group per thread): acc = g + e; the tile's winners (entries [ts[t], ts[t + 1]) of the
// prepared message, in ascending order) take their values from acc, and e = acc with +0 there.
// ---------------------------------------------------------------------------------------------
static_assert(kAggTile == 4u * kNT, "one float4 group per thread");

template <int GDT>
__global__ __launch_bounds__(kNT) void k_randk_apply(int32_t d, int32_t K, const uint32_t* ts, const uint32_t* idx,
                                                     const void* g, float* e, float* val) {
  __shared__ __align__(16) int32_t slot[kAggTile];  // element -> its winner's message entry, or -1
  const uint32_t t = blockIdx.x, lo = t * kAggTile, hi = min((uint32_t)d, lo + kAggTile);
  const uint32_t i0 = lo + threadIdx.x * 4u;
  const uint32_t ja = ts[t], jb = min(ts[t + 1], (uint32_t)K);
  const bool whole = hi - lo == kAggTile;
  const int nv = i0 < hi ? (int)min(4u, hi - i0) : 0;
  float gv[4], ev[4];
  if (whole) {
    load4gf<GDT>(g, i0, gv);
    load4f(e, i0, ev);
  } else {
    load4g<GDT>(g, i0, nv, gv);
    load4(e, i0, nv, ev);
  }
  *reinterpret_cast<int4*>(&slot[threadIdx.x * 4u]) = make_int4(-1, -1, -1, -1);
  __syncthreads();
  for (uint32_t j = ja + threadIdx.x; j < jb; j += kNT) {
    const uint32_t x = idx[j] - lo;
    if (x < kAggTile) slot[x] = (int32_t)j;
  }
  __syncthreads();
  const int4 sl = *reinterpret_cast<const int4*>(&slot[threadIdx.x * 4u]);
  const int32_t s4[4] = {sl.x, sl.y, sl.z, sl.w};
  float a[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    a[q] = gv[q] + ev[q];
    if (s4[q] >= 0) {
      val[s4[q]] = a[q];
      a[q] = 0.0f;
    }
  }
  if (whole) store4(e, i0, 4, a);
  else store4(e, i0, nv, a);
}

// Shared block starts: the column sums of the W workers' values (worker order, from +0.0).
__global__ __launch_bounds__(kNT) void k_shared_sum(int32_t W, int32_t K, const float* val, float* sum) {
  const uint32_t j = blockIdx.x * kNT + threadIdx.x;
  if (j < (uint32_t)K) sum[j] = column_sum(val, W, K, j);
}

// Standard SGD's exchange (no compression): out = (sum over workers in order, from +0.0) / W of
// the dense gradients g[W][d].  Two float4 groups per thread, one in each half of the groups, and
// the loads of kDenseBatch workers in flight together (16 workers on ResNet-50's d: 287 us, 76 %
// of 8 TB/s, against 305 us with one group and 8 loads in flight, 296 us with one group and 16).
constexpr int kDenseBatch = 16;
__global__ __launch_bounds__(kNT) void k_dense_average(int32_t d, int32_t W, const float* g, int average,
                                                       float* out) {
  const uint32_t ngr = ((uint32_t)d + 3u) / 4u;
  const uint32_t half = (ngr + 1u) / 2u;
  const uint32_t t = blockIdx.x * kNT + threadIdx.x;
  if (t >= half) return;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t gi = t + (uint32_t)h * half;
    if (gi >= ngr) break;
    const uint32_t i0 = gi * 4u;
    const int nv = (int)min(4u, (uint32_t)d - i0);
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int w0 = 0; w0 < W; w0 += kDenseBatch) {
      float v[kDenseBatch][4];
#pragma unroll
      for (int u = 0; u < kDenseBatch; ++u)
        if (w0 + u < W) load4(g + (size_t)(w0 + u) * d, i0, nv, v[u]);
#pragma unroll
      for (int u = 0; u < kDenseBatch; ++u)
        if (w0 + u < W)
#pragma unroll
          for (int q = 0; q < 4; ++q) s[q] += v[u][q];
    }
    const bool pow2 = (W & (W - 1)) == 0;
    const float inv = 1.0f / (float)W;
    float o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = average ? agg_scale(s[q], W, pow2, inv) : s[q];
    store4(out, i0, nv, o);
  }
}

// ---------------------------------------------------------------------------------------------
// Selection pipeline (top-k, random-k)
// KIND 0 = top-k: key' = magnitude bits of the value, the k largest are sent.
// KIND 1 = random-k: key' = ~Philox key, so the k smallest random keys have the largest key'.
// Among equal key', lower indices are sent first.
// ---------------------------------------------------------------------------------------------
template <int KIND>
__device__ __forceinline__ uint32_t sel_key(uint32_t idx, float val, uint32_t o, int l, uint32_t step,
                                            uint32_t s0, uint32_t s1) {
  if constexpr (KIND == 0) return mag_key(val);
  else return ~randk_key(idx - o, (uint32_t)l, step, s0, s1);
}

constexpr int kBatch = 8;             // independent loads in flight per thread in the selection passes
constexpr uint32_t kListLds = 8192;    // listed candidates held in LDS by k_select
constexpr uint32_t kRowsLds = 16384;   // rows per segment whose list additions k_select counts in LDS
constexpr uint32_t kRankList = 256;    // lists up to this size are ranked directly (no radix levels)
constexpr uint32_t kBigK = 1u << 20;   // layouts with a k_l this large count row winners in parallel
constexpr int32_t kBigRows = 16384;    // ... and so do layouts with a segment of more rows than this
constexpr uint32_t kSelPer = 8;        // rows per k_select thread held in registers
constexpr uint32_t kHistDirect = 32;   // rows with more candidates below the last bin histogram them in LDS first
constexpr int kHCopies = 16;           // copies of each candidate histogram (row r adds to copy r % 16)
constexpr uint32_t kDiagCount = 4u;    // diagnostics: the row counts of a segment did not add up to k_l
// R_IT of a top-k segment on a many-row layout whose threshold key T is shared by more listed
// candidates than win: k_rowcount counts each row's keys equal to T, k_rowtie finds the last
// winner among them (R_NEED of them win, in index order) and writes the real R_IT.
constexpr uint32_t kTieRows = 0xFFFFFFFEu;

// Workgroup-wide AND and OR of per-thread values; `lds` holds 2 * kSelNT / 64 words.
__device__ __forceinline__ void block_and_or(uint32_t& a, uint32_t& o, uint32_t* lds) {
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) {
    a &= __shfl_xor(a, s, 64);
    o |= __shfl_xor(o, s, 64);
  }
  constexpr int nw = kSelNT / 64;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) {
    lds[wid] = a;
    lds[nw + wid] = o;
  }
  __syncthreads();
  a = 0xFFFFFFFFu;
  o = 0u;
#pragma unroll
  for (int w = 0; w < nw; ++w) {
    a &= lds[w];
    o |= lds[nw + w];
  }
  __syncthreads();
}

// Calls fn(f, keys[f]) for every f < n, in a strided order with kBatch loads in flight.
template <int B = kBatch, typename K, typename F>
__device__ __forceinline__ void for_keys(const K& keys, uint32_t n, F fn) {
  for (uint32_t base = 0; base < n; base += (uint32_t)kSelNT * B) {
    uint32_t k[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const uint32_t f = base + (uint32_t)u * kSelNT + threadIdx.x;
      k[u] = f < n ? keys[f] : 0u;
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const uint32_t f = base + (uint32_t)u * kSelNT + threadIdx.x;
      if (f < n) fn(f, k[u]);
    }
  }
}

// A list in global memory, a wavefront per sub-list: the position within a sub-list is the address,
// where indexing the concatenation searched the sub-list bounds for every key (BERT flat at 10 %
// with bf16 values: the selection kernel's sweeps of a 211,000-key list took 97 us that way), and
// no sub-list waits for another (swept one after another by the whole workgroup, 38,000 keys kept
// two loads per thread in flight).  fn(f, key) gets the position f in the concatenation; fn2(f, key,
// address) also where the key lies in the list arrays.
static_assert(kSubLists == kSelNT / 64, "a wavefront per sub-list");
template <int B = kBatch, typename F>
__device__ __forceinline__ void for_keys2(const SubLists& L, F fn2) {
  const uint32_t c = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  uint32_t m0 = 0, m1 = 0;  // the bounds of sub-list c, selected without indexing M
#pragma unroll
  for (int x = 0; x <= kSubLists; ++x) {
    if (x == (int)c) m0 = L.M[x];
    if (x == (int)c + 1) m1 = L.M[x];
  }
  const uint32_t nc = m1 - m0;
  const size_t at = L.base + (size_t)c * L.q;
  const uint32_t* a = L.arr + at;
  for (uint32_t base = 0; base < nc; base += 64u * B) {
    uint32_t k[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const uint32_t j = base + (uint32_t)u * 64u + lane;
      k[u] = j < nc ? a[j] : 0u;
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const uint32_t j = base + (uint32_t)u * 64u + lane;
      if (j < nc) fn2(m0 + j, k[u], at + j);
    }
  }
}
template <int B = kBatch, typename F>
__device__ __forceinline__ void for_keys(const SubLists& L, uint32_t n, F fn) {
  (void)n;  // = L.M[kSubLists]
  for_keys2<B>(L, [&](uint32_t f, uint32_t k, size_t) { fn(f, k); });
}

// Exact selection over the whole segment (used when the candidates cannot contain the answer):
// radix levels over the keys of all d_l elements, then an index-ordered emission.
template <int KIND>
__device__ void slow_select(const Tables& T, int l, const float* data, float* e_zero, uint32_t* out_idx,
                            float* out_val, uint32_t s0, uint32_t s1, uint32_t step, uint32_t* hist, uint32_t* lds) {
  const uint32_t o = (uint32_t)T.seg_off[l], n = (uint32_t)T.seg_off[l + 1] - o;
  const uint32_t P = (uint32_t)T.seg_P[l], kl = (uint32_t)T.seg_k[l];
  // random-k keys depend on the position only: without data (a selection prepared ahead of the
  // step) only the indices are written
  auto keyat = [&](uint32_t j) -> uint32_t {
    return sel_key<KIND>(o + j, KIND == 1 && !data ? 0.0f : data[o + j], o, l, step, s0, s1);
  };
  uint32_t prefix = 0, need = kl;
  int known = 0;
  while (known < 32) {
    const int w = min(11, 32 - known);
    const int shift = 32 - known - w;
    for (int b = threadIdx.x; b < (1 << w); b += kSelNT) hist[b] = 0;
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < n; j += kSelNT) {
      const uint32_t k = keyat(j);
      if (known == 0 || (k >> (32 - known)) == (prefix >> (32 - known)))
        atomicAdd(&hist[(k >> shift) & ((1u << w) - 1u)], 1u);
    }
    __syncthreads();
    uint32_t above;
    const int bin = block_resolve<kSelNT>(hist, 1 << w, need, lds, above);
    prefix |= (uint32_t)max(bin, 0) << shift;
    need -= above;
    known += w;
  }
  const uint32_t Tk = prefix, r = need;
  uint32_t run_a = 0, run_b = 0;
  for (uint32_t j0 = 0; j0 < n; j0 += kSelNT) {
    const uint32_t j = j0 + threadIdx.x;
    uint32_t a = 0, b = 0;
    if (j < n) {
      const uint32_t k = keyat(j);
      a = k > Tk;
      b = k == Tk;
    }
    uint32_t tot;
    const uint32_t ex = block_excl_scan<kSelNT>(a | (b << 16), lds, tot);
    const uint32_t ea = run_a + (ex & 0xFFFFu), eb = run_b + (ex >> 16);
    if ((a || (b && eb < r)) && ea + min(eb, r) < kl) {
      const uint32_t pos = P + ea + min(eb, r);
      out_idx[pos] = o + j;
      if (out_val) out_val[pos] = data[o + j];
      if (e_zero) e_zero[o + j] = 0.0f;
    }
    run_a += tot & 0xFFFFu;
    run_b += tot >> 16;
  }
}

// ---------------------------------------------------------------------------------------------
// Workgroup helpers of the per-segment kernels (kSelNT threads)
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t block_max_u32(uint32_t v, uint32_t* lds) {
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) v = max(v, (uint32_t)__shfl_xor(v, s, 64));
  constexpr int nw = kSelNT / 64;
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  v = 0;
#pragma unroll
  for (int w = 0; w < nw; ++w) v = max(v, lds[w]);
  __syncthreads();
  return v;
}

// Position of the r-th (1-based) entry equal to x among keys[0, m), in position order.  Each
// wave owns a contiguous share of the positions; `lds` holds kSelNT / 64 words.
template <typename K>
__device__ __forceinline__ uint32_t block_nth_equal(const K& keys, uint32_t m, uint32_t x, uint32_t r, uint32_t* lds) {
  __shared__ uint32_t s_pos;
  constexpr int NW = kSelNT / 64;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t W0 = (uint32_t)(((uint64_t)m * wid) / NW), W1 = (uint32_t)(((uint64_t)m * (wid + 1)) / NW);
  uint32_t cnt = 0;
  for (uint32_t b = W0; b < W1; b += 64) {
    const uint32_t f = b + lane;
    cnt += (uint32_t)__popcll(__ballot(f < W1 && keys[f] == x));
  }
  if (lane == 0) lds[wid] = cnt;
  if (threadIdx.x == 0) s_pos = m;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wid; ++w) before += lds[w];
  if (before < r && r <= before + cnt) {  // wave-uniform: this wave holds the r-th match
    uint32_t run = before;
    for (uint32_t b = W0; b < W1; b += 64) {
      const uint32_t f = b + lane;
      const bool t = f < W1 && keys[f] == x;
      const uint64_t mk = __ballot(t);
      const uint32_t c = (uint32_t)__popcll(mk);
      if (run + c >= r) {
        if (t && run + lanes_below(mk) + 1 == r) s_pos = f;
        break;
      }
      run += c;
    }
  }
  __syncthreads();
  const uint32_t p = s_pos;
  __syncthreads();
  return p;
}

// The r-th smallest idx[j] (r >= 1, indices distinct) among the j < m with keys[j] == x: radix
// levels over ~idx, whose largest values are the smallest indices.
template <typename K, typename I>
__device__ __forceinline__ uint32_t block_nth_smallest_tie(const K& keys, const I& idx, uint32_t m, uint32_t x,
                                           uint32_t r, uint32_t* hist, uint32_t* lds) {
  uint32_t prefix = 0, need = r;
  int known = 0;
  while (known < 32) {
    const int w = min(11, 32 - known);
    const int shift = 32 - known - w;
    for (int b = threadIdx.x; b < (1 << w); b += kSelNT) hist[b] = 0;
    __syncthreads();
    const uint32_t pmask = known == 0 ? 0u : (0xFFFFFFFFu << (32 - known));
    for (uint32_t j = threadIdx.x; j < m; j += kSelNT) {
      if (keys[j] == x) {
        const uint32_t v = ~idx[j];
        if ((v & pmask) == (prefix & pmask)) atomicAdd(&hist[(v >> shift) & ((1u << w) - 1u)], 1u);
      }
    }
    __syncthreads();
    uint32_t above;
    const int bin = block_resolve<kSelNT>(hist, 1 << w, need, lds, above);
    prefix |= (uint32_t)max(bin, 0) << shift;
    need -= above;
    known += w;
  }
  return ~prefix;
}

// Candidate histogram bin of a top-k key >= A (higher bins hold larger keys).  Bin 0 holds the
// key A alone, so that a threshold landing on a value shared by very many elements (exact zeros,
// say) is recognised as a pure tie; larger keys go to 1 + ((key - A - 1) >> sh), clamped to the
// last bin.
__device__ __forceinline__ uint32_t cand_bin(uint32_t key, uint32_t A, uint32_t sh) {
  return key == A ? 0u : 1u + min((key - A - 1u) >> sh, (uint32_t)kHBins - 2u);
}

// The least key of the last bin (a key the bins cannot reach: 2^32 - 1, above every magnitude).
__device__ __forceinline__ uint32_t last_bin_key(uint32_t A, uint32_t sh) {
  const uint64_t t = (uint64_t)A + 1u + ((uint64_t)(kHBins - 2u) << sh);
  return (uint32_t)min<uint64_t>(t, 0xFFFFFFFFull);
}

// Magnitude keys of acc read in place (a row's elements equal to A are counted, not stored).
struct AccKeys {
  const float* p;
  __device__ __forceinline__ uint32_t operator[](uint32_t f) const { return mag_key(p[f]); }
};

// The first and one past the last element of a row.
__device__ __forceinline__ void row_bounds(const Tables& T, uint32_t row, uint32_t& lo, uint32_t& hi) {
  uint32_t o = 0, e_ = (uint32_t)T.d, tb = row * kTile;
  if (T.L > 1) {
    const uint4 rr = reinterpret_cast<const uint4*>(T.row_rec)[row];
    o = rr.y;
    e_ = rr.z;
    tb = rr.w;
  }
  lo = max(o, tb);
  hi = min(e_, tb + kTile);
}

// LDS histogram add of one key per active lane: the lanes whose bin is the first active lane's
// add together with one atomic, the others one by one.  Sample keys crowd a few bins (BERT's
// gradients: a histogram of 65,536 of them took 20 us with an atomic per key, same-address
// atomics of one wavefront being serialised; the sample selection 36 -> 28 us this way).
__device__ __forceinline__ void hist_add_peel(uint32_t* h, uint32_t b) {
  const uint32_t b0 = __builtin_amdgcn_readfirstlane(b);
  const uint64_t same = __ballot(b == b0);
  if (b != b0) atomicAdd(&h[b], 1u);
  else if ((threadIdx.x & 63u) == (uint32_t)(__ffsll((long long)same) - 1)) atomicAdd(&h[b0], (uint32_t)__popcll(same));
}

// ---------------------------------------------------------------------------------------------
// Top-k sample
// ---------------------------------------------------------------------------------------------
// One workgroup of kSampleRun threads per run: a segment of up to kExactMax elements is sampled
// whole (runs of consecutive positions).  A larger one, given s = runs * kSampleRun samples by the
// layout (a share of its samples in proportion to its size, at least kSampleMinRuns runs), is
// split into s strata of equal length (to within one element) and sampled once in each, at a
// pseudo-random position inside the stratum (stratified sampling): every part of the segment, a
// small tensor of large values inside a flat gradient included, is represented in proportion to
// its size, and the count of sampled keys above a value varies no more than a simple random
// sample's would (runs of contiguous elements, by contrast, sample a handful of clusters: a small
// tensor is either missed or over-represented many times).  Sample q = run * kSampleRun + thread;
// the runs of a sampled segment also clear its candidate histogram (kHCopies * kHBins words).
static_assert(kExactMax % kSelNT == 0, "whole sample keys per thread");
static_assert(2 * kRankList <= kHBins, "the ranked entries (64-bit words) of an exact segment fit a histogram array");

// Positions 0, 1, ... as the indices of keys held in position order.
struct LocalPos {
  __device__ uint32_t operator[](uint32_t f) const { return f; }
};
template <typename K, typename I>
__device__ __forceinline__ void list_threshold_ao(const K& key, const I& idx, uint32_t m, uint32_t need,
                                                  uint32_t kand, uint32_t kor, uint32_t* hist, uint32_t* lds,
                                                  uint64_t* g, uint32_t& T_out, uint32_t& IT_out,
                                                  uint32_t* defer_need = nullptr);
template <int GDT, bool FUSED>
__global__ __launch_bounds__(kSampleRun) void k_sample_gather(Tables T, WSel ws0, Batch BT) {
  const WSel ws = ws_at(ws0, (uint64_t)blockIdx.y * BT.ws);
  const void* g = BT.g[blockIdx.y];
  const float* src = BT.src[blockIdx.y];
  const uint32_t r = blockIdx.x;
  // a table lookup: one round trip instead of a binary search's chain (none for one segment)
  const int l = T.L == 1 ? 0 : T.run_seg[r];
  const uint32_t o = (uint32_t)T.seg_off[l], n = (uint32_t)T.seg_off[l + 1] - o;
  const uint32_t q = r - (uint32_t)T.seg_ro[l];
  uint32_t i;
  bool in = true;
  if (n <= (uint32_t)kExactMax) {
    const uint32_t j = q * kSampleRun + threadIdx.x;
    in = j < n;
    i = o + j;
  } else {
    const uint32_t ns = ((uint32_t)T.seg_ro[l + 1] - (uint32_t)T.seg_ro[l]) * kSampleRun;  // samples
    const uint32_t sq = q * kSampleRun + threadIdx.x;  // the stratum
    const uint32_t a = (uint32_t)(((uint64_t)sq * n) / ns);
    const uint32_t b = (uint32_t)(((uint64_t)(sq + 1u) * n) / ns);
    const uint32_t x = philox(make_uint4(sq, 0u, 0u, kSampleTag | (uint32_t)l), 0u, 0u).x;
    i = o + a + __umulhi(x, b - a);  // uniform in [a, b): b > a because ns <= n (runs <= n / kSampleRun)
    for (uint32_t h = sq; h < (uint32_t)(kHCopies * kHBins); h += ns) ws.hist[(size_t)l * kHCopies * kHBins + h] = 0u;
  }
  // the overflow pool's counters start from zero (the first kernel of a top-k step)
  if (r == 0 && threadIdx.x < (unsigned)kPools) *pcnt_of(ws, threadIdx.x) = 0u;
  uint32_t key = 0;
  if (in) {
    float a;
    if constexpr (FUSED) a = load1g<GDT>(g, i) + src[i];
    else a = src[i];
    key = mag_key(a);
  }
  ws.samp[(size_t)r * kSampleRun + threadIdx.x] = key;
}

// Per segment (one workgroup) the candidate rule of the streaming pass:
//  * at most kExactMax elements: the exact k_l-th largest key T over the whole segment and the
//    bound I (one past the index of the last tie sent; ties go to lower indices); the candidates
//    are then exactly the winners (mode 1).
//  * larger segments: A = the lower edge of the bin of the top 11 key bits that holds the
//    srank-th largest sampled key (srank: the expected rank of the k_l-th key in the sample plus
//    a margin); every key >= A is a candidate.  The candidates are histogrammed in bins of 2^sh
//    keys above A, sh chosen so that the range up to the urank-th sampled key (the expected rank
//    minus the margin) spans about 1024 bins: the k_l-th key very likely falls inside it, and the
//    bins there are as narrow as the sample allows (mode 0).
// R_Z (seg_zc): the key from which the pass stores +0, near the k_l-th largest.  With kMidRank and more
// samples expected above it the two edges are close and their middle in key space does (BERT flat at
// 1 %, 164 of them: the emission 16.5 us; by the rank below 27, where the residual gathers under the
// threshold inside one bin).  With fewer the upper edge lies far off (at ten, at the sample's largest
// key) and the middle left most winners below it: there R_Z is the expected rank's own key, interpolated
// in its bin (BERT per layer at 1.5 %: the emission 33 -> 31 us, ResNet-50 per layer at 3 % 14.5 -> 10.9).
constexpr uint32_t kMidRank = 64;
__global__ __launch_bounds__(kSelNT) void k_sample_select(Tables T, WSel ws0, Batch BT) {
  const WSel ws = ws_at(ws0, (uint64_t)blockIdx.y * BT.ws);
  __shared__ uint32_t keys[kExactMax];
  __shared__ uint32_t hist[kHBins];
  __shared__ __align__(8) uint32_t hist2[kHBins];
  __shared__ uint32_t lds[2 * kSelNT / 64];
  const int l = blockIdx.x;
  const uint32_t o = (uint32_t)T.seg_off[l], n = (uint32_t)T.seg_off[l + 1] - o;
  const uint32_t* sk = ws.samp + (size_t)T.seg_ro[l] * kSampleRun;
  uint32_t* R = res_of(ws, l);
  if (n <= (uint32_t)kExactMax) {
    uint32_t kand = 0xFFFFFFFFu, kor = 0u;
    for_keys<kExactMax / kSelNT>(sk, n, [&](uint32_t f, uint32_t k) {
      keys[f] = k;
      kand &= k;
      kor |= k;
    });
    block_and_or(kand, kor, lds);  // its barriers also publish keys[]
    // the k_l best of the segment's keys (positions as indices): hist2 holds the ranked entries
    uint32_t Tk, IT;
    list_threshold_ao(keys, LocalPos{}, n, (uint32_t)T.seg_k[l], kand, kor, hist, lds,
                      reinterpret_cast<uint64_t*>(hist2), Tk, IT);
    const uint32_t it = IT == 0xFFFFFFFFu ? IT : o + IT;  // every tie wins, or one past the last
    if (threadIdx.x == 0) {
      R[R_A] = Tk;
      R[R_IA] = it;
      R[R_T] = Tk;
      R[R_IT] = it;
      R[R_MODE] = 1;
      R[R_SLOW] = 0;
      R[R_OVF] = 0;
    }
    return;
  }
  // sampled: bins of the top 11 key bits (8 exponent + 3 mantissa bits)
  const uint32_t ns = ((uint32_t)T.seg_ro[l + 1] - (uint32_t)T.seg_ro[l]) * kSampleRun;  // samples
  for (int b = threadIdx.x; b < kHBins; b += kSelNT) hist[b] = 0;
  __syncthreads();
  // Samples of up to NK keys per thread stay in registers through the refinements (a 65,536-key sample
  // read again for each edge: BERT flat at 10 %, 27.1 us for this kernel, 22.7 now); larger ones are read
  // again.
  auto rule = [&](auto per) {
    constexpr int NK = decltype(per)::value;
    uint32_t k[NK > 0 ? NK : 1];
    if constexpr (NK > 0) {
#pragma unroll
      for (int u = 0; u < NK; ++u) {
        const uint32_t f = (uint32_t)u * kSelNT + threadIdx.x;
        k[u] = f < ns ? sk[f] : 0u;
      }
    }
    // every sampled key in turn, f < ns
    auto each = [&](auto fn) {
      if constexpr (NK > 0) {
#pragma unroll
        for (int u = 0; u < NK; ++u)
          if ((uint32_t)u * kSelNT + threadIdx.x < ns) fn(k[u]);
      } else {
        for_keys(sk, ns, [&](uint32_t, uint32_t x) { fn(x); });
      }
    };
    uint32_t kmax = 0u;
    // (the enlarged samples of dense layouts: the peeled add; a 16,384-key sample of ResNet-50's
    // gradients took 1 us longer with it than with an atomic per key)
    each([&](uint32_t x) {
      if constexpr (NK == 0 || NK > kSampleTotal / kSelNT) hist_add_peel(hist, x >> 20);
      else atomicAdd(&hist[x >> 20], 1u);
      kmax = max(kmax, x);
    });
    __syncthreads();
    kmax = block_max_u32(kmax, lds);
    // Key edge of the rank-th largest sampled key: the lower (or upper) edge of its top-11-bit bin,
    // refined by the next 11 bits when that bin holds more than 64 sampled keys (concentrated
    // values: an unrefined edge could take up to the whole bin's keys as candidates beyond the
    // rank, which the candidate pool is not sized for).  Both ranks' bins come from one scan of
    // the histogram.
    const uint32_t rank = (uint32_t)T.seg_srank[l], urank = (uint32_t)T.seg_urank[l];
    int bin_t, bin_u;
    uint32_t above_t, above_u;
    block_resolve2<kSelNT>(hist, kHBins, rank < ns ? rank : 0u, urank, lds, bin_t, above_t, bin_u, above_u);
    auto rank_edge = [&](int bin, uint32_t above, uint32_t rk, bool upper) -> uint32_t {
      if (bin < 0) return 0u;
      if (hist[bin] <= 64u) return ((uint32_t)bin + (upper ? 1u : 0u)) << 20;
      for (int b = threadIdx.x; b < kHBins; b += kSelNT) hist2[b] = 0;
      __syncthreads();
      each([&](uint32_t x) {
        if ((x >> 20) == (uint32_t)bin) atomicAdd(&hist2[(x >> 9) & (kHBins - 1)], 1u);
      });
      __syncthreads();
      uint32_t above2;
      const int bin2 = block_resolve<kSelNT>(hist2, kHBins, rk - above, lds, above2);
      return ((uint32_t)bin << 20) + (((uint32_t)max(bin2, 0) + (upper ? 1u : 0u)) << 9);
    };
    // rank >= sample size: every element is a candidate
    const uint32_t thr = rank < ns ? rank_edge(bin_t, above_t, rank, false) : 0u;
    // the bins resolve the range up to the upper edge of where the k-th key very likely lies
    uint32_t top = rank_edge(bin_u, above_u, urank, true);
    if (top <= thr || top > kmax) top = kmax;
    const uint32_t span = top - thr;
    // the least shift whose bins 1 .. kHBins - 2 hold the span (2^11 - 2 of them: span < 2^b gives at
    // most 2^10 bins with a shift of b - 10, and one bit less where that still fits)
    uint32_t sh = span < 1024u ? 0u : (uint32_t)(32 - __clz(span)) - 10u;
    if (sh && (span >> (sh - 1u)) < (uint32_t)kHBins - 2u) --sh;
    uint32_t z = thr + (top - thr) / 2u;
    const uint32_t mid = (uint32_t)((uint64_t)ns * (uint32_t)T.seg_k[l] / n);
    if (T.seg_zc[l] && mid - 1u < kMidRank - 1u) {  // uniform
      uint32_t above_m;
      const int bin_m = block_resolve<kSelNT>(hist, kHBins, mid, lds, above_m);
      // (the sample holds more than mid keys: the bin is there and not empty)
      const uint32_t below = ((2u * (mid - above_m) - 1u) << 19) / hist[bin_m];  // from the bin's upper edge
      z = max((((uint32_t)bin_m + 1u) << 20) - below, thr);
    }
    if (threadIdx.x == 0) {
      R[R_A] = thr;
      R[R_Z] = z + 1u;
      R[R_IA] = 0xFFFFFFFFu;
      R[R_SH] = sh;
      R[R_MODE] = 0;
      R[R_SLOW] = 0;
      R[R_OVF] = 0;
    }
  };
  if (ns <= 4u * kSelNT) rule(std::integral_constant<int, 4>{});
  else if (ns <= (uint32_t)kSampleTotal) rule(std::integral_constant<int, kSampleTotal / kSelNT>{});
  else if (ns <= (uint32_t)kSampleCap) rule(std::integral_constant<int, kSampleCap / kSelNT>{});
  else rule(std::integral_constant<int, 0>{});
}

// ---------------------------------------------------------------------------------------------
// Streaming pass: fused accumulate + candidate test + ordered compaction into the row's slot
// (+ top-k: candidate histogram).  One workgroup of kStrNT threads per row.
// ---------------------------------------------------------------------------------------------
// Threads per workgroup of the streaming selection pass: two float4 groups per thread (a row of
// kTile elements per workgroup).  Measured per pass on ResNet-50 flat, top-k / random-k: 256
// threads (4 groups each) 52.0 / 52.2 us, 512 threads 50.5 / 51.0, 1024 threads 53.1 / 55.8 (one
// barrier across 16 wavefronts holds the whole row back).
constexpr int kStrNT = 512;
constexpr int kStrW = kStrNT / 64;     // its wavefronts

// Its LDS.
template <int KIND>
struct StreamLds {
  uint32_t wt[16];                          // candidates by group and wavefront (group-major)
  uint32_t tie[8];                          // top-k: elements equal to A, and candidates of the last bin << 16
  uint32_t cert[8];                         // random-k: certain winners by wavefront
  uint32_t und;                             // random-k, direct lists: undecided candidates listed so far
  uint32_t cb;                              // the row's first pool entry (a reservation in the overflow pool)
  uint32_t hist[KIND == 0 ? kHBins : 1];
};

// The pass is close to being bound by its instructions (a row's 48 KB pass a CU in about 4700 cycles),
// so what a row's lanes share is kept in scalar registers: candidate sets as lane masks (a compare's
// own result), counts as their population counts.  WHOLE: the row is a whole data tile (all but a
// segment's ends): no element is masked.  Candidates take six bytes (value, place in the tile), top-k's
// keys being the values' magnitudes.  Against per-lane flags, masks on every row and twelve-byte
// candidates: 1e9 elements at 1 %, random-k, bf16 1727 -> 1602 us (10.1 GB, 1575 us at the 6.4 TB/s
// that plain streaming reaches); BERT per layer at 1 %, top-k, bf16 216 -> 198 us (172), flat at 10 %
// 264 -> 234 us (219); ResNet-18 per layer at 1 %, random-k 27.6 -> 25.7 us (22).
// (Measured and slower: candidates staged in LDS and stored by coalesced instructions, with the
// histogram cleared and counted before the row's barrier, BERT per layer 210 -> 218 us, for its two
// more barriers; histogram rows of up to 256 keys added to global memory without LDS, 218 -> 395 us.)
template <int KIND, int GDT, bool FUSED, bool ZC, bool DIRECT, bool WHOLE>
__device__ __forceinline__ void stream_row(const Tables& T, const void* g, const float* src, float* acc_out, uint32_t s0,
                                           uint32_t s1, uint32_t step, const WSel& ws, StreamLds<KIND>& S, uint32_t row,
                                           int l, uint32_t o, uint32_t tb, uint32_t lo, uint32_t hi, uint32_t cb,
                                           uint32_t scap) {
  constexpr int kSR = (int)kTile / (4 * kStrNT);  // float4 groups per thread
  static_assert(kSR * kStrW == 16 && kStrW == 8, "a row's counts fit 16 lanes");
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wid = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  uint32_t* R = res_of(ws, l);
  uint32_t mode = 1, A = 0, IA = 0, sh = 0, ulo = 0, tlast = 0;
  bool zc = false;           // top-k, fused: +0 stored at the candidates from key zk on, not acc
  uint32_t zk = 0xFFFFFFFFu;
  if constexpr (KIND == 0) {
    mode = R[R_MODE];
    A = R[R_A];
    IA = R[R_IA];
    sh = R[R_SH];
    zc = ZC && FUSED && T.seg_zc[l] != 0u;
    if (zc) zk = R[R_Z];
  } else {
    tlast = (uint32_t)(T.seg_tau[l] - 1u);  // the largest candidate key
    ulo = T.seg_ulo[l];
    // the counters of k_collect_randk start from zero (this kernel completes before it runs)
    if (!DIRECT && tb == o / kTile * kTile) {
      if (threadIdx.x < kSubLists) *lcnt_of(ws, l, threadIdx.x) = 0u;
      else if (threadIdx.x < 2 * kSubLists) *scnt_of(ws, l, threadIdx.x - kSubLists) = 0u;
      else if (threadIdx.x == 2 * kSubLists) R[R_OVF] = 0u;
    }
  }
  float v[kSR][4];
  uint32_t vm[kSR];
  uint32_t i0[kSR];
#pragma unroll
  for (int r = 0; r < kSR; ++r) {
    i0[r] = tb + (uint32_t)(r * kStrNT + threadIdx.x) * 4u;
    vm[r] = WHOLE ? 0xFu : group_mask(i0[r], lo, hi);
  }
  auto in = [&](int r, int q) { return WHOLE || ((vm[r] >> q) & 1u); };
  auto store = [&](int r, const float x[4]) {
    if constexpr (WHOLE) store4(acc_out, i0[r], 4, x);
    else store4m(acc_out, i0[r], vm[r], x);
  };
  float gv[kSR][4];
  const bool data = !(KIND == 1 && !FUSED && !src);  // none: a random-k selection prepared ahead of the step
#pragma unroll
  for (int r = 0; r < kSR; ++r) {
    if constexpr (FUSED) {
      if constexpr (WHOLE) load4gf<GDT>(g, i0[r], gv[r]);
      else load4gm<GDT>(g, i0[r], vm[r], gv[r]);
    }
    if (data) {
      if constexpr (WHOLE) load4f(src, i0[r], v[r]);
      else load4m(src, i0[r], vm[r], v[r]);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[r][q] = 0.0f;
    }
  }
  // random-k: the Philox keys of the thread's elements depend on positions only; they are computed
  // while the thread's loads are in flight
  uint32_t uk[KIND == 1 ? kSR : 1][4];
  if constexpr (KIND == 1) {
#pragma unroll
    for (int r = 0; r < kSR; ++r) {
      if ((o & 3u) == 0) {  // the float4 group is one Philox block
        uint4 x = make_uint4(0u, 0u, 0u, 0u);
        if (vm[r]) x = philox(make_uint4((i0[r] - o) >> 2, 0u, step, kRandkTag | (uint32_t)l), s0, s1);
#pragma unroll
        for (int q = 0; q < 4; ++q) uk[r][q] = word(x, q);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) uk[r][q] = in(r, q) ? randk_key(i0[r] + q - o, (uint32_t)l, step, s0, s1) : 0u;
      }
    }
  }
  uint64_t cm[kSR][4];   // the wavefront's candidates
  uint64_t wm[KIND == 1 ? kSR : 1][4];  // random-k: those that are certain winners (key below ulo)
  uint32_t n[kSR];       // their number
  uint32_t ncert = 0, ntie = 0, nlast = 0;
  const uint32_t top = ZC ? last_bin_key(A, sh) : 0xFFFFFFFFu;
#pragma unroll
  for (int r = 0; r < kSR; ++r) {
    if constexpr (FUSED) {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[r][q] = gv[r][q] + v[r][q];
      if (KIND == 0 && !zc) store(r, v[r]);
    }
    n[r] = 0;
    float z[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      bool c;
      if constexpr (KIND == 0) {
        // sampled segments: keys above A are stored, keys equal to A (the tie bin: exact zeros, say,
        // which may be most of a segment) only counted; exact segments: the winner rule itself
        const uint32_t k = mag_key(v[r][q]);
        const uint64_t gt = __ballot(in(r, q) && k > A), eq = __ballot(in(r, q) && k == A);
        cm[r][q] = gt;
        if (mode == 0) {
          ntie += (uint32_t)__popcll(eq);
          if constexpr (ZC) nlast += (uint32_t)__popcll(__ballot(in(r, q) && k >= top));
        } else if (eq) {
          cm[r][q] = gt | __ballot(in(r, q) && k == A && i0[r] + q < IA);
        }
        c = k >= zk;  // (above A: a candidate)
      } else {
        c = in(r, q) && uk[r][q] <= tlast;
        cm[r][q] = __ballot(c);
        wm[r][q] = __ballot(in(r, q) && uk[r][q] < ulo);
        ncert += (uint32_t)__popcll(wm[r][q]);
      }
      n[r] += (uint32_t)__popcll(cm[r][q]);
      z[q] = c ? 0.0f : v[r][q];
    }
    // +0 stored at the candidates, whose losers the emission restores: random-k (the window's losers
    // are few, about 6 sqrt(k_l) + 32 of a segment; zeroing the winners afterwards instead wrote
    // single words into lines long evicted from the caches: 1e9 elements at 10 %, 1.9 of the
    // emission's 2.3 ms) and top-k segments with seg_zc, there from the key R_Z on, where the k_l-th key
    // is expected.  The exact path puts them all back first.
    if (FUSED && (KIND == 1 || zc)) store(r, z);
    if (lane == 0) S.wt[r * kStrW + wid] = n[r];
  }
  if (lane == 0) {
    if constexpr (KIND == 1) S.cert[wid] = ncert;
    else S.tie[wid] = ntie | (nlast << 16);  // (a wavefront has 512 elements)
  }
  if (KIND == 1 && threadIdx.x == 0) S.und = 0;
  __syncthreads();
  // the row's candidates go to its static slot, or, when there are more than it holds, to entries
  // reserved in the overflow pool; a row that does not fit is dropped and its segment takes the
  // exact path (the histogram still counts its candidates)
  const uint32_t cnt16 = S.wt[lane & 15u], side = KIND == 0 ? S.tie[lane & 7u] : S.cert[lane & 7u];
  const uint32_t inc = row16_incl_scan(cnt16);
  const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)inc, 15);
  const uint32_t all = row8_sum(side);  // ties | last << 16; certain winners
  if (tot > scap) {
    if (threadIdx.x == 0) S.cb = pool_reserve(ws, row, tot);
    __syncthreads();
    cb = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.cb);
  }
  const bool dropped = cb == kDropped;
  if (threadIdx.x == 0) {
    if (T.L > 1 || tot > scap) ws.coff[row] = cb;
    ws.counts[row] = tot;
    if (KIND == 1) ws.rcnt[row] = all;  // its certain winners (key below ulo)
  }
  if (dropped) {
    if constexpr (KIND == 0) {
      if (threadIdx.x == 0) atomicOr(&R[R_OVF], 1u);
    }
    if (FUSED && (KIND == 1 || zc)) {
      // the candidates' values were stored as +0 above; without the candidates the exact path
      // cannot restore them, so they are stored again now
#pragma unroll
      for (int r = 0; r < kSR; ++r) store(r, v[r]);
    }
  }
  uint32_t* gh = KIND == 0 ? ws.hist + ((size_t)l * kHCopies + (row % kHCopies)) * kHBins : nullptr;
  if (KIND == 0 && mode == 0 && threadIdx.x == 0) {
    // the ties are the histogram's bin 0
    const uint32_t tie = all & 0xFFFFu, last = all >> 16;
    ws.rtie[row] = tie;
    if (tie) atomicAdd(gh, tie);
    if (ZC && last) atomicAdd(gh + kHBins - 1, last);
  }
#pragma unroll
  for (int r = 0; r < kSR; ++r) {
    if (n[r] && !dropped) {  // uniform
      uint32_t pos = cb + (uint32_t)__builtin_amdgcn_readlane((int)(inc - cnt16), (int)(r * kStrW + wid));
#pragma unroll
      for (int q = 0; q < 4; ++q) pos += lanes_below(cm[r][q]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (__builtin_amdgcn_inverse_ballot_w64(cm[r][q])) {
          const uint32_t x = i0[r] - tb + q;
          const bool certain = KIND == 1 && __builtin_amdgcn_inverse_ballot_w64(wm[r][q]);
          ws.cand_loc[pos] = (uint16_t)(certain ? x | kCertain : x);
          ws.cand_val[pos] = v[r][q];
          if (KIND == 1 && !certain) {
            const uint32_t key = ~uk[r][q];
            ws.cand_key[pos] = key;
            if constexpr (DIRECT) {
              // direct lists: (key', index) pairs at the row's pool entries in the pair array (fewer
              // than its candidates)
              const uint32_t p = atomicAdd(&S.und, 1u);
              ws.pairs[(size_t)cb + p] = make_uint2(key, tb + x);
            }
          }
          ++pos;
        }
      }
    }
  }
  if constexpr (KIND == 0) {
    const uint32_t below = tot - (ZC ? all >> 16 : 0u);  // candidates below the last bin (without ZC: all)
    if (mode == 0 && below) {
      if (below > kHistDirect) {  // many: count them in LDS, then one atomic per used bin
        for (int b = threadIdx.x; b < kHBins; b += kStrNT) S.hist[b] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSR; ++r)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (n[r] && __builtin_amdgcn_inverse_ballot_w64(cm[r][q])) {
              const uint32_t k = mag_key(v[r][q]);
              if (!ZC || k < top) atomicAdd(&S.hist[cand_bin(k, A, sh)], 1u);
            }
        __syncthreads();
        for (int b = threadIdx.x; b < kHBins; b += kStrNT) {
          const uint32_t c = S.hist[b];
          if (c) atomicAdd(&gh[b], c);
        }
      } else {
#pragma unroll
        for (int r = 0; r < kSR; ++r)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (n[r] && __builtin_amdgcn_inverse_ballot_w64(cm[r][q])) {
              const uint32_t k = mag_key(v[r][q]);
              if (!ZC || k < top) atomicAdd(&gh[cand_bin(k, A, sh)], 1u);
            }
      }
    }
  }
}

// ZC: some top-k segment of the layout has seg_zc (the form without it has no such test, nor the last
// bin's count by ballot: the last bin holds most of a dense segment's candidates, few of the others').
// DIRECT: random-k with direct lists (T.rk_direct).
template <int KIND, int GDT, bool FUSED, bool ZC = false, bool DIRECT = false>
__global__ __launch_bounds__(kStrNT) void k_stream_sel(Tables T, const void* g, const float* src, float* acc_out,
                                                    uint32_t s0, uint32_t s1, uint32_t step, WSel ws) {
  __shared__ StreamLds<KIND> S;
  const uint32_t row = blockIdx.x;
  // the row's segment and bounds: arithmetic on one segment, else one record load (the data loads
  // wait for the bounds only, not for a chain through the segment tables)
  int l = 0;
  uint32_t o = 0, e_ = (uint32_t)T.d, tb = row * kTile;
  uint32_t cb, scap;  // the row's static slot (several segments: loaded with the row's record)
  if (T.L > 1) {
    const uint4 rr = reinterpret_cast<const uint4*>(T.row_rec)[row];
    cb = ws.soff[row];
    scap = ws.soff[row + 1];
    l = (int)rr.x;
    o = rr.y;
    e_ = rr.z;
    tb = rr.w;
    scap -= cb;
  } else {
    static_slot(T, ws, row, cb, scap);
  }
  const uint32_t lo = max(o, tb), hi = min(e_, tb + kTile);
  if (lo == tb && hi == tb + kTile)
    stream_row<KIND, GDT, FUSED, ZC, DIRECT, true>(T, g, src, acc_out, s0, s1, step, ws, S, row, l, o, tb, lo, hi, cb, scap);
  else
    stream_row<KIND, GDT, FUSED, ZC, DIRECT, false>(T, g, src, acc_out, s0, s1, step, ws, S, row, l, o, tb, lo, hi, cb, scap);
}

// Top-k, per segment: the histogram bin B holding the k_l-th best candidate and how many winners
// it still has to give; fewer than k_l candidates in all marks the segment for the exact path.
__global__ __launch_bounds__(kSelNT) void k_resolve(Tables T, WSel ws0, Batch BT) {
  const WSel ws = ws_at(ws0, (uint64_t)blockIdx.y * BT.ws);
  __shared__ uint32_t hist[kHBins];
  __shared__ uint32_t lds[2 * kSelNT / 64];
  const int l = blockIdx.x;
  uint32_t* R = res_of(ws, l);
  // the segment's mode and every copy of its histogram in one round trip (a segment of mode 1 has
  // no histogram: its loads read the unused copies and are dropped)
  constexpr int kPer = kHBins / kSelNT;
  static_assert(kHBins % kSelNT == 0, "whole bins per thread");
  const uint32_t mode = R[R_MODE], ovf = R[R_OVF];
  const uint32_t* gh = ws.hist + (size_t)l * kHCopies * kHBins;
  uint32_t c[kPer][kHCopies];
#pragma unroll
  for (int u = 0; u < kPer; ++u)
#pragma unroll
    for (int x = 0; x < kHCopies; ++x) c[u][x] = gh[x * kHBins + u * kSelNT + threadIdx.x];
  if (mode != 0) return;
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    uint32_t sum = 0;
#pragma unroll
    for (int x = 0; x < kHCopies; ++x) sum += c[u][x];
    hist[u * kSelNT + threadIdx.x] = sum;
  }
  __syncthreads();
  const uint32_t kl = (uint32_t)T.seg_k[l];
  uint32_t above;
  const int bin = block_resolve<kSelNT>(hist, kHBins, kl, lds, above);
  if (threadIdx.x < kSubLists) *lcnt_of(ws, l, threadIdx.x) = 0;
  if (ovf) {
    // A row's candidates did not fit the workspace (the sample put A far below the k_l-th key), but
    // the histogram counted them all: the rows collect again the keys of bins >= B only (those
    // above bin B are certain, bin B's are listed), as a retry (below) does.  With one segment the
    // pool's parts start again from empty (every row is collected again), unless the pass stored
    // +0 at the candidates: the rows then read their old candidates to put them back into acc, so
    // those must stay where they are.  The threshold bin being the key A itself, or the retry
    // switched off: the exact path.
    const uint32_t A = R[R_A], sh = R[R_SH];
    if (bin < 1 || !T.tk_retry) {
      if (threadIdx.x == 0) {
        R[R_SLOW] = 1;
        R[R_RETRY] = 0;
        atomicOr(ws.diag, kDiagSlowPath);
      }
      return;
    }
    if (T.L == 1 && !T.seg_zc[l] && threadIdx.x < (unsigned)kPools) *pcnt_of(ws, threadIdx.x) = 0u;
    if (threadIdx.x == 0) {
      const uint32_t b = (uint32_t)bin;
      R[R_A2] = A + ((b - 1u) << sh);  // keys above it: bins >= B
      R[R_A] = b < (uint32_t)kHBins - 1u ? A + 1u + (b << sh) : 0xFFFFFFFFu;  // first key of bin B + 1
      R[R_NEED] = kl - above;
      R[R_B] = 1u;  // not the tie bin: the listed candidates are ranked
      R[R_RETRY] = 1u;
      R[R_OVF] = 0u;
      atomicOr(ws.diag, kDiagRetry);
    }
    return;
  }
  if (bin >= 0) {
    if (threadIdx.x == 0) {
      R[R_B] = (uint32_t)bin;
      R[R_NEED] = kl - above;
      R[R_RETRY] = 0;
    }
    return;
  }
  // Fewer than k_l candidates: the sample misjudged the density above A.  The retry threshold A2
  // is read from the same sample, at the rank where the density actually found (N keys above A
  // against s sampled ones) predicts 4 k_l + 256 keys above it; its rows then collect every key
  // above A2 again and count those equal to it (k_collect), and k_select falls back to the exact
  // whole-segment path only if those are still fewer than k_l.
  uint32_t mine = 0;
#pragma unroll
  for (int u = 0; u < kPer; ++u) mine += hist[u * kSelNT + threadIdx.x];
  uint32_t N;
  (void)block_excl_scan<kSelNT>(mine, lds, N);
  const uint32_t A = R[R_A];
  const uint32_t ns = ((uint32_t)T.seg_ro[l + 1] - (uint32_t)T.seg_ro[l]) * kSampleRun;
  const uint32_t* sk = ws.samp + (size_t)T.seg_ro[l] * kSampleRun;
  __syncthreads();
  for (int b = threadIdx.x; b < kHBins; b += kSelNT) hist[b] = 0;
  __syncthreads();
  uint32_t above_a = 0;
  for_keys(sk, ns, [&](uint32_t, uint32_t k) {
    atomicAdd(&hist[k >> 20], 1u);
    above_a += k >= A ? 1u : 0u;
  });
  uint32_t sA;
  (void)block_excl_scan<kSelNT>(above_a, lds, sA);  // its barriers also publish hist
  // (at least the rank where the sample alone predicts 4 k_l + 64 keys, in case its top was the
  // only part it misjudged; only that rank when fewer than 8 sampled keys reach A: the scale
  // N / s is then too noisy to use, and too large a threshold would overflow the candidate pool)
  const uint32_t n_seg = (uint32_t)T.seg_off[l + 1] - (uint32_t)T.seg_off[l];
  const uint64_t plain = (((uint64_t)4 * kl + 64u) * ns + n_seg - 1u) / n_seg;
  const uint64_t want = sA >= 8u ? ((uint64_t)4 * kl + 256u) * (uint64_t)sA : 0u;
  const uint64_t ratio = (want + max(N, 1u) - 1u) / max(N, 1u);
  const uint32_t r2 = (uint32_t)min<uint64_t>((uint64_t)ns, max(plain, ratio));
  uint32_t a2above;
  const int b2 = block_resolve<kSelNT>(hist, kHBins, r2, lds, a2above);
  const uint32_t A2 = b2 < 0 || r2 >= ns ? 0u : min(A, (uint32_t)b2 << 20);
  if (threadIdx.x == 0) {
    if (!T.tk_retry || A2 >= A) {
      R[R_SLOW] = 1;
      R[R_RETRY] = 0;
      atomicOr(ws.diag, kDiagSlowPath);
    } else {
      R[R_RETRY] = 1u;
      R[R_A2] = A2;
      R[R_NEED] = kl - N;
      R[R_B] = 1u;  // not the tie bin: the listed candidates are ranked
      atomicOr(ws.diag, kDiagRetry);
    }
  }
}

// Top-k candidate retry, one wavefront per row: the row's keys are read again from acc and every
// key > A2 becomes a candidate, in index order, in the row's static slot or, if more, in entries
// reserved in the overflow pool; those >= A (the first candidates) are certain winners, those in
// (A2, A) go to the segment's list, and the keys equal to A2 are counted (ties, taken by index if
// the list falls short).  A row or a list that does not fit marks the segment for the exact path.
__device__ __forceinline__ void collect_retry(const Tables& T, const WSel& ws, const Batch& BT, uint32_t row, int l,
                                              uint32_t* R) {
  const uint32_t lane = threadIdx.x & 63;
  const float* acc = BT.g[blockIdx.y] ? BT.e[blockIdx.y] : BT.src[blockIdx.y];
  uint32_t o = 0, e_ = (uint32_t)T.d, tb = row * kTile;
  if (T.L > 1) {
    const uint4 rr = reinterpret_cast<const uint4*>(T.row_rec)[row];
    o = rr.y;
    e_ = rr.z;
    tb = rr.w;
  }
  const uint32_t lo = max(o, tb), hi = min(e_, tb + kTile);
  const uint32_t A = R[R_A], A2 = R[R_A2];
  const uint32_t r0 = (uint32_t)T.seg_cbase[l], c = (row - r0) % kSubLists, lq = T.seg_lq[l];
  const size_t sb = sublist_base(T, l, c);
  if (BT.g[blockIdx.y] && T.seg_zc[l]) {
    // the pass stored +0 at the row's candidates: their values go back into acc first (a dropped
    // row's pass stored acc itself), made visible to this wavefront's reads below (a fence for the
    // device writes back the whole L2 of an XCD, the row's own stores need none of that)
    float* accw = BT.e[blockIdx.y];
    const uint32_t oc = ws.counts[row];
    const uint32_t oco = row_entry(T, ws, row, oc, ws.coff[row]);
    if (oco != kDropped)
      for (uint32_t j = lane; j < oc; j += 64) accw[tb + ws.cand_loc[(size_t)oco + j]] = ws.cand_val[(size_t)oco + j];
    __threadfence_block();
  }
  // pass 1: how many (above A2, and equal)
  uint32_t n = 0, nt = 0;
  for (uint32_t i0 = lo; i0 < hi; i0 += 64) {
    const uint32_t i = i0 + lane;
    const uint32_t k = i < hi ? mag_key(acc[i]) : 0u;
    n += (uint32_t)__popcll(__ballot(i < hi && k > A2));
    nt += (uint32_t)__popcll(__ballot(i < hi && k == A2));
  }
  if (lane == 0) ws.rtie[row] = nt;
  uint32_t cb, scap;
  static_slot(T, ws, row, cb, scap);
  if (n > scap) {
    uint32_t at = 0;
    if (lane == 0) at = pool_reserve(ws, row, n);
    cb = __shfl(at, 0, 64);
  }
  if (lane == 0) ws.coff[row] = cb;
  if (cb == kDropped) {
    if (lane == 0) atomicOr(&R[R_OVF], 1u);
    return;
  }
  // pass 2: the candidates and the list
  uint16_t* cloc = ws.cand_loc + cb;
  float* cval = ws.cand_val + cb;
  uint32_t m = 0, na = 0;
  for (uint32_t i0 = lo; i0 < hi; i0 += 64) {
    const uint32_t i = i0 + lane;
    const float v = i < hi ? acc[i] : 0.0f;
    const uint32_t key = mag_key(v);
    const bool take = i < hi && key > A2, cert = take && key >= A, lst = take && !cert;
    const uint64_t bt = __ballot(take), bl = __ballot(lst);
    if (take) {
      const uint32_t pos = m + lanes_below(bt);
      cloc[pos] = (uint16_t)(i - tb);
      cval[pos] = v;
    }
    m += (uint32_t)__popcll(bt);
    na += (uint32_t)__popcll(__ballot(cert));
    const uint32_t nl = (uint32_t)__popcll(bl);
    if (nl) {
      uint32_t base = 0;
      if (lane == 0) base = atomicAdd(lcnt_of(ws, l, c), nl);
      base = __shfl(base, 0, 64);
      const uint32_t t = base + lanes_below(bl);
      if (lst && t < lq) {  // a full sub-list is seen by k_select (its count exceeds lq)
        const size_t p = sb + t;
        ws.list_key[p] = key;
        ws.list_idx[p] = i;
      }
    }
  }
  if (lane == 0) {
    ws.counts[row] = m;
    ws.rcnt[row] = na;
  }
}

constexpr uint32_t kCollectBuf = 512;  // listed candidates a wavefront of k_collect stages in LDS
// Chunks of 64 candidates loaded together: four where a wavefront has one row (BERT flat at 10 %, over 400
// candidates a row: 24.8 -> 20.9 us), one in a batch (16 workers on ResNet-50: 27.7 us, 28.4 with four).
constexpr uint32_t collect_chunks(uint32_t rows) { return rows == 1u ? 4u : 1u; }

// Top-k, per row: candidates certain to win (above bin B of a histogrammed segment) are counted, the
// undecided ones (inside it) go to the segment's list, in any order: the selection over the list does
// not depend on it; row r appends to sub-list r % kSubLists, which spreads the atomics on the list
// counters.  One wavefront per kCollectRows rows: their segments, candidate counts and, of one
// segment, first candidates are loaded together; counts come from ballots, and the listed candidates
// are staged in LDS.
template <uint32_t kCollectRows>
__global__ __launch_bounds__(kNT) void k_collect(Tables T, WSel ws0, Batch BT) {
  const WSel ws = ws_at(ws0, (uint64_t)blockIdx.y * BT.ws);
  __shared__ uint32_t s_lk[kNT / 64][kCollectBuf], s_li[kNT / 64][kCollectBuf];
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  // a wavefront's rows lie far apart: crowded rows (a layer of large values) are neighbours, and one
  // wavefront with several of them would hold the kernel up
  const uint32_t stride = ((uint32_t)T.nrows + kCollectRows - 1u) / kCollectRows;
  const uint32_t row0 = blockIdx.x * (kNT / 64) + (threadIdx.x >> 6);
  if (row0 >= stride) return;
  int ls[kCollectRows];
  uint32_t cnts[kCollectRows], cofs[kCollectRows];
  constexpr uint32_t kU = collect_chunks(kCollectRows);
  float v0[kCollectRows][kU];
  // one segment: its record read once, in the first round trip (k_collect does not write it; read
  // per row, each row's fields waited for again after the previous row's list stores)
  uint32_t r_skip = 0, r_retry = 0, r_A = 0, r_sh = 0, r_B = 0;
  if (T.L == 1) {
    const uint32_t* R0 = res_of(ws, 0);
    r_skip = R0[R_SLOW] | R0[R_MODE];
    r_retry = R0[R_RETRY];
    r_A = R0[R_A];
    r_sh = R0[R_SH];
    r_B = R0[R_B];
  }
#pragma unroll
  for (uint32_t r = 0; r < kCollectRows; ++r) {
    const uint32_t row = min(row0 + r * stride, (uint32_t)T.nrows - 1u);
    ls[r] = T.L == 1 ? 0 : T.row_seg[row];  // one segment: no load before the segment's record
    cnts[r] = ws.counts[row];
    cofs[r] = ws.coff[row];
    // one segment: the first values of the row's static slot, in the same round trip (used if the
    // row's candidates are there; past the count: unused, and not loaded past the slot)
    const uint32_t cap0 = T.L == 1 ? min(ws.S, (uint32_t)T.d - row * kTile) : 0u;
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) v0[r][u] = 64u * u + lane < cap0 ? ws.cand_val[(size_t)row * ws.S + 64u * u + lane] : 0.0f;
  }
#pragma unroll
  for (uint32_t r = 0; r < kCollectRows; ++r) {
    const uint32_t row = row0 + r * stride;
    if (row >= (uint32_t)T.nrows) break;
    const int l = ls[r];
    uint32_t* R = res_of(ws, l);
    const bool one = T.L == 1;
    if (one ? r_skip != 0 : (R[R_SLOW] || R[R_MODE])) continue;
    if (one ? r_retry != 0 : R[R_RETRY] != 0) {
      collect_retry(T, ws, BT, row, l, R);
      continue;
    }
    const uint32_t A = one ? r_A : R[R_A], sh = one ? r_sh : R[R_SH], B = one ? r_B : R[R_B];
    const uint32_t co = row_entry(T, ws, row, cnts[r], cofs[r]);
    if (co == kDropped) continue;  // the segment takes the exact path
    // keys from k2 on (the first of bin B + 1) are certain winners, those from k1 on (bin B's first)
    // undecided and listed.  Tie bin (B = 0, the key A alone, whose elements the pass only counted):
    // every stored candidate is a certain winner and nothing is listed
    const uint32_t k2 = B + 1u < (uint32_t)kHBins ? A + 1u + (B << sh) : 0xFFFFFFFFu;
    const uint32_t k1 = B ? A + 1u + ((B - 1u) << sh) : k2;
    const uint32_t cnt = cnts[r];
    const float* cv = ws.cand_val + co;
    const uint16_t* ci = ws.cand_loc + co;
    const bool v0_ok = one && co == row * ws.S;
    const uint32_t r0 = (uint32_t)T.seg_cbase[l], c = (row - r0) % kSubLists, lq = T.seg_lq[l];
    const size_t sb = sublist_base(T, l, c);
    const uint32_t tb = row_tile(T, row);
    // The row's listed candidates are staged in the wavefront's LDS buffer and written out with
    // one reservation of list space per row (or per full buffer).  An atomic per chunk of 64
    // candidates, each waited for, on the 16 sub-list counters took 92-141 us to collect BERT flat
    // at 10 % with bf16 values (211,000 equal keys in the threshold bin); staged, 30 us.
    uint32_t na = 0, nb = 0;  // certain winners; listed candidates in the buffer (uniform)
    auto flush = [&]() {
      uint32_t base = 0;
      if (lane == 0) base = atomicAdd(lcnt_of(ws, l, c), nb);
      base = __shfl(base, 0, 64);
      for (uint32_t x = lane; x < nb; x += 64) {
        const uint32_t t = base + x;
        if (t < lq) {  // a full sub-list is seen by k_select (its count exceeds lq)
          ws.list_key[sb + t] = s_lk[wv][x];
          ws.list_idx[sb + t] = s_li[wv][x];
        }
      }
      nb = 0;
    };
    float vn[kU];
    auto fetch = [&](uint32_t j0) {
#pragma unroll
      for (uint32_t u = 0; u < kU; ++u) vn[u] = j0 + 64u * u + lane < cnt ? cv[j0 + 64u * u + lane] : 0.0f;
    };
    if (v0_ok) {
#pragma unroll
      for (uint32_t u = 0; u < kU; ++u) vn[u] = v0[r][u];
    } else {
      fetch(0);
    }
#pragma unroll 1
    for (uint32_t j0 = 0; j0 < cnt; j0 += 64u * kU) {
      uint32_t k[kU];
#pragma unroll
      for (uint32_t u = 0; u < kU; ++u) k[u] = mag_key(vn[u]);
      if (cnt - j0 > 64u * kU) fetch(j0 + 64u * kU);  // the next chunks' values, in flight
#pragma unroll
      for (uint32_t u = 0; u < kU; ++u) {
        if (j0 + 64u * u >= cnt) break;
        const uint32_t left = cnt - j0 - 64u * u;
        const uint64_t there = left >= 64u ? ~0ull : (1ull << left) - 1ull;
        const uint64_t b2 = __ballot(k[u] >= k2) & there, bu = __ballot(k[u] >= k1) & there & ~b2;
        na += (uint32_t)__popcll(b2);
        const uint32_t nu = (uint32_t)__popcll(bu);
        if (nu == 0) continue;
        if (nb + nu > kCollectBuf) flush();
        if (__builtin_amdgcn_inverse_ballot_w64(bu)) {
          const uint32_t x = nb + lanes_below(bu);
          s_lk[wv][x] = k[u];
          s_li[wv][x] = tb + ci[j0 + 64u * u + lane];
        }
        nb += nu;
      }
    }
    if (nb) flush();
    if (lane == 0) ws.rcnt[row] = na;
  }
}

// Random-k without direct lists, per row: the undecided candidates ([ulo, tau)) go to the segment's
// sub-lists, the certain winners are added to the segment's counters.  A wavefront looks at rw rows'
// counts (a lane each) and reads the candidates of those that hold an undecided one only (1e9 elements
// at 1 %: one row in seven; every candidate's key read and tested took 65 us).  Those rows are read one
// after another, four loads in flight, so rw is as large as leaves kCollectWaves wavefronts: at 64 rows
// each, 2100 rows of 380 candidates made 33 wavefronts and the step took 257 us, now 64 (8.6e6 elements at
// 9.4 %; 36.6e6 at 0.33 %: 119 us, now 98; 1e9 at 1 % keeps 64 rows).
constexpr uint32_t kCollectWaves = 2048;
inline uint32_t collect_rows(uint64_t rows) {
  uint32_t rw = 64;
  while (rw > 1u && rows / rw < kCollectWaves) rw /= 2u;
  return rw;
}
constexpr uint32_t kCollectWide = 1024;  // segments of at least this many rows: a wavefront reserves list space once
__global__ __launch_bounds__(kNT) void k_collect_randk(Tables T, WSel ws0, Batch BT, uint32_t rw) {
  const WSel ws = ws_at(ws0, (uint64_t)blockIdx.y * BT.ws);
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = blockIdx.x * (kNT / 64) + (threadIdx.x >> 6), row0 = wave * rw;
  if (row0 >= (uint32_t)T.nrows) return;
  const uint32_t row = min(row0 + lane, (uint32_t)T.nrows - 1u);
  const bool has = lane < rw && row0 + lane < (uint32_t)T.nrows;
  int l = 0;
  uint32_t cnt = 0, cert = 0, co = kDropped, tb = 0, sub = 0;
  if (has) {
    l = T.L == 1 ? 0 : T.row_seg[row];
    cnt = ws.counts[row];
    cert = ws.rcnt[row];
    tb = row_tile(T, row);
    co = row_entry(T, ws, row, cnt, ws.coff[row]);
    sub = (row - (uint32_t)T.seg_cbase[l]) % kSubLists;
    if (co == kDropped) atomicOr(&res_of(ws, l)[R_OVF], 1u);
  }
  const int l0 = __builtin_amdgcn_readfirstlane(l);  // (the first row: lane 0 has one)
  if (__ballot(has && l != l0) == 0) {  // rows of one segment: one addition
    const uint32_t s = wave_incl_scan(cert);
    if (lane == 63 && s) atomicAdd(scnt_of(ws, l0, wave % kSubLists), s);
  } else if (has && cert) {
    atomicAdd(scnt_of(ws, l, sub), cert);
  }
  const bool list = has && co != kDropped && cnt > cert;
  uint32_t at = 0;
  // (the 16 counters take one atomic at a time, about 15 ns each)
  if (__ballot(has && l != l0) == 0 && (uint32_t)(T.seg_cbase[l0 + 1] - T.seg_cbase[l0]) >= kCollectWide) {
    const uint32_t und = list ? cnt - cert : 0u, inc = wave_incl_scan(und);
    const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    sub = wave % kSubLists;
    if (all && lane == 0) at = atomicAdd(lcnt_of(ws, l0, sub), all);
    at = (uint32_t)__builtin_amdgcn_readlane((int)at, 0) + inc - und;
  } else if (list) {
    at = atomicAdd(lcnt_of(ws, l, sub), cnt - cert);
  }
  uint64_t todo = __ballot(list);
  while (todo) {
    const int j = __ffsll((long long)todo) - 1;
    todo &= todo - 1;
    const int rl = __builtin_amdgcn_readlane(l, j);
    const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)cnt, j), c0 = (uint32_t)__builtin_amdgcn_readlane((int)co, j);
    const uint32_t t0 = (uint32_t)__builtin_amdgcn_readlane((int)tb, j), lq = T.seg_lq[rl];
    const size_t sb = sublist_base(T, rl, (uint32_t)__builtin_amdgcn_readlane((int)sub, j));
    uint32_t p = (uint32_t)__builtin_amdgcn_readlane((int)at, j);
    for (uint32_t f0 = 0; f0 < n; f0 += 256) {
      uint32_t x[4], k[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t f = f0 + (uint32_t)u * 64u + lane;
        x[u] = f < n ? ws.cand_loc[(size_t)c0 + f] : kCertain;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t f = f0 + (uint32_t)u * 64u + lane;
        k[u] = !(x[u] & kCertain) ? ws.cand_key[(size_t)c0 + f] : 0u;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint64_t b = __ballot(!(x[u] & kCertain));
        const uint32_t t = p + lanes_below(b);
        if (!(x[u] & kCertain) && t < lq) {  // a full sub-list is seen by k_select (its count exceeds lq)
          ws.list_key[sb + t] = k[u];
          ws.list_idx[sb + t] = t0 + x[u];
        }
        p += (uint32_t)__popcll(b);
      }
    }
  }
}

// An entry to be ranked as one 64-bit word: key' in the high half and the complement of the index
// in the low half, so that one unsigned comparison orders entries by key' descending, then index
// ascending.  The word 0 (key' 0 with index 2^32 - 1, which no element has) beats no entry; it
// pads a ranked list to rank_pad(m) words, the stride of the ranking loop.
__device__ __forceinline__ uint64_t rank_word(uint32_t key, uint32_t idx) {
  return ((uint64_t)key << 32) | (uint64_t)(~idx);
}
__device__ __forceinline__ uint32_t rank_pad(uint32_t m) { return (m + 63u) & ~63u; }

// The need-th best (1 <= need <= m <= kRankList) of m entries held in LDS as rank words, padded
// with zero words up to rank_pad(m): every entry counts the entries that beat it.  An entry is
// shared by 4, 8 or 16 threads (as many as the workgroup's threads allow for m entries), each
// comparing against every 4th, 8th or 16th entry, four loads in flight per pass.  Gives its key'
// and one past its index.
__device__ __forceinline__ void rank_select(const uint64_t* g, uint32_t m, uint32_t need, uint32_t& T_out,
                                            uint32_t& IT_out) {
  static_assert(kRankList * 4 <= kSelNT, "four threads per ranked entry");
  __shared__ uint32_t s_t, s_it;
  const uint32_t lg = m <= kSelNT / 16 ? 4u : (m <= kSelNT / 8 ? 3u : 2u);  // log2 threads per entry
  const uint32_t tpe = 1u << lg;
  const uint32_t e = threadIdx.x >> lg, part = threadIdx.x & (tpe - 1u);
  uint32_t rank = 0;
  uint64_t v = 0;
  if (e < m) {
    v = g[e];
    // j0 + 3 tpe stays below m rounded up to 4 tpe, which divides 64: inside the padding
    for (uint32_t j0 = part; j0 < m; j0 += 4u * tpe) {
      uint64_t w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = g[j0 + (uint32_t)u * tpe];
#pragma unroll
      for (int u = 0; u < 4; ++u) rank += w[u] > v ? 1u : 0u;
    }
  }
  // the entry's threads are adjacent lanes of one wavefront
  rank += __shfl_xor(rank, 1, 64);
  rank += __shfl_xor(rank, 2, 64);
  if (lg >= 3u) rank += __shfl_xor(rank, 4, 64);
  if (lg >= 4u) rank += __shfl_xor(rank, 8, 64);
  if (e < m && part == 0 && rank == need - 1) {
    s_t = (uint32_t)(v >> 32);
    s_it = ~(uint32_t)v + 1u;
  }
  __syncthreads();
  T_out = s_t;
  IT_out = s_it;
  __syncthreads();
}

// The need best of the m listed candidates (key' descending, then index ascending; 1 <= need <=
// m): the key' T of the last winner and one past its index (every listed winner is key' > T, or
// key' == T with index below that bound).  Radix levels of 11 bits narrow the key' range until
// the bin holding the need-th best has at most kRankList entries; those are gathered and ranked.
// kand / kor: the AND and the OR of the m keys (needed when m > kRankList).
template <typename K, typename I>
__device__ __forceinline__ void list_threshold_ao(const K& key, const I& idx, uint32_t m, uint32_t need,
                                                  uint32_t kand, uint32_t kor, uint32_t* hist, uint32_t* lds,
                                                  uint64_t* g, uint32_t& T_out, uint32_t& IT_out,
                                                  uint32_t* defer_need) {
  __shared__ uint32_t s_n;
  if (m <= kRankList) {
    for (uint32_t j = threadIdx.x; j < rank_pad(m); j += kSelNT) g[j] = j < m ? rank_word(key[j], idx[j]) : 0ull;
    __syncthreads();
    rank_select(g, m, need, T_out, IT_out);
    return;
  }
  const uint32_t diff = kand ^ kor;
  uint32_t prefix = kand, known = 32;  // all keys equal: nothing to resolve
  uint32_t cnt = m;
  if (diff) {
    const int h = 31 - __clz(diff);
    prefix = h == 31 ? 0u : (kand & (0xFFFFFFFFu << (h + 1)));
    known = (uint32_t)(31 - h);
    while (known < 32 && cnt > kRankList) {
      const int w = min(11, 32 - (int)known);
      const int shift = 32 - (int)known - w;
      for (int b = threadIdx.x; b < (1 << w); b += kSelNT) hist[b] = 0;
      __syncthreads();
      const uint32_t pmask = known == 0 ? 0u : (0xFFFFFFFFu << (32 - known));
      const uint32_t want = prefix & pmask;
      for_keys(key, m, [&](uint32_t, uint32_t k) {
        if ((k & pmask) == want) atomicAdd(&hist[(k >> shift) & ((1u << w) - 1u)], 1u);
      });
      __syncthreads();
      uint32_t above;
      const int bin = block_resolve<kSelNT>(hist, 1 << w, need, lds, above);
      cnt = hist[max(bin, 0)];
      __syncthreads();
      prefix |= (uint32_t)max(bin, 0) << shift;
      need -= above;
      known += (uint32_t)w;
    }
  }
  if (cnt <= kRankList) {  // gather the entries sharing the resolved prefix and rank them
    const uint32_t pmask = known == 0 ? 0u : (known >= 32 ? 0xFFFFFFFFu : (0xFFFFFFFFu << (32 - known)));
    const uint32_t want = prefix & pmask;
    if (threadIdx.x == 0) s_n = 0;
    for (uint32_t j = cnt + threadIdx.x; j < rank_pad(cnt); j += kSelNT) g[j] = 0ull;  // the gather fills [0, cnt)
    __syncthreads();
    for_keys(key, m, [&](uint32_t f, uint32_t k) {
      if ((k & pmask) == want) {
        const uint32_t p = atomicAdd(&s_n, 1u);
        g[p] = rank_word(k, idx[f]);
      }
    });
    __syncthreads();
    rank_select(g, cnt, need, T_out, IT_out);
    return;
  }
  // more than kRankList entries share the full key': ties ordered by index (with defer_need, the
  // caller resolves them: IT_out = kTieRows, *defer_need = how many of them win)
  T_out = prefix;
  if (need >= cnt) {
    IT_out = 0xFFFFFFFFu;
  } else if (defer_need) {
    IT_out = kTieRows;
    *defer_need = need;
  } else {
    IT_out = block_nth_smallest_tie(key, idx, m, prefix, need, hist, lds) + 1u;
  }
}

template <typename K>
__device__ __forceinline__ void list_threshold(const K& key, const K& idx, uint32_t m, uint32_t need,
                                               uint32_t* hist, uint32_t* lds, uint64_t* g,
                                               uint32_t& T_out, uint32_t& IT_out, uint32_t* defer_need = nullptr) {
  uint32_t kand = 0xFFFFFFFFu, kor = 0u;
  if (m > kRankList) {
    for_keys(key, m, [&](uint32_t, uint32_t k) {
      kand &= k;
      kor |= k;
    });
    block_and_or(kand, kor, lds);
  }
  list_threshold_ao(key, idx, m, need, kand, kor, hist, lds, g, T_out, IT_out, defer_need);
}

// Random-k, a list in global memory: its keys u = ~key' are uniform over [ulo, uhi], so the need-th
// smallest of m lies within a few standard deviations of its expected rank.  The keys of that band go
// to LDS (their number and that of the keys below it counted on the way), and the answer is found
// among them.  False when the band missed it (six deviations: a chance below 10^-8) or does not fit;
// the general search over the list follows.  1e9 elements at 1 %, 38,000 listed: the select kernel
// 94 -> 57 us.  (Lists in LDS gain nothing from a band: ranking one directly in place of the radix
// level took 11.8 us like before on flat 2^20 at 1 %.)
__device__ __forceinline__ bool band_threshold(const SubLists& lk, const SubLists& li, uint32_t m, uint32_t need,
                                               uint32_t ulo, uint32_t uhi, uint32_t* s_key, uint32_t* s_idx,
                                               uint32_t cap, uint32_t* hist, uint32_t* lds, uint64_t* g,
                                               uint32_t& T_out, uint32_t& IT_out) {
  __shared__ uint32_t s_in, s_below;
  const double span = (double)(uhi - ulo) + 1.0, per = span / (double)m;
  const float x = (float)need / (float)m;
  const double h = 6.0f * sqrtf(fmaxf((float)m * x * (1.0f - x), 0.0f)) + 8.0f;
  const uint32_t b0 = ulo + (uint32_t)fmin(fmax(((double)need - h) * per, 0.0), span - 1.0);
  const uint32_t b1 = ulo + (uint32_t)fmin(fmax(((double)need + h) * per, 0.0), span - 1.0);
  if (threadIdx.x == 0) s_in = s_below = 0u;
  __syncthreads();
  uint32_t below = 0;
  for_keys2(lk, [&](uint32_t, uint32_t k, size_t at) {
    const uint32_t u = ~k;
    below += u < b0 ? 1u : 0u;
    if (u >= b0 && u <= b1) {
      const uint32_t p = atomicAdd(&s_in, 1u);
      if (p < cap) {
        s_key[p] = k;
        s_idx[p] = li.arr[at];
      }
    }
  });
  if (below) atomicAdd(&s_below, below);
  __syncthreads();
  const uint32_t n = s_in, before = s_below;
  __syncthreads();
  if (n > cap || need <= before || need > before + n) return false;  // uniform
  list_threshold(s_key, s_idx, n, need - before, hist, lds, g, T_out, IT_out);
  return true;
}

// Per segment: the exact threshold among the listed candidates, then every row's message offset;
// or the exact whole-segment path when the candidates cannot hold the answer.  Independent loads
// are issued together (record, sub-list sizes, the rows' counts) to keep the chain of dependent
// memory round trips short.  BIG (layouts with a very large k_l or very many rows): the threshold, and
// the list's winners added to their rows' counts with global atomics (the listed candidates are few
// beside the winners, so that counting every row's winners again, 22 us on BERT flat at 10 % and 55 us
// on 1e9 elements at 1 %, is not needed); k_rowsum turns the counts into offsets over many workgroups.
// SMALL: segments of at most kSmallRows rows, random-k on direct layouts only, lists expected to fit
// kSmallList entries.  PAIR: 64 registers a thread, so that two workgroups fit a CU (8 workers' random-k
// steps on ResNet-18's 62 layers, 496 workgroups: 24.7 -> 20.7 us).  Random-k spills 32 registers there;
// launches that give no CU a second workgroup (kCUs) take the form without PAIR, 87 registers and no
// spill.  Steps with PAIR / without: random-k per layer at 1 %, ResNet-50's 161 workgroups 72.8 / 66.6 us,
// ResNet-18's 62 43.0 / 40.0, 4 workers' 248 127.8 / 120.4; 5 workers' 310, with the larger form's one
// workgroup to a CU, 156.9 / 157.8.  Top-k spills nothing with PAIR and measures the same.
constexpr uint32_t kSmallList = 4096, kSmallRows = 4096;
constexpr uint32_t kCUs = 256;
template <int KIND, bool BIG, bool SMALL = false, bool PAIR = false>
__global__ __launch_bounds__(kSelNT, PAIR ? 8 : 4) void k_select(Tables T, WSel ws0, uint32_t* out_idx, float* out_val,
                                                   uint32_t step, Batch BT) {
  const WSel ws = ws_at(ws0, (uint64_t)blockIdx.y * BT.ws);
  float* e_zero = BT.e[blockIdx.y];
  const float* data = BT.g[blockIdx.y] ? BT.e[blockIdx.y] : BT.src[blockIdx.y];  // acc
  out_idx = shifted(out_idx, (uint64_t)blockIdx.y * BT.msg * 4u);
  out_val = out_val ? shifted(out_val, (uint64_t)blockIdx.y * BT.msg * 4u) : nullptr;
  const uint32_t s0 = BT.seed_lo[blockIdx.y], s1 = BT.seed_hi[blockIdx.y];
  constexpr uint32_t kPer = SMALL ? kSmallRows / kSelNT : kSelPer;  // rows per thread held in registers (more are re-read)
  __shared__ uint32_t hist[kHBins];
  __shared__ uint32_t lds[3 * kSelNT / 64];
  constexpr uint32_t kCap = SMALL ? kSmallList : kListLds, kRowCap = SMALL ? kSmallRows : kRowsLds;
  __shared__ uint32_t s_key[kCap];
  __shared__ uint32_t s_idx[kCap];
  __shared__ uint32_t s_add[BIG ? 1 : kRowCap];
  __shared__ uint64_t s_g[kRankList];
  const int l = blockIdx.x;
  uint32_t* R = res_of(ws, l);
  // (one segment: no table loads before the rows' loads)
  const uint32_t r0 = T.L == 1 ? 0u : (uint32_t)T.seg_cbase[l];
  const uint32_t nr = T.L == 1 ? (uint32_t)T.nrows : (uint32_t)T.seg_cbase[l + 1] - r0;
  const uint32_t kl = T.L == 1 ? (uint32_t)T.K : (uint32_t)T.seg_k[l];
  const uint32_t per = (nr + kSelNT - 1) / kSelNT;
  const uint32_t a = min(nr, threadIdx.x * per), b = min(nr, a + per);
  const uint32_t* rc = ws.rcnt + r0;
  const uint32_t* cc = ws.counts + r0;
  // round trip 1: record, sub-list sizes, row counts
  bool slow = false, listed = true;
  uint32_t need = 0, mU = 0, exU = 0, ovf = 0;
  if constexpr (KIND == 0) {
    slow = R[R_SLOW] != 0;
    listed = R[R_MODE] == 0;
    need = R[R_NEED];
    ovf = R[R_OVF];
  }
  const bool direct = KIND == 1 && (SMALL || T.rk_direct);
  const uint32_t lq = T.seg_lq[l];
  uint32_t lc[kSubLists];
#pragma unroll
  for (int c = 0; c < kSubLists; ++c) lc[c] = direct ? 0u : *lcnt_of(ws, l, (uint32_t)c);
  bool lfull = false;  // a sub-list overflowed its region
#pragma unroll
  for (int c = 0; c < kSubLists; ++c) lfull |= lc[c] > lq;
  // top-k candidate retry whose list holds fewer than the `need` winners: every listed candidate
  // wins, and the rest are the first elements equal to A2 (counted per row, not stored)
  bool retry_ties = false;
  if constexpr (KIND == 0) {
    // a row or a sub-list that did not fit the workspace: the exact path
    if (!slow) {
      uint32_t m = 0;
#pragma unroll
      for (int c = 0; c < kSubLists; ++c) m += lc[c];
      retry_ties = listed && R[R_RETRY] && m < need;
      if (retry_ties) need -= m;
      if (ovf || (listed && lfull)) {
        slow = true;
        __syncthreads();  // every thread has read R_SLOW before it is set
        if (threadIdx.x == 0) {
          R[R_SLOW] = 1u;
          atomicOr(ws.diag, kDiagSlowPath);
        }
      }
    }
  }
  const bool counted = KIND == 1 && !direct;  // (the pass counted the certain winners by segment)
  // random-k: the rows' first pool entries (one segment: the static slot, r * S, unless the row
  // holds more candidates than it, so only those rows' entries are loaded)
  const uint32_t* ro = ws.coff + r0;
  auto first_entry = [&](uint32_t x, uint32_t cnt) -> uint32_t {
    const uint32_t row = r0 + x;
    return cnt > min(ws.S, (uint32_t)T.d - row * kTile) ? ro[x] : row * ws.S;
  };
  uint32_t cr[kPer], cn[kPer], co[kPer];
#pragma unroll
  for (uint32_t x = 0; x < kPer; ++x) {
    cr[x] = !(counted && BIG) && a + x < b ? rc[a + x] : 0u;
    cn[x] = !counted && a + x < b ? cc[a + x] : 0u;
    co[x] = KIND == 1 && T.L > 1 && !counted && a + x < b ? ro[a + x] : 0u;
  }
  if (KIND == 1 && T.L == 1 && !counted) {
#pragma unroll
    for (uint32_t x = 0; x < kPer; ++x)
      if (a + x < b) co[x] = first_entry(a + x, cn[x]);
  }
  if constexpr (KIND == 1) {
    // random-k: the certain winners S (keys below ulo) and the candidates N decide whether the
    // window [ulo, tau) holds the k_l-th smallest key (also counted: rows whose candidates did not
    // fit the workspace)
    uint32_t S, N, dropped;
    if (counted) {
      uint32_t m = 0;
      S = 0;
#pragma unroll
      for (int c = 0; c < kSubLists; ++c) {
        S += *scnt_of(ws, l, (uint32_t)c);
        m += lc[c];
      }
      N = S + m;
      dropped = R[R_OVF];
    } else {
      uint32_t sv[3] = {0u, 0u, 0u};
#pragma unroll
      for (uint32_t x = 0; x < kPer; ++x) {
        sv[0] += cr[x];
        sv[1] += cn[x];
        sv[2] += co[x] == kDropped ? 1u : 0u;
      }
      for (uint32_t x = a + kPer; x < b; ++x) {
        const uint32_t c = cc[x];
        sv[0] += rc[x];
        sv[1] += c;
        sv[2] += (T.L == 1 ? first_entry(x, c) : ro[x]) == kDropped ? 1u : 0u;
      }
      uint32_t ex[3], tot[3];
      block_excl_scan_n<kSelNT, 3>(sv, lds, ex, tot);
      S = tot[0];
      N = tot[1];
      dropped = tot[2];
      exU = ex[1] - ex[0];
    }
    // direct lists: the rows' undecided candidates (counts - certain) must fit the LDS list;
    // sub-lists: every one its region
    slow = S > kl || N < kl || dropped != 0 || (direct ? N - S > kCap : lfull);
    need = kl - S;
    mU = N - S;
    if (threadIdx.x == 0) {
      R[R_SLOW] = slow ? 1u : 0u;
      if (slow) atomicOr(ws.diag, kDiagSlowPath);
    }
  }
  // The streaming pass stored +0 at candidates (random-k: all; top-k segments with seg_zc): the
  // exact path needs acc there, which the candidates keep (a row whose candidates did not fit
  // stored acc there itself).  Uniform.
  auto restore_candidates = [&]() {
    if (!e_zero || (KIND == 0 && !T.seg_zc[l])) return;
    for (uint32_t x = a; x < b; ++x) {
      const uint32_t cnt = cc[x], tb = row_tile(T, r0 + x);
      const uint32_t sl = T.L == 1 ? first_entry(x, cnt) : ro[x];
      if (sl == kDropped) continue;
      for (uint32_t j = 0; j < cnt; ++j)
        e_zero[tb + (ws.cand_loc[(size_t)sl + j] & (kTile - 1u))] = ws.cand_val[(size_t)sl + j];
    }
    __threadfence();
    __syncthreads();
  };
  if (slow) {
    restore_candidates();
    slow_select<KIND>(T, l, data, e_zero, out_idx, out_val, s0, s1, step, hist, lds);
    return;
  }
  const bool rows_lds = nr <= kRowCap;
  bool tie = false;
  bool done = KIND == 1;  // many rows: the rows' winner counts are complete
  if constexpr (KIND == 0) tie = listed && (R[R_B] == 0 || retry_ties);
  if (tie) {
    // The threshold bin is the key A alone, whose elements the streaming pass counted per row but
    // did not store (a retry: the key A2, counted by k_collect): every stored candidate wins, and
    // the first `need` of the elements equal to it, in index order.  A scan of the rows' tie counts
    // finds the row of the last winner, and one pass over that row's elements in acc the winner
    // itself.  The rows with winning ties are emitted from acc (all their elements are scanned
    // there: counts = the row's length, flagged kAccRow).
    __shared__ uint32_t s_row, s_rank;
    const uint32_t* rt = ws.rtie + r0;
    uint32_t tl[kPer], st = 0;
#pragma unroll
    for (uint32_t x = 0; x < kPer; ++x) {
      tl[x] = a + x < b ? rt[a + x] : 0u;
      st += tl[x];
    }
    for (uint32_t x = a + kPer; x < b; ++x) st += rt[x];
    uint32_t totT;
    uint32_t before = block_excl_scan<kSelNT>(st, lds, totT);
    if (totT < need) {  // a retry with too few ties (the tie bin itself holds at least `need`)
      if (threadIdx.x == 0) {
        R[R_SLOW] = 1u;
        atomicOr(ws.diag, kDiagSlowPath);
      }
      restore_candidates();
      slow_select<KIND>(T, l, data, e_zero, out_idx, out_val, s0, s1, step, hist, lds);
      return;
    }
    uint32_t* rcw = ws.rcnt + r0;
    if (retry_ties) {
      // a retry counted only its certain winners per row: all the row's candidates win here
#pragma unroll
      for (uint32_t x = 0; x < kPer; ++x) cr[x] = cn[x];
      for (uint32_t x = a + kPer; x < b; ++x) rcw[x] = cc[x];
    }
    for (uint32_t x = a; x < b; ++x) {
      uint32_t t = 0;  // tl[x - a] by unrolled selects (a dynamic index would put tl in scratch)
      if (x - a < kPer) {
#pragma unroll
        for (uint32_t y = 0; y < kPer; ++y)
          if (y == x - a) t = tl[y];
      } else {
        t = rt[x];
      }
      const uint32_t take = min(t, need > before ? need - before : 0u);
      if (before < need && need <= before + t) {
        s_row = x;
        s_rank = need - before;
      }
      if (take) {
        uint32_t lo, hi;
        row_bounds(T, r0 + x, lo, hi);
        // the row's own candidate count moves to rtie (the emission finds its candidates with it)
        uint32_t oc = 0;
        if (x - a < kPer) {
#pragma unroll
          for (uint32_t y = 0; y < kPer; ++y)
            if (y == x - a) oc = cn[y];
        } else {
          oc = cc[x];
        }
        ws.rtie[r0 + x] = oc;
        ws.counts[r0 + x] = (hi - lo) | kAccRow;
      }
      if (x - a < kPer) {
        uint32_t now = 0;
#pragma unroll
        for (uint32_t y = 0; y < kPer; ++y)
          if (y == x - a) {
            cr[y] += take;
            now = cr[y];
          }
        // (many-row layouts: k_rowcount keeps the winner count of a row emitted from acc)
        if (take) rcw[x] = now;
      } else {
        rcw[x] += take;  // re-read by this thread below
      }
      before += t;
    }
    __syncthreads();
    uint32_t lo, hi;
    row_bounds(T, r0 + s_row, lo, hi);
    const uint32_t A = retry_ties ? R[R_A2] : R[R_A];
    if (e_zero && T.seg_zc[l] && !R[R_RETRY]) {
      // the pass stored +0 at this row's candidates: back to acc before its elements are searched
      // (+0 has the key of a tie at A = 0)
      const uint32_t row = r0 + s_row, oc = ws.rtie[row], tb = row_tile(T, row);
      const uint32_t co = row_entry(T, ws, row, oc, ws.coff[row]);
      if (co != kDropped)
        for (uint32_t j = threadIdx.x; j < oc; j += kSelNT) e_zero[tb + ws.cand_loc[(size_t)co + j]] = ws.cand_val[(size_t)co + j];
      // this workgroup's reads only: a fence for the device writes back the L2 that the pass has just
      // filled with e (this kernel on BERT per layer at 1.2 %, a gradient of zeros: 56 -> 15 us)
      __threadfence_block();
      __syncthreads();
    }
    const uint32_t p = block_nth_equal(AccKeys{data + lo}, hi - lo, A, s_rank, lds);
    if (threadIdx.x == 0) {
      R[R_T] = A;
      R[R_IT] = lo + p + 1u;
    }
  }
  if (listed && !tie) {
    const uint32_t o = (uint32_t)T.seg_off[l];
    SubLists lk, li;
    lk.arr = ws.list_key;
    li.arr = ws.list_idx;
    lk.base = li.base = T.seg_lbase[l];
    lk.q = li.q = lq;
    uint32_t m = 0;
#pragma unroll
    for (int c = 0; c < kSubLists; ++c) {
      lk.M[c] = li.M[c] = m;
      m += lc[c];
    }
    lk.M[kSubLists] = li.M[kSubLists] = m;
    if (direct) m = mU;
    const bool in_lds = (KIND == 1 && SMALL) || m <= kCap;  // (direct lists fit, else the segment is slow)
    // top-k, list staged in LDS: the AND and OR of its keys, taken as they pass through
    uint32_t sand = 0xFFFFFFFFu, sor = 0u;
    if (direct) {
      // round trip 2 (direct lists; every row of the segment is one of kPer per thread): each
      // thread notes the pool entries of its rows' undecided candidates at their list positions,
      // then the pairs are fetched, all loads in flight together
      uint32_t f = exU;
#pragma unroll
      for (uint32_t x = 0; x < kPer; ++x) {
        if (a + x < b)
          for (uint32_t t = 0; t < cn[x] - cr[x]; ++t) s_key[f++] = co[x] + t;
      }
      __syncthreads();
      for (uint32_t f0 = 0; f0 < m; f0 += (uint32_t)kSelNT * 4u) {
        uint2 pr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t fu = f0 + (uint32_t)u * kSelNT + threadIdx.x;
          pr[u] = make_uint2(0u, 0u);
          if (fu < m) {
            const uint32_t at = s_key[fu];
            pr[u] = ws.pairs[at];
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t fu = f0 + (uint32_t)u * kSelNT + threadIdx.x;
          if (fu < m) {
            s_key[fu] = pr[u].x;
            s_idx[fu] = pr[u].y;
          }
        }
      }
    } else if (in_lds) {
      // round trip 2: the listed candidates
      for (uint32_t f0 = 0; f0 < m; f0 += (uint32_t)kSelNT * 4u) {
        uint32_t kx[4], ix[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t f = f0 + (uint32_t)u * kSelNT + threadIdx.x;
          kx[u] = f < m ? lk[f] : 0u;
          ix[u] = f < m ? li[f] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t f = f0 + (uint32_t)u * kSelNT + threadIdx.x;
          if (f < m) {
            s_key[f] = kx[u];
            s_idx[f] = ix[u];
            sand &= kx[u];
            sor |= kx[u];
          }
        }
      }
    }
    if (!BIG && rows_lds)
      for (uint32_t x = threadIdx.x; x < nr; x += kSelNT) s_add[x] = 0;
    __syncthreads();
    // need == 0 (random-k only): the certain winners, keys below ulo, are all the winners
    uint32_t Tk = KIND == 1 ? ~T.seg_ulo[l] : 0u, IT = 0;
    // many-row top-k layouts: ties at the threshold key are ordered by index through the rows
    // (a list of millions of equal keys, as bf16 gradients give, took one workgroup 7-14 ms)
    uint32_t tneed = 0;
    uint32_t* defer = KIND == 0 && BIG ? &tneed : nullptr;
    if (need > 0) {
      if constexpr (KIND == 1) {
        // random-k: every listed key' = ~u has u in [ulo, tau), so its bits above the highest one
        // in which ~(tau - 1) and ~ulo differ are theirs: the prefix the AND / OR sweep over the
        // list finds (1.2 us on ResNet-50 flat) comes from the window itself
        const uint32_t klo = ~(uint32_t)(T.seg_tau[l] - 1u), khi = ~T.seg_ulo[l];
        if (in_lds) list_threshold_ao(s_key, s_idx, m, need, klo, khi, hist, lds, s_g, Tk, IT, defer);
        else if (!band_threshold(lk, li, m, need, ~khi, ~klo, s_key, s_idx, kCap, hist, lds, s_g, Tk, IT))
          list_threshold_ao(lk, li, m, need, klo, khi, hist, lds, s_g, Tk, IT, defer);
      } else if (in_lds) {
        // (the AND / OR taken while staging the list spares a sweep over it: 1.1 us on ResNet-50)
        if (m > kRankList) block_and_or(sand, sor, lds);
        list_threshold_ao(s_key, s_idx, m, need, sand, sor, hist, lds, s_g, Tk, IT, defer);
      } else {
        list_threshold(lk, li, m, need, hist, lds, s_g, Tk, IT, defer);
      }
      // the list's winners join their rows' counts (many rows, top-k: a list that fits LDS, else the
      // rows are counted again by k_rowcount)
      const uint32_t c0 = o / kTile;
      if constexpr (BIG) done = IT != kTieRows && (KIND == 1 || in_lds);
      auto join = [&](uint32_t i) {
        if (!BIG && rows_lds) atomicAdd(&s_add[i / kTile - c0], 1u);
        else atomicAdd(&ws.rcnt[r0 + (i / kTile - c0)], 1u);
      };
      if (!BIG || done) {
        if (in_lds) {
          for (uint32_t j = threadIdx.x; j < m; j += kSelNT) {
            const uint32_t k = s_key[j], i = s_idx[j];
            if (k > Tk || (k == Tk && i < IT)) join(i);
          }
        } else {
          for_keys2(lk, [&](uint32_t, uint32_t k, size_t at) {
            if (k >= Tk) {
              const uint32_t i = li.arr[at];
              if (k > Tk || i < IT) join(i);
            }
          });
        }
      }
    }
    if (threadIdx.x == 0) {
      R[R_T] = Tk;
      R[R_IT] = IT;
      if (IT == kTieRows) R[R_NEED] = tneed;
    }
    if (!BIG && !rows_lds) {
      // the additions went to global memory: order them before re-reading the counts
      __threadfence();
      __syncthreads();
#pragma unroll
      for (uint32_t x = 0; x < kPer; ++x) cr[x] = a + x < b ? rc[a + x] : 0u;
    }
    __syncthreads();
  }
  if constexpr (BIG) {
    if (KIND == 0 && threadIdx.x == 0) R[R_DONE] = done ? 1u : 0u;
    return;
  }
  // row offsets: exclusive scan of the rows' winner counts (mode 1: every candidate wins)
  const uint32_t* cnt = listed ? rc : cc;
  const bool add = listed && rows_lds && !tie;
  uint32_t w[kPer], sum = 0;
#pragma unroll
  for (uint32_t x = 0; x < kPer; ++x) {
    w[x] = (listed ? cr[x] : cn[x]) + (add && a + x < b ? s_add[a + x] : 0u);
    sum += w[x];
  }
  for (uint32_t x = a + kPer; x < b; ++x) sum += cnt[x] + (add ? s_add[x] : 0u);
  uint32_t tot;
  const uint32_t ex = block_excl_scan<kSelNT>(sum, lds, tot);
  uint32_t run = (uint32_t)T.seg_P[l] + ex;
  uint32_t* roff = ws.roff + r0;
#pragma unroll
  for (uint32_t x = 0; x < kPer; ++x) {
    if (a + x < b) roff[a + x] = run;
    run += w[x];
  }
  for (uint32_t x = a + kPer; x < b; ++x) {
    roff[x] = run;
    run += cnt[x] + (add ? s_add[x] : 0u);
  }
  if (threadIdx.x == 0 && tot != kl) atomicOr(ws.diag, kDiagCount);
}

// Top-k, many rows, per row of a segment whose list did not fit k_select's LDS (or whose ties or
// retry change the rows' counts): how many of the row's candidates win.  One wavefront per row,
// kRowcountU chunks of 64 candidates loaded together, counts by ballots.
constexpr uint32_t kRowcountU = 4;
__global__ __launch_bounds__(kNT) void k_rowcount(Tables T, WSel ws0, Batch BT) {
  const WSel ws = ws_at(ws0, (uint64_t)blockIdx.y * BT.ws);
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t row = blockIdx.x * (kNT / 64) + (threadIdx.x >> 6);
  if (row >= (uint32_t)T.nrows) return;
  const int l = T.L == 1 ? 0 : T.row_seg[row];
  const uint32_t* R = res_of(ws, l);
  if (R[R_SLOW] || R[R_MODE] || R[R_DONE]) return;
  const uint32_t cw = ws.counts[row], cnt = cw & ~kAccRow;
  // a row emitted from acc (winning ties): k_select wrote its winner count (its stored candidates,
  // which all win, and the ties it takes)
  if (cw & kAccRow) return;
  const uint32_t co = row_entry(T, ws, row, cnt, ws.coff[row]), tb = row_tile(T, row);
  uint32_t won = 0, tie = 0;
  const uint32_t Tk = R[R_T], IT = R[R_IT];
  const bool defer = IT == kTieRows;  // ties at T resolved by k_rowtie: count them apart
  const float* cv = ws.cand_val + co;
  const uint16_t* ci = ws.cand_loc + co;
  for (uint32_t j0 = 0; j0 < cnt; j0 += 64u * kRowcountU) {
    float v[kRowcountU];
#pragma unroll
    for (uint32_t u = 0; u < kRowcountU; ++u) {
      const uint32_t j = j0 + 64u * u + lane;
      v[u] = j < cnt ? cv[j] : 0.0f;
    }
#pragma unroll
    for (uint32_t u = 0; u < kRowcountU; ++u) {
      const uint32_t j = j0 + 64u * u + lane, k = mag_key(v[u]);
      const bool in = j < cnt;
      // (the index only for a key equal to the threshold key)
      const bool w = in && (k > Tk || (!defer && k == Tk && tb + ci[j] < IT));
      won += (uint32_t)__popcll(__ballot(w));
      tie += (uint32_t)__popcll(__ballot(in && defer && k == Tk));
    }
  }
  if (lane == 0) {
    ws.rcnt[row] = won;
    if (defer) ws.rtie[row] = tie;
  }
}

// Magnitude keys of a row's stored candidates.
struct CandKeys {
  const float* v;
  __device__ __forceinline__ uint32_t operator[](uint32_t f) const { return mag_key(v[f]); }
};

// Top-k, many rows, per segment whose threshold key T is shared by more candidates than win (R_IT =
// kTieRows): a scan of the rows' counts of keys equal to T (tiles of kSelNT * 8 rows: coalesced loads
// into LDS, eight consecutive rows per thread, a workgroup scan) finds the row where the R_NEED-th
// falls, then that tie inside the row's candidates (stored in index order) gives R_IT, and the rows
// before it add all their ties to their winners, the row itself the ties up to that one.
__global__ __launch_bounds__(kSelNT) void k_rowtie(Tables T, WSel ws0, Batch BT) {
  const WSel ws = ws_at(ws0, (uint64_t)blockIdx.y * BT.ws);
  constexpr uint32_t kU = 8, kTl = kSelNT * kU;
  __shared__ uint32_t lds[2 * kSelNT / 64];
  __shared__ uint32_t s_c[kTl + kTl / 32];
  __shared__ uint32_t s_row, s_rank;
  auto pad = [](uint32_t i) { return i + (i >> 5); };
  const int l = blockIdx.x;
  const uint32_t* R = res_of(ws, l);
  if (R[R_SLOW] || R[R_MODE] || R[R_IT] != kTieRows) return;
  const uint32_t r0 = (uint32_t)T.seg_cbase[l], nr = (uint32_t)T.seg_cbase[l + 1] - r0;
  uint32_t* cnt = ws.rcnt + r0;
  const uint32_t* rt = ws.rtie + r0;
  const uint32_t need = R[R_NEED], Tk = R[R_T];
  if (threadIdx.x == 0) {
    s_row = nr;
    s_rank = 0;
  }
  uint32_t before = 0;  // ties in earlier tiles
  for (uint32_t t0 = 0; t0 < nr; t0 += kTl) {
    uint32_t v[kU];
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) {
      const uint32_t x = t0 + u * kSelNT + threadIdx.x;
      v[u] = x < nr ? rt[x] : 0u;
    }
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) s_c[pad(u * kSelNT + threadIdx.x)] = v[u];
    __syncthreads();
    uint32_t sum = 0;
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) {
      v[u] = s_c[pad(threadIdx.x * kU + u)];
      sum += v[u];
    }
    uint32_t tot;
    uint32_t run = before + block_excl_scan<kSelNT>(sum, lds, tot);
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) {
      if (run < need && need <= run + v[u]) {
        s_row = t0 + threadIdx.x * kU + u;
        s_rank = need - run;
      }
      run += v[u];
    }
    before += tot;
    __syncthreads();
  }
  __syncthreads();
  // the s_rank-th key equal to T among the row's candidates (index order): the last winner
  const uint32_t sr = s_row, srank = s_rank;
  if (sr < nr) {
    const uint32_t row = r0 + sr, c = ws.counts[row];
    const uint32_t co = row_entry(T, ws, row, c, ws.coff[row]);
    const uint32_t p = block_nth_equal(CandKeys{ws.cand_val + co}, c, Tk, srank, lds);
    if (threadIdx.x == 0) res_of(ws, l)[R_IT] = row_tile(T, row) + ws.cand_loc[(size_t)co + p] + 1u;
  }
  for (uint32_t x = threadIdx.x; x < nr && x <= sr; x += kSelNT) cnt[x] += x < sr ? rt[x] : srank;
}

// Many rows: the winners of each of at most kRowBlocks blocks of `rows` consecutive rows (a multiple of
// kRowsumT; one workgroup each), and every row's winners before it in its block.  A segment's rows
// hold k_l winners in all, so a row's message position is the winners of all the rows before it,
// whichever segments they belong to.  (One workgroup walking all rows took 63 us over the 244,141
// rows of 1e9 elements.)
constexpr uint32_t kRowsumT = kNT * 8u;
template <int KIND>
__global__ __launch_bounds__(kNT) void k_rowsum(Tables T, WSel ws0, Batch BT, uint32_t rows) {
  const WSel ws = ws_at(ws0, (uint64_t)blockIdx.y * BT.ws);
  __shared__ uint32_t lds[kNT / 64];
  const uint32_t b0 = blockIdx.x * rows, b1 = min((uint32_t)T.nrows, b0 + rows);
  uint32_t run = 0;
  for (uint32_t t0 = b0; t0 < b1; t0 += kRowsumT) {
    const uint32_t x0 = t0 + threadIdx.x * 8u;
    uint32_t c[8], sum = 0;
    if (x0 + 8u <= b1) {  // rows start at multiples of eight
      const uint4 p = *reinterpret_cast<const uint4*>(ws.rcnt + x0), q = *reinterpret_cast<const uint4*>(ws.rcnt + x0 + 4);
      c[0] = p.x; c[1] = p.y; c[2] = p.z; c[3] = p.w;
      c[4] = q.x; c[5] = q.y; c[6] = q.z; c[7] = q.w;
    } else {
#pragma unroll
      for (uint32_t u = 0; u < 8u; ++u) c[u] = x0 + u < b1 ? ws.rcnt[x0 + u] : 0u;
    }
#pragma unroll
    for (uint32_t u = 0; u < 8u; ++u) {
      const uint32_t x = x0 + u;
      if (x < b1) {
        const int l = T.L == 1 ? 0 : T.row_seg[x];
        const uint32_t* R = res_of(ws, l);
        // the exact path wrote its segment's message: its first row stands for all
        if (R[R_SLOW]) c[u] = x == (uint32_t)T.seg_cbase[l] ? (uint32_t)T.seg_k[l] : 0u;
        else if (KIND == 0 && R[R_MODE]) c[u] = ws.counts[x];  // every candidate wins
      }
      sum += c[u];
    }
    uint32_t tot;
    uint32_t at = run + block_excl_scan<kNT>(sum, lds, tot);
#pragma unroll
    for (uint32_t u = 0; u < 8u; ++u) {
      if (x0 + u < b1) ws.roff[x0 + u] = at;
      at += c[u];
    }
    run += tot;
  }
  if (threadIdx.x == 0) ws.bsum[blockIdx.x] = run;
}

// The sum of the first b blocks' winners (uniform b; one wavefront).
__device__ __forceinline__ uint32_t rows_before(const WSel& ws, uint32_t b) {
  uint32_t s = 0;
#pragma unroll
  for (uint32_t u = 0; u < kRowBlocks / 64u; ++u) {
    const uint32_t j = u * 64u + (threadIdx.x & 63u);
    if (j < b) s += ws.bsum[j];
  }
  return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(s), 63);
}

// Emission: per row, the winners in index order to the message at the row's offset, and e = +0
// there.  One wavefront per RW consecutive rows: lanes j < RW hold row j's count, offset and
// threshold; the rows' candidates are laid out one after another over the 64 lanes (a wave prefix
// of the counts; each lane finds its row by a binary search over those lanes), so a wavefront
// serves its rows in one or a few passes of 64 candidates, the next pass's loads in flight while
// the current one is written.  A winner's position is its row's offset plus the row's winners
// before it: earlier passes (kept by the row's lane) and a ballot count over the row's lanes in
// this pass.  RW = 2 to 16 for random-k, by the candidates of a row; for top-k, whose rows in the
// layers of largest magnitude hold hundreds, 2 for a batch and 4 on a very large sparse layout (one row
// to a wavefront: k_emit_row).  A top-k row with winning ties (flagged kAccRow) takes its elements in
// acc as its candidates.  The step's last kernel, it also clears the overflow pool's counters for the
// next step.
template <int KIND, uint32_t RW, bool ONE>
__global__ __launch_bounds__(kNT) void k_emit(Tables T, WSel ws0, uint32_t* out_idx, float* out_val, Batch BT,
                                              int cand_zeroed, uint32_t block_rows) {
  constexpr bool ACC_ROWS = KIND == 0;
  static_assert(RW >= 1 && RW <= 64 && (RW & (RW - 1)) == 0, "one lane per row, a power of two");
  const WSel ws = ws_at(ws0, (uint64_t)blockIdx.y * BT.ws);
  float* e_zero = BT.e[blockIdx.y];
  out_idx = shifted(out_idx, (uint64_t)blockIdx.y * BT.msg * 4u);
  out_val = out_val ? shifted(out_val, (uint64_t)blockIdx.y * BT.msg * 4u) : nullptr;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t row0 = (blockIdx.x * (kNT / 64) + (threadIdx.x >> 6)) * RW;
  if (row0 >= (uint32_t)T.nrows) return;
  // lane j < RW: row row0 + j (rows past the end and rows of exact-path segments count 0)
  if (blockIdx.x == 0 && threadIdx.x < (unsigned)kPools) *pcnt_of(ws, threadIdx.x) = 0u;
  const uint32_t myrow = row0 + lane;
  const bool has_row = lane < RW && myrow < (uint32_t)T.nrows;
  uint32_t cnt = 0, off = 0, Tk = 0, IT = 0, pend = 0, co = 0, in_acc = 0;
  // zk: the pass stored +0 at this row's candidates (random-k, fused: all, zk = 0; top-k segments with
  // seg_zc, unless a candidate retry put acc back: those of keys from zk on): losers among them get
  // their values back, winners among the others +0.  A row emitted from acc whose candidates are +0
  // first puts them back (rst, ocnt and oco: its own candidates).
  constexpr uint32_t kNoZ = 0xFFFFFFFFu;  // none (above every magnitude)
  uint32_t zk = kNoZ, rst = 0, ocnt = 0, oco = 0, pbeg = 0, tb = 0;
  bool last_row = false;  // of its segment
  if (has_row) {
    const int l = ONE ? 0 : T.row_seg[myrow];  // one segment: no load before the record
    const uint32_t* R = res_of(ws, l);
    cnt = ws.counts[myrow];
    co = ws.coff[myrow];
    off = ws.roff[myrow];
    pbeg = (uint32_t)T.seg_P[l];
    pend = (uint32_t)T.seg_P[l + 1];
    tb = row_tile(T, myrow);
    last_row = T.L == 1 ? myrow + 1u == (uint32_t)T.nrows : myrow + 1u == (uint32_t)T.seg_cbase[l + 1];
    Tk = R[R_T];
    IT = R[R_IT];
    const bool zrow = e_zero && (cand_zeroed || (ACC_ROWS && T.seg_zc[l] && !R[R_RETRY]));
    if (ACC_ROWS && (cnt & kAccRow)) {  // the row's first element in acc
      if (zrow) {
        ocnt = ws.rtie[myrow];
        oco = row_entry(T, ws, myrow, ocnt, co);
        rst = oco != kDropped ? 1u : 0u;
      }
      uint32_t hi;
      row_bounds(T, myrow, co, hi);
      cnt &= ~kAccRow;
      in_acc = 1u;
    } else {
      co = row_entry(T, ws, myrow, cnt, co);
      if (zrow) zk = KIND == 0 ? R[R_Z] : 0u;
    }
    if (R[R_SLOW]) {
      cnt = 0;
      rst = 0;
      last_row = false;
    }
  }
  if (block_rows) {  // (a wavefront's rows lie in one block)
    const uint32_t before = rows_before(ws, row0 / block_rows);
    off += before;
  }
  const float* acc = BT.g[blockIdx.y] ? BT.e[blockIdx.y] : BT.src[blockIdx.y];
  if (ACC_ROWS && __ballot(rst != 0u)) {  // wave-uniform
    for (uint32_t u = 0; u < RW; ++u) {
      const uint32_t n = __shfl(rst, (int)u, 64) ? __shfl(ocnt, (int)u, 64) : 0u;
      const uint32_t b0 = __shfl(oco, (int)u, 64);
      const uint32_t t0 = __shfl(tb, (int)u, 64);
      for (uint32_t j = lane; j < n; j += 64) e_zero[t0 + ws.cand_loc[(size_t)b0 + j]] = ws.cand_val[(size_t)b0 + j];
    }
    __threadfence_block();  // before the wavefront reads the rows' elements from acc
  }
  const uint32_t incl = wave_incl_scan(cnt);
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
  const uint32_t pre = incl - cnt;  // this lane's row: first flattened candidate
  const uint32_t copre = co - pre;
  // what lane r holds of row r: the same for every row of one segment (lane 0 has a row)
  auto of_row = [&](uint32_t x, uint32_t r) -> uint32_t {
    return ONE ? (uint32_t)__builtin_amdgcn_readfirstlane((int)x) : (uint32_t)__shfl(x, (int)r, 64);
  };
  auto tile_of = [&](uint32_t r) -> uint32_t { return ONE ? (row0 + r) * kTile : (uint32_t)__shfl(tb, (int)r, 64); };
  // The wave's loop; the form that tests for rows emitted from acc runs only in a wave holding one.
  auto run = [&](auto acc_rows) {
    constexpr bool AR = decltype(acc_rows)::value;
    // flattened candidate f -> its row lane r (the last row lane with pre_r <= f; for f < total that
    // row's count is nonzero, so f lies inside it) and its entry: a pool entry, or an element of acc
    auto locate = [&](uint32_t f, uint32_t& r, uint32_t& sl, bool& ia) {
      r = 0;
#pragma unroll
      for (uint32_t step = RW / 2; step >= 1; step >>= 1) {
        const uint32_t p = __shfl(pre, (int)(r + step), 64);
        if (f < total && p <= f) r += step;
      }
      sl = __shfl(copre, (int)r, 64) + f;
      ia = AR && __shfl(in_acc, (int)r, 64) != 0u;
    };
    // the entry's key', its element within the row's tile (with kCertain where it wins anyhow) and value
    auto fetch = [&](uint32_t sl, uint32_t t0, bool ia, uint32_t& k, uint32_t& i, float& v) {
      if (AR && ia) {
        v = acc[sl];
        i = sl - t0;
      } else {
        v = ws.cand_val[sl];
        i = ws.cand_loc[sl];
      }
      if constexpr (KIND == 0) k = mag_key(v);
      else k = sl;  // the key is loaded for an undecided candidate only, when its pass comes
    };
    uint32_t done = 0;  // this lane's row: winners emitted in earlier passes
    uint32_t r, sl;
    bool ia;
    locate(lane, r, sl, ia);
    uint32_t k = 0, i = 0;
    float v = 0.0f;
    {
      const uint32_t t0 = tile_of(r);
      if (lane < total) fetch(sl, t0, ia, k, i, v);
    }
    for (uint32_t f0 = 0; f0 < total; f0 += 64) {
      const uint32_t f = f0 + lane;
      const bool in = f < total;
      const uint32_t rpre = __shfl(pre, (int)r, 64);
      const uint32_t rTk = of_row(Tk, r), rIT = of_row(IT, r);
      const uint32_t roffr = __shfl(off + done, (int)r, 64);
      // (one segment: no row's candidates are +0 where another's are not, but a row emitted from acc)
      const uint32_t rpend = of_row(pend, r), rzk = ONE && !AR ? of_row(zk, r) : (uint32_t)__shfl(zk, (int)r, 64);
      const uint32_t rpbeg = of_row(pbeg, r);
      const bool certain = KIND == 1 && (i & kCertain);
      uint32_t ck = k;
      if constexpr (KIND == 1) ck = in && !certain ? ws.cand_key[k] : 0u;
      const uint32_t ci = tile_of(r) + (i & (kTile - 1u));
      const float cv = v;
      // the next pass's candidates, in flight while this pass is written
      uint32_t rn = 0, sn = 0;
      bool ian = false;
      locate(f + 64, rn, sn, ian);
      const uint32_t tn = tile_of(rn);
      if (f + 64 < total) fetch(sn, tn, ian, k, i, v);
      const bool win = in && (certain || ck > rTk || (ck == rTk && ci < rIT));
      const bool zeroed = KIND == 0 ? ck >= rzk : rzk == 0u;
      const uint64_t bw = __ballot(win);
      // this pass's lanes of row r before this lane: [lo_r, lane)
      const uint32_t lo_r = rpre > f0 ? rpre - f0 : 0u;
      const uint64_t below = (lane ? (~0ull >> (64 - lane)) : 0ull) & ~((lo_r ? (~0ull >> (64 - lo_r)) : 0ull));
      const uint32_t pos = roffr + (uint32_t)__popcll(bw & below);
      if (win && pos - rpbeg < rpend - rpbeg) {
        out_idx[pos] = ci;
        if (out_val) out_val[pos] = cv;
        if (e_zero && !zeroed) e_zero[ci] = 0.0f;
      }
      if (e_zero && zeroed && in && !win) e_zero[ci] = cv;  // a losing candidate stored as +0: its value
      // each row lane adds its winners of this pass
      if (has_row) {
        const uint32_t a = pre > f0 ? pre - f0 : 0u, z = incl > f0 ? min(incl - f0, 64u) : 0u;
        if (z > a) {
          const uint64_t m = (z == 64 ? ~0ull : (~0ull >> (64 - z))) & ~(a ? (~0ull >> (64 - a)) : 0ull);
          done += (uint32_t)__popcll(bw & m);
        }
      }
      r = rn;
    }
    if (block_rows && last_row && off + done != pend) atomicOr(ws.diag, kDiagCount);
  };
  if (ACC_ROWS && __ballot(in_acc != 0u)) run(std::true_type{});
  else run(std::false_type{});
}

// The same, one row per wavefront, for rows of many candidates: everything that the row's lanes share is
// kept in scalar registers, kRowU chunks of 64 candidates loaded together, the next ones in flight while
// they are written (a wait for loads also waits for the stores before it: BERT flat at 10 % 54.3 -> 52.1 us
// against one chunk ahead).
constexpr uint32_t kRowU = 4;
template <int KIND>
__global__ __launch_bounds__(kNT) void k_emit_row(Tables T, WSel ws0, uint32_t* out_idx, float* out_val, Batch BT,
                                                  int cand_zeroed, uint32_t block_rows) {
  const WSel ws = ws_at(ws0, (uint64_t)blockIdx.y * BT.ws);
  float* e_zero = BT.e[blockIdx.y];
  out_idx = shifted(out_idx, (uint64_t)blockIdx.y * BT.msg * 4u);
  out_val = out_val ? shifted(out_val, (uint64_t)blockIdx.y * BT.msg * 4u) : nullptr;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t row = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kNT / 64) + (threadIdx.x >> 6)));
  if (row >= (uint32_t)T.nrows) return;
  if (blockIdx.x == 0 && threadIdx.x < (unsigned)kPools) *pcnt_of(ws, threadIdx.x) = 0u;
  const int l = T.L == 1 ? 0 : T.row_seg[row];
  const uint32_t* R = res_of(ws, l);
  // one segment: the first candidates of the row's static slot, in the same round trip as its counts
  // (used if the row's candidates are there)
  const uint32_t cap0 = T.L == 1 ? min(ws.S, (uint32_t)T.d - row * kTile) : 0u;
  float vn[kRowU];
  uint32_t xn[kRowU];
#pragma unroll
  for (uint32_t u = 0; u < kRowU; ++u) {
    const uint32_t j = 64u * u + lane;
    vn[u] = j < cap0 ? ws.cand_val[(size_t)row * ws.S + j] : 0.0f;
    xn[u] = j < cap0 ? ws.cand_loc[(size_t)row * ws.S + j] : 0u;
  }
  const uint32_t cw = ws.counts[row], Tk = R[R_T], IT = R[R_IT], tb = row_tile(T, row);
  const uint32_t pbeg = (uint32_t)T.seg_P[l], pend = (uint32_t)T.seg_P[l + 1];
  uint32_t off = ws.roff[row];
  if (R[R_SLOW]) return;
  if (block_rows) off += rows_before(ws, row / block_rows);
  const bool zrow = e_zero && (cand_zeroed || (KIND == 0 && T.seg_zc[l] && !R[R_RETRY]));
  const bool in_acc = KIND == 0 && (cw & kAccRow);
  uint32_t cnt = cw & ~kAccRow, co = 0;
  const float* acc = BT.g[blockIdx.y] ? BT.e[blockIdx.y] : BT.src[blockIdx.y];
  if (in_acc) {
    if (zrow) {  // its own candidates' values go back into acc first
      const uint32_t oc = ws.rtie[row], oco = row_entry(T, ws, row, oc, ws.coff[row]);
      if (oco != kDropped)
        for (uint32_t j = lane; j < oc; j += 64) e_zero[tb + ws.cand_loc[(size_t)oco + j]] = ws.cand_val[(size_t)oco + j];
      __threadfence_block();  // before the wavefront reads the row's elements from acc
    }
    uint32_t hi;
    row_bounds(T, row, co, hi);
  } else {
    co = row_entry(T, ws, row, cnt, ws.coff[row]);
  }
  const bool restore = zrow && !in_acc;  // the pass stored +0 at candidates (top-k: of keys from zk on)
  const uint32_t zk = KIND == 0 && restore ? R[R_Z] : 0xFFFFFFFFu;
  auto fetch = [&](uint32_t j0) {  // lane's candidates of kRowU chunks
#pragma unroll
    for (uint32_t u = 0; u < kRowU; ++u) {
      const uint32_t j = j0 + 64u * u + lane;
      if (j < cnt) {
        vn[u] = in_acc ? acc[co + j] : ws.cand_val[(size_t)co + j];
        xn[u] = in_acc ? co + j - tb : ws.cand_loc[(size_t)co + j];
      }
    }
  };
  if (!(cap0 && !in_acc && co == row * ws.S)) fetch(0);
  uint32_t done = 0;
#pragma unroll 1
  for (uint32_t j0 = 0; j0 < cnt; j0 += 64u * kRowU) {
    float v[kRowU];
    uint32_t x[kRowU], k[kRowU];
#pragma unroll
    for (uint32_t u = 0; u < kRowU; ++u) {
      v[u] = vn[u];
      x[u] = xn[u];
      k[u] = mag_key(v[u]);
      if constexpr (KIND == 1) {
        const uint32_t j = j0 + 64u * u + lane;
        k[u] = j < cnt && !(x[u] & kCertain) ? ws.cand_key[(size_t)co + j] : 0u;
      }
    }
    if (cnt - j0 > 64u * kRowU) fetch(j0 + 64u * kRowU);  // in flight while these chunks are written
#pragma unroll
    for (uint32_t u = 0; u < kRowU; ++u) {
      if (j0 + 64u * u >= cnt) break;
      const uint32_t left = cnt - j0 - 64u * u;
      const uint64_t there = left >= 64u ? ~0ull : (1ull << left) - 1ull;
      const uint32_t i = tb + (x[u] & (kTile - 1u));
      uint64_t bw = __ballot(k[u] > Tk);
      const uint64_t eq = __ballot(k[u] == Tk) & there;
      if (eq) bw |= __ballot(k[u] == Tk && i < IT);
      if constexpr (KIND == 1) bw |= __ballot((x[u] & kCertain) != 0u);
      bw &= there;
      const uint32_t at = off + done;  // the chunk's first winner
      const uint32_t pos = at + lanes_below(bw);
      done += (uint32_t)__popcll(bw);
      // (a chunk's positions lie in the segment's part of the message unless its counts are wrong)
      const bool safe = at >= pbeg && off + done <= pend;
      const bool zeroed = KIND == 0 ? k[u] >= zk : restore;
      if (safe && __builtin_amdgcn_inverse_ballot_w64(bw)) {
        out_idx[pos] = i;
        if (out_val) out_val[pos] = v[u];
        if (e_zero && !zeroed) e_zero[i] = 0.0f;  // a winner not stored as +0
      }
      if (restore && zeroed && __builtin_amdgcn_inverse_ballot_w64(there & ~bw)) e_zero[i] = v[u];  // a loser that was
    }
  }
  if (block_rows && lane == 0) {
    const bool last = T.L == 1 ? row + 1u == (uint32_t)T.nrows : row + 1u == (uint32_t)T.seg_cbase[l + 1];
    if (last && off + done != pend) atomicOr(ws.diag, kDiagCount);
  }
}

}  // namespace efs
