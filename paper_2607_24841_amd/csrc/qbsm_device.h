// Device helpers shared by the product kernels: spike expansion, staged
// epilogue operands, weight-skip statistics.
#pragma once

#include "common.h"

namespace nmdlm {

constexpr int kMaxEpiTokens = 128;      // row-block tokens whose residual words are staged
static_assert(kMaxEpiTokens >= 8 * 16, "every tile's residual words are staged (RT <= 8)");

__device__ __forceinline__ uint32_t expand4(uint32_t nib) {
  // 4 bits -> 4 bytes of 0/1 (bit i -> byte i); the shifted copies of the
  // nibble do not overlap, so the multiply adds no carries.
  return (nib * 0x00204081u) & 0x01010101u;
}

__device__ __forceinline__ v4i a_operand(uint32_t b16) {
  return v4i{(int)expand4(b16 & 0xFu), (int)expand4((b16 >> 4) & 0xFu),
             (int)expand4((b16 >> 8) & 0xFu), (int)expand4(b16 >> 12)};
}

// Epilogue operands staged in LDS at kernel entry, so that the epilogue
// issues no dependent global load.
struct EpiStage {
  int bias[64];
  int theta[64];
  unsigned long long resid[kMaxEpiTokens];  // [t * Mb + token]
  signed char lut[256];                     // activation table (EPI_QNL_IF)
  uint32_t vbits[NMDLM_MAX_T * 64];         // channel-major output: token bits per (t, column)
};

// The epilogue operands one thread stages (at most one of each kind per
// thread: 64 columns, T * Mb <= kMaxEpiTokens residual words, 256 table
// bytes), loaded into registers first so that the staging loads of a kernel
// are all in flight together.  The loads take clamped (valid) addresses and
// no per-lane condition; the conditions are applied when the values are
// stored, so that no load is waited for before the last one is issued.
struct EpiRegs {
  int bias, theta_ch, theta_seg;
  unsigned long long resid;
  int lut;
};

template <int NT>
__device__ __forceinline__ EpiRegs epi_load(const QbsmArgs& a, int tid, int x, int y) {
  static_assert(NT >= 256 && NT >= kMaxEpiTokens, "one staged item of each kind per thread");
  EpiRegs r{0, 0, 0, 0ull, 0};
  // each kind is loaded by the waves that hold one of its items (a
  // wave-uniform test), every lane of such a wave at a valid address
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nc = min(x * 64 + (tid & 63), a.N - 1);
  if (wv == 0) {
    if (a.bias) r.bias = a.bias[nc];
    if (a.theta_vec) r.theta_ch = a.theta_vec[nc];
  }
  if (a.mode == EPI_IF || a.mode == EPI_QNL_IF)
    r.theta_seg = a.seg[a.nseg > 1 ? div_small(x * 64, a.inv_segw) : 0].theta;
  if (a.resid && wv * 64 < a.T * a.Mb) {  // T * Mb <= 16 * RT <= kMaxEpiTokens
    const int i = min(tid, a.T * a.Mb - 1);
    const int t = div_small(i, a.inv_mb), m = min(y * a.Mb + (i - t * a.Mb), a.M - 1);
    r.resid = a.resid[t * a.rld_t + (int64_t)m * a.rld_m + x];
  }
  if (a.mode == EPI_QNL_IF && wv < 4) r.lut = (int)(signed char)a.lut[tid & 255];
  return r;
}

template <int NT>
__device__ __forceinline__ void epi_store(const QbsmArgs& a, EpiStage& ep, const EpiRegs& r, int tid,
                                          int x, int y) {
  if (tid < 64) {
    const bool nv = x * 64 + tid < a.N;
    ep.bias[tid] = nv ? r.bias : 0;
    // firing threshold of each column: per channel, else the segment's
    ep.theta[tid] = a.theta_vec ? (nv ? r.theta_ch : 1) : r.theta_seg;
  }
  if (a.resid && tid < a.T * a.Mb) {
    const int t = div_small(tid, a.inv_mb), m = y * a.Mb + (tid - t * a.Mb);
    ep.resid[tid] = m < a.M ? r.resid : 0ull;
  }
  if (a.mode == EPI_QNL_IF && tid < 256) ep.lut[tid] = (signed char)r.lut;
  for (int i = tid; i < NMDLM_MAX_T * 64; i += NT) ep.vbits[i] = 0u;
}

// ------------------------------------------------- weight-skip statistics
// The statistics of a product are those of the whole block: the number of
// input rows (channels) active in the union of all its spike rows.  Workgroup
// (0,0,0) computes them between the barriers the product already has, so they
// add no round trip at the end of the kernel:
//   stats_slice  (with the staging loads) this thread's OR over a slice of
//                the union sources: the producer's partial unions when given,
//                else the spike rows (a product whose own union already is
//                the block union counts that instead)
//   stats_merge  (after the first barrier) ORs the slices into sStat
//   stats_count  (after a later barrier) adds the popcounts into sCnt
//   stats_write  (after a later barrier) thread 0 stores the record
// OR of src[r][w] (r < nsrc, row stride Kw) over a slice of the rows: with
// NT >= Kw, thread tid takes word tid % Kw and rows tid / Kw, + NT / Kw, ...,
// so that few loads per thread are all in flight together.
template <int NT>
__device__ __forceinline__ unsigned long long or_slice(const uint64_t* src, int nsrc, int Kw,
                                                       int tid) {
  unsigned long long u = 0ull;
  if (NT < Kw) return u;
  const float inv_kw = 1.0f / (float)Kw;
  const int slices = div_small(NT, inv_kw), s0 = div_small(tid, inv_kw), w = tid - s0 * Kw;
  if (s0 >= slices) return u;
  int r = s0;
  for (; r + 3 * slices < nsrc; r += 4 * slices)
    u |= src[(size_t)r * Kw + w] | src[(size_t)(r + slices) * Kw + w] |
         src[(size_t)(r + 2 * slices) * Kw + w] | src[(size_t)(r + 3 * slices) * Kw + w];
  for (; r < nsrc; r += slices) u |= src[(size_t)r * Kw + w];
  return u;
}

// dst[w] = OR of the slices (dst cleared before the barrier that precedes
// this call); bits of the last word past K are dropped with last_mask.
template <int NT>
__device__ __forceinline__ void or_merge(unsigned long long* dst, const uint64_t* src, int nsrc,
                                         int Kw, int tid, unsigned long long u,
                                         unsigned long long last_mask) {
  if (NT >= Kw) {
    const float inv_kw = 1.0f / (float)Kw;
    const int slices = div_small(NT, inv_kw), s0 = div_small(tid, inv_kw), w = tid - s0 * Kw;
    if (w == Kw - 1) u &= last_mask;
    if (s0 < slices && u) atomicOr(&dst[w], u);
  } else {
    // more words than threads: each thread ORs every source of its words
    for (int w = tid; w < Kw; w += NT) {
      unsigned long long v = 0ull;
      for (int r = 0; r < nsrc; ++r) v |= src[(size_t)r * Kw + w];
      dst[w] = (w == Kw - 1) ? (v & last_mask) : v;  // the only writer of word w
    }
  }
}

template <int NT>
__device__ __forceinline__ unsigned long long stats_slice(const QbsmArgs& a, int Kw, int tid) {
  if (a.dense) return 0ull;
  return a.upart ? or_slice<NT>(a.upart, a.nparts, Kw, tid) : or_slice<NT>(a.S, a.T * a.M, Kw, tid);
}

template <int NT>
__device__ __forceinline__ void stats_merge(const QbsmArgs& a, unsigned long long* sStat, int Kw,
                                            int tid, unsigned long long u) {
  if (a.dense) return;
  if (a.upart) or_merge<NT>(sStat, a.upart, a.nparts, Kw, tid, u, ~0ull);
  else or_merge<NT>(sStat, a.S, a.T * a.M, Kw, tid, u, ~0ull);
}

template <int NT>
__device__ __forceinline__ void stats_count(const QbsmArgs& a, const unsigned long long* sStat,
                                            int* sCnt, int Kw, int tid, int lane) {
  const unsigned long long last_mask = (a.K & 63) ? (1ull << (a.K & 63)) - 1ull : ~0ull;
  int cnt = 0;
  if (a.dense) {
    cnt = tid == 0 ? a.K : 0;
  } else {
    for (int w = tid; w < Kw; w += NT) {
      const unsigned long long u = sStat[w];
      cnt += __popcll((w == Kw - 1) ? (u & last_mask) : u);
    }
  }
  for (int o = kWave / 2; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
  if (lane == 0 && cnt) atomicAdd(sCnt, cnt);
}

__device__ __forceinline__ void stats_write(const QbsmArgs& a, int total) {
  a.stats->k_total = a.K;
  a.stats->k_active = total;
  a.stats->n = a.N;
  a.stats->weight_bytes = (int64_t)total * (int64_t)a.N;
}

// The whole count by one workgroup that has nothing else to do: the union of
// the sources' rows in sU [Kw], sixteen rows of a thread's word in flight.
template <int NT>
__device__ __forceinline__ void stats_alone(const QbsmArgs& a, unsigned long long* sU, int* sCnt, int Kw, int tid,
                            int lane) {
  if (tid == 0) *sCnt = 0;
  for (int w = tid; w < Kw; w += NT) sU[w] = 0ull;
  __syncthreads();
  if (!a.dense) {
    const uint64_t* src = a.upart ? a.upart : a.S;
    const int nsrc = a.upart ? a.nparts : a.T * a.M;
    const int per = min(Kw, NT), slices = NT / per, s0 = tid / per;
    for (int w = tid - s0 * per; w < Kw && s0 < slices; w += per) {
      unsigned long long u = 0ull;
      for (int r = s0; r < nsrc; r += 16 * slices) {
        unsigned long long v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = src[(size_t)min(r + k * slices, nsrc - 1) * Kw + w];
#pragma unroll
        for (int k = 0; k < 16; ++k) u |= v[k];
      }
      if (u) atomicOr(&sU[w], u);
    }
    __syncthreads();
  }
  stats_count<NT>(a, sU, sCnt, Kw, tid, lane);
  __syncthreads();
  if (tid == 0) stats_write(a, *sCnt);
}


}  // namespace nmdlm
