// Attention on spike operands: binary-binary scores (popcount of AND), table
// weights, integer-normalised weighted sum of binary values.
//
//   s = popcount(Q_i AND K_j) per head;  p = lut[s] in [0, 255]
//   num[i,c] = sum_j p_ij V[j,c];  den[i] = sum_j p_ij
//   a[i,c] = floor(256 * num / den)   (0 if den = 0)
//
// Both products run on v_mfma_i32_16x16x64_i8, exact in int32: the scores as
// a 0/1-byte product of key and query bits over the head's channels, the
// weighted sum with p - 128 (signed byte) against the value bits expanded to
// bytes, to which 128 * (number of ones of V[.,c]) is added back.  A sum is at
// most 255 per key: below 2^31 up to NMDLM_MAX_KEYS keys.
#include <algorithm>

#include "common.h"

namespace nmdlm {

static_assert(255LL * NMDLM_MAX_KEYS < 1LL << 31, "sums of table weights fit int32");

// floor(256 * num / den) for 0 <= num <= den (0 when den = 0): from 65536 keys
// on, in 64 bits.  (num and den themselves stay below 2^31 up to
// NMDLM_MAX_KEYS keys of weight 255.)
__device__ __forceinline__ int32_t attn_norm(int num, int den) {
  return den <= 0 ? 0 : (int32_t)((256LL * num) / den);
}

// The same for four numerators over one denominator and fewer than 65536 keys
// (num and den below 2^24, exact as floats): k = 256 / den, lowered by 2^-20 of
// itself, more than the rounding errors of the reciprocal and the two products
// (4 units of 2^-24), so the truncated estimate is the floor or one below it; the
// remainder 256 num - q den, one rounding of an exact value, decides which.
// An empty denominator (num = 0) counts as one.
__device__ __forceinline__ v4i attn_norm4(v4i num, int den_i) {
  const float den = (float)max(den_i, 1);
  const float k = __builtin_amdgcn_rcpf(den) * (256.0f - 0x1p-12f);
  v4i a;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float n = (float)num[e];
    const float q = __builtin_truncf(n * k);
    a[e] = (int)q + (__builtin_fmaf(-q, den, 256.0f * n) >= den ? 1 : 0);
  }
  return a;
}

// ---------------------------------------------------------------------------
// One wave's share of the attention of 16*QG queries of one head and
// timestep: 64-key chunks, each lane (g = lane/16, c = lane%16).
//
// Scores: the A operand of tile u (u = 0..3) holds 16 keys, row r = key
// 16*(r/4) + 4u + r%4 of the chunk, the B operand the 16 queries; the result
// of lane (g, c) is then the scores of query c with keys 16g + 4u + e, so over
// the four tiles a lane owns the 16 consecutive keys 16g .. 16g+15 of its
// query: the operand the weighted sum wants, with no exchange.  A lane's key
// bits (dh = 128: dword g of the row, two k-steps; dh = 64: 16-bit piece g)
// become bytes in place as bits & (0x01010101 << i), of value 2^i; the query's
// byte is 2^(3-i), so a score arrives times 8, the byte offset into the table.
// The order of the channels differs from the memory order, the same way for
// keys and queries.
//
// Weights: the table sits in LDS four times, the entry p - 128 shifted to byte
// 0..3 of a dword, so a P operand dword is four reads and two ORs; scores less
// than 32 apart fall in different banks, equal scores broadcast.
//
// Weighted sum: A = the value bits of 16 channels (rows), B = P (columns =
// queries): lane (g, c) accumulates query c, channels 16n + 4g + e.  Value
// bits h (16 keys of a channel) become bytes as (x >> i) & 0x01010101 of
// x = h | h << 12: byte b of dword i is key i + {0, 8, 4, 12}[b], and P is
// packed to match.
//
// Per 32 queries and chunk (QG = 2, dh = 128) that is 125 vector instructions
// and 32 MFMAs, where scoring by popcounts took 350 vector instructions per 16
// queries; the key and value expansions (100 of the 125) are shared by the QG
// query groups.  Bound by LDS, whose indexed path is busy 51% of the cycles (a third of
// that conflicts of the table reads, 32 of them a chunk), and by instruction issue;
// the matrix cores are busy 37% (counters of the call below).
// T = 4, 16 heads of 128, 2048 queries x 2048 keys: 213 -> 76 us (1.8 POP/s).
// ---------------------------------------------------------------------------
typedef uint32_t __attribute__((may_alias)) u32_alias;
typedef uint16_t __attribute__((may_alias)) u16_alias;
typedef int __attribute__((may_alias)) i32_alias;
typedef v4i __attribute__((may_alias)) v4i_alias;
constexpr uint32_t kByteOnes = 0x01010101u;
constexpr int kAttnStages = 3;    // chunks of a wave in LDS
constexpr int kLutEntries = 132;  // scores 0..128, padded to a multiple of four

// Entry s of the table, 8 bytes (a score arrives times 8, as a byte offset):
// the byte lut[s] - 128 at byte positions 2h and 2h + 1 of two dwords, h = 0, 1
// the half of the table.
struct AttnLut {
  int e[2][kLutEntries][2];
};
constexpr int kLutLoads = (kLutEntries + 63) / 64;  // for a workgroup of one wave
struct LutRegs {
  uint8_t v[kLutLoads];
};
// loads at clamped places, without a condition, to leave with the others
__device__ __forceinline__ LutRegs load_lut(const uint8_t* __restrict__ lut, int tid, int nth) {
  LutRegs r;
#pragma unroll
  for (int k = 0; k < kLutLoads; ++k) r.v[k] = lut[min(tid + k * nth, kLutEntries - 1)];
  return r;
}
__device__ __forceinline__ void fill_lut(AttnLut& sLut, const LutRegs& r, int tid, int nth) {
#pragma unroll
  for (int k = 0; k < kLutLoads; ++k) {
    const int i = tid + k * nth;
    if (i < kLutEntries) {
      const uint32_t v = (uint32_t)r.v[k] ^ 0x80u;
#pragma unroll
      for (int b = 0; b < 4; ++b) sLut.e[b >> 1][i][b & 1] = (int)(v << (8 * b));
    }
  }
}

__device__ __forceinline__ v4i bytes16(uint32_t x) {  // (x >> i) & ones, i = 0..3
  return v4i{(int)(x & kByteOnes), (int)((x >> 1) & kByteOnes), (int)((x >> 2) & kByteOnes),
             (int)((x >> 3) & kByteOnes)};
}
// key bits in place (values 2^i) and the query bits that make every product 8
__device__ __forceinline__ v4i key_bytes(uint32_t x) {
  return v4i{(int)(x & kByteOnes), (int)(x & (kByteOnes << 1)), (int)(x & (kByteOnes << 2)),
             (int)(x & (kByteOnes << 3))};
}
__device__ __forceinline__ v4i query_bytes(uint32_t x) {
  const v4i b = bytes16(x);
  return v4i{b[0] << 3, b[1] << 2, b[2] << 1, b[3]};
}

// A wave's LDS buffer for the chunk being scored: its 64 key rows, in the
// order the tiles take them, and one value word per channel.
template <int DHW>
struct AttnStage {
  uint64_t k[64 * DHW];
  uint64_t v[DHW * 64];
};

// What a lane loads of a chunk: key row `lane`, the value words of channels
// lane and lane + 64 (whole rows and words: adjacent lanes at adjacent
// addresses, where fetching the operand pieces directly cost 400 cache
// accesses per chunk and set the kernel's time).
template <int DHW>
struct AttnChunk {
  uint64_t k[DHW], v[DHW];
};

template <int DHW, int QG>
struct AttnWave {
  static constexpr int NT = DHW * 4;
  v4i q[QG][DHW];
  v4i acc[QG][NT];
  int den[QG];  // sum of p - 128 of query c over this lane's keys
  int cnt[NT];  // ones of channel 16n + c over this lane's keys

  // query rows iq0 + 16u + c (clamped to the last valid row), channels of head h
  __device__ __forceinline__ static void load_queries(uint32_t (&raw)[QG],
                                                      const uint64_t* __restrict__ qrow, int dw,
                                                      int iq0, int mlast, int g, int c) {
#pragma unroll
    for (int u = 0; u < QG; ++u) {
      const uint64_t* p = qrow + (size_t)min(iq0 + 16 * u + c, mlast) * dw;
      if constexpr (DHW == 2) raw[u] = reinterpret_cast<const u32_alias*>(p)[g];
      else raw[u] = reinterpret_cast<const u16_alias*>(p)[g];
    }
  }
  __device__ __forceinline__ void init(const uint32_t (&raw)[QG]) {
#pragma unroll
    for (int u = 0; u < QG; ++u) {
      const uint32_t w = raw[u];
      if constexpr (DHW == 2) {
        q[u][0] = query_bytes(w);
        q[u][1] = query_bytes(w >> 4);
      } else {
        q[u][0] = query_bytes(w | (w << 12));
      }
      den[u] = 0;
#pragma unroll
      for (int n = 0; n < NT; ++n) acc[u][n] = v4i{0, 0, 0, 0};
    }
#pragma unroll
    for (int n = 0; n < NT; ++n) cnt[n] = 0;
  }

  // kb: key row 0 of the timestep at this head's words; vb: value word 0 of
  // the timestep at this head's channels.  The cache capacity is a multiple
  // of 64, so every row of a chunk holds memory (rows past C+M are masked).
  __device__ __forceinline__ static void load(AttnChunk<DHW>& ch, const uint64_t* __restrict__ kb,
                                              const uint64_t* __restrict__ vb, int dw, int d, int jc,
                                              int lane) {
    const uint64_t* kr = kb + (size_t)jc * 64 * dw;
    const uint64_t* vr = vb + (size_t)jc * d;
#pragma unroll
    for (int w = 0; w < DHW; ++w) {
      ch.k[w] = kr[(uint32_t)(lane * dw + w)];
      ch.v[w] = vr[(uint32_t)(w * 64 + lane)];
    }
  }

  // the chunk into LDS
  __device__ __forceinline__ static void put(const AttnChunk<DHW>& ch, AttnStage<DHW>& st, int lane) {
    const int slot = ((lane >> 2) & 3) * 16 + (lane >> 4) * 4 + (lane & 3);
#pragma unroll
    for (int w = 0; w < DHW; ++w) {
      st.k[slot * DHW + w] = ch.k[w];
      st.v[w * 64 + lane] = ch.v[w];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }

  // tile u's key is row c of the tile, its bits dword g of the row (dh = 128)
  // or 16-bit piece g (dh = 64)
  __device__ __forceinline__ static void key_pieces(const AttnStage<DHW>& st, uint32_t (&k)[4], int g,
                                                    int c) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if constexpr (DHW == 2) k[u] = reinterpret_cast<const u32_alias*>(st.k)[(u * 16 + c) * 4 + g];
      else k[u] = reinterpret_cast<const u16_alias*>(st.k)[(u * 16 + c) * 4 + g];
    }
  }
  // the bits of channel 16n + c over keys 16g .. 16g+15
  __device__ __forceinline__ static void value_pieces(const AttnStage<DHW>& st, uint32_t (&v)[NT], int g,
                                                      int c) {
#pragma unroll
    for (int n = 0; n < NT; ++n) v[n] = reinterpret_cast<const u16_alias*>(st.v)[(n * 16 + c) * 4 + g];
  }

  // 8 * scores of the chunk's keys
  __device__ __forceinline__ void scores(const uint32_t (&k)[4], v4i (&s)[QG][4]) const {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      v4i k0, k1;
      if constexpr (DHW == 2) {
        k0 = key_bytes(k[u]);
        k1 = key_bytes(k[u] >> 4);
      } else {
        k0 = key_bytes(k[u] | (k[u] << 12));
      }
#pragma unroll
      for (int w = 0; w < QG; ++w)
        s[w][u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(k0, q[w][0], v4i{0, 0, 0, 0}, 0, 0, 0);
      if constexpr (DHW == 2) {
#pragma unroll
        for (int w = 0; w < QG; ++w)
          s[w][u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(k1, q[w][1], s[w][u], 0, 0, 0);
      }
    }
  }

  // table bytes in place of the scores (tile u's at byte {0, 2, 1, 3}[u])
  __device__ __forceinline__ static void lookup(v4i (&s)[QG][4], const char* lb) {
#pragma unroll
    for (int w = 0; w < QG; ++w)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int b = u == 1 ? 2 : (u == 2 ? 1 : u);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          s[w][u][e] = *reinterpret_cast<const int*>(lb + kLutEntries * 8 * (b >> 1) + 4 * (b & 1) + s[w][u][e]);
      }
  }

  __device__ __forceinline__ static void pack(const v4i (&s)[QG][4], v4i (&p)[QG]) {
#pragma unroll
    for (int w = 0; w < QG; ++w) p[w] = s[w][0] | s[w][1] | s[w][2] | s[w][3];
  }

  __device__ __forceinline__ void weigh(const uint32_t (&v)[NT], const v4i (&p)[QG]) {
#pragma unroll
    for (int w = 0; w < QG; ++w)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        den[w] = __builtin_amdgcn_sdot4(p[w][i], (int)kByteOnes, den[w], false);
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const uint32_t h = v[n];
      cnt[n] += __popc(h);
      const v4i va = bytes16(h | (h << 12));
#pragma unroll
      for (int w = 0; w < QG; ++w)
        acc[w][n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(va, p[w], acc[w][n], 0, 0, 0);
    }
  }

  // the chunks jc0, jc0 + step, ... < nch (jc0 < nch).  Two chunks are in
  // work: while the weighted sum of one runs, the table reads of the next are
  // in flight, and the loads of the one after that.  Only the last chunk of
  // the context can be partial.
  __device__ __forceinline__ void run(const uint64_t* __restrict__ kb, const uint64_t* __restrict__ vb,
                                      int dw, int d, int J, int nch, int jc0, int step,
                                      const AttnLut& sLut, AttnStage<DHW>* st, int lane,
                                      int g, int c, const AttnChunk<DHW>& first,
                                      AttnChunk<DHW> nxt) {
    const char* lb = reinterpret_cast<const char*>(&sLut);
    int jc = jc0;
    AttnStage<DHW>*s0 = st, *s1 = st + 1, *s2 = st + 2;  // chunks j - 1, j, j + 1
    v4i s[QG][4], p[QG];
    uint32_t k[4], v[NT];
    put(first, *s0, lane);
    key_pieces(*s0, k, g, c);
    put(nxt, *s1, lane);
    load(nxt, kb, vb, dw, d, min(jc + 2 * step, nch - 1), lane);
    scores(k, s);
    lookup(s, lb);
    key_pieces(*s1, k, g, c);
    pack(s, p);
    for (jc += step; jc < nch; jc += step) {
      value_pieces(*s0, v, g, c);
      scores(k, s);
      __builtin_amdgcn_sched_barrier(0);
      lookup(s, lb);
      put(nxt, *s2, lane);
      load(nxt, kb, vb, dw, d, min(jc + 2 * step, nch - 1), lane);
      key_pieces(*s2, k, g, c);
      weigh(v, p);
      __builtin_amdgcn_sched_barrier(0);
      pack(s, p);
      AttnStage<DHW>* const t = s0;
      s0 = s1;
      s1 = s2;
      s2 = t;
    }
    value_pieces(*s0, v, g, c);
    const int jl = jc - step;
    if (jl * 64 + 64 > J) {  // wave-uniform
      const int nvalid = J - (jl * 64 + 16 * g);  // of this lane's 16 keys
      const uint32_t vm = nvalid >= 16 ? 0xFFFFu : (nvalid <= 0 ? 0u : ((1u << nvalid) - 1u));
      const v4i m = bytes16(vm | (vm << 12)) * 0xFF;
#pragma unroll
      for (int w = 0; w < QG; ++w) p[w] &= m;
#pragma unroll
      for (int n = 0; n < NT; ++n) v[n] &= vm;
    }
    weigh(v, p);
#pragma unroll
    for (int w = 0; w < QG; ++w) {  // over the four lane groups
      den[w] += __shfl_xor(den[w], 16);
      den[w] += __shfl_xor(den[w], 32);
    }
    // 128 * the ones of each channel over the wave's keys, added to the sums
    // of channels 16n + 4g + e (the counts change lanes through the stage)
#pragma unroll
    for (int n = 0; n < NT; ++n) cnt[n] += __shfl_xor(cnt[n], 16);
#pragma unroll
    for (int n = 0; n < NT; ++n) cnt[n] += __shfl_xor(cnt[n], 32);
    char* sc = reinterpret_cast<char*>(st);
#pragma unroll
    for (int n = 0; n < NT; ++n)  // the four lane groups store the same values
      *reinterpret_cast<i32_alias*>(sc + 64 * n + 4 * c) = 128 * cnt[n];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const v4i x = *reinterpret_cast<const v4i_alias*>(sc + 64 * n + 16 * g);
#pragma unroll
      for (int w = 0; w < QG; ++w) acc[w][n] += x;
    }
  }
};

// valid keys of the chunks jc0, jc0 + step, ... < nch
__device__ __forceinline__ int keys_of(int jc0, int step, int nch, int J) {
  if (jc0 >= nch) return 0;
  const int n = (nch - 1 - jc0) / step + 1;
  return n * 64 - (((nch - 1 - jc0) % step == 0) ? nch * 64 - J : 0);
}

// ---------------------------------------------------------------------------
// k_attn: scores and weighted sums of one (head, 16 queries, timestep), the
// chunks shared by NW waves whose sums meet in LDS; the IF of the output
// follows in its own kernel.  For grids too small for one wave per 16 queries
// (the denoising step's): every load of a short context is in flight at once.
//
// grid (H, n_seq * ceil(M/16), T), M queries per sequence, rows of q and
// a_out sequence-major (n_seq * M per timestep), the caches of sequence s at
// s * seq_words words past kc / vt.
//
// dh = 128 takes 129 registers, one too many for two workgroups on a CU.  WPE = 4
// (waves per SIMD) holds it to 128, an address pair of the chunk loop spilled: for
// grids of more workgroups than CUs (T = 8, 133 x 773 keys, 12 heads 28.0 -> 23.2 us; 101 x
// 899, 16 heads 28.2 -> 23.2); smaller ones lose 4% by the spill.  The
// entries stand at 1 KB, as the products' do: at 256 bytes the same code took 0.2 us more.
// ---------------------------------------------------------------------------
template <int DHW, int NW, int WPE>
__global__ __launch_bounds__(NW * 64, WPE) __attribute__((aligned(1024)))
void k_attn(const uint64_t* __restrict__ q,
            const uint64_t* __restrict__ kc,
            const uint64_t* __restrict__ vt, int64_t cap,
            int T, int M, int C, int H,
            const uint8_t* __restrict__ lut,
            int32_t* __restrict__ a_out, int n_seq,
            int64_t seq_words) {
  constexpr int DH = DHW * 64;
  constexpr int NT = DH / 16;
  constexpr int NTH = NW * 64;
  __shared__ AttnLut sLut;
  __shared__ v4i sNum[NT * 64];  // [tile n][lane]: query c, channels 16n + 4g + e
  __shared__ int sDen[16];
  __shared__ AttnStage<DHW> sStage[kAttnStages * NW];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, c = lane & 15;
  // neighbouring heads share key lines: consecutive logical ids, head fastest
  const int nwg = gridDim.x * gridDim.y * gridDim.z;
  const int lid = xcd_order(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), nwg);
  const int h = lid % gridDim.x, qbg = (lid / gridDim.x) % gridDim.y,
            t = lid / (gridDim.x * gridDim.y);
  const int qbps = gridDim.y / n_seq;               // query blocks per sequence
  const int sq = qbg / qbps, qb = qbg - sq * qbps;  // sequence, block within it
  const int Mt = n_seq * M, r0 = sq * M;            // rows per timestep, first row of sq
  const int d = H * DH, dw = d / 64;
  const int J = C + M;
  const int nch = (J + 63) / 64;
  const uint64_t* kb = kc + sq * seq_words + (size_t)t * cap * dw + h * DHW;
  const uint64_t* vb = vt + sq * seq_words + (size_t)t * (cap / 64) * d + h * DH;

  AttnChunk<DHW> first, next;
  // every load of the prologue leaves before the first is waited for
  const LutRegs lr = load_lut(lut, tid, NTH);
  uint32_t qraw[1];
  AttnWave<DHW, 1>::load_queries(qraw, q + ((size_t)t * Mt + r0) * dw + h * DHW, dw, qb * 16, M - 1, g, c);
  AttnWave<DHW, 1>::load(first, kb, vb, dw, d, min(wave, nch - 1), lane);
  AttnWave<DHW, 1>::load(next, kb, vb, dw, d, min(wave + NW, nch - 1), lane);
  __builtin_amdgcn_sched_barrier(0);
  AttnWave<DHW, 1> w;
  w.init(qraw);
  fill_lut(sLut, lr, tid, NTH);
  for (int i = tid; i < NT * 64; i += NTH) sNum[i] = v4i{0, 0, 0, 0};
  if (tid < 16) sDen[tid] = 0;
  __syncthreads();
  if (wave < nch) {  // wave-uniform
    w.run(kb, vb, dw, d, J, nch, wave, NW, sLut, &sStage[kAttnStages * wave], lane, g, c, first, next);
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const v4i x = w.acc[0][n];
#pragma unroll
      for (int e = 0; e < 4; ++e) atomicAdd(reinterpret_cast<int*>(&sNum[n * 64 + lane]) + e, x[e]);
    }
    if (g == 0) atomicAdd(&sDen[c], w.den[0] + 128 * keys_of(wave, NW, nch, J));
  }
  __syncthreads();

  const bool small = J < 65536;
  for (int i = tid; i < NT * 64; i += NTH) {
    const int n = i >> 6, lc = i & 15, lg = (i >> 4) & 3;
    const int iq = qb * 16 + lc;
    if (iq >= M) continue;
    const v4i x = sNum[i];
    const int den = sDen[lc];
    v4i a;
    if (small) {
      a = attn_norm4(x, den);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = attn_norm(x[e], den);
    }
    int32_t* o = a_out + ((size_t)t * Mt + r0 + iq) * d + h * DH + n * 16 + 4 * lg;
    if ((reinterpret_cast<uintptr_t>(a_out) & 15) == 0) {  // uniform
      *reinterpret_cast<v4i*>(o) = a;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = a[e];
    }
  }
}

// ---------------------------------------------------------------------------
// k_attn_if: attention followed by the IF neuron of its output, in one kernel.
// Workgroup = one head and 16*QG queries, wave = (timestep, part): the parts of
// a timestep (PARTS, QG = 1: grids that leave SIMDs idle) take its chunks in
// turn and add their sums in LDS; without parts a wave takes all chunks of its
// timestep and normalises its sums itself.  The sums or currents meet in LDS
// (16 queries at a time, over the chunks' stages) and the waves share the
// tiles of 16 channels for the IF recurrence over t, the spike words and the
// token's union over t.  a_out (the currents) and s_out are each optional.
// No currents go through memory (64 MB written and read at the 2048-token
// prompt below) and there is no launch between the two.
// ---------------------------------------------------------------------------
struct AttnIfArgs {
  const uint64_t* q;
  const uint64_t* kc;
  const uint64_t* vt;
  int64_t cap;
  int T, M, C, H, n_seq, parts;
  int64_t seq_words;
  const uint8_t* lut;
  int32_t theta;
  int32_t* a_out;
  uint64_t* s_out;
  uint64_t* u_out;
};

template <int DHW, int QG, bool PARTS>
__global__ __launch_bounds__(64 * NMDLM_MAX_T) void k_attn_if(AttnIfArgs a) {
  constexpr int DH = DHW * 64;
  constexpr int NT = DHW * 4;
  static_assert(!PARTS || QG == 1, "parts: one query group");
  __shared__ AttnLut sLut;
  __shared__ int sDen[PARTS ? NMDLM_MAX_T : 1][16];
  __shared__ uint32_t sWord[NMDLM_MAX_T][16][2 * DHW];  // halves of the spike words
  // the waves' stages, then (chunks done) the sums [T][NT][64]
  extern __shared__ v4i sNum[];
  AttnStage<DHW>* sStage = reinterpret_cast<AttnStage<DHW>*>(sNum);

  const int nth = blockDim.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = nth >> 6;
  const int g = lane >> 4, c = lane & 15;
  const int nwg = gridDim.x * gridDim.y;
  const int lid = xcd_order(blockIdx.x + gridDim.x * blockIdx.y, nwg);
  const int h = lid % gridDim.x, qbg = lid / gridDim.x;
  const int qbps = gridDim.y / a.n_seq;
  const int sq = qbg / qbps, qb = qbg - sq * qbps;
  const int Mt = a.n_seq * a.M, r0 = sq * a.M;
  const int d = a.H * DH, dw = d / 64;
  const int J = a.C + a.M, nch = (J + 63) / 64;
  const int np = PARTS ? a.parts : 1;
  const int t = PARTS ? wave / np : wave, part = wave - t * np;
  const uint64_t* kb = a.kc + sq * a.seq_words + (size_t)t * a.cap * dw + h * DHW;
  const uint64_t* vb = a.vt + sq * a.seq_words + (size_t)t * (a.cap / 64) * d + h * DH;

  AttnChunk<DHW> first, next;
  // every load of the prologue leaves before the first is waited for
  const LutRegs lr = load_lut(a.lut, tid, nth);
  uint32_t qraw[QG];
  AttnWave<DHW, QG>::load_queries(qraw, a.q + ((size_t)t * Mt + r0) * dw + h * DHW, dw, qb * 16 * QG,
                                  a.M - 1, g, c);
  AttnWave<DHW, QG>::load(first, kb, vb, dw, d, min(part, nch - 1), lane);
  AttnWave<DHW, QG>::load(next, kb, vb, dw, d, min(part + np, nch - 1), lane);
  __builtin_amdgcn_sched_barrier(0);
  AttnWave<DHW, QG> w;
  w.init(qraw);
  fill_lut(sLut, lr, tid, nth);
  __syncthreads();
  if (!PARTS || part < nch)  // wave-uniform
    w.run(kb, vb, dw, d, J, nch, part, np, sLut, &sStage[kAttnStages * wave], lane, g, c, first, next);
  __syncthreads();  // the stages are read
  if constexpr (PARTS) {
    for (int i = tid; i < a.T * NT * 64; i += nth) sNum[i] = v4i{0, 0, 0, 0};
    for (int i = tid; i < a.T * 16; i += nth) (&sDen[0][0])[i] = 0;
    __syncthreads();
  }
  const bool small = J < 65536;
  const bool vec = (reinterpret_cast<uintptr_t>(a.a_out) & 15) == 0;

#pragma unroll
  for (int u = 0; u < QG; ++u) {
    if (u > 0) __syncthreads();  // the previous group's currents and words are read
    const int iq0 = (qb * QG + u) * 16, iq = iq0 + c;
    for (int i = tid; i < a.T * 32 * DHW; i += nth) (&sWord[0][0][0])[i] = 0u;
    if constexpr (PARTS) {
      if (part < nch) {
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            atomicAdd(reinterpret_cast<int*>(&sNum[(t * NT + n) * 64 + lane]) + e, w.acc[u][n][e]);
        if (g == 0) atomicAdd(&sDen[t][c], w.den[u] + 128 * keys_of(part, np, nch, J));
      }
    } else {
      const int den = w.den[u] + 128 * J;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        v4i x;
        if (small) {
          x = attn_norm4(w.acc[u][n], den);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = attn_norm(w.acc[u][n][e], den);
        }
        sNum[(t * NT + n) * 64 + lane] = x;
      }
    }
    __syncthreads();
    for (int n = wave; n < NT; n += nwaves) {
      v4i V = v4i{0, 0, 0, 0};  // at most 256 T
      for (int t0 = 0; t0 < a.T; t0 += 4) {
        v4i cur[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int tt = min(t0 + k, a.T - 1);
          cur[k] = sNum[(tt * NT + n) * 64 + lane];
          if constexpr (PARTS) {
            const int den = sDen[tt][c];
            if (small) {
              cur[k] = attn_norm4(cur[k], den);
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) cur[k][e] = attn_norm(cur[k][e], den);
            }
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int tt = t0 + k;
          if (tt >= a.T) break;  // uniform
          if (a.a_out && iq < a.M) {
            int32_t* o = a.a_out + ((size_t)tt * Mt + r0 + iq) * d + h * DH + n * 16 + 4 * g;
            if (vec) {
              *reinterpret_cast<v4i*>(o) = cur[k];
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) o[e] = cur[k][e];
            }
          }
          uint32_t bits = 0u;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            V[e] += cur[k][e];
            const bool s = V[e] >= a.theta;
            if (s) V[e] -= a.theta;
            bits |= (uint32_t)s << e;
          }
          // tile n's 16 bits of the query's word, four from each lane group
          atomicOr(&sWord[tt][c][n >> 1], bits << (16 * (n & 1) + 4 * g));
        }
      }
    }
    if (!a.s_out) continue;  // uniform
    __syncthreads();
    for (int i = tid; i < 16 * DHW * a.T; i += nth) {
      const int k = i % DHW, m = (i / DHW) % 16, tt = i / (16 * DHW);
      if (iq0 + m < a.M)
        a.s_out[((size_t)tt * Mt + r0 + iq0 + m) * dw + h * DHW + k] =
            sWord[tt][m][2 * k] | (uint64_t)sWord[tt][m][2 * k + 1] << 32;
    }
    if (a.u_out)
      for (int i = tid; i < 16 * DHW; i += nth) {
        const int k = i % DHW, m = i / DHW;
        uint64_t uor = 0ull;
        for (int tt = 0; tt < a.T; ++tt) uor |=
            sWord[tt][m][2 * k] | (uint64_t)sWord[tt][m][2 * k + 1] << 32;
        if (iq0 + m < a.M) a.u_out[(size_t)(r0 + iq0 + m) * dw + h * DHW + k] = uor;
      }
  }
}

template <int DHW, int QG, bool PARTS = false>
static nmdlm_status attn_if_launch(const AttnIfArgs& a, hipStream_t st) {
  const dim3 grid(a.H, a.n_seq * ((a.M + 16 * QG - 1) / (16 * QG)));
  const size_t dyn = std::max((size_t)a.T * DHW * 4 * 64 * sizeof(v4i),
                              a.T * a.parts * kAttnStages * sizeof(AttnStage<DHW>));
  if (dyn > 57344 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_if<DHW, QG, PARTS>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn) != hipSuccess)
    return NMDLM_ERR_HIP;
  hipLaunchKernelGGL((k_attn_if<DHW, QG, PARTS>), grid, dim3(64 * a.T * a.parts), (uint32_t)dyn, st, a);
  return hip_status();
}

// Which kernel, all measured with spikes out, H = 16 unless said, dh = 64 / 128:
//  * 32 queries a wave (QG = 2) halve the expansions and the staging per
//    query but need two such waves per SIMD: T = 4, 2048 x 2048 keys 45.8 / 75.3
//    us against 80.3 / 93.6 with 16; 600 x 1200 keys 20.2 / 29.0 against
//    19.5 / 27.4.
//  * Parts: where the waves of 16 queries leave SIMDs idle.  T = 1 (four; the
//    parts also share the epilogue of what would be a workgroup of one wave):
//    H = 8, 32 x 700 keys, dh = 128 7.4 us against 10.7; 1000 x 2000 9.5 / 13.7
//    against 14.5 / 22.6; 4 x 480, dh = 64 4.8 against 6.3.  T = 2 (four) from 7 / 4
//    chunks on: 7 chunks 6.0 / 7.8 against 6.1 / 8.8, 4 chunks of 64: 5.7 against
//    5.4.  Below 12 chunks only while the parts run at once: T = 1, 300 workgroups, 10
//    chunks, dh = 128 9.7 against 11.1, 672 workgroups, 6 chunks, dh = 64 7.9 against 7.4.
//    T = 3, 4 (two) from 12: 256 x 1256 11.7 / 15.6 against 11.2 / 15.8; 9 chunks 8.8
//    against 7.5.
//  * k_attn and the IF kernel, a second launch and the currents through
//    memory, where few workgroups would each walk a long context.  From 128
//    workgroups on never (256 x 1256 keys 17.2 / 31.0 against 11.2 / 15.8); below,
//    from 12 chunks on, when a wave walks more than 6: T = 4, 32 x 1056 keys,
//    dh = 128 11.5 us against 13.7 (8032 keys: 20 against 63).  With few of them (up
//    to one workgroup of k_attn per CU) also for shorter walks, by the chunk's
//    cost (kWalk): inside a step, graph time, T = 4, dh = 128, 6 chunks 7.5 against
//    8.3, 11 chunks 8.4 against 11.0; T = 8, dh = 64 5 chunks 7.5 against 7.7, 8 chunks
//    7.5 against 8.8; T = 8, dh = 128 3 chunks 7.6 against 8.4, 8 chunks 8.5 against 11.7.
//    A call by itself pays the host's pace for the second launch (11.3 us a call
//    against 8.3): T = 4, dh = 128, 11 chunks 11.2 against 10.7; T = 8, 7 chunks 11.1 against
//    11.4, 11 chunks 10.5 against 14.2.
constexpr int kAttnNW = 8;           // waves per workgroup of k_attn
constexpr int kPartsMinChunks = 12;
constexpr int kFusedMaxWalk = 6;     // chunks per wave of few workgroups with parts
constexpr long long kFusedMinWgs = 128;
constexpr long long kFullWaves = 2048;  // two waves per SIMD
// longest walk in one kernel with at most kOneRound workgroups of k_attn:
// [step][dh / 64 - 1][T = 1, 2 | 3, 4 | 5, 6 | 7, 8] (T = 1, 2: as with parts)
constexpr long long kOneRound = 256;  // one workgroup of k_attn per CU
constexpr int kWalk[2][2][4] = {{{11, 11, 11, 11}, {11, 11, 6, 6}}, {{11, 11, 5, 5}, {11, 5, 2, 1}}};

AttnRoute attn_route(const AttnCall& c) {
  const long long heads = (long long)c.H * c.n_seq;
  const long long wgs = heads * ((c.M + 15) / 16);
  const int nch = (c.C + c.M + 63) / 64, w = c.dh / 64 - 1;
  AttnRoute r{1, 1, false};
  if (c.M >= 32 && heads * ((c.M + 31) / 32) * c.T >= kFullWaves) {
    r.groups = 2;
    return r;
  }
  if (nch >= kPartsMinChunks) {
    if (wgs * c.T < kFullWaves) r.parts = c.T <= 2 ? 4 : (c.T <= 4 ? 2 : 1);
  } else if (wgs * c.T <= kFullWaves / 4 && (c.T == 1 || (c.T == 2 && nch >= (w ? 4 : 7)))) {
    r.parts = 4;
  }
  if (c.fused || wgs >= kFusedMinWgs) return r;
  const int walk = (nch + r.parts - 1) / r.parts;
  r.split = (nch >= kPartsMinChunks && walk > kFusedMaxWalk) ||
            (wgs * c.T <= kOneRound && walk > kWalk[c.step][w][(c.T - 1) / 2]);
  return r;
}

template <int DHW>
static nmdlm_status launch_attention_dh(const AttnCall& c, hipStream_t st) {
  const AttnRoute r = attn_route(c);
  const AttnIfArgs a{c.q, c.k_cache, c.vt_cache, c.cap, c.T, c.M, c.C, c.H, c.n_seq, r.parts,
                     c.seq_words, c.lut, c.theta, c.a_out, c.s_out, c.u_out};
  if (r.groups == 2) return attn_if_launch<DHW, 2>(a, st);
  if (!r.split) return r.parts > 1 ? attn_if_launch<DHW, 1, true>(a, st) : attn_if_launch<DHW, 1>(a, st);
  int32_t* const cur = c.a_out ? c.a_out : c.a_scratch;
  const dim3 grid(c.H, c.n_seq * ((c.M + 15) / 16), c.T);
  const auto fn = (long long)grid.x * grid.y * grid.z > kOneRound ? k_attn<DHW, kAttnNW, DHW == 2 ? 4 : 1>
                                                                  : k_attn<DHW, kAttnNW, 1>;
  hipLaunchKernelGGL(fn, grid, dim3(kAttnNW * 64), 0, st, c.q, c.k_cache, c.vt_cache, c.cap, c.T, c.M, c.C,
                     c.H, c.lut, cur, c.n_seq, c.seq_words);
  const nmdlm_status rc = hip_status();
  if (rc != NMDLM_OK || !c.s_out) return rc;
  return launch_if(cur, c.T, c.n_seq * c.M, c.H * c.dh, c.theta, nullptr, nullptr, nullptr, c.s_out,
                   st, c.u_out);
}

nmdlm_status launch_attention(const AttnCall& c, hipStream_t st) {
  if (c.n_seq < 1) return NMDLM_ERR_INVALID_ARG;
  if (c.dh == 64) return launch_attention_dh<1>(c, st);
  if (c.dh == 128) return launch_attention_dh<2>(c, st);
  return NMDLM_ERR_UNSUPPORTED;
}

}  // namespace nmdlm
