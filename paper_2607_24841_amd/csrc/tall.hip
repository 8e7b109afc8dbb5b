// The spike product over many rows (prefills, steps over many sequences):
// a plain int8 contraction over the blocked weight copy, with the neurons in
// the epilogue.
#include <hip/hip_ext.h>

#include "qbsm_device.h"

namespace nmdlm {

constexpr int kTallRows = 128;   // block rows per workgroup
constexpr int kTallTiles = 4;    // 64-column tiles per workgroup, one per wave
constexpr int kTallWords = 4;    // words (of 64 input channels) per LDS stage
constexpr int kTallStage = kTallWords * (kTallRows / 16) * 64;  // 16-byte A operands per stage

// Channel-major output of a tile's 64 columns (lane = column): token bits per
// (step, column) in ep.vbits, written run by run (see token_run).
__device__ __forceinline__ void tall_channel_major(const QbsmArgs& a, const EpiStage& ep,
                                                   const SpikeSeg& seg, int segi, int lane, int n0,
                                                   int y) {
  if (n0 + lane >= a.N) return;
  const int ch = n0 + lane - segi * a.seg_w;
  const int yb = y * a.Mb, ntok = min(a.Mb, a.M - yb);
  const bool bytes = whole_bytes(seg, a.Mb);
  for (int ml = 0; ml < ntok;) {  // uniform
    const TokenRun r = token_run(seg, yb + ml, ntok - ml);
    const uint32_t keep = r.n >= 32 ? 0xFFFFFFFFu : ((1u << r.n) - 1u);
    uint64_t* base = seg.ptr + (int64_t)r.seq * seg.ld_s + (int64_t)ch * seg.ld_m;
    for (int t = 0; t < a.T; ++t) {
      const uint32_t bits = (ep.vbits[t * 64 + lane] >> ml) & keep;
      uint64_t* row = base + t * seg.ld_t;
      if (bytes) {
        for (int b = 0; b < (r.n + 7) >> 3; ++b) {
          const int pb = (r.pos >> 3) + b;
          reinterpret_cast<uint8_t*>(row + (int64_t)(pb >> 3) * seg.ld_p)[pb & 7] =
              (uint8_t)(bits >> (8 * b));
        }
      } else {
        const int o = r.pos & 63;
        unsigned long long* w = reinterpret_cast<unsigned long long*>(row + (int64_t)(r.pos >> 6) * seg.ld_p);
        const uint64_t m1 = o ? (uint64_t)keep >> (64 - o) : 0ull;
        atomicAnd(w, ~((uint64_t)keep << o));
        if (bits) atomicOr(w, (unsigned long long)((uint64_t)bits << o));
        if (m1) {
          const uint64_t b1 = (uint64_t)bits >> (64 - o);
          atomicAnd(w + seg.ld_p, ~m1);
          if (b1) atomicOr(w + seg.ld_p, (unsigned long long)b1);
        }
      }
    }
    ml += r.n;
  }
}

// The membranes of a lane's neurons (tall_epilogue): sb[t KB + k] takes, at
// bit 4e + v, the sign of V - theta (set: no spike) of row 16k + 4g + e,
// column 4c + v of step t.
template <int T, bool QNL, bool RES>
__device__ __forceinline__ void tall_integrate(const v4i (&acc)[8][4], const EpiStage& ep, int shift,
                                               int theta, int g, int c, uint32_t (&sb)[8]) {
  constexpr int KB = 8 / T;
  constexpr int Mb = 16 * KB;
  const uint8_t* rb = reinterpret_cast<const uint8_t*>(ep.resid) + 32 * g + (c >> 1);
#pragma unroll
  for (int k = 0; k < KB; ++k)
#pragma unroll
    for (int e = 3; e >= 0; --e) {
      uint32_t rn[T];  // residual bits of the four columns
#pragma unroll
      for (int t = 0; t < T; ++t)
        rn[t] = RES ? (uint32_t)rb[(t * Mb + 16 * k + e) * 8] >> (4 * (c & 1)) : 0u;
      int I[4][T];
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int t = 0; t < T; ++t) {
          I[v][t] = acc[t * KB + k][v][e];
          if constexpr (QNL) I[v][t] = (int)ep.lut[min(127, max(-128, I[v][t] >> shift)) & 0xFF];
        }
#pragma unroll
      for (int v = 3; v >= 0; --v) {
        int V = 0;
#pragma unroll
        for (int t = 0; t < T; ++t) {
          V += I[v][t];
          if constexpr (RES) V += theta & ((int)(rn[t] << (31 - v)) >> 31);
          const int d = V - theta;
          sb[t * KB + k] = __builtin_amdgcn_alignbit(sb[t * KB + k], (uint32_t)d, 31);
          V = d >= 0 ? d : V;
        }
      }
      __builtin_amdgcn_sched_barrier(0);  // four neurons at a time (registers)
    }
}

// The first `left` of four neighbouring values of a row, in one store where all
// four are inside (rows need not start at 16 bytes: the store asks for 4).  A wave
// then writes 256 contiguous bytes of four rows; four stores of a dword a lane, 16
// bytes apart, took most of the epilogue (currents, rows x K x N: 1760 x 197 x 5244 27.3
// -> 14.4 us, 7295 x 148 x 8193 101 -> 57, 2196 x 2360 x 18747 138 -> 117).
typedef float v4f __attribute__((ext_vector_type(4)));
template <typename E, typename V>
__device__ __forceinline__ void store4(E* p, V x, int left) {
  if (left >= 4) {
    struct __attribute__((packed, aligned(4), may_alias)) Any { V v; };
    reinterpret_cast<Any*>(p)->v = x;
  } else {
#pragma unroll
    for (int v = 0; v < 3; ++v)
      if (v < left) p[v] = x[v];
  }
}

// Epilogue of one wave's 128 x 64 tile from its accumulators: acc[q][v][e] of
// lane (g, c) is tile row 16q + 4g + e, column 4c + v.  With row blocks of
// Mb = 128 / T tokens (T = 1, 2, 4, 8), row t Mb + m lies in q = t KB + m / 16
// with 4g + e = m % 16, so a lane holds all T currents of its neurons (tokens
// 16k + 4g + e, k < KB = 8 / T) and integrates them in registers, in 32 bits
// (the launcher's bounds keep every membrane below 2^31), five or so
// instructions a step: the sign of V - theta is the spike bit (inverted),
// shifted into the 16 bits of the lane's 4 rows x 4 columns.  (With the 64-bit
// membrane of the other kernels the epilogue took as long as 16 words of K.)
template <int T>
__device__ __forceinline__ void tall_epilogue(const QbsmArgs& a, const v4i (&acc)[8][4], EpiStage& ep,
                                              uint32_t* lds, int lane, int x, int y) {
  constexpr int KB = 8 / T;
  constexpr int Mb = 16 * KB;
  const int g = lane >> 4, c = lane & 15;
  const int n0 = x * 64;
  if (a.mode == EPI_HEAD || a.mode == EPI_CUR) {
    const bool head = a.mode == EPI_HEAD;
    float sc[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) sc[v] = head && n0 + 4 * c + v < a.N ? a.scale[n0 + 4 * c + v] : 0.f;
#pragma unroll
    for (int k = 0; k < KB; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = y * Mb + 16 * k + 4 * g + e;
        if (m >= a.M) continue;
        const int n = n0 + 4 * c;
        if (n >= a.N) continue;
        if (head) {
          v4f x;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            int sum = 0;
#pragma unroll
            for (int t = 0; t < T; ++t) sum += acc[t * KB + k][v][e];
            x[v] = (float)sum * sc[v];
          }
          store4(a.logits + (size_t)m * a.N + n, x, a.N - n);
        } else {
#pragma unroll
          for (int t = 0; t < T; ++t) {
            v4i x;
#pragma unroll
            for (int v = 0; v < 4; ++v) x[v] = acc[t * KB + k][v][e] + ep.bias[4 * c + v];
            store4(a.cur_out + ((size_t)t * a.M + m) * a.N + n, x, a.N - n);
          }
        }
      }
    return;
  }
  const int segi = a.nseg == 1 ? 0 : div_small(n0, a.inv_segw);
  const SpikeSeg seg = a.seg[segi];
  const int wseg = (n0 - segi * a.seg_w) >> 6;
  const bool qnl = a.mode == EPI_QNL_IF, res = a.resid != nullptr;
  const int theta = seg.theta;
  // sb[t KB + k]: bit 4e + v = no spike of row 16k + 4g + e, column 4c + v
  uint32_t sb[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) sb[i] = 0u;
  if (qnl) {
    if (res) tall_integrate<T, true, true>(acc, ep, a.lut_shift, theta, g, c, sb);
    else tall_integrate<T, true, false>(acc, ep, a.lut_shift, theta, g, c, sb);
  } else {
    if (res) tall_integrate<T, false, true>(acc, ep, 0, theta, g, c, sb);
    else tall_integrate<T, false, false>(acc, ep, 0, theta, g, c, sb);
  }
  // spikes; columns past N have none
  const int ncol = a.N - (n0 + 4 * c);
  const uint32_t cm = ncol >= 4 ? 0xFFFFu : (ncol <= 0 ? 0u : ((1u << ncol) - 1u) * 0x1111u);
#pragma unroll
  for (int i = 0; i < 8; ++i) sb[i] = ~sb[i] & cm;
  if (seg.transposed) {  // row blocks of at most 32 tokens (T >= 4)
    if constexpr (Mb <= 32) {
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          uint32_t bits = 0u;
#pragma unroll
          for (int k = 0; k < KB; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              bits |= ((sb[t * KB + k] >> (4 * e + v)) & 1u) << (16 * k + 4 * g + e);
          if (bits) atomicOr(&ep.vbits[t * 64 + 4 * c + v], bits);
        }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      tall_channel_major(a, ep, seg, segi, lane, n0, y);
    }
    return;
  }
  // natural words: 16 bits per (q, g, c) in LDS, [q][g][c]; the word of row
  // 16q + 4g + e is the nibbles e of the 16 columns' pieces
  uint16_t* pc = reinterpret_cast<uint16_t*>(lds);
#pragma unroll
  for (int i = 0; i < 8; ++i) pc[i * 64 + lane] = (uint16_t)sb[i];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  uint64_t u = 0ull;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int i = lane + 64 * j, t = i / Mb, m = y * Mb + (i - t * Mb);  // i = tile row
    const int sh = 4 * (i & 3);
    uint64_t word = 0ull;
#pragma unroll
    for (int cc = 0; cc < 16; ++cc)
      word |= (uint64_t)((pc[(i >> 2) * 16 + cc] >> sh) & 0xFu) << (4 * cc);
    if (m < a.M) {
      const int64_t mo = seg.seq_len > 0
                             ? (int64_t)(m / seg.seq_len) * seg.ld_s + (int64_t)(m % seg.seq_len) * seg.ld_m
                             : (int64_t)m * seg.ld_m;
      seg.ptr[t * seg.ld_t + mo + wseg] = word;
      u |= word;
    }
  }
  if (a.u_out) {
    // partial union of the tile's output word over the row block
    for (int o = kWave / 2; o > 0; o >>= 1) u |= __shfl_xor(u, o);
    if (lane == 0) a.u_out[(size_t)y * a.u_ld + x] = u;
  }
}

// Workgroup = 4 waves, tile = 128 block rows x 256 columns; wave j takes the
// 64-column tile 4x + j over every word of K, 32 MFMAs per word.
//
// Weights come straight from the blocked copy, four 16-byte loads per lane
// and word, four words in flight: 128 rows a tile keep them at 32 bytes a
// clock and CU at the matrix cores' peak (64-row tiles need the 64 that the
// cache delivers).  The spikes, one bit per element in memory, are expanded to
// 0/1 bytes once per workgroup (a wave of its own expansions spends 12 vector
// instructions per four MFMAs on them): stages of kTallWords words in LDS, in
// operand order (a lane's operand is one 16-byte read, no bank conflicts), two
// stages, one barrier per stage; each thread expands the eight 16-bit pieces
// of two words of one row, a piece per half word of products.  Every word is
// read and multiplied: over 128 rows a word of 64 channels has its spike.
//
// Bound by the matrix cores in the loop and by the chain of loads before it and the
// neurons after it, some 8 us a round of the chip: over the whole kernel the matrix
// cores are busy 50-57% of the cycles of a prefill's products (K = 2048 and 8192), 31-37%
// at K = 1024 (counters).
// Rows x K x N, T = 4, against 64-row tiles: 8192 x 2048 x 6144 118 -> 80 us
// (2.6 POP/s), 8192 x 8192 x 2048 253 -> 96 (2.9), 8192 x 1024 x 3072 40 -> 29,
// 2048 x 1024 x 4096 20.7 -> 14.1; T = 8, 5552 x 1024 x 3072 52 -> 29.
template <int T>
__global__ __launch_bounds__(256, 2) __attribute__((aligned(1024))) void k_qbsm_tall(QbsmArgs a) {
  __shared__ EpiStage ep[kTallTiles];
  __shared__ int sStatCnt;
  extern __shared__ v4i sA[];  // [2][kTallWords][8][64] A operands; then the epilogue's words
  touch_kernargs<sizeof(QbsmArgs)>();
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int x, y, z;
  tile_coords_inv(x, y, z, a.inv_gy, a.inv_gxy);
  constexpr int Mb = kTallRows / T;
  const int Kw = (a.K + 63) >> 6;
  const int gx = (a.N + 63) >> 6;
  const int xs = x * kTallTiles + wave;

  // staging: row tid % 128, words 2 (tid / 128) and + 1 of a stage
  const int srow = tid & (kTallRows - 1), shalf = tid / kTallRows;
  const int sm = y * Mb + srow % Mb;
  const uint64_t* sp = a.S + (size_t)((srow / Mb) * a.M + min(sm, a.M - 1)) * Kw;
  const bool sv = sm < a.M;
  // element (word w, row r): operand (w * 8 + r / 16) * 64 + 16 g + r % 16
  v4i* const sdst = sA + (2 * shalf * 8 + (srow >> 4)) * 64 + (srow & 15);
  auto load_spikes = [&](int w0, uint64_t (&s)[2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int w = w0 + 2 * shalf + j;
      const uint64_t v = sp[min(w, Kw - 1)];
      s[j] = (sv && w < Kw) ? v : 0ull;
    }
  };
  auto expand_piece = [&](const uint64_t (&s)[2], int buf, int p) {  // piece p of 8
    const uint32_t h = (uint32_t)(s[p >> 2] >> (16 * (p & 3))) & 0xFFFFu;
    sdst[buf * kTallStage + (p >> 2) * 8 * 64 + (p & 3) * 16] = a_operand(h);
  };
  const char* Wbb = reinterpret_cast<const char*>(a.Wb) + (size_t)min(xs, gx - 1) * 4096;  // uniform
  const size_t wstep = (size_t)gx * 4096;
  auto load_b = [&](int w, v4i (&b)[4]) {
    const char* p = Wbb + (size_t)min(w, Kw - 1) * wstep;
#pragma unroll
    for (int v = 0; v < 4; ++v) b[v] = *reinterpret_cast<const v4i*>(p + (uint32_t)(v * 1024 + lane * 16));
  };

  uint64_t s[2];
  v4i b[kTallWords][4];
  load_spikes(0, s);
  EpiRegs er[kTallTiles];
#pragma unroll
  for (int j = 0; j < kTallTiles; ++j) er[j] = epi_load<256>(a, tid, min(x * kTallTiles + j, gx - 1), y);
  __builtin_amdgcn_sched_barrier(0);  // every load above is issued before the first use
#pragma unroll
  for (int j = 0; j < kTallTiles; ++j)
    epi_store<256>(a, ep[j], er[j], tid, min(x * kTallTiles + j, gx - 1), y);
#pragma unroll
  for (int i = 0; i < kTallWords; ++i) load_b(i, b[i]);
#pragma unroll
  for (int p = 0; p < 8; ++p) expand_piece(s, 0, p);
  load_spikes(kTallWords, s);
  __syncthreads();

  v4i acc[8][4];
#pragma unroll
  for (int q = 0; q < 8; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[q][v] = v4i{0, 0, 0, 0};
  int buf = 0;
  for (int w0 = 0; w0 < Kw; w0 += kTallWords, buf ^= 1) {
    // operand 8 i + q: word i, row group q; three reads ahead of the products,
    // in this order (left to itself the compiler reads each operand just
    // before its products and waits for it)
    const v4i* src = sA + buf * kTallStage + lane;
    v4i af[4];
#pragma unroll
    for (int q = 0; q < 3; ++q) af[q] = src[q * 64];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kTallWords; ++i) {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int o = 8 * i + q;
        if (o + 3 < 8 * kTallWords) af[(o + 3) & 3] = src[(o + 3) * 64];
#pragma unroll
        for (int v = 0; v < 4; ++v)
          acc[q][v] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[o & 3], b[i][v], acc[q][v], 0, 0, 0);
        if ((q & 3) == 1) expand_piece(s, buf ^ 1, 2 * i + (q >> 2));  // of the next stage
        if ((q & 3) != 1) __builtin_amdgcn_sched_barrier(0);
      }
      load_b(w0 + i + kTallWords, b[i]);
      __builtin_amdgcn_sched_barrier(0);
    }
    load_spikes(w0 + 2 * kTallWords, s);
    __syncthreads();
  }

  if (xs < gx)
    tall_epilogue<T>(a, acc, ep[wave], reinterpret_cast<uint32_t*>(sA) + wave * 512, lane, xs, y);

  if (a.stats && x == 0 && y == 0) {  // uniform
    // active rows of the whole block's union
    __syncthreads();
    stats_alone<256>(a, reinterpret_cast<unsigned long long*>(sA), &sStatCnt, Kw, tid, lane);
  }
}

constexpr size_t kTallLds = 2 * kTallStage * sizeof(v4i);
static_assert(kTallLds >= NMDLM_MAX_K / 64 * 8, "the statistics' union fits the stages");

bool tall_fits(const QbsmCall& c) {
  const bool spikes = c.mode == EPI_IF || c.mode == EPI_QNL_IF;
  if (!c.Wb || c.s_neg || !(c.T == 1 || c.T == 2 || c.T == 4 || c.T == 8)) return false;
  if (!spikes) return c.mode == EPI_CUR || c.mode == EPI_HEAD;
  // 32-bit membranes: |V| <= T (127 K + 2 theta) < 2^31 at T = 8, K = 65536
  if (c.cur_out || c.bias || c.theta_vec) return false;
  for (int i = 0; i < c.nseg; ++i)
    if (c.seg[i].theta > (1 << 26) || (c.seg[i].transposed && kTallRows / c.T > 32)) return false;
  return true;
}

nmdlm_status launch_tall(const QbsmArgs& a, int gx, int gy, hipStream_t st, hipEvent_t e0,
                         hipEvent_t e1) {
  const dim3 grid((gx + kTallTiles - 1) / kTallTiles, gy);
  void (*fn)(QbsmArgs) = a.T == 8 ? k_qbsm_tall<8> : a.T == 4 ? k_qbsm_tall<4>
                         : a.T == 2 ? k_qbsm_tall<2> : k_qbsm_tall<1>;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)kTallLds) != hipSuccess)
    return NMDLM_ERR_HIP;
  hipExtLaunchKernelGGL(fn, grid, dim3(256), (uint32_t)kTallLds, st, e0, e1, 0, a);
  return hip_status();
}

}  // namespace nmdlm
