// Host-side queries for the tests: the choice of a product's kernel (a test of
// one kernel states that its sizes reach it) and the runs in which a row block
// is stored channel-major.  Not part of the installed header; nothing is
// launched and no GPU is needed.
#include "common.h"

using namespace nmdlm;

extern "C" {

struct nmdlm_plan_query {
  int32_t mode;  // EpiMode
  int32_t T, M, K, N;
  int32_t blocked, bias, cur, theta_vec, ternary;  // presence of each
  int32_t theta;
  int32_t transposed;  // three segments of N / 3 columns, the last channel-major
  int32_t pos0, seq_len;
  uint32_t flags;
};
struct nmdlm_plan_answer {
  int32_t status, kernel;  // nmdlm_status, QbsmKernel
  int32_t rows, tokens, row_blocks, splits, waves;
};

void nmdlm_internal_plan(const nmdlm_plan_query* q, nmdlm_plan_answer* out) {
  // pointers are only tested for presence
  char* const some = reinterpret_cast<char*>(256);
  QbsmCall c{};
  c.T = q->T;
  c.M = q->M;
  c.K = q->K;
  c.N = q->N;
  c.ldw = q->N;
  c.mode = q->mode;
  c.Wb = q->blocked ? reinterpret_cast<int8_t*>(some) : nullptr;
  c.bias = q->bias ? reinterpret_cast<int32_t*>(some) : nullptr;
  c.cur_out = q->cur ? reinterpret_cast<int32_t*>(some) : nullptr;
  c.theta_vec = q->theta_vec ? reinterpret_cast<int32_t*>(some) : nullptr;
  c.s_neg = q->ternary ? reinterpret_cast<uint64_t*>(some) : nullptr;
  c.nseg = q->transposed ? 3 : 1;
  c.seg_w = q->transposed ? q->N / 3 : 1 << 30;
  for (int i = 0; i < kMaxSeg; ++i) c.seg[i].theta = q->theta;
  c.seg[2].transposed = q->transposed;
  c.seg[2].pos0 = q->pos0;
  c.seg[1].seq_len = c.seg[2].seq_len = c.seq_len = q->seq_len;
  c.flags = q->flags;
  Carver cv{some, 0, (size_t)-1, true};
  QbsmScratch scr;
  carve_qbsm_scratch(cv, qbsm_limits_single(q->T, q->M, q->K, q->N), &scr);
  const QbsmPlan p = plan_qbsm(c, scr);
  *out = nmdlm_plan_answer{p.status, p.kernel, 16 * p.RT, p.Mb, p.gy, p.P, p.NW};
}

// The route of an attention call: 16-query groups of a wave, waves per timestep,
// 1 when attention and IF are two kernels.
void nmdlm_internal_attn_route(int T, int M, int C, int H, int dh, int n_seq, int fused, int step,
                               int32_t* out) {
  AttnCall c{};
  c.T = T;
  c.M = M;
  c.C = C;
  c.H = H;
  c.dh = dh;
  c.n_seq = n_seq;
  c.fused = fused != 0;
  c.step = step != 0;
  const AttnRoute r = attn_route(c);
  out[0] = r.groups;
  out[1] = r.parts;
  out[2] = r.split ? 1 : 0;
}

// The runs of row block y of M tokens into out[4 i ..]: sequence, first position,
// tokens, 1 when stored in bytes.  Returns their number.
int nmdlm_internal_token_runs(int pos0, int seq_len, int Mb, int M, int y, int32_t* out) {
  SpikeSeg seg{};
  seg.pos0 = pos0;
  seg.seq_len = seq_len;
  const int yb = y * Mb, ntok = M - yb < Mb ? M - yb : Mb;
  int n = 0;
  for (int ml = 0; ml < ntok; ++n) {
    const TokenRun r = token_run(seg, yb + ml, ntok - ml);
    const int32_t v[4] = {r.seq, r.pos, r.n, whole_bytes(seg, Mb) ? 1 : 0};
    for (int i = 0; i < 4; ++i) out[4 * n + i] = v[i];
    ml += r.n;
  }
  return n;
}

}  // extern "C"
