// Filtered link-prediction ranks (Sec. 5.4, filtered protocol): every held-out
// triple (s, r, d) is ranked against all entities on both sides,
//   destination side  1 + #{d' != d : (s, r, d') not known, f(s, r, d') >= f(s, r, d)}
//   source side       1 + #{s' != s : (s', r, d) not known, f(s', r, d) >= f(s, r, d)}
// with f(s, r, d) = sim(g(x_s, theta_r), x_d) (Sec. 3.1).
//
// The candidate scores of a block of queries form one matrix product
// S = Q . T^T against a candidate table T, both as row pieces
// (kernels_score.hip):
//   destination side  Q = g(x_s) (dot) or its unit vector (cos); T = the
//                     entity table (unit rows for cos);
//   source side       Q = g*(x_d) (dot, the adjoint: <g(x), y> = <x, g*(y)>;
//                     translation adds the per-query constant <theta_r, x_d>)
//                     or the unit x_d (cos); T = the entity table (dot) or the
//                     unit rows of g(x) under the single relation (cos).
//   reciprocal predicates: the source side's Q = g(x_d, theta_{r+R}) (a unit
//                     vector for cos) against the entity table, and its own
//                     positive score sim(Q, x_s), which replaces the
//                     destination side's in pos once that side is counted.
// The product's epilogue compares each score with the query's positive one and
// leaves a bit per score and the bits' number per row and 64 columns, 32 times
// fewer bytes than the scores.  The count kernel adds those up and takes back
// the known triples' candidates by testing the same bits, so that the count
// and the filter correction agree element by element.  Measured at 50,000
// queries against 15,000 entities, d = 400, both sides: 4.5 ms of kernels, 3.6 of
// them the product, at 1.06 PFLOP/s (12.0 ms with stored float32 scores).
#include <algorithm>

#include "kernels.h"
#include "pieces.h"
#include "row_ops.h"

namespace {

// row i of a table or query block, written as pieces by the wave that holds it
__device__ __forceinline__ void store_pieces(const StepGeom& g, const Row& x, RankRows t, int64_t i, bool cplx, int lane) {
  const int e = pieces::scale_exponent(pieces::row_absmax(x));
  pieces::store_row(x, pieces::scale_of(e), t.p + i * g.pld, g.d, g.dh, cplx, lane);
  if (lane == 0) t.is[i] = pieces::inverse_scale_of(e);
}

// candidate tables: one wave per candidate row
__global__ __launch_bounds__(256) void rank_tables_kernel(StepGeom g, const float* emb, const float* relp,
                                                          const float* relT, const int32_t* cand, int64_t n_col,
                                                          RankRows T0, RankRows T1) {
  __shared__ float stage[4][512];
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_col) return;
  const bool cplx = g.op == OP_COMPLEX;
  Row x;
  row_load(x, emb + (cand ? (int64_t)cand[row] : row) * g.d, g.d, cplx, lane);
  if (g.cmp == CMP_DOT) {
    store_pieces(g, x, T0, row, cplx, lane);
    return;
  }
  Row xh = x;
  row_normalize(xh);
  store_pieces(g, xh, T0, row, cplx, lane);
  if (T1.p) {
    // cos with a non-identity operator: one relation, applied to every source candidate
    Row gx;
    if (g.op == OP_LINEAR) {
      mat_apply(gx, relT, x, stage[threadIdx.x >> 6], g.d, lane);   // A x
    } else {
      Row th;
      row_load(th, relp, g.d, cplx, lane);
      gx = op_forward(g.op, x, th);
    }
    row_normalize(gx);
    store_pieces(g, gx, T1, row, cplx, lane);
  }
}

// queries of rows [e0, e0 + rows) for one side; side 0 also writes the
// positive score p_e = f(s, r, d), computed as pbg_score_edges does, and the
// source side with reciprocal predicates its own
__global__ __launch_bounds__(256) void rank_queries_kernel(StepGeom g, const float* emb, const float* relp,
                                                           const float* relT, const int32_t* src,
                                                           const int32_t* rel, const int32_t* dst,
                                                           int64_t e0, int rows, int side, RankRows Q,
                                                           float* pos, float* bias) {
  __shared__ float stage[4][512];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int q = blockIdx.x * 4 + w;
  if (q >= rows) return;
  const int64_t e = e0 + q;
  const bool cplx = g.op == OP_COMPLEX;
  const int d = g.d;
  const int r = rel ? rel[e] : 0;
  Row x, y, th;
  row_load(x, emb + (int64_t)src[e] * d, d, cplx, lane);
  row_load(y, emb + (int64_t)dst[e] * d, d, cplx, lane);
  if (g.op != OP_IDENTITY && g.op != OP_LINEAR) row_load(th, relp + (int64_t)r * g.dr, d, cplx, lane);
  else row_zero(th);
  if (side == 0) {
    Row gq;
    if (g.op == OP_LINEAR) mat_apply(gq, relT + (int64_t)r * d * d, x, stage[w], d, lane);   // A x
    else gq = op_forward(g.op, x, th);
    if (g.cmp == CMP_COS) {
      row_normalize(gq);
      row_normalize(y);
    }
    const float p = row_dot(gq, y);
    store_pieces(g, gq, Q, q, cplx, lane);
    if (lane == 0) {
      pos[e] = p;
      bias[q] = 0.0f;
    }
  } else if (g.recip) {
    Row k;
    if (g.op == OP_LINEAR) {
      mat_apply(k, relT + (int64_t)(r + g.R) * d * d, y, stage[w], d, lane);   // A_{r+R} y
    } else {
      Row tr;
      if (g.op != OP_IDENTITY) row_load(tr, relp + (int64_t)(r + g.R) * g.dr, d, cplx, lane);
      else row_zero(tr);
      k = op_forward(g.op, y, tr);
    }
    if (g.cmp == CMP_COS) {
      row_normalize(k);
      row_normalize(x);
    }
    const float p1 = row_dot(k, x);
    store_pieces(g, k, Q, q, cplx, lane);
    if (lane == 0) {
      pos[e] = p1;
      bias[q] = 0.0f;
    }
  } else {
    Row k;
    float bs = 0.0f;
    if (g.cmp == CMP_COS) {
      k = y;
      row_normalize(k);
    } else if (g.op == OP_LINEAR) {
      mat_apply(k, relp + (int64_t)r * d * d, y, stage[w], d, lane);                       // A^T y
    } else if (g.op == OP_TRANSLATION) {
      k = y;
      bs = row_dot(th, y);
    } else {
      k = op_adjoint(g.op, y, th);
    }
    store_pieces(g, k, Q, q, cplx, lane);
    if (lane == 0) bias[q] = bs;
  }
}

// first index in [lo, hi) whose (a, b) key is not below (ka, kb)
__device__ int64_t lower_bound2(const int32_t* a, const int32_t* b, int64_t lo, int64_t hi, int32_t ka,
                                int32_t kb) {
  while (lo < hi) {
    const int64_t mid = lo + ((hi - lo) >> 1);
    const bool less = a[mid] < ka || (a[mid] == ka && b[mid] < kb);
    if (less) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// A workgroup ranks 64 queries.  The hit counts of four queries are one word:
// sixteen threads cover the 64 queries, the sixteen groups of them share the
// column blocks.  Each query's range of candidates to take back is searched by
// a thread of its own (a search is a chain of loads); the ranges, a few long
// ones among many short, are then one list that all threads share.  (A wave
// per query, one query after another: 272 us a side at the sizes above.)
__global__ __launch_bounds__(256) void rank_count_kernel(RankCount a) {
  __shared__ uint32_t cnt[16][64];
  __shared__ uint32_t back[64];      // candidates taken back
  __shared__ int64_t range[2][64];   // first candidate and end of each query's range
  __shared__ int64_t sum[64];        // lengths of the ranges up to and with each query's
  __shared__ int32_t true_id[64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int q0 = blockIdx.x * 64;
  {
    const int grp = tid >> 4, c4 = 4 * (tid & 15);
    const int64_t ldm = 16 * (int64_t)a.RB;   // a multiple of 256: the word lies inside
    uint32_t n[4] = {0u, 0u, 0u, 0u};
    for (int nb = grp; nb < a.n_blk; nb += 16) {
      const uint32_t v = *(const uint32_t*)(a.hits + nb * ldm + q0 + c4);
#pragma unroll
      for (int k = 0; k < 4; ++k) n[k] += (v >> (8 * k)) & 0xFFu;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) cnt[grp][c4 + k] = n[k];
  }
  if (tid < 128) {
    const int end = tid >> 6, q = q0 + lane;
    int64_t at = 0;
    if (q < a.rows) {
      const int64_t e = a.e0 + q;
      const int32_t s = a.src[e], d = a.dst[e];
      if (end) true_id[lane] = a.side == 0 ? d : s;
      if (a.cand)   // the true entity's places in the list
        at = lower_bound2(a.cand, a.cand, 0, a.n_cand, a.side == 0 ? d : s, end ? INT32_MAX : INT32_MIN);
      else if (a.n_known > 0)   // known triples sharing (s, r) (side 0) or (d, r) (side 1)
        at = lower_bound2(a.ka, a.kb, 0, a.n_known, a.side == 0 ? s : d, (a.rel ? a.rel[e] : 0) + end);
    }
    range[end][lane] = at;
  }
  auto hit = [&](int i, int64_t col) {
    const int q = q0 + i;
    const uint32_t v = a.bits[((col >> 4) * a.RB + (q >> 4)) * 8 + ((q >> 3) & 1) * 4 + (q & 3)];
    return (v >> (16 * ((q >> 2) & 1) + (int)(col & 15))) & 1u;
  };
  __syncthreads();
  if (tid < 64) {
    int64_t n = range[1][lane] - range[0][lane];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t v = __shfl_up(n, o, 64);
      n += lane >= o ? v : 0;
    }
    sum[lane] = n;
    // without a list the true entity's column is its id
    back[lane] = !a.cand && q0 + lane < a.rows ? hit(lane, true_id[lane]) : 0u;
  }
  __syncthreads();
  for (int64_t f = tid; f < sum[63]; f += 256) {
    int i = 0;   // the first query whose sum exceeds f
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
      if (sum[i + o - 1] <= f) i += o;
    const int64_t lo = range[0][i], k = range[1][i] - (sum[i] - f);
    uint32_t h;
    if (a.cand) {
      h = hit(i, a.cand_at[k]);
    } else {
      const int32_t t = a.kc[k];
      h = t != true_id[i] && (k == lo || a.kc[k - 1] != t) ? hit(i, t) : 0u;   // duplicates once
    }
    if (h) atomicAdd(&back[i], 1u);
  }
  __syncthreads();
  if (tid < 64 && q0 + tid < a.rows) {
    uint32_t c = 1u - back[tid];
#pragma unroll
    for (int k = 0; k < 16; ++k) c += cnt[k][tid];
    a.ranks[(a.side == 0 ? 0 : a.n_eval) + a.e0 + q0 + tid] = (int32_t)c;
  }
}

// MRR and Hits@10 over the ranks, in a fixed order (fp64): sums of
// RANK_METRIC_BLOCKS workgroups, then theirs (as ranks == NULL).  (One
// workgroup over 100,000 ranks: 124 us.)
__global__ __launch_bounds__(256) void rank_metrics_kernel(const int32_t* ranks, int64_t n, const double* part,
                                                           double* out) {
  __shared__ double s_rr[256];
  __shared__ double s_h[256];
  double rr = 0.0, h = 0.0;
  if (ranks) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
      const int32_t k = ranks[i];
      rr += 1.0 / (double)k;
      h += k <= 10 ? 1.0 : 0.0;
    }
  } else if ((int)threadIdx.x < RANK_METRIC_BLOCKS) {
    rr = part[2 * threadIdx.x];
    h = part[2 * threadIdx.x + 1];
  }
  s_rr[threadIdx.x] = rr;
  s_h[threadIdx.x] = h;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      s_rr[threadIdx.x] += s_rr[threadIdx.x + o];
      s_h[threadIdx.x] += s_h[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double inv = ranks || n <= 0 ? 1.0 : (double)n;
    out[2 * blockIdx.x] = s_rr[0] / inv;
    out[2 * blockIdx.x + 1] = s_h[0] / inv;
  }
}

// known-triple sort: keys of one field through the current permutation
__global__ void perm_keys_kernel(const int32_t* field, const uint32_t* perm, int64_t n, uint32_t* keys,
                                 uint32_t* vals_init) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = vals_init ? i : (int64_t)perm[i];
    keys[i] = field ? (uint32_t)field[j] : 0u;
    if (vals_init) vals_init[i] = (uint32_t)i;
  }
}

__global__ void gather3_kernel(const uint32_t* perm, const int32_t* a, const int32_t* b, const int32_t* c,
                               int64_t n, int32_t* oa, int32_t* ob, int32_t* oc) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = perm[i];
    oa[i] = a[j];
    ob[i] = b ? b[j] : 0;
    oc[i] = c[j];
  }
}

int grid_of(int64_t n) {
  int64_t b = (n + 255) / 256;
  if (b < 1) b = 1;
  if (b > 16384) b = 16384;
  return (int)b;
}

}  // namespace

void launch_rank_tables(const StepGeom& g, const float* emb, const float* relp, const float* relT,
                        const int32_t* cand, int64_t n_col, RankRows T0, RankRows T1, hipStream_t s) {
  if (n_col <= 0) return;
  rank_tables_kernel<<<(unsigned)((n_col + 3) / 4), 256, 0, s>>>(g, emb, relp, relT, cand, n_col, T0, T1);
}

void launch_rank_queries(const StepGeom& g, const float* emb, const float* relp, const float* relT,
                         const int32_t* src, const int32_t* rel, const int32_t* dst, int64_t e0, int rows,
                         int side, RankRows Q, float* pos, float* bias, hipStream_t s) {
  if (rows <= 0) return;
  rank_queries_kernel<<<(rows + 3) / 4, 256, 0, s>>>(g, emb, relp, relT, src, rel, dst, e0, rows, side, Q,
                                                     pos, bias);
}

void launch_rank_count(const RankCount& a, hipStream_t s) {
  if (a.rows <= 0) return;
  rank_count_kernel<<<(a.rows + 63) / 64, 256, 0, s>>>(a);
}

void launch_rank_metrics(const int32_t* ranks, int64_t n, double* out, hipStream_t s) {
  rank_metrics_kernel<<<RANK_METRIC_BLOCKS, 256, 0, s>>>(ranks, n, nullptr, out + 2);
  rank_metrics_kernel<<<1, 256, 0, s>>>(nullptr, n, out + 2, out);
}

void launch_perm_keys(const int32_t* field, const uint32_t* perm, int64_t n, uint32_t* keys,
                      uint32_t* vals_init, hipStream_t s) {
  if (n <= 0) return;
  perm_keys_kernel<<<grid_of(n), 256, 0, s>>>(field, perm, n, keys, vals_init);
}

void launch_gather3(const uint32_t* perm, const int32_t* a, const int32_t* b, const int32_t* c, int64_t n,
                    int32_t* oa, int32_t* ob, int32_t* oc, hipStream_t s) {
  if (n <= 0) return;
  gather3_kernel<<<grid_of(n), 256, 0, s>>>(perm, a, b, c, n, oa, ob, oc);
}
