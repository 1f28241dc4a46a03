// Loss values and per-edge gradients of a step (Sec. 3.1 losses): the
// finalisation's workgroup body.
#pragma once

#include "kernels.h"
#include "device_common.h"

// ---- row scales of the ranking backward --------------------------------------
// The rows of nn and of qk differ by powers of two, and an fp16 scale holds 30
// of them, so rows far below a (chunk, side)'s largest go to further levels:
// level l takes rows 30 l to 30 l + 29 binades below it with scale
// 2^(e - e_max + 30 l + 15), the others with 0.  The backward sums a level at a
// time, so a large row that an edge does not select costs it nothing.  (Rows of
// zeros belong to no level; one level is the rule.)  Each of the chunk's nblk
// workgroups finds the four largest and smallest exponents again (a few
// thousand floats that the L2 holds; one atomic maximum a row in the gather
// cost it twenty times its own time) and writes its share of the scales.
__device__ __forceinline__ void row_scales(const StepGeom& g, const StepBufs& b, int c, int Cc, int blk, int nblk) {
  constexpr int WAVES = FIN_THREADS / PBG_WAVE;
  __shared__ float ends[4][WAVES][2];   // of the scales and of the negated ones, rows of zeros apart
  const int Nc = Cc + g.U;
  auto scales = [&](int k) {
    const int z = c * 2 + (k & 1);
    return k < 2 ? b.pn_is + (int64_t)z * g.N : b.pq_is + (int64_t)z * g.C;
  };
  // each thread's first rows of all four, on their way together (a small step
  // has no others)
  const int own = blk * FIN_THREADS + threadIdx.x;
  float first[4], mine[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int rows = k < 2 ? Nc : Cc;
    first[k] = (int)threadIdx.x < rows ? scales(k)[threadIdx.x] : PIECES_ZERO_ROW;
    mine[k] = own < rows ? scales(k)[own] : 0.0f;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float* is = scales(k);
    const int rows = k < 2 ? Nc : Cc;
    float hi = 0.0f, lo = -INFINITY;
    auto add = [&](float x) {
      hi = fmaxf(hi, x);
      lo = fmaxf(lo, x == PIECES_ZERO_ROW ? -INFINITY : -x);
    };
    add(first[k]);
#pragma unroll 4
    for (int t = threadIdx.x + FIN_THREADS; t < rows; t += FIN_THREADS) add(is[t]);
    hi = group16_max(hi);
    lo = group16_max(lo);
    hi = fmaxf(hi, __shfl_xor(hi, 16, PBG_WAVE));
    lo = fmaxf(lo, __shfl_xor(lo, 16, PBG_WAVE));
    hi = fmaxf(hi, __shfl_xor(hi, 32, PBG_WAVE));
    lo = fmaxf(lo, __shfl_xor(lo, 32, PBG_WAVE));
    if ((threadIdx.x & 63) == 0) {
      ends[k][threadIdx.x >> 6][0] = hi;
      ends[k][threadIdx.x >> 6][1] = lo;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const bool nn = k < 2;
    const int z = c * 2 + (k & 1), rows = nn ? Nc : Cc;
    const float* is = scales(k);
    float hi = ends[k][0][0], lo = ends[k][0][1];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
      hi = fmaxf(hi, ends[k][w][0]);
      lo = fmaxf(lo, ends[k][w][1]);
    }
    const int top = (int)(__float_as_uint(hi) >> 23) + 14;
    // no row but rows of zeros: one level of zeros
    const int levels = lo == -INFINITY ? 1 : (top - ((int)(__float_as_uint(-lo) >> 23) + 14)) / 30 + 1;
    if (blk == 0 && threadIdx.x == 0) (nn ? b.pn_top : b.pq_top)[z] = make_int2(top, levels);
    const int ld = nn ? g.ks_n : g.ks_q;
    uint16_t* ks = (nn ? b.nks : b.qks) + (int64_t)z * KS_LEVELS * ld;
    for (int t = own; t < rows; t += nblk * FIN_THREADS) {
      const float x = t == own ? mine[k] : is[t];
      int ex = x == PIECES_ZERO_ROW ? 0 : 30 + (int)(__float_as_uint(x) >> 23) + 14 - top;
      for (int l = 0; l < levels; ++l, ex += 30) ks[(int64_t)l * ld + t] = (uint16_t)(ex > 0 && ex <= 30 ? ex << 10 : 0);
    }
  }
}

// ---- per-edge dL/dp, translation bias gradient, losses ------------------------
// Workgroup blk of chunk c (FIN_THREADS rows): writes its share of the chunk
// loss to parts[c * nblk + blk].
__device__ __forceinline__ void finalize_block(const StepGeom& g, const StepBufs& b, int softmax_scales,
                                               double* parts, int c, int blk, int nblk) {
  const int Cc = chunk_edges(g, c);
  double acc = 0.0;
  const int e = blk * FIN_THREADS + threadIdx.x;
  if (g.pieces == PIECES_SCALED && g.loss == LOSS_RANKING) row_scales(g, b, c, Cc, blk, nblk);
  if (e < Cc) {
    const int64_t ce = (int64_t)c * g.C + e;
    const float p = b.pos[pos_index(g, c, 0, e)];
    const float p1 = b.pos[pos_index(g, c, 1, e)];   // p itself without reciprocal predicates
    float l0 = 0.f, l1 = 0.f, d0 = 0.f, d1 = 0.f;
    // column tiles with candidates of this chunk (merged: side 1's in-chunk
    // tiles, then its uniform ones)
    const int bn = g.pieces != PIECES_NONE ? PBG_PART_BN : PBG_SCORE_BN;
    const int n0 = (Cc + g.U + bn - 1) / bn;
    const int n1 = g.dq_has_dn ? (Cc + bn - 1) / bn + (g.U + bn - 1) / bn : n0;
    if (g.loss != LOSS_SOFTMAX) {
      const float* r0 = b.rowpart + ((int64_t)(c * 2 + 0) * g.C + e) * g.nct * 2;
      const float* r1 = b.rowpart + ((int64_t)(c * 2 + 1) * g.C + e) * g.nct * 2;
#pragma unroll 8
      for (int ct = 0; ct < n0; ++ct) {
        const float2 a0 = *(const float2*)(r0 + 2 * ct);
        l0 += a0.x;
        d0 += a0.y;
      }
#pragma unroll 8
      for (int ct = 0; ct < n1; ++ct) {
        const float2 a1 = *(const float2*)(r1 + 2 * ct);
        l1 += a1.x;
        d1 += a1.y;
      }
    }
    double loss;
    float dp, dp1 = 0.f, dsum1;
    float side_loss[2];
    if (g.recip) {
      // each side with its own positive score
      const float ps[2] = {p, p1};
      const float ls[2] = {l0, l1}, dsn[2] = {d0, d1};
      float dps[2];
      loss = 0.0;
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        const float pp = ps[side];
        if (g.loss == LOSS_RANKING) {
          side_loss[side] = ls[side];
          dps[side] = -dsn[side];
        } else if (g.loss == LOSS_LOGISTIC) {
          side_loss[side] = ls[side] + softplusf(-pp);
          dps[side] = sigmoidf(pp) - 1.0f;
        } else {
          const float* rp = b.rowpart + ((int64_t)(c * 2 + side) * g.C + e) * g.nct * 2;
          float M = pp;
          for (int ct = 0; ct < n0; ++ct) M = fmaxf(M, rp[2 * ct]);
          float Z = expf(pp - M);
          for (int ct = 0; ct < n0; ++ct) {
            const float mx = rp[2 * ct];
            if (mx > -INFINITY) Z += rp[2 * ct + 1] * expf(mx - M);
          }
          const float lse = M + logf(Z);
          if (softmax_scales) {
            float* rs = b.rowscale + (int64_t)(c * 2 + side) * g.nct * g.C + e;
            for (int ct = 0; ct < n0; ++ct) {
              const float mx = rp[2 * ct];
              rs[(int64_t)ct * g.C] = mx > -INFINITY ? expf(mx - lse) : 0.0f;
            }
          }
          side_loss[side] = lse - pp;
          dps[side] = expf(pp - lse) - 1.0f;
        }
        loss += (double)side_loss[side];
      }
      dp = dps[0];
      dp1 = dps[1];
      dsum1 = 0.0f;   // no translation bias: both queries carry the operator
    } else if (g.loss == LOSS_RANKING) {
      loss = (double)l0 + (double)l1;
      dp = -(d0 + d1);
      dsum1 = d1;
      side_loss[0] = l0;
      side_loss[1] = l1;
    } else if (g.loss == LOSS_LOGISTIC) {
      const float sp = softplusf(-p);
      loss = (double)l0 + (double)l1 + 2.0 * (double)sp;
      dp = 2.0f * (sigmoidf(p) - 1.0f);
      dsum1 = d1;
      side_loss[0] = l0 + sp;
      side_loss[1] = l1 + sp;
    } else {
      // log-sum-exp of each side's row over {p} and its valid candidates, from
      // the per-tile (max M, sum exp(s - M)) partials; each tile's sum is then
      // replaced by exp(M - lse), which turns the stored exp(s - M) into dS
      float lse[2];
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        const float* rp = b.rowpart + ((int64_t)(c * 2 + side) * g.C + e) * g.nct * 2;
        float M = p;
        for (int ct = 0; ct < n0; ++ct) M = fmaxf(M, rp[2 * ct]);
        float Z = expf(p - M);
        for (int ct = 0; ct < n0; ++ct) {
          const float mx = rp[2 * ct];
          if (mx > -INFINITY) Z += rp[2 * ct + 1] * expf(mx - M);
        }
        lse[side] = M + logf(Z);
        if (softmax_scales) {
          float* rs = b.rowscale + (int64_t)(c * 2 + side) * g.nct * g.C + e;
          for (int ct = 0; ct < n0; ++ct) {
            const float mx = rp[2 * ct];
            rs[(int64_t)ct * g.C] = mx > -INFINITY ? expf(mx - lse[side]) : 0.0f;
          }
        }
      }
      const float lse0 = lse[0], lse1 = lse[1];
      loss = ((double)lse0 - p) + ((double)lse1 - p);
      const float s0 = expf(p - lse0), s1 = expf(p - lse1);
      dp = (s0 - 1.0f) + (s1 - 1.0f);
      dsum1 = 1.0f - s1;
      side_loss[0] = lse0 - p;
      side_loss[1] = lse1 - p;
    }
    if (b.rowloss) {
      b.rowloss[(int64_t)(c * 2 + 0) * g.C + e] = side_loss[0];
      b.rowloss[(int64_t)(c * 2 + 1) * g.C + e] = side_loss[1];
    }
    if (g.cweight) {
      // the chunk's relation weight multiplies the edge's loss and every
      // gradient (the contractions' share is scaled as they store it)
      const float w = wave_uniform(g.cweight[c]);
      loss *= (double)w;
      dp *= w;
      dp1 *= w;
      dsum1 *= w;
    }
    b.dpos[pos_index(g, c, 0, e)] = dp;
    if (g.recip) b.dpos[pos_index(g, c, 1, e)] = dp1;
    b.dsum1[ce] = dsum1;
    acc += loss;
  }
  // fixed-order block reduction of this workgroup's share of the chunk loss
  __shared__ double red[FIN_THREADS];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = FIN_THREADS / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) parts[(int64_t)c * nblk + blk] = red[0];
}

