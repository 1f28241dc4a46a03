// Backward of the logistic and softmax losses: dQ = dS . N and dN = dS^T . Q
// with dS a float32 matrix (softmax: exp(s - block maximum), completed by the
// row's scale of its 64-column block as it is staged) and the rows of N and Q
// as pieces (pieces.h).  dS is split into two fp16 pieces too: three plane
// products, as in the score.
//
// dS spans many binades (a softmax probability may be 2^-40, and a row update
// does not depend on its gradient's size), and with per-row scales (dot) the
// rows of B carry different powers of two, which are multiplied into dS.  So
// every output row has a power of two of its own that puts the largest of its
// factors so far in [2^10, 2^15): a slice that exceeds it lowers the power and
// rescales the accumulators.  A factor is then held to 2^-35 of the row's
// largest, whatever that is.
//
// A workgroup computes 128 x 16 NB outputs, four waves of 32 rows over all
// columns.  B rows move global -> LDS as they lie in memory and are read
// through the transposing LDS reads; dS goes through registers (scale, split)
// into LDS: k-contiguous rows for dQ, its rows as they are for dN, whose
// fragments are read transposed as well.  A wave stages the dS of its own
// rows, so only B needs a barrier and A a single stage.  Wide tiles (NB = 13)
// read dS half as often where the rows are long: at d = 400 two column tiles
// instead of four.
//
// Measured a step in traces: softmax, d = 400, 40 chunks of 1,000 edges and
// 1,000 uniform negatives 1,065 us; logistic, d = 100, as many chunks 346 us.
// (With one fixed power for all rows, A staged by the whole workgroup between
// two barriers and the B fragments read just before their products 1,020 and
// 404 us.)  A slice costs a wave 1,250 cycles of products at NB = 13 and about
// 140 vector instructions; the rest is the wait for dS, which comes from memory
// once a column tile.
#include <algorithm>

#include "kernels.h"
#include "pieces.h"

namespace {

using namespace pieces;

constexpr int BK = 32, BT = 128;

constexpr int row_blocks(int nb) { return nb <= 2 ? 1 : (nb <= 4 ? 2 : (nb <= 8 ? 4 : 8)); }

template <int NB>
struct ValueSmem {
  static constexpr int BL = row_blocks(NB);
  uint16_t B[2][BK * 64 * BL];
  uint16_t A[BT * 64];
};

// Powers of two of the output rows' factors: the largest so far times the
// power lies in [2^10, 2^11) when it is set and below 2^15 until the next.
constexpr float kFactorLimit = 32768.0f;
// the power for a largest factor m; the smallest exponents share one (2^122)
__device__ __forceinline__ float factor_scale(float m) {
  return 0.0625f * scale_of(scale_exponent(m));
}
// 1 / x, x a power of two
__device__ __forceinline__ float inverse_power(float x) { return __uint_as_float((254u << 23) - __float_as_uint(x)); }

// Multiplies the accumulators by a factor a row.  The lanes hold the wave's 32
// rows' factors as they stage them: COL the four rows 4 (lane % 8) .. + 3, else
// rows lane / 4 and lane / 4 + 16.
template <int NB, bool COL>
__device__ __forceinline__ void scale_rows(v4f mine, v4f (&acc)[2][NB], int lane) {
  const int g = lane >> 4;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    v4f x;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      x[r] = COL ? __shfl(mine[r], 4 * i + g, PBG_WAVE) : __shfl(mine[i], 4 * (4 * g + r), PBG_WAVE);
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] *= x;
  }
}

// four floats at any multiple of four bytes
__device__ __forceinline__ v4f load4(const float* p) {
  typedef float u4f __attribute__((ext_vector_type(4), aligned(4)));
  return *(const u4f*)p;
}

// one k-run of a tile.  COL: A[m][k] = dS[k][m], else dS[m][k].  kf: the scale
// of each row of B (SCALED).  Leaves the sums undone of the rows' powers.
template <int NB, bool COL, bool SOFTMAX, bool SCALED>
__device__ __forceinline__ void value_run(const ValueArgs& a, const float* ds, const float* rs, const float* kf,
                                          const uint16_t* brows, int m0, int M, int K, int n0,
                                          ValueSmem<NB>& sm, v4f (&acc)[2][NB], int w, int lane) {
  constexpr int BL = row_blocks(NB);
  const int l16 = lane & 15, g = lane >> 4;
  const int nk = (K + BK - 1) / BK;
  if (nk <= 0) return;
  const rsrc_t rb = make_rsrc(brows);
  uint32_t ob[BL];
  int brow[BL];
#pragma unroll
  for (int i = 0; i < BL; ++i) {
    int word, col;
    kr_lane<BL>(w + 4 * i, lane, brow[i], word, col);
    ob[i] = (n0 & ~31) + col < a.dh ? (uint32_t)(((int64_t)brow[i] * a.ld + 2 * (n0 & ~31) + word) * 2) : kOob;
  }
  auto load_b = [&](int buf, int kt) {
    const bool tail = (kt + 1) * BK > K;
#pragma unroll
    for (int i = 0; i < BL; ++i)
      dma16(rb, sm.B[buf] + (w + 4 * i) * 512, (tail && kt * BK + brow[i] >= K) ? kOob : ob[i], kt * BK * a.ld * 2);
  };
  // The wave's dS of a slice, as it lies: COL the rows k = arow + 8 q of columns
  // 4 (lane % 8) .. + 3 (half a wave the even ones: their stores to LDS fall in
  // distinct banks), else eight k from 8 (lane % 4) of the rows arow + 16 q.
  // Offsets count from the slice's first row (COL) or the
  // wave's: a matrix of any size.
  v4f pa[4];
  float f[4];      // COL: factor of each k row; else: of the two rows
  v4f fk[2];       // SCALED, not COL: factors of the eight k
  const int x0 = m0 + 32 * w;   // the wave's first output row
  const int arow = COL ? 2 * ((lane >> 3) & 3) + (lane >> 5) : lane >> 2, acol = COL ? 4 * (lane & 7) : 8 * (lane & 3);
  const int k4 = (K + 3) & ~3;
  uint32_t oa[COL ? 4 : 2];
#pragma unroll
  for (int q = 0; q < (COL ? 4 : 2); ++q) {
    const bool in = COL ? x0 + acol < a.lds : x0 + arow + 16 * q < M;
    oa[q] = in ? (uint32_t)(((int64_t)(arow + (COL ? 8 : 16) * q) * a.lds + acol) * 4) : kOob;
  }
  const float* abase = COL ? ds + x0 : ds + (int64_t)x0 * a.lds;
  auto load_a = [&](int kt) {
    const int k0 = kt * BK;
    if (COL) {
      const rsrc_t rd = make_rsrc(abase + (int64_t)k0 * a.lds);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = k0 + arow + 8 * q;
        const bool in = k < K;
        pa[q] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rd, in ? oa[q] : kOob, 0, 0));
        const int kk = in ? k : 0;
        f[q] = SOFTMAX ? rs[(int64_t)min(x0 >> 6, a.nct - 1) * a.C + kk] : 1.0f;
        if (SCALED) f[q] *= kf[kk];
      }
    } else {
      const rsrc_t rd = make_rsrc(abase);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
          pa[2 * q + h] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(
                                                      rd, k0 + acol + 4 * h < k4 ? oa[q] + 16 * h : kOob, 4 * k0, 0));
        const int m = x0 + arow + 16 * q;
        f[q] = SOFTMAX ? rs[(int64_t)(k0 >> 6) * a.C + (m < M ? m : 0)] : 1.0f;
      }
      if (SCALED) {   // past the rows: finite, and dS is zero there
        fk[0] = load4(kf + k0 + acol);
        fk[1] = load4(kf + k0 + acol + 4);
      }
    }
  };
  // the powers of this lane's rows: COL of its four columns, else of its two rows
  v4f sc;
#pragma unroll
  for (int c = 0; c < 4; ++c) sc[c] = factor_scale(0.0f);
  auto factors = [&](v4f (&v)[4]) {
    if (COL) {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = pa[q] * f[q] * sc;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v[q] = pa[q] * (f[q >> 1] * sc[q >> 1]);
        if (SCALED) v[q] *= fk[q & 1];
      }
    }
  };
  // splits the factors into LDS
  auto split_a = [&](const v4f (&v)[4]) {
    if (COL) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = arow + 8 * q;
        uint32_t h0, l0, h1, l1;
        split2_pair(v[q].x, v[q].y, h0, l0);
        split2_pair(v[q].z, v[q].w, h1, l1);
        const uint32_t at = 64 * 4 * k + (acol & 15);   // 16-bit words
        const uint32_t pr = 4 * w + (acol >> 4);
        *(uint2*)(sm.A + at + 16 * (pr ^ kr_f<4>(k))) = make_uint2(h0, h1);
        *(uint2*)(sm.A + at + 16 * ((pr + 2) ^ kr_f<4>(k))) = make_uint2(l0, l1);
      }
    } else {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int m = 32 * w + arow + 16 * q;
        u32x4 h, l;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          uint32_t h0, l0, h1, l1;
          split2_pair(v[2 * q + k].x, v[2 * q + k].y, h0, l0);
          split2_pair(v[2 * q + k].z, v[2 * q + k].w, h1, l1);
          h[2 * k] = h0;
          h[2 * k + 1] = h1;
          l[2 * k] = l0;
          l[2 * k + 1] = l1;
        }
        *(u32x4*)(sm.A + kc_slot(m, 0, lane & 3)) = h;
        *(u32x4*)(sm.A + kc_slot(m, 1, lane & 3)) = l;
      }
    }
  };
  // lowers the powers of the rows whose largest factor of the slice exceeds
  // theirs; the accumulators follow
  auto lower_powers = [&]() {
    v4f m = {0.f, 0.f, 0.f, 0.f};
    if (COL) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = 0; c < 4; ++c) m[c] = fmaxf(m[c], pa[q][c] * f[q]);
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int o = 8; o < 64; o <<= 1) m[c] = fmaxf(m[c], __shfl_xor(m[c], o, PBG_WAVE));
    } else {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        float t = 0.0f;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            float x = pa[2 * q + h][c] * f[q];
            if (SCALED) x *= fk[h][c];
            t = fmaxf(t, x);
          }
        t = fmaxf(t, __shfl_xor(t, 1, PBG_WAVE));
        m[q] = fmaxf(t, __shfl_xor(t, 2, PBG_WAVE));
      }
    }
    v4f ratio;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float old = sc[c];
      if (m[c] * old >= kFactorLimit) sc[c] = factor_scale(m[c]);
      ratio[c] = sc[c] * inverse_power(old);
    }
    scale_rows<NB, COL>(ratio, acc, lane);
  };
  auto store_a = [&]() {
    v4f v[4];
    factors(v);
    float top = v[0].x;   // ahead of the split, which takes the registers over
#pragma unroll
    for (int q = 0; q < 16; ++q) top = fmaxf(top, v[q >> 2][q & 3]);
    split_a(v);
    // rare past the first slices, so the slice is simply written again
    if (__any(top >= kFactorLimit)) {
      lower_powers();
      factors(v);
      __asm__ volatile("" ::: "memory");
      split_a(v);
    }
    __asm__ volatile("" ::: "memory");   // the wave's own fragment reads follow
  };
  const bool odd = (n0 & 16) != 0;
  const int rho = l16 >> 2;
  const uint32_t b0 = lds_offset(sm.B) + kr_address<BL>(8 * g + rho, l16);
  const uint32_t b1 = lds_offset(sm.B) + kr_address<BL>(8 * g + 4 + rho, l16);
  const uint32_t a0 = lds_offset(sm.A) + kr_address<4>(8 * g + rho, l16);
  const uint32_t a1 = lds_offset(sm.A) + kr_address<4>(8 * g + 4 + rho, l16);
  const int as[2] = {kc_slot(32 * w + l16, 0, g), kc_slot(32 * w + l16, 1, g)};

  load_b(0, 0);
  load_a(0);
  store_a();
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    wait_loads();
    __syncthreads();
    if (kt + 1 < nk) {
      load_b(buf ^ 1, kt + 1);
      load_a(kt + 1);
    }
    v8h af[2][2];   // [plane][row block]
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (COL) {
          const uint32_t x = 32u * (4 * w + 2 * p + i);
          af[p][i] = kr_fragment(a0 ^ x, a1 ^ x);
        } else {
          af[p][i] = *(const v8h*)(sm.A + as[p] + 16 * 64 * i);
        }
      }
    // a block's fragments are read while the one before it is multiplied (read
    // and awaited block by block, the LDS's latency was a third of the time)
    const uint32_t bb = buf * (uint32_t)sizeof(sm.B[0]);
    v8h bf[2][2];   // [block parity][plane]
    auto read_b = [&](int j) {
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const uint32_t x = 32u * ((NB & 1) && odd ? kr_pair(j + 1, p) : kr_pair(j, p));
        bf[j & 1][p] = kr_fragment((b0 + bb) ^ x, (b1 + bb) ^ x);
      }
    };
    read_b(0);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (j + 1 < NB) read_b(j + 1);
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[q == 0][i], bf[j & 1][q == 1], acc[i][j], 0, 0, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, (COL ? 8 : 4) + 4, 0);   // LDS reads
#pragma unroll
    for (int j = 0; j + 1 < NB; ++j) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // a matrix instruction
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    }
    __asm__ volatile("" ::: "memory");   // the wave has read this slice's A
    if (kt + 1 < nk) store_a();
  }
  // the powers undone
#pragma unroll
  for (int c = 0; c < 4; ++c) sc[c] = inverse_power(sc[c]);
  scale_rows<NB, COL>(sc, acc, lane);
}

template <int NB, bool SOFTMAX, bool SCALED>
__global__ __launch_bounds__(256, 2) void value_backward_kernel(ValueArgs a, int tiles_q, int tiles_n, int tiles_d,
                                                                int nq) {
  __shared__ __align__(16) ValueSmem<NB> sm;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool dq = (int)blockIdx.x < nq;
  const int id = dq ? blockIdx.x : blockIdx.x - nq;
  const int nwg = dq ? nq : gridDim.x - nq;
  // all tiles of one (chunk, side) on one XCD
  const int q8 = nwg >> 3, r8 = nwg & 7, xcd = id & 7;
  const int lid = xcd * q8 + min(xcd, r8) + (id >> 3);
  const int td = lid % tiles_d;
  int rest = lid / tiles_d;
  const int tiles = dq ? tiles_q : tiles_n;
  const int tm = rest % tiles;
  rest /= tiles;
  const int c = rest >> 1, side = rest & 1, z = rest;
  const int Cc = a.cstart ? wave_uniform(a.cstart[c + 1] - a.cstart[c]) : min(a.C, a.m_step - c * a.C);
  const int Nc = Cc + a.U;
  const int n0 = td * 16 * NB, m0 = tm * BT, M = dq ? Cc : Nc;
  if (m0 >= M) return;
  v4f acc[2][NB];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  const float* ds = a.ds + (int64_t)z * a.C * a.lds;
  const float* rs = SOFTMAX ? a.rowscale + (int64_t)z * a.nct * a.C : nullptr;
  float f = SCALED ? 1.0f : 0x1p-15f;   // unit rows are held times 2^15
  if (dq)
    value_run<NB, false, SOFTMAX, SCALED>(a, ds, rs, SCALED ? a.ni + (int64_t)z * (a.C + a.U) : nullptr,
                                          a.N + c * a.n_cs + side * a.n_ss, m0, M, Nc, n0, sm, acc, w, lane);
  else
    value_run<NB, true, SOFTMAX, SCALED>(a, ds, rs, SCALED ? a.qi + (int64_t)z * a.C : nullptr,
                                         a.Q + c * a.q_cs + side * a.q_ss, m0, M, Cc, n0, sm, acc, w, lane);
  if (a.cscale) f *= wave_uniform(a.cscale[c]);
  float* C = dq ? a.dq + c * a.dq_cs + side * a.dq_ss : a.dn + c * a.dn_cs + side * a.dn_ss;
  const int l16 = lane & 15, g = lane >> 4;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + 32 * w + 16 * i + 4 * g + r;
      if (m >= M) continue;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int n = n0 + 16 * j + l16;
        if (n < a.dp) C[(int64_t)m * a.dp + n] = acc[i][j][r] * f;
      }
    }
}

template <int NB>
void launch_value_nb(const ValueArgs& a, int nchunks, hipStream_t s) {
  const int tiles_d = (a.dp + 16 * NB - 1) / (16 * NB);
  const int tiles_q = (a.C + BT - 1) / BT, tiles_n = (a.C + a.U + BT - 1) / BT;
  const int64_t nq = (int64_t)tiles_q * tiles_d * 2 * nchunks, nn = (int64_t)tiles_n * tiles_d * 2 * nchunks;
  const unsigned grid = (unsigned)(nq + nn);
  if (a.rowscale) {
    if (a.ni) value_backward_kernel<NB, true, true><<<grid, 256, 0, s>>>(a, tiles_q, tiles_n, tiles_d, (int)nq);
    else value_backward_kernel<NB, true, false><<<grid, 256, 0, s>>>(a, tiles_q, tiles_n, tiles_d, (int)nq);
  } else {
    if (a.ni) value_backward_kernel<NB, false, true><<<grid, 256, 0, s>>>(a, tiles_q, tiles_n, tiles_d, (int)nq);
    else value_backward_kernel<NB, false, false><<<grid, 256, 0, s>>>(a, tiles_q, tiles_n, tiles_d, (int)nq);
  }
}

}  // namespace

void launch_value_backward(const ValueArgs& a, int nchunks, hipStream_t s) {
  if (nchunks <= 0) return;
  // the fewest column tiles; among equals the fewest 16-column blocks
  const int nb = (a.dp + 15) / 16;
  if (nb <= 2) launch_value_nb<2>(a, nchunks, s);
  else if (nb <= 4) launch_value_nb<4>(a, nchunks, s);
  else if (nb <= 7) launch_value_nb<7>(a, nchunks, s);
  else if (nb <= 8 || (nb + 12) / 13 == (nb + 7) / 8) launch_value_nb<8>(a, nchunks, s);
  else launch_value_nb<13>(a, nchunks, s);
}
