// Backward of the logistic and softmax losses: dQ = dS . N and dN = dS^T . Q
// with dS a float32 matrix (softmax: exp(s - block maximum), completed by the
// row's scale of its 64-column block as it is staged) and the rows of N and Q
// as pieces (pieces.h).  dS is split into two fp16 pieces too, times 2^15 and
// the losses' own power of two: three plane products, as in the score.
//
// A workgroup computes 128 x 16 NB outputs, four waves of 32 rows over all
// columns.  B rows move global -> LDS as they lie in memory and are read
// through the transposing LDS reads; dS goes through registers (scale, split)
// into LDS: k-contiguous rows for dQ, its rows as they are for dN, whose
// fragments are read transposed as well.  Wide tiles (NB = 13) read dS half
// as often where the rows are long: at d = 400 two column tiles instead of
// four.
//
// With per-row scales (dot) the rows of B carry different powers of two; the
// factor that makes them equal (2^(e_k - e_max), from the finalisation) is
// multiplied into dS with the rest.
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
  static constexpr int AB = NB <= 8 ? 2 : 1;   // stages of A (one where B takes the room of two)
  uint16_t B[2][BK * 64 * BL];
  uint16_t A[AB][BT * 64];
};

// one k-run of a tile.  COL: A[m][k] = dS[k][m], else dS[m][k].
template <int NB, bool COL, bool SOFTMAX, bool SCALED>
__device__ __forceinline__ void value_run(const ValueArgs& a, const float* ds, const float* rs, const float* kf,
                                          const uint16_t* brows, int m0, int M, int K, float afac, int n0,
                                          ValueSmem<NB>& sm, v4f (&acc)[2][NB], int w, int lane) {
  constexpr int BL = row_blocks(NB), AB = ValueSmem<NB>::AB;
  const int tid = threadIdx.x, l16 = lane & 15, g = lane >> 4;
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
  // dS of a slice: COL four k rows (tid / 32 + 8 q) of four columns, else two
  // rows (tid / 4 + 64 q) of eight k.  Offsets count from the slice's (COL) or
  // the tile's first row: dS may hold more than 4 GiB
  v4f pa[4];
  float f[4];      // COL: factor of each row; else: factors of the two rows
  v4f fk[2];       // SCALED, not COL: factors of the eight k
  const int xcol = 4 * (tid & 31), xrow = tid >> 2, kq = 8 * (tid & 3);
  const int k4 = (K + 3) & ~3;
  auto load_a = [&](int kt) {
    const int k0 = kt * BK;
    const rsrc_t rd = make_rsrc(ds + (int64_t)(COL ? k0 : m0) * a.lds);
    if (COL) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = k0 + (tid >> 5) + 8 * q;
        const bool in = k < K;
        pa[q] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(
                                            rd, in && m0 + xcol < a.lds ? (uint32_t)(((k - k0) * a.lds + m0 + xcol) * 4) : kOob, 0, 0));
        const int kk = in ? k : 0;
        f[q] = afac;
        if (SOFTMAX) f[q] *= rs[(int64_t)min((m0 + xcol) >> 6, a.nct - 1) * a.C + kk];
        if (SCALED) f[q] *= kf[kk];
      }
    } else {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int m = m0 + xrow + 64 * q;
#pragma unroll
        for (int h = 0; h < 2; ++h)
          pa[2 * q + h] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(
                                                      rd, m < M && k0 + kq + 4 * h < k4 ? (uint32_t)(((m - m0) * a.lds + k0 + kq + 4 * h) * 4) : kOob, 0, 0));
        f[q] = afac;
        if (SOFTMAX) f[q] *= rs[(int64_t)(k0 >> 6) * a.C + (m < M ? m : 0)];
      }
      if (SCALED) {
        fk[0] = *(const v4f*)(kf + k0 + kq);
        fk[1] = *(const v4f*)(kf + k0 + kq + 4);
      }
    }
  };
  auto store_a = [&](int buf) {
    if (COL) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = (tid >> 5) + 8 * q;
        const v4f v = pa[q] * f[q];
        uint32_t h0, l0, h1, l1;
        split2_pair(v.x, v.y, h0, l0);
        split2_pair(v.z, v.w, h1, l1);
        const uint32_t at = 64 * 4 * k + (xcol & 15);   // 16-bit words
        const uint32_t pr = 4 * (xcol >> 5) + ((xcol >> 4) & 1);
        *(uint2*)(sm.A[buf] + at + 16 * (pr ^ kr_f<4>(k))) = make_uint2(h0, h1);
        *(uint2*)(sm.A[buf] + at + 16 * ((pr + 2) ^ kr_f<4>(k))) = make_uint2(l0, l1);
      }
    } else {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int m = xrow + 64 * q;
        u32x4 h, l;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          v4f v = pa[2 * q + k] * f[q];
          if (SCALED) v *= fk[k];
          uint32_t h0, l0, h1, l1;
          split2_pair(v.x, v.y, h0, l0);
          split2_pair(v.z, v.w, h1, l1);
          h[2 * k] = h0;
          h[2 * k + 1] = h1;
          l[2 * k] = l0;
          l[2 * k + 1] = l1;
        }
        *(u32x4*)(sm.A[buf] + kc_slot(m, 0, tid & 3)) = h;
        *(u32x4*)(sm.A[buf] + kc_slot(m, 1, tid & 3)) = l;
      }
    }
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
  store_a(0);
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1, abuf = AB == 2 ? buf : 0;
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
          const uint32_t x = 32u * (4 * w + 2 * p + i), ab = abuf * (uint32_t)sizeof(sm.A[0]);
          af[p][i] = kr_fragment((a0 + ab) ^ x, (a1 + ab) ^ x);
        } else {
          af[p][i] = *(const v8h*)(sm.A[abuf] + as[p] + 16 * 64 * i);
        }
      }
    const uint32_t bb = buf * (uint32_t)sizeof(sm.B[0]);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      v8h bf[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const uint32_t x = 32u * ((NB & 1) && odd ? kr_pair(j + 1, p) : kr_pair(j, p));
        bf[p] = kr_fragment((b0 + bb) ^ x, (b1 + bb) ^ x);
      }
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[q == 0][i], bf[q == 1], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) {
      if (AB == 1) __syncthreads();   // every wave has read this slice's A
      store_a(AB == 2 ? buf ^ 1 : 0);
    }
  }
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
  // logistic: dS carries 1 / (candidates - 1), whose power of two is taken out
  const int lk = SOFTMAX || Nc < 2 ? 0 : 31 - __builtin_clz(Nc - 1);
  const float afac = ldexpf(1.0f, (SCALED ? 0 : 15) + lk);
  float f = ldexpf(1.0f, -30 - lk);
  if (dq) {
    value_run<NB, false, SOFTMAX, SCALED>(a, ds, rs, SCALED ? a.nkf + (int64_t)z * a.ks_n : nullptr,
                                          a.N + c * a.n_cs + side * a.n_ss, m0, M, Nc, afac, n0, sm, acc, w, lane);
    if (SCALED) f = ldexpf(1.0f, a.nmax[z] - 156 - lk);
  } else {
    value_run<NB, true, SOFTMAX, SCALED>(a, ds, rs, SCALED ? a.qkf + (int64_t)z * a.ks_q : nullptr,
                                         a.Q + c * a.q_cs + side * a.q_ss, m0, M, Cc, afac, n0, sm, acc, w, lane);
    if (SCALED) f = ldexpf(1.0f, a.qmax[z] - 156 - lk);
  }
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
    if (a.nkf) value_backward_kernel<NB, true, true><<<grid, 256, 0, s>>>(a, tiles_q, tiles_n, tiles_d, (int)nq);
    else value_backward_kernel<NB, true, false><<<grid, 256, 0, s>>>(a, tiles_q, tiles_n, tiles_d, (int)nq);
  } else {
    if (a.nkf) value_backward_kernel<NB, false, true><<<grid, 256, 0, s>>>(a, tiles_q, tiles_n, tiles_d, (int)nq);
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
