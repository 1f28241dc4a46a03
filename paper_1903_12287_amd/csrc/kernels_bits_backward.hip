// Ranking backward: dQ = dS . N and dN = dS^T . Q with dS (0 or 1) as bits
// (the blocks that the score kernel leaves, BitsView in kernels.h) and the
// rows of N and Q as pieces (pieces.h).
//
// A workgroup computes 64 IM x 16 NB outputs: four waves of 16 IM rows, each
// over all columns, so that every row's bits are expanded by one wave only.
// The rows of the B operand (k) move global -> LDS as they lie in memory, and
// the matrix fragments (eight k of one column) come out of the transposing
// LDS reads of gfx950, so no transposed copy of the pieces exists.  A slice
// is 32 k: two stages in LDS, one barrier per slice.
//
// With float32 operands a set bit is the fp16 number 2^-14 (bit 10 alone), so
// that the sum of two bits (the merged in-chunk block below), 2^-13, is an
// integer add of the patterns.  (The denormals 2^-24 and 2^-23 would need no
// shift, but the matrix instruction aligns their products by their unnormalised
// exponent and loses ten bits of the sums.)  With per-row scales (dot) each
// k's bit is multiplied by its row's scale relative to the chunk's largest row.
// Where rows differ by more than an fp16 number holds, the scales come in
// levels of 30 binades (finalize_body.h) and the run over k is made once a
// level, the smallest rows' first, the accumulators carried from one to the
// next: a row counts unless it is some 140 binades below the largest.
//
// Merged in-chunk block (cos without reciprocal predicates: the queries of a
// side are the other side's candidates): with B0 the bits of side 0 and B1
// those of side 1's in-chunk block, stored transposed in the same places,
//   dQ0 + dN1 of edge e   = sum_t (B0[e][t] + B1[e][t]) N0[t] over t < Cc,
//                           then B0 alone over the uniform candidates;
//   dQ1 + dN0 of edge i   = sum_e (B0[e][i] + B1[e][i]) N1[e] over e < Cc,
//                           then side 1's uniform bits times N1.
#include <algorithm>

#include "kernels.h"
#include "pieces.h"

namespace {

using namespace pieces;

constexpr int BK = 32;

// how a set bit (or the sum of two) becomes the matrix operand
enum { A_UNIT = 0, A_SCALED = 1 };

// a set bit as it enters the integer sums of a pair
constexpr uint32_t one_bits(int mode) { return mode == A_UNIT ? 0x04000400u : 0x00010001u; }

// 128-byte blocks (32 columns, both planes) of a B row
constexpr int row_blocks(int nb) { return nb <= 2 ? 1 : (nb <= 4 ? 2 : 4); }

template <int NB, int IM>
struct BitsSmem {
  static constexpr int BL = row_blocks(NB);
  uint16_t B[2][BK * 64 * BL];
  uint32_t bits[2][2][64 * IM];   // [stage][plane]: 32 k of 64 IM rows (or columns)
  u32x4 lut[256];                 // byte -> eight 16-bit 0 / one_bits
};

// one run over k of a tile: dS rows (ROW: A[m][k] = bit (row m, column k)) or
// columns (COL: A[m][k] = bit (row k, column m)) times rows of B
struct BitsPhase {
  const uint32_t* p0;   // bit blocks of the first plane, of the second (merged, k < kmerge)
  const uint32_t* p1;
  int RB;               // row blocks per column block
  int CB;               // column blocks
  int blk;              // first row block (ROW) or column block (COL) of the tile
  const uint16_t* B;    // the B rows
  int K, kmerge;
  const uint16_t* ks;   // A_SCALED: fp16 scale of each k, [levels][ld_ks]
  int ld_ks, levels;
};

template <int NB, int IM>
struct BitsLoader {
  static constexpr int BL = row_blocks(NB);   // moves per wave: 4 BL of 1 KB over four waves
  rsrc_t rb, r0, r1;
  uint32_t ob[BL];
  int row[BL];
  uint32_t obits;
  int w, lane, ld, K, kmerge, bstep;

  template <bool COL, bool MERGE>
  __device__ __forceinline__ void begin(const BitsPhase& p, int ld_, int n0, int dh, int w_, int lane_) {
    w = w_;
    lane = lane_;
    ld = ld_;
    K = p.K;
    kmerge = p.kmerge;
    rb = make_rsrc(p.B);
#pragma unroll
    for (int i = 0; i < BL; ++i) {
      int word, col;
      kr_lane<BL>(w + 4 * i, lane, row[i], word, col);
      // an odd NB starts every other tile in the middle of a block
      ob[i] = (n0 & ~31) + col < dh ? (uint32_t)(((int64_t)row[i] * ld + 2 * (n0 & ~31) + word) * 2) : kOob;
    }
    r0 = make_rsrc(p.p0);
    if (MERGE) r1 = make_rsrc(p.p1);
    // 16 bytes (half a block) a lane; 32 IM... lanes of one move cover the slice
    if (!COL) {
      const int per = 8 * IM;                      // halves per column block
      const int cb = lane / per, rb_ = (lane % per) >> 1, half = lane & 1;
      obits = (cb < 2 && p.blk + rb_ < p.RB) ? (uint32_t)(((cb * p.RB + p.blk + rb_) * 8 + 4 * half) * 4) : kOob;
      bstep = 2 * p.RB * 32;                       // two column blocks a slice
    } else {
      const int cb = lane >> 2, rb_ = (lane >> 1) & 1, half = lane & 1;
      obits = (cb < 4 * IM && p.blk + cb < p.CB) ? (uint32_t)((((p.blk + cb) * p.RB + rb_) * 8 + 4 * half) * 4) : kOob;
      bstep = 2 * 32;                              // two row blocks a slice
    }
  }

  template <bool MERGE>
  __device__ __forceinline__ void slice(BitsSmem<NB, IM>& sm, int buf, int kt) const {
    const int k0 = kt * BK;
    // the slice's bits: 32 x 64 IM bits = 64 IM words, 16 IM lanes of 16 bytes
    if (w == 3 && (IM == 4 || lane < 16 * IM)) dma16(r0, sm.bits[buf][0], obits, kt * bstep);
    if (MERGE && w == 2 && k0 < kmerge && (IM == 4 || lane < 16 * IM)) dma16(r1, sm.bits[buf][1], obits, kt * bstep);
    const bool tail = k0 + BK > K;
#pragma unroll
    for (int i = 0; i < BL; ++i)
      dma16(rb, sm.B[buf] + (w + 4 * i) * 512, (tail && k0 + row[i] >= K) ? kOob : ob[i], k0 * ld * 2);
  }
};

__device__ __forceinline__ uint32_t pk_mul_u16(uint32_t a, uint32_t b) {
  typedef unsigned short us2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, (us2)(__builtin_bit_cast(us2, a) * __builtin_bit_cast(us2, b)));
}

template <int NB, int IM, int MODE, bool COL, bool MERGE>
__device__ __forceinline__ void bits_phase(const BitsPhase& p, int ld, int n0, int dh, BitsSmem<NB, IM>& sm,
                                           v4f (&acc)[IM][NB], int w, int lane) {
  constexpr int BL = row_blocks(NB);
  const int l16 = lane & 15, g = lane >> 4;
  const int nk = (p.K + BK - 1) / BK;
  if (nk <= 0) return;
  const bool odd = (n0 & 16) != 0;
  BitsLoader<NB, IM> ld_;
  ld_.template begin<COL, MERGE>(p, ld, n0, dh, w, lane);
  ld_.template slice<MERGE>(sm, 0, 0);
  // this lane's rows of the transposing reads: k in natural order for ROW;
  // for COL in the order of the words' fields, 0 4 1 5 | 2 6 3 7
  const int rho = l16 >> 2;
  const int row0 = 8 * g + (COL ? (rho >> 1) + 4 * (rho & 1) : rho);
  const int row1 = row0 + (COL ? 2 : 4);
  const uint32_t b0 = lds_offset(sm.B) + kr_address<BL>(row0, l16);
  const uint32_t b1 = lds_offset(sm.B) + kr_address<BL>(row1, l16);
  // ROW: the byte of row 16 i + l16 of the wave, k = 8 g .. + 7; COL: the four
  // words of rows 8 g .. + 7 of column block i of the wave
  const uint32_t boff = COL ? (uint32_t)(((w * IM * 2 + (g >> 1)) * 8 + 4 * (g & 1)) * 4)
                            : (uint32_t)((((g >> 1) * 4 * IM + w * IM) * 8 + 4 * (l16 >> 3) + (l16 & 3)) * 4 +
                                         2 * ((l16 >> 2) & 1) + (g & 1));
  constexpr int bstride = COL ? 64 : 32;   // bytes between the wave's fragments
  // COL: column l16 is bits l16 and 16 + l16 of a word; rotated to the place
  // of a 1 in the two halves
  constexpr uint32_t kBit = one_bits(MODE);
  const uint32_t crot = (uint32_t)(l16 + (MODE == A_UNIT ? 22 : 0)) & 31u;
  u32x4 ks = {0u, 0u, 0u, 0u};
  const int nit = MODE == A_SCALED ? nk * p.levels : nk;   // slices of all levels
  const uint16_t* lks = p.ks;                              // the level's scales
  if (MODE == A_SCALED) {
    lks += (int64_t)(p.levels - 1) * p.ld_ks;
    ks = *(const u32x4*)(lks + 8 * g);
  }
  int lkt = 0;   // slice of the level
  for (int it = 0; it < nit; ++it) {
    const int kt = MODE == A_SCALED ? lkt : it;
    const int buf = it & 1;
    wait_loads();
    __syncthreads();
    const bool merged = MERGE && kt * BK < p.kmerge;
    u32x4 scl = ks;   // scales of the slice's k, in the lane's order
    if (MODE == A_SCALED && COL)
      scl = (u32x4){(ks.x & 0xFFFFu) | (ks.z << 16), (ks.x >> 16) | (ks.z & 0xFFFF0000u),
                    (ks.y & 0xFFFFu) | (ks.w << 16), (ks.y >> 16) | (ks.w & 0xFFFF0000u)};
    const char* bp0 = (const char*)sm.bits[buf][0] + boff;
    const char* bp1 = (const char*)sm.bits[buf][1] + boff;
    v8h af[IM];
#pragma unroll
    for (int i = 0; i < IM; ++i) {
      u32x4 v;
      if (COL) {
        v = *(const u32x4*)(bp0 + i * bstride);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = __builtin_amdgcn_alignbit(v[q], v[q], crot) & kBit;
      } else {
        v = sm.lut[*(const uint8_t*)(bp0 + i * bstride)];
      }
      if (MERGE && merged) {
        u32x4 x;
        if (COL) {
          x = *(const u32x4*)(bp1 + i * bstride);
#pragma unroll
          for (int q = 0; q < 4; ++q) x[q] = __builtin_amdgcn_alignbit(x[q], x[q], crot) & kBit;
        } else {
          x = sm.lut[*(const uint8_t*)(bp1 + i * bstride)];
        }
        v += x;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (MODE == A_SCALED) v[q] = pk_mul_u16(v[q], scl[q]);
      }
      af[i] = __builtin_bit_cast(v8h, v);
    }
    const bool level_ends = MODE == A_SCALED && kt + 1 == nk;
    if (MODE == A_SCALED) {
      lkt = level_ends ? 0 : kt + 1;
      if (level_ends) lks -= p.ld_ks;
    }
    if (it + 1 < nit) {
      ld_.template slice<MERGE>(sm, buf ^ 1, MODE == A_SCALED ? lkt : it + 1);
      if (MODE == A_SCALED) ks = *(const u32x4*)(lks + lkt * BK + 8 * g);
    }
    const uint32_t bb = buf * sizeof(sm.B[0]);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      v8h bf[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint32_t x = 32u * ((NB & 1) && odd ? kr_pair(j + 1, q) : kr_pair(j, q));
        bf[q] = kr_fragment((b0 + bb) ^ x, (b1 + bb) ^ x);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int i = 0; i < IM; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[i], bf[q], acc[i][j], 0, 0, 0);
    }
    if (level_ends && it + 1 < nit) {
#pragma unroll
      for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] *= 0x1p-30f;
    }
  }
}

// The tile's outputs; rows below mlo and from M on are not written.
template <int NB, int IM>
__device__ __forceinline__ void store_tile(float* C, int ldc, int m0, int mlo, int M, int n0, int N, float f,
                                           const v4f (&acc)[IM][NB], int w, int lane) {
  const int l16 = lane & 15, g = lane >> 4;
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + 16 * (IM * w + i) + 4 * g + r;
      if (m < mlo || m >= M) continue;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int n = n0 + 16 * j + l16;
        if (n < N) C[(int64_t)m * ldc + n] = acc[i][j][r] * f;
      }
    }
}

// Work of chunk c: dQ tiles of both sides, then dN tiles (long runs over k
// first).  MERGED: dN only for the uniform candidates.
template <int NB, int IM, int MODE, bool MERGED>
__global__ __launch_bounds__(256, 2) void bits_backward_kernel(BitsArgs a, int tiles_q, int tiles_n, int tiles_d,
                                                               int nq) {
  __shared__ __align__(16) BitsSmem<NB, IM> sm;
  constexpr int BT = 64 * IM;
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
  const int c = rest >> 1, side = rest & 1;
  const int Cc = a.cstart ? wave_uniform(a.cstart[c + 1] - a.cstart[c]) : min(a.C, a.m_step - c * a.C);
  const int Nc = Cc + a.U;
  const int n0 = td * 16 * NB;
  const int first = (!dq && MERGED) ? (Cc & ~15) : 0;   // dN starts at the uniform candidates' block
  const int m0 = first + tm * BT;
  const int M = dq ? Cc : Nc;
  if (m0 >= M) return;
  if (tid < 256) {
    u32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = ((((tid >> (2 * q)) & 3) * 0x8001u) & 0x10001u) * (one_bits(MODE) & 0xFFFFu);
    sm.lut[tid] = v;   // visible after the first slice's barrier
  }
  v4f acc[IM][NB];
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};

  const uint32_t* bs = a.bits0 + c * a.bits_cs + side * a.bits_ss;
  const uint16_t* nrows = a.N + c * a.n_cs + side * a.n_ss;   // candidates of this side
  const uint16_t* qrows = a.Q + c * a.q_cs + side * a.q_ss;   // queries of this side
  const int CB = a.CB;
  float f = a.unscale;
  // the scales of the rows of B
  const uint16_t* ks = nullptr;
  const int ld_ks = dq ? a.ks_n : a.ks_q;
  int levels = 1;
  if (MODE == A_SCALED) {
    const int z = 2 * c + side;
    ks = (dq ? a.nks : a.qks) + (int64_t)z * KS_LEVELS * ld_ks;
    const int2 t = (dq ? a.ntop : a.qtop)[z];
    f = ldexpf(1.0f, wave_uniform(t.x) - 156);
    levels = wave_uniform(t.y);
  }
  if (dq) {
    if (MERGED && side == 1) {
      // in-chunk block by columns, then the uniform candidates by rows
      const BitsPhase p{a.bits0 + c * a.bits_cs, a.bits1 + c * a.bits1_cs, a.RB, a.CB1, m0 >> 4, nrows, Cc,
                        Cc, nullptr, 0, 1};
      bits_phase<NB, IM, MODE, true, true>(p, a.ld, n0, a.dh, sm, acc, w, lane);
      __syncthreads();   // the stages are free again
      const BitsPhase u{bs, nullptr, a.RB, CB, m0 >> 4, nrows + (int64_t)Cc * a.ld, a.U, 0, nullptr, 0, 1};
      bits_phase<NB, IM, MODE, false, false>(u, a.ld, n0, a.dh, sm, acc, w, lane);
    } else {
      const BitsPhase p{bs, MERGED ? a.bits1 + c * a.bits1_cs : nullptr, a.RB, CB, m0 >> 4, nrows, Nc,
                        MERGED ? Cc : 0, ks, ld_ks, levels};
      bits_phase<NB, IM, MODE, false, MERGED>(p, a.ld, n0, a.dh, sm, acc, w, lane);
    }
  } else {
    const bool uni = MERGED && side == 1;   // side 1's bits hold the uniform columns only
    const BitsPhase p{bs, nullptr, a.RB, CB, (uni ? m0 - first : m0) >> 4, qrows, Cc, 0, ks, ld_ks, levels};
    bits_phase<NB, IM, MODE, true, false>(p, a.ld, n0, a.dh, sm, acc, w, lane);
  }
  // the chunk's relation weight scales its gradients (powers of two aside, an
  // ordinary float32 product)
  if (a.cscale) f *= wave_uniform(a.cscale[c]);
  if (dq) {
    store_tile<NB, IM>(a.dq + c * a.dq_cs + side * a.dq_ss, a.dp, m0, 0, M, n0, a.dp, f, acc, w, lane);
  } else {
    // MERGED, side 1: the matrix starts at the first uniform candidate
    const int shift = (MERGED && side == 1) ? Cc - first : 0;
    store_tile<NB, IM>(a.dn + c * a.dn_cs + side * a.dn_ss, a.dp, m0 + shift, MERGED ? Cc : 0, M, n0, a.dp, f, acc, w,
                       lane);
  }
}

template <int NB, int IM, int MODE, bool MERGED>
void launch_bits_t(const BitsArgs& a, int nchunks, hipStream_t s) {
  constexpr int BT = 64 * IM;
  const int tiles_d = (a.dp + 16 * NB - 1) / (16 * NB);
  const int tiles_q = (a.C + BT - 1) / BT;
  const int rows_n = MERGED ? a.U + 15 : a.C + a.U;
  const int tiles_n = (rows_n + BT - 1) / BT;
  const int64_t nq = (int64_t)tiles_q * tiles_d * 2 * nchunks, nn = (int64_t)tiles_n * tiles_d * 2 * nchunks;
  bits_backward_kernel<NB, IM, MODE, MERGED><<<(unsigned)(nq + nn), 256, 0, s>>>(a, tiles_q, tiles_n, tiles_d,
                                                                                    (int)nq);
}

template <int NB, int IM>
void launch_bits_nb(const BitsArgs& a, int nchunks, hipStream_t s) {
  if (a.merged) launch_bits_t<NB, IM, A_UNIT, true>(a, nchunks, s);
  else if (a.nks) launch_bits_t<NB, IM, A_SCALED, false>(a, nchunks, s);
  else launch_bits_t<NB, IM, A_UNIT, false>(a, nchunks, s);
}

template <int NB>
void launch_bits_im(const BitsArgs& a, int nchunks, hipStream_t s) {
  // 256-row tiles; 128-row ones where a chunk's rows would leave most of a
  // tall tile empty
  if (a.C > 128 || a.U > 256) launch_bits_nb<NB, 4>(a, nchunks, s);
  else launch_bits_nb<NB, 2>(a, nchunks, s);
}

}  // namespace

void launch_bits_backward(const BitsArgs& a, int nchunks, hipStream_t s) {
  if (nchunks <= 0) return;
  // columns per tile: the fewest 16-column blocks over all column tiles
  const int nb = (a.dp + 15) / 16;
  if (nb <= 2) launch_bits_im<2>(a, nchunks, s);
  else if (nb <= 4) launch_bits_im<4>(a, nchunks, s);
  else if ((nb + 6) / 7 * 7 < (nb + 7) / 8 * 8) launch_bits_im<7>(a, nchunks, s);
  else launch_bits_im<8>(a, nchunks, s);
}
