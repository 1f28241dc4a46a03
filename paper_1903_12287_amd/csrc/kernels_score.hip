// Score contraction of a step's chunks with the loss epilogue on its
// accumulators (Sec. 4.3 batched negatives: the score block of a chunk is one
// product, S = Q . N^T), float32 operands as row pieces (pieces.h): three
// plane products.
//
// Workgroups of WR x 2 waves walk 64 WR x 128 tiles (64 x 64 a wave), one
// workgroup a CU: eight waves (WR = 4), or four where a chunk has few edges.
// A workgroup's slices of 32 k, across all of its tiles, are one stream
// through three stages of LDS: while a slice is multiplied, the next one's
// fragments are read from LDS and the two after that are on their way from
// memory (global -> LDS without registers), one barrier per slice.  Tiles
// of a chunk go to one XCD so that its L2 holds the operands.  Measured at 40
// chunks of 1,000 edges and 1,000 uniform negatives, d = 128: 143 us in unit
// rows (the three-piece bf16 kernel before it 230 us), 172 us in scaled ones
// at d = 100 (254 us), in traces.
//
// What bounds it: matrix and vector instructions of a SIMD barely overlap on
// gfx950 (measured), so a tile costs their sum: per wave and slice 48 products
// (768 cycles), per tile 470 vector instructions of the epilogue (880 where
// it serves both sides).
#include <algorithm>

#include "kernels.h"
#include "pieces.h"

namespace {

using namespace pieces;

constexpr int BN = 128, BK = 32, STAGES = 3;

// What the candidates' scales give to the queries' (SCALED; the ranks take
// theirs through the exponent): an accumulator times a candidate's scale must
// not overflow where the score does not.  2^-23 is the most that the smallest
// scale, 2^-126, can give.
constexpr float kColShare = 0x1p-23f;

struct ScoreTile {
  int c, side, tm, tn, m0, n0, M, N, Cc;
  int64_t nrow0;   // candidate row of column 0
};

// division by a launch constant: m = ceil(2^32 / d); the product's high word is
// the quotient or one more
struct Divider {
  uint32_t d, m;
};
__device__ __forceinline__ int divide(Divider v, int x, int& rest) {
  int q = v.d == 1 ? x : (int)(((uint64_t)(uint32_t)x * v.m) >> 32);
  rest = x - q * (int)v.d;
  if (rest < 0) {
    --q;
    rest += (int)v.d;
  }
  return q;
}

// tiles of a launch: rows of tiles, column tiles of side 0 and of side 1
struct TileGrid {
  int per0, total;      // side 0's tiles of a chunk, all tiles
  int tiles_m;
  uint32_t band_m;      // reciprocal of four rows of tiles (Divider)
  Divider chunk, tn0, tn1;
};

// A plain product's tiles go in bands of four tile rows, column by column: the
// 32 tiles an XCD works on at a time take 4 panels of A and 8 of B (3.5 MB at
// 400 elements, its L2 4 MB) and not 1 and 32 (7.3 MB).
__device__ __forceinline__ void band_tile(const TileGrid& tg, int r, int& tm, int& tn) {
  int rest;
  const int band = divide(Divider{4 * tg.tn0.d, tg.band_m}, r, rest);
  const int h = min(4, tg.tiles_m - 4 * band);
  tn = rest / h;
  tm = 4 * band + rest - tn * h;
}

// The tile `id` of the launch; false: nothing to compute.  With share, side 0
// spans all candidates and side 1 the uniform ones only.
template <int BM>
__device__ __forceinline__ bool score_tile(const ScoreArgs& a, const TileGrid& tg, int id, ScoreTile& t) {
  int r;
  t.c = divide(tg.chunk, id, r);
  t.side = r >= tg.per0 ? 1 : 0;
  if (t.side) t.tm = divide(tg.tn1, r - tg.per0, t.tn);
  else if (a.Mfix > 0) band_tile(tg, r, t.tm, t.tn);
  else t.tm = divide(tg.tn0, r, t.tn);
  t.m0 = t.tm * BM;
  t.n0 = t.tn * BN;
  t.nrow0 = 0;
  if (a.Mfix > 0) {
    t.Cc = t.M = a.Mfix;
    t.N = a.Nfix;
  } else {
    if (a.cstart) t.Cc = wave_uniform(a.cstart[t.c + 1] - a.cstart[t.c]);
    else t.Cc = min(a.C, a.m_step - t.c * a.C);
    t.M = t.Cc;
    t.N = t.Cc + a.U;
    if (a.share && t.side) {
      t.N = a.U;
      t.nrow0 = t.Cc;
    }
  }
  return t.m0 < t.M && t.n0 < t.N;
}

template <int WR>
struct ScoreSmem {
  uint16_t A[STAGES][64 * WR * 64];
  uint16_t B[STAGES][BN * 64];
  float nthr[64 * WR];     // negated thresholds in the accumulators' scale, row and column scales
  float scl[64 * WR];
  float nthr1[BN];
  float cscl[BN];
  float thr[64 * WR];      // margin - p + bias of the rows and (shared tiles) of the columns
  float thr1[BN];
};

// moves a tile's slices: 8 WR moves of A and 16 of B over 2 WR waves
template <int WR>
struct SliceLoader {
  static constexpr int NB = 8 / WR;   // B moves per wave
  static constexpr int PER_SLICE = 4 + NB;
  rsrc_t ra, rb;
  uint32_t oa[4], ob[NB];
  int w, kq, dh;

  __device__ __forceinline__ void tile(const ScoreArgs& a, const ScoreTile& t, int w_, int lane) {
    w = w_;
    kq = 8 * (kc_lane_group(lane) & 3);
    dh = a.dh;
    // offsets count from the tile's first row: operands of any number of rows
    ra = make_rsrc(a.A + t.c * a.a_cs + t.side * a.a_ss + (int64_t)t.m0 * a.ld);
    rb = make_rsrc(a.B + t.c * a.b_cs + t.side * a.b_ss + (t.nrow0 + t.n0) * a.ld);
#pragma unroll
    for (int j = 0; j < 4; ++j) oa[j] = kc_offset(w + 2 * WR * j, a.ld, 0, t.M - t.m0, lane);
#pragma unroll
    for (int j = 0; j < NB; ++j) ob[j] = kc_offset(w + 2 * WR * j, a.ld, 0, t.N - t.n0, lane);
  }
  __device__ __forceinline__ void none() {
#pragma unroll
    for (int j = 0; j < 4; ++j) oa[j] = kOob;
#pragma unroll
    for (int j = 0; j < NB; ++j) ob[j] = kOob;
  }
  __device__ __forceinline__ void slice(ScoreSmem<WR>& sm, int stage, int kt) const {
    // the last slice may reach past the rows' elements
    const bool off = kt * BK + kq >= dh;
#pragma unroll
    for (int j = 0; j < 4; ++j) dma16(ra, sm.A[stage] + (w + 2 * WR * j) * 512, off ? kOob : oa[j], 128 * kt);
#pragma unroll
    for (int j = 0; j < NB; ++j) dma16(rb, sm.B[stage] + (w + 2 * WR * j) * 512, off ? kOob : ob[j], 128 * kt);
  }
};

struct Frags {
  v8h a[2][4], b[2][4];
};

template <int WR>
__device__ __forceinline__ void read_frags(const ScoreSmem<WR>& sm, int stage, const int (&fa)[2], const int (&fb)[2],
                                           Frags& f) {
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f.a[p][i] = *(const v8h*)(sm.A[stage] + fa[p] + 16 * 64 * i);
      f.b[p][i] = *(const v8h*)(sm.B[stage] + fb[p] + 16 * 64 * i);
    }
}

// acc += a slice (l h', h l', h h' of the row pairs, the small products first) while the next slice's
// fragments are read and the slice two further on is fetched, a read or a
// fetch between every two products.  (Issued together at the
// slice's start, the reads and fetches of all waves kept the LDS and the
// address unit busy for 1,000 cycles before the first product: 2,550 cycles a
// slice, 1,536 of them products.)
template <int WR>
__device__ __forceinline__ void multiply(const Frags& f, v4f (&acc)[4][4], ScoreSmem<WR>& sm, int stage,
                                         const int (&fa)[2], const int (&fb)[2], Frags& next,
                                         const SliceLoader<WR>& ld, int lstage, int lkt) {
  read_frags<WR>(sm, stage, fa, fb, next);
  ld.slice(sm, lstage, lkt);
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(f.a[q == 0][i], f.b[q == 1][j], acc[i][j], 0, 0, 0);
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);   // matrix instructions
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // an LDS read
  }
#pragma unroll
  for (int k = 0; k < SliceLoader<WR>::PER_SLICE; ++k) {
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // a fetch
  }
}

// -inf in the accumulators past the batch's rows and columns and on the masked
// diagonal (no threshold is below it)
__device__ __forceinline__ void mask_tile(const ScoreTile& t, v4f (&acc)[4][4], int wm, int wn, int lane) {
  const int l16 = lane & 15, g = lane >> 4;
  const int nd = t.nrow0 == 0 ? t.n0 : -0x40000000;   // side 1's uniform candidates have no diagonal
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int n = 64 * wn + 16 * j + l16;
    const bool off = t.n0 + n >= t.N;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = t.m0 + 64 * wm + 16 * i + 4 * g + r;
        if (off || nd + n == m || m >= t.M) acc[i][j][r] = -INFINITY;
      }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// lane (i, j, r)'s words of a wave's block of hits: its place in a bit plane,
// and the hits of row 16 (l16 / 4) + 4 g + l16 % 4 over the 64 columns
__device__ __forceinline__ int64_t hit_words(const ScoreArgs& a, const ScoreTile& t, int wm, int wn, int lane) {
  const int rb = ((t.m0 + 64 * wm) >> 4) + (lane >> 4), cb = ((t.n0 + 64 * wn) >> 4) + ((lane >> 2) & 3);
  return ((int64_t)cb * a.RB + rb) * 8 + (lane & 3);
}
__device__ __forceinline__ uint32_t row_hits(uint32_t wlo, uint32_t whi, int lane) {
  const int l16 = lane & 15, g = lane >> 4;
  // the four fields of the lane, then over the four j
  uint32_t n4 = __builtin_popcount(wlo & 0xFFFFu) | (__builtin_popcount(wlo >> 16) << 8) |
                (__builtin_popcount(whi & 0xFFFFu) << 16) | (__builtin_popcount(whi >> 16) << 24);
  n4 += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)n4, 0x124, 0xF, 0xF, false);   // row_ror:4
  n4 += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)n4, 0x128, 0xF, 0xF, false);   // row_ror:8
  const uint32_t n = (uint32_t)__shfl((int)n4, 16 * (l16 >> 2) + (l16 & 3), PBG_WAVE);
  return (n >> (8 * g)) & 0xFFu;
}

// Ranking loss of a tile: hit = [s > -(margin - p + bias)].  The ballot of an
// accumulator register holds 16 columns of four rows; the 64 ballots of the
// wave's block are deposited one per lane and stored as two 4-byte words a
// lane: 16 x 16 blocks of eight words, [half][r], whose 16-bit fields are rows
// 8 half + r and 8 half + 4 + r (BitsView in kernels.h).  SHARED: the tile is
// also the transposed tile of side 1 (rows n, columns m): its hits go to the
// second plane in the same place, its row sums are this tile's column sums.
// Row partials (hinge sum, hits) are written per 64 columns, each wave its own.
// Elements that count for neither hold -inf (mask_tile).
template <bool SHARED, bool SCALED, int WR>
__device__ __forceinline__ void bits_epilogue(const ScoreArgs& a, const ScoreTile& t, v4f (&acc)[4][4],
                                              ScoreSmem<WR>& sm, int wm, int wn, int lane) {
  const int l16 = lane & 15, g = lane >> 4;
  uint32_t wlo = 0, whi = 0, xlo = 0, xhi = 0;
  float mine = 0.0f;   // row sum of row 16 (l16 / 4) + 4 g + l16 % 4
  float ls1[4] = {0.f, 0.f, 0.f, 0.f};
  uint32_t c1[4] = {0u, 0u, 0u, 0u};
  float nthr1[4], cscl[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (SHARED) nthr1[j] = sm.nthr1[64 * wn + 16 * j + l16];
    if (SCALED) cscl[j] = sm.cscl[64 * wn + 16 * j + l16];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int mb = 64 * wm + 16 * i + 4 * g;
    const v4f nthr = *(const v4f*)&sm.nthr[mb];
    float ls[4] = {-0.0f, -0.0f, -0.0f, -0.0f};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      // four ballots before their uses, in scalar registers of their own: an
      // instruction that reads one right behind the compare would wait
      float s[4];
      uint64_t mk[4], mk1[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[r] = SCALED ? acc[i][j][r] * cscl[j] : acc[i][j][r];
        mk[r] = __ballot(s[r] > nthr[r]);
        if (SHARED) mk1[r] = __ballot(s[r] > nthr1[j]);
      }
      __asm__ volatile("" : "+s"(mk[0]), "+s"(mk[1]), "+s"(mk[2]), "+s"(mk[3]));
      if (SHARED) __asm__ volatile("" : "+s"(mk1[0]), "+s"(mk1[1]), "+s"(mk1[2]), "+s"(mk1[3]));
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int idx = (i * 4 + j) * 4 + r;
        wlo = writelane((uint32_t)mk[r], idx, wlo);
        whi = writelane((uint32_t)(mk[r] >> 32), idx, whi);
        ls[r] += __builtin_amdgcn_inverse_ballot_w64(mk[r]) ? s[r] : 0.0f;
        if (SHARED) {
          const bool hit1 = __builtin_amdgcn_inverse_ballot_w64(mk1[r]);
          xlo = writelane((uint32_t)mk1[r], idx, xlo);
          xhi = writelane((uint32_t)(mk1[r] >> 32), idx, xhi);
          ls1[j] += hit1 ? s[r] : 0.0f;
          c1[j] += hit1 ? 1u : 0u;
        }
      }
      // the sums are taken here and not after the loop, so that the ballots of
      // only a few registers are live at a time (scalar registers)
      __asm__ volatile("" : "+v"(ls[0]), "+v"(ls[1]), "+v"(ls[2]), "+v"(ls[3]));
      if (SHARED) __asm__ volatile("" : "+v"(ls1[j]), "+v"(c1[j]));
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float s = group16_sum(ls[r]);
      mine = l16 == 4 * i + r ? s : mine;   // every lane of the group holds the row's sum
    }
  }
  {
    const int64_t at = hit_words(a, t, wm, wn, lane);
    uint32_t* d = a.bits0 + t.c * a.bits_cs + t.side * a.bits_ss + at;
    d[0] = wlo;
    d[4] = whi;
    if (SHARED) {
      uint32_t* d1 = a.bits1 + t.c * a.bits1_cs + at;
      d1[0] = xlo;
      d1[4] = xhi;
    }
    const float c = (float)row_hits(wlo, whi, lane);
    const int row = 64 * wm + 16 * (l16 >> 2) + 4 * g + (l16 & 3), m = t.m0 + row;
    const int nb = t.n0 / 64 + wn;   // column block of 64
    if (m < t.M && 64 * nb < t.N) {
      // merged: side 1's in-chunk blocks come first
      const int slot = a.share && t.side == 1 ? (t.Cc + 63) / 64 + nb : nb;
      float2* rp = (float2*)a.rowpart + ((int64_t)(t.c * 2 + t.side) * a.C + m) * a.nct + slot;
      *rp = make_float2(fmaf(sm.thr[row], c, mine * sm.scl[row]), c);
    }
  }
  if (SHARED) {
    float ms = 0.0f, mc = 0.0f;   // lane 16 j + l16: column 16 j + l16
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float s = ls1[j];
      float c = (float)c1[j];
      s += __shfl_xor(s, 16, PBG_WAVE);
      c += __shfl_xor(c, 16, PBG_WAVE);
      s += __shfl_xor(s, 32, PBG_WAVE);
      c += __shfl_xor(c, 32, PBG_WAVE);
      ms = g == j ? s : ms;
      mc = g == j ? c : mc;
    }
    const int n = t.n0 + 64 * wn + lane, mblk = t.m0 / 64 + wm;
    if (n < t.M && 64 * mblk < t.M) {
      float2* rp = (float2*)a.rowpart + ((int64_t)(t.c * 2 + 1) * a.C + n) * a.nct + mblk;
      *rp = make_float2(fmaf(sm.thr1[64 * wn + lane], mc, ms * a.unscale), mc);
    }
  }
}

__device__ __forceinline__ int power_of(float scale) { return (int)(__float_as_uint(scale) >> 23) - 127; }

// Candidates at or above the positive score, [s + bias >= p], as bits (the
// layout of bits_epilogue; columns past N are 0) and their number per row and
// 64 columns.  The scales go through the exponent, exact for rows of any
// magnitude.
template <int WR>
__device__ __forceinline__ void rank_epilogue(const ScoreArgs& a, const ScoreTile& t, v4f (&acc)[4][4],
                                              const ScoreSmem<WR>& sm, int wm, int wn, int lane) {
  const int l16 = lane & 15, g = lane >> 4;
  uint32_t wlo = 0, whi = 0;
  int ce[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) ce[j] = power_of(sm.cscl[64 * wn + 16 * j + l16]);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int mb = 64 * wm + 16 * i + 4 * g;
    const v4f scl = *(const v4f*)&sm.scl[mb];
    const v4f bias = *(const v4f*)&sm.nthr[mb];
    const v4f p = *(const v4f*)&sm.thr[mb];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool in = t.n0 + 64 * wn + 16 * j + l16 < t.N;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float s = ldexpf(acc[i][j][r], ce[j] + power_of(scl[r])) + bias[r];
        uint64_t mk = __ballot(in && s >= p[r]);
        __asm__ volatile("" : "+s"(mk));
        const int idx = (i * 4 + j) * 4 + r;
        wlo = writelane((uint32_t)mk, idx, wlo);
        whi = writelane((uint32_t)(mk >> 32), idx, whi);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  uint32_t* d = a.bits0 + hit_words(a, t, wm, wn, lane);
  d[0] = wlo;
  d[4] = whi;
  const uint32_t c = row_hits(wlo, whi, lane);
  const int m = t.m0 + 64 * wm + 16 * (l16 >> 2) + 4 * g + (l16 & 3), nb = t.n0 / 64 + wn;
  if (64 * nb < t.N) a.hits[(int64_t)nb * (16 * a.RB) + m] = (uint8_t)c;   // rows past M: never read
}

// Logistic: dS = sigmoid(s) / K and the row's losses softplus(s) / K; softmax:
// exp(s - M), M the row's maximum over the block's 64 columns, and (M, row
// sum).  Float32 rows to Cm (zeros off the valid set), row partials per 64
// columns.  Masked elements hold -inf.
template <int EPI, bool SCALED, int WR>
__device__ __forceinline__ void value_epilogue(const ScoreArgs& a, const ScoreTile& t, v4f (&acc)[4][4],
                                               const ScoreSmem<WR>& sm, int wm, int wn, int lane) {
  const int l16 = lane & 15, g = lane >> 4;
  const int Nc = t.Cc + a.U;
  const float kinv = Nc > 1 ? 1.0f / (float)(Nc - 1) : 0.0f;
  float cscl[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) cscl[j] = SCALED ? sm.cscl[64 * wn + 16 * j + l16] : 1.0f;
  float m0 = 0.0f, m1 = 0.0f;   // this lane's row: 16 (l16 / 4) + 4 g + l16 % 4
  float* base = a.Cm + t.c * a.c_cs + t.side * a.c_ss;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int mb = 64 * wm + 16 * i + 4 * g;
    const v4f scl = *(const v4f*)&sm.scl[mb];
    const v4f bias = *(const v4f*)&sm.thr[mb];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = t.m0 + mb + r;
      float s[4], v0 = 0.0f, v1 = 0.0f;
#pragma unroll
      for (int j = 0; j < 4; ++j) s[j] = (SCALED ? acc[i][j][r] * cscl[j] : acc[i][j][r]) * scl[r] + bias[r];
      float* row = base + (int64_t)m * a.ldc;
      if (EPI == EPI_LOSS) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float sg, sp;
          logistic_pair(s[j], sg, sp);
          s[j] = sg * kinv;
          v0 += sp * kinv;
          v1 += s[j];
        }
        v0 = group16_sum(v0);
        v1 = group16_sum(v1);
      } else {
        v0 = group16_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          s[j] = v0 > -INFINITY ? expf(s[j] - v0) : 0.0f;
          v1 += s[j];
        }
        v1 = group16_sum(v1);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = t.n0 + 64 * wn + 16 * j + l16;
        if (m < t.M && n < a.ldc) row[n] = s[j];
      }
      const bool own = l16 == 4 * i + r;
      m0 = own ? v0 : m0;
      m1 = own ? v1 : m1;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  const int m = t.m0 + 64 * wm + 16 * (l16 >> 2) + 4 * g + (l16 & 3), nb = t.n0 / 64 + wn;
  if (m < t.M && 64 * nb < t.N)
    *((float2*)a.rowpart + ((int64_t)(t.c * 2 + t.side) * a.C + m) * a.nct + nb) = make_float2(m0, m1);
}

// EPI_STORE: the scores as float32 rows in Cm
template <bool SHARED, int WR>
__device__ __forceinline__ void store_epilogue(const ScoreArgs& a, const ScoreTile& t, v4f (&acc)[4][4],
                                               const ScoreSmem<WR>& sm, int wm, int wn, int lane) {
  const int l16 = lane & 15, g = lane >> 4;
  float* Cm = a.Cm + t.c * a.c_cs + t.side * a.c_ss;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const v4f scl = *(const v4f*)&sm.scl[64 * wm + 16 * i + 4 * g];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = t.m0 + 64 * wm + 16 * i + 4 * g + r;
      if (m >= t.M) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = t.n0 + 64 * wn + 16 * j + l16;
        const float s = (acc[i][j][r] * sm.cscl[64 * wn + 16 * j + l16]) * scl[r];
        if (n < t.N) Cm[(int64_t)m * a.ldc + t.nrow0 + n] = s;
        if (SHARED && n < t.M) (a.Cm + t.c * a.c_cs + a.c_ss)[(int64_t)n * a.ldc + m] = s;
      }
    }
  }
}

// SCALED: rows with scales of their own (dot); never shared
template <int EPI, bool SCALED, int WR>
__global__ __launch_bounds__(128 * WR, WR / 2) void score_kernel(ScoreArgs a, TileGrid tg) {
  constexpr int BM = 64 * WR;
  __shared__ __align__(16) ScoreSmem<WR> sm;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w >> 1, wn = w & 1;
  const int l16 = lane & 15, g = lane >> 4;
  // an XCD's workgroups (blockIdx.x % 8) walk a contiguous range of tiles
  const int x = blockIdx.x & 7, step = gridDim.x >> 3;
  const int hi = (int)((int64_t)tg.total * (x + 1) / 8);
  const int first = (int)((int64_t)tg.total * x / 8) + (blockIdx.x >> 3);
  auto next_tile = [&](int& id, ScoreTile& t) {
    for (; id < hi; id += step)
      if (score_tile<BM>(a, tg, id, t)) {
        id += step;
        return true;
      }
    return false;
  };
  const int nk = (a.dh + BK - 1) / BK;
  const int fa[2] = {kc_slot(64 * wm + l16, 0, g), kc_slot(64 * wm + l16, 1, g)};
  const int fb[2] = {kc_slot(64 * wn + l16, 0, g), kc_slot(64 * wn + l16, 1, g)};

  // the stream of slices: its tile and k as the loads see them.  Past the last
  // tile the loads go on with offsets that read zeros, so that the number in
  // flight is always the same.
  SliceLoader<WR> ld;
  int lid = first, lkt = 0, lstage = 0;
  {
    ScoreTile t;
    if (!next_tile(lid, t)) return;
    ld.tile(a, t, w, lane);
  }
  auto loaded = [&]() {
    lstage = lstage == STAGES - 1 ? 0 : lstage + 1;
    if (++lkt == nk) {
      lkt = 0;
      ScoreTile t;
      if (next_tile(lid, t)) ld.tile(a, t, w, lane);
      else ld.none();
    }
  };
  ld.slice(sm, lstage, lkt);
  loaded();
  ld.slice(sm, lstage, lkt);
  loaded();
  wait_loads();
  lds_barrier();
  ld.slice(sm, lstage, lkt);
  loaded();
  Frags fr, fr2;
  read_frags<WR>(sm, 0, fa, fb, fr);
  int stage = 1;   // the stage of the next slice's fragments

  ScoreTile cur;
  int id = first;
  while (next_tile(id, cur)) {
    const bool shared = !SCALED && a.share && cur.side == 0 && cur.n0 < cur.M;
    // per-row values in the first half of the threads, per-column ones (side
    // 1's positive scores for shared tiles, the candidates' scales) in the
    // second: loaded here, spread through LDS before the epilogue.  Past the
    // batch: whatever the padded buffers hold.
    const bool col = tid >= BM;
    const int own = col ? tid - BM : tid;
    float p = 0.0f, bias = 0.0f, scl = 1.0f;
    if (EPI == EPI_RANK) p = a.pos[cur.m0 + own % BM];
    if (EPI == EPI_LOSS_BITS)
      p = a.pos[(int64_t)(cur.c * a.pos_sides + (a.pos_sides - 1) * cur.side) * a.C +
                (col ? min(cur.n0, a.C) + (own & (BN - 1)) : cur.m0 + own)];
    if (SCALED)
      scl = col ? a.ib[cur.c * a.ib_cs + cur.side * a.ib_ss + cur.nrow0 + cur.n0 + (own & (BN - 1))]
                : a.ia[cur.c * a.ia_cs + cur.side * a.ia_ss + cur.m0 + own];
    if (SCALED && EPI != EPI_STORE && a.bias && (EPI == EPI_RANK || cur.side == 1))
      bias = a.bias[(int64_t)cur.c * a.C + (col ? 0 : cur.m0 + own)];
    v4f acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
    const float thr = (a.margin - p) + bias;
    // multiplies the slice whose fragments `now` holds while the next one's
    // are read: the next slice has landed for every wave (the one after it may
    // be in flight), and every wave has read the fragments of this one
    auto advance = [&](const Frags& now, Frags& next) {
      __builtin_amdgcn_s_waitcnt(0x0F70 | SliceLoader<WR>::PER_SLICE);
      lds_barrier();
      multiply<WR>(now, acc, sm, stage, fa, fb, next, ld, lstage, lkt);
      loaded();
      stage = stage == STAGES - 1 ? 0 : stage + 1;
    };
    // the per-row and per-column values into LDS, past the first barrier of
    // the tile (every wave has left the last tile's epilogue) and before the
    // last
    auto spread = [&]() {
      if (!col) {
        sm.scl[own] = !SCALED ? a.unscale : (EPI == EPI_RANK ? scl : scl * (1.0f / kColShare));
        if (EPI == EPI_LOSS || EPI == EPI_SOFTMAX_EXP) sm.thr[own] = bias;
        if (EPI == EPI_RANK) {
          sm.thr[own] = p;
          sm.nthr[own] = bias;
        }
        if (EPI == EPI_LOSS_BITS) {   // the scale's inverse is exact: a power of two
          sm.thr[own] = thr;
          sm.nthr[own] = cur.m0 + own < cur.M ? -thr * (SCALED ? __builtin_amdgcn_rcpf(scl) * kColShare : a.iunscale) : INFINITY;
        }
      } else if (own < BN) {
        sm.cscl[own] = cur.n0 + own >= cur.N ? 1.0f   // the masked -inf stay so
                       : (SCALED && EPI != EPI_RANK ? scl * kColShare : scl);
        if (EPI == EPI_LOSS_BITS) {
          sm.thr1[own] = thr;
          sm.nthr1[own] = cur.n0 + own < cur.M ? -thr * a.iunscale : INFINITY;
        }
      }
    };
    // in pairs, so that the two fragment sets swap without being copied
    for (int kt = 0; kt + 1 < nk; kt += 2) {
      advance(fr, fr2);
      if (kt == 0) spread();
      advance(fr2, fr);
    }
    if (nk & 1) {
      advance(fr, fr2);
      if (nk == 1) {
        // rows of at most 32 elements: the rounding of so short a sum does not
        // hide the product of the two low planes, so it is added too
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fr.a[1][i], fr.b[1][j], acc[i][j], 0, 0, 0);
      }
      fr = fr2;
    }
    if (nk == 1) {
      spread();
      lds_barrier();
    }
    if (EPI == EPI_STORE) {
      if (shared) store_epilogue<true, WR>(a, cur, acc, sm, wm, wn, lane);
      else store_epilogue<false, WR>(a, cur, acc, sm, wm, wn, lane);
    } else if (EPI == EPI_RANK) {
      rank_epilogue<WR>(a, cur, acc, sm, wm, wn, lane);
    } else {
      const bool diag = cur.nrow0 == 0 && cur.m0 < cur.n0 + BN && cur.n0 < cur.m0 + BM;
      if (diag || cur.n0 + BN > cur.N || (shared && cur.m0 + BM > cur.M)) mask_tile(cur, acc, wm, wn, lane);
      if (EPI == EPI_LOSS || EPI == EPI_SOFTMAX_EXP) value_epilogue<EPI, SCALED, WR>(a, cur, acc, sm, wm, wn, lane);
      else if (!SCALED && shared) bits_epilogue<true, SCALED, WR>(a, cur, acc, sm, wm, wn, lane);
      else bits_epilogue<false, SCALED, WR>(a, cur, acc, sm, wm, wn, lane);
    }
  }
  wait_loads();   // nothing may land in LDS after the workgroup has left it
}

template <int EPI, bool SCALED, int WR>
void launch_wr(const ScoreArgs& a, int batches, hipStream_t s) {
  const int M = a.Mfix > 0 ? a.Mfix : a.C, N = a.Mfix > 0 ? a.Nfix : a.C + a.U;
  const int tiles_m = (M + 64 * WR - 1) / (64 * WR);
  const int tn0 = (N + BN - 1) / BN;
  const int tn1 = a.nsides < 2 ? 0 : (a.share ? (a.U + BN - 1) / BN : tn0);
  const int64_t total = (int64_t)batches * tiles_m * (tn0 + tn1);
  if (total <= 0) return;
  // one workgroup a CU on 256 CUs, in multiples of the eight XCDs
  const int grid = (int)std::min<int64_t>(256, (total + 7) / 8 * 8);
  auto divider = [](int d) {
    return Divider{(uint32_t)std::max(d, 1), d <= 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d)};
  };
  const TileGrid tg{tiles_m * tn0, (int)total, tiles_m, divider(4 * tn0).m, divider(tiles_m * (tn0 + tn1)), divider(tn0), divider(tn1)};
  score_kernel<EPI, SCALED, WR><<<grid, 128 * WR, 0, s>>>(a, tg);
}

// four waves where no chunk fills more than their 128 rows.  Not by the
// average: relation-grouped chunks of about 70 edges (500 uniform negatives,
// d = 200) took 135 us with 128-row tiles, 100 us with 256-row ones, whose
// eight waves keep twice the loads in flight.
bool few(const ScoreArgs& a) { return (a.Mfix > 0 ? a.Mfix : a.C) <= 128; }

template <int EPI, bool SCALED>
void launch_few(const ScoreArgs& a, int batches, hipStream_t s) {
  few(a) ? launch_wr<EPI, SCALED, 2>(a, batches, s) : launch_wr<EPI, SCALED, 4>(a, batches, s);
}

template <int EPI>
void launch_t(const ScoreArgs& a, int batches, hipStream_t s) {
  if (a.ia) launch_few<EPI, true>(a, batches, s);
  else launch_few<EPI, false>(a, batches, s);
}

}  // namespace

void launch_score(const ScoreArgs& a, int epi, int nchunks, hipStream_t s) {
  if (nchunks <= 0) return;
  if (epi == EPI_LOSS_BITS) launch_t<EPI_LOSS_BITS>(a, nchunks, s);
  else if (epi == EPI_LOSS) launch_t<EPI_LOSS>(a, nchunks, s);
  else if (epi == EPI_SOFTMAX_EXP) launch_t<EPI_SOFTMAX_EXP>(a, nchunks, s);
  else if (epi == EPI_RANK) launch_few<EPI_RANK, true>(a, nchunks, s);
  else launch_t<EPI_STORE>(a, nchunks, s);
}
