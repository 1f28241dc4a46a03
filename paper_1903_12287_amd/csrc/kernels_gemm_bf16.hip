// bfloat16 inputs / float32 accumulation for the three chunk contractions
// (Sec. 4.3 batched negatives; the score block of a chunk is one product).
//
//   forward  S  = Q  . N^T  :  A = Q    [e][f],  B = N   [t][f]
//   dQ       dQ = dS . N    :  A = dS   [e][t],  B = N^T [f][t]
//   dN       dN = dS^T . Q  :  A = dS^T [t][e],  B = Q^T [f][e]
// The B operands are contiguous along k: the bf16 copies of Q and N and their
// transposes are produced once per step (LDS-tiled transpose).  The A operand
// of the backward products is dS itself, read in place: for the ranking loss
// from its bit matrix (rows for dQ, columns for dN), otherwise from bf16 dS
// rows (transposed on the way into LDS for dN), so no copy of dS^T exists.
//
// Layout and schedule follow the float32 kernel: 256-thread workgroups of
// 2 x 2 waves on 128 x BN tiles, buffer loads with hardware zero-fill,
// register prefetch one k-slice ahead, double-buffered LDS tiles and all
// tiles of one batch on one XCD.  A slice is 32 deep, one
// v_mfma_f32_16x16x32_bf16 step: lane L feeds A[L % 16][8 (L / 16) + i] and
// B[8 (L / 16) + i][L % 16], i = 0..7, one 16-byte LDS read each; the
// accumulator holds D[4 (L / 16) + r][L % 16] in register r.
// LDS tiles are [row][k], 32 bf16 (64 bytes) per row with no padding: the
// 16-byte group q of row x is kept at group q ^ (((x >> 1) ^ ((x >> 3) & 1)) & 3),
// which repeats every 16 rows.
// A fragment read (16 consecutive rows, one group each) then touches every
// 16-byte bank group once, whether the LDS serves 16 lanes over 64 banks or
// 8 lanes over 32 banks per cycle, and so do the tile stores (four groups of
// consecutive rows).
#include <algorithm>

#include "kernels.h"
#include "device_common.h"

namespace {

constexpr int BM = 128;
constexpr int BK = 32;          // k per slice = bf16 elements per LDS tile row
constexpr uint32_t OOB = 0x80000000u;

typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A buffer descriptor must be wave-uniform.  Tile base addresses are, but
// their 64-bit products are formed on the vector unit, and a descriptor left
// in vector registers would make the compiler wrap every load that uses it in
// a loop over lanes; reading the address back from the first lane keeps it
// scalar.
__device__ __forceinline__ rsrc_t make_rsrc(const void* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), (short)0, 0x7FFFFFF0, 0x00020000);
}
__device__ __forceinline__ u32x4 bload16(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
}

__device__ __forceinline__ float bf16_to_f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint16_t f_to_bf16(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

// two floats -> one packed bf16 pair (a in the low half), round to nearest even
__device__ __forceinline__ uint32_t f2_to_bf16x2(float a, float b) {
  return __builtin_bit_cast(uint32_t, (bf16x2_t){(__bf16)a, (__bf16)b});
}

__device__ __forceinline__ int pick_dim(int sel, int fixed, int Cc, int Nc) {
  return sel == DIM_CC ? Cc : (sel == DIM_NC ? Nc : fixed);
}

// element offset of the 16-byte group q of row x in a swizzled LDS tile
__device__ __forceinline__ int swz(int x, int q) {
  return x * BK + ((q ^ (((x >> 1) ^ ((x >> 3) & 1)) & 3)) << 3);
}

// two bits t (0..3) -> the packed bf16 pair (bit 0 low, bit 1 high) of 0.0 / 1.0:
// t * 0x8001 puts bit 0 at bit 0 and bit 1 at bit 16, and 0x3F80 is 1.0
__device__ __forceinline__ uint32_t bit_pair(uint32_t t) { return ((t * 0x8001u) & 0x10001u) * 0x3F80u; }

// One operand tile of TX rows x BK k as LDS [row][k] bf16 (swizzled); each
// thread moves TX * BK / 8 / 256 groups of eight elements per slice.  Loaded
// words stay raw in registers until the store, after the slice's matrix work.
//   GA_KC        global [x][k] bf16, ld elements, k contiguous (zero-padded to 8)
//   GA_MC        global [k][x] bf16, x contiguous: eight x of one k go to eight
//                tile rows
//   GA_BITS_ROW  bit matrix (dsb layout), tile row x = matrix row, k = column
//   GA_BITS_COL  bit matrix, tile row x = matrix column, k = matrix row; the
//                words of eight consecutive rows of one word column are 16
//                contiguous bytes (row pitch a multiple of 8)
template <int TX, int MODE>
struct TileH {
  static constexpr int LOADS = TX * BK / 8 / 256;
  static constexpr int SIZE = TX * BK;

  // offsets of rows count from the tile's (GA_KC) or the slice's (GA_MC) first
  // row: dS may hold more than 4 GiB
  __device__ __forceinline__ static void load(u32x4* r, const uint16_t* p, int ld, int x0, int xdim, int k0, int kdim,
                                              int tid) {
    const rsrc_t rs = make_rsrc(p + (MODE == GA_KC ? (int64_t)x0 * ld : (MODE == GA_MC ? (int64_t)k0 * ld : 0)));
#pragma unroll
    for (int q = 0; q < LOADS; ++q) {
      const int f = tid + 256 * q;
      uint32_t off = OOB;
      if (MODE == GA_MC) {
        const int k = f / (TX / 8), xq = f % (TX / 8);
        const int gk = k0 + k, gx = x0 + 8 * xq;
        if (gk < kdim && gx < ((xdim + 7) & ~7)) off = (uint32_t)((k * ld + gx) * 2);
        r[q] = bload16(rs, off);
      } else {
        const int x = f >> 2, kq = f & 3;
        const int gx = x0 + x, gk = k0 + 8 * kq;
        if (MODE == GA_KC) {
          if (gx < xdim && gk < ((kdim + 7) & ~7)) off = (uint32_t)((x * ld + gk) * 2);
          r[q] = bload16(rs, off);
        } else if (MODE == GA_BITS_ROW) {
          if (gx < xdim && gk < ((kdim + 7) & ~7)) off = (uint32_t)(((int64_t)(gk >> 4) * ld + gx) * 2);
          const uint32_t w = __builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0);
          r[q] = (u32x4){w, 0u, 0u, 0u};
        } else {
          if (gx < ((xdim + 7) & ~7) && gk < kdim) off = (uint32_t)(((int64_t)(gx >> 4) * ld + gk) * 2);
          r[q] = bload16(rs, off);
        }
      }
    }
  }

  __device__ __forceinline__ static void store(uint16_t* s, const u32x4* r, int tid, int x0, int k0, int kdim) {
#pragma unroll
    for (int q = 0; q < LOADS; ++q) {
      const int f = tid + 256 * q;
      if (MODE == GA_MC) {
        const int k = f / (TX / 8), xq = f % (TX / 8);
        const u32x4 v = r[q];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int x = 8 * xq + i;
          s[swz(x, k >> 3) + (k & 7)] = (uint16_t)((i & 1) ? (v[i >> 1] >> 16) : (v[i >> 1] & 0xFFFFu));
        }
      } else {
        const int x = f >> 2, kq = f & 3;
        u32x4 v = r[q];
        if (MODE == GA_BITS_ROW) {
          // bits of columns k0 + 8 kq + 0..7 -> four packed bf16 pairs
          const uint32_t bits = v.x >> ((8 * kq) & 15);
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = bit_pair(__builtin_amdgcn_ubfe(bits, 2 * i, 2));
        } else if (MODE == GA_BITS_COL) {
          // bit b of the words of rows gk .. gk + 7 (two rows per dword)
          const int b = (x0 + x) & 15;
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = ((v[i] >> b) & 0x00010001u) * 0x3F80u;
          const int nv = kdim - (k0 + 8 * kq);   // rows from nv on lie outside the chunk
          if (nv < 8) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] &= (2 * i + 1 < nv) ? 0xFFFFFFFFu : (2 * i < nv ? 0xFFFFu : 0u);
          }
        }
        *(u32x4*)(s + swz(x, kq)) = v;
      }
    }
  }
};

// LDS of one workgroup: the A and B tiles (two buffers), row partials
template <int BN>
struct SmemH {
  uint16_t As[2][BM * BK];
  uint16_t Bs[2][BN * BK];
  float red[2][BM][2];
  float rowv[2][BM];
};

// Position of a workgroup's TM x BN tile (TM = 128 rows unless stated): `id` numbers the workgroup among
// the nwg of its product (hardware order) and is remapped so that all tiles of
// one batch (chunk, side) run on one XCD.
struct TileGeo {
  int c, side, Nc, M, N, K, m0, n0, tn;
};

// false: nothing to compute (the tile lies beyond this batch's rows, or beyond
// its columns, where a loss epilogue still leaves neutral row partials)
template <int BN, int EPI, int TM = BM>
__device__ __forceinline__ bool tile_geo(const GemmArgsH& a, int tiles_n, int tiles_m, int nwg, int id,
                                         TileGeo& t) {
  const int q8 = nwg >> 3, r8 = nwg & 7, xcd = id & 7;
  const int lid = xcd * q8 + min(xcd, r8) + (id >> 3);
  t.tn = lid % tiles_n;
  const int rest = lid / tiles_n;
  const int tm = rest % tiles_m;
  const int z = rest / tiles_m;
  t.c = z / a.nsides;
  t.side = z - t.c * a.nsides;
  int Cc = a.C;
  t.Nc = a.C + a.U;
  if (a.cstart) {
    Cc = wave_uniform(a.cstart[t.c + 1] - a.cstart[t.c]);
    t.Nc = Cc + a.U;
  } else if (a.m_step > 0) {
    Cc = min(a.C, a.m_step - t.c * a.C);
    t.Nc = Cc + a.U;
  }
  t.M = pick_dim(a.mdim, a.Mfix, Cc, t.Nc);
  t.N = pick_dim(a.ndim, a.Nfix, Cc, t.Nc);
  t.K = pick_dim(a.kdim, a.Kfix, Cc, t.Nc);
  t.m0 = tm * TM;
  t.n0 = t.tn * BN;
  if (t.m0 >= t.M) return false;
  if (t.n0 >= t.N) {
    const int tid = threadIdx.x;
    if (EPI != EPI_STORE && tid < TM && t.m0 + tid < t.M) {
      float* rp = a.rowpart + (((int64_t)(t.c * 2 + t.side) * a.C + t.m0 + tid) * a.nct + t.tn) * 2;
      rp[0] = EPI == EPI_SOFTMAX_STATS ? -INFINITY : 0.0f;
      rp[1] = 0.0f;
    }
    return false;
  }
  return true;
}

// per-row values of the tile for the loss epilogues, read once at the start
// of the tile while its first operands load: the hinge threshold
// margin - p + bias (-inf for rows past the batch) for the ranking bits, else
// the positive score p and the bias
template <int EPI, int TM = BM>
__device__ __forceinline__ void load_rowv(const GemmArgsH& a, const TileGeo& t, float (&rowv)[2][TM]) {
  const int tid = threadIdx.x;
  if (tid < TM) {
    const int m = t.m0 + tid;
    const bool mrow = m < t.M;
    const int64_t o = (int64_t)t.c * a.C + m;
    // row of pos: chunk c (pos_sides = 1), or chunk c and side (pos_sides = 2);
    // arithmetic rather than a select keeps the tile loop free of spills
    const int64_t op = (int64_t)(t.c * a.pos_sides + (a.pos_sides - 1) * t.side) * a.C + m;
    const float p = mrow ? a.pos[op] : 0.0f;
    const float bm = (mrow && a.bias && t.side == 1) ? a.bias[o] : 0.0f;
    if (EPI == EPI_LOSS_BITS) {
      rowv[0][tid] = mrow ? a.margin - p + bm : -INFINITY;
    } else {
      rowv[0][tid] = p;
      rowv[1][tid] = bm;
    }
  }
}

// Ranking loss rows of a tile (MASKED: the tile holds columns past the batch
// or the masked diagonal).  Hinge z = s + margin - p, dS = [z > 0]; each lane
// group's ballot word is the bit-matrix word of its row for these 16 columns
// and its population count that row's share of the dS row sum.
template <int BN, bool MASKED, int TM = BM>
__device__ __forceinline__ void bits_rows(const GemmArgsH& a, const TileGeo& t, v4f (&acc)[TM / 32][BN / 32],
                                          float (&red)[2][TM][2], const float (&rowv)[2][TM]) {
  constexpr int WN = BN / 2, WMR = TM / 2;
  constexpr int JN = WN / 16, IM = TM / 32;
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int wm = w >> 1, wn = w & 1;
  const int l16 = lane & 15, g = lane >> 4;
  const int colb = t.n0 + WN * wn + l16;
  const int wcol0 = (t.n0 + WN * wn) >> 4;
  // the words of four consecutive rows are adjacent (word-column major)
  uint16_t* dbase = a.dsb + t.c * a.cb_cs + t.side * a.cb_ss + (int64_t)wcol0 * a.ldcb + t.m0 + WMR * wm + 4 * g;
#pragma unroll
  for (int i = 0; i < IM; ++i) {
    const int mb = WMR * wm + 16 * i + 4 * g;   // first of this lane group's four rows
    const v4f thr = *(const v4f*)&rowv[0][mb];
    float ls[4] = {-0.0f, -0.0f, -0.0f, -0.0f};   // -0 + x is x: the first add folds away
    uint32_t cnt[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < JN; ++j) {
      uint32_t wd[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        // s + thr > 0 exactly when s > -thr (an IEEE sum is positive exactly
        // when the exact sum is), so the compare needs no add; the hinge sum
        // of the row is the sum of its selected scores plus thr per bit
        const float s = acc[i][j][r];
        bool hit = s > -thr[r];
        if (MASKED) {
          const int n = colb + 16 * j;
          if (n >= t.N || n == t.m0 + mb + r) hit = false;
        }
        const uint64_t mk = __ballot(hit);
        ls[r] += hit ? s : 0.0f;   // one select on the compare already made
        wd[r] = (uint32_t)(mk >> (16 * g)) & 0xFFFFu;
        cnt[r] += __builtin_popcount(wd[r]);
      }
      if (l16 == 0 && t.m0 + mb < t.M && wcol0 + j < a.nwcb)
        *(uint2*)(dbase + (int64_t)j * a.ldcb + 16 * i) = make_uint2(wd[0] | (wd[1] << 16), wd[2] | (wd[3] << 16));
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v0 = group16_sum(ls[r]);
      if (l16 == 0) {
        red[wn][mb + r][0] = fmaf(thr[r], (float)cnt[r], v0);   // rows past the batch: unused
        red[wn][mb + r][1] = (float)cnt[r];
      }
    }
  }
}

// logistic loss (dS rows in bf16 or float32) and softmax statistics (raw
// scores + per-tile max and sum of exp) rows of a tile
template <int BN, int EPI, bool MASKED, int TM = BM>
__device__ __forceinline__ void value_rows(const GemmArgsH& a, const TileGeo& t, v4f (&acc)[TM / 32][BN / 32],
                                           float (&red)[2][TM][2], const float (&rowv)[2][TM]) {
  constexpr int WN = BN / 2, WMR = TM / 2;
  constexpr int JN = WN / 16, IM = TM / 32;
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int wm = w >> 1, wn = w & 1;
  const int l16 = lane & 15, g = lane >> 4;
  const int c = t.c, side = t.side, M = t.M, N = t.N, m0 = t.m0;
  const int colb = t.n0 + WN * wn + l16;
  const float kinv = (t.Nc - 1 > 0) ? 1.0f / (float)(t.Nc - 1) : 0.0f;
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ml = WMR * wm + 16 * i + 4 * g + r;
      const int m = m0 + ml;
      const bool mrow = m < M;
      const float p = rowv[0][ml];
      const float bm = rowv[1][ml];
      const int64_t orow = c * a.c_cs + side * a.c_ss + (int64_t)m * a.ldc;
      float v0, v1;
      if (EPI == EPI_LOSS) {
        float lsum = 0.0f, dsum = 0.0f;
#pragma unroll
        for (int j = 0; j < JN; ++j) {
          const int n = colb + 16 * j;
          const float s = acc[i][j][r] + bm;
          const bool valid = mrow && !(MASKED && (n >= N || n == m));
          float dsv = 0.0f;
          if (valid) {
            if (a.loss == LOSS_RANKING) {
              const float zz = a.margin - p + s;
              if (zz > 0.0f) {
                dsv = 1.0f;
                lsum += zz;
              }
            } else {
              float sg, sp;
              logistic_pair(s, sg, sp);
              dsv = sg * kinv;
              lsum += sp * kinv;
            }
          }
          dsum += dsv;
          if (mrow && n < a.ldc) {
            if (a.dsh) a.dsh[orow + n] = f_to_bf16(dsv);
            else a.Cm[orow + n] = dsv;
          }
        }
        v0 = group16_sum(lsum);
        v1 = group16_sum(dsum);
      } else {  // EPI_SOFTMAX_STATS
        float mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < JN; ++j) {
          const int n = colb + 16 * j;
          const float s = acc[i][j][r] + bm;
          if (mrow && !(MASKED && (n >= N || n == m))) mx = fmaxf(mx, s);
          if (mrow && n < a.ldc) a.Cm[orow + n] = s;
        }
        mx = group16_max(mx);
        float se = 0.0f;
#pragma unroll
        for (int j = 0; j < JN; ++j) {
          const int n = colb + 16 * j;
          if (mrow && !(MASKED && (n >= N || n == m))) se += expf(acc[i][j][r] + bm - mx);
        }
        v0 = mx;
        v1 = group16_sum(se);
      }
      if (l16 == 0) {
        red[wn][ml][0] = v0;
        red[wn][ml][1] = v1;
      }
    }
}

// Stores the tile (EPI_STORE) or runs the loss epilogue on it: dS leaves as
// bits (ranking), as bf16 rows (logistic, when dsh is set) or float32 rows in
// Cm, or the raw float32 scores go to Cm for the softmax row pass; row
// partials (loss, dS sum / max, sum exp) are combined over the tile's two
// column halves and written per column tile.
template <int BN, int EPI, int TM = BM>
__device__ __forceinline__ void tile_epilogue(const GemmArgsH& a, const TileGeo& t, v4f (&acc)[TM / 32][BN / 32],
                                              float (&red)[2][TM][2], const float (&rowv)[2][TM]) {
  constexpr int WN = BN / 2, WMR = TM / 2;
  constexpr int JN = WN / 16, IM = TM / 32;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = tid >> 6;
  const int wm = w >> 1, wn = w & 1;
  const int l16 = lane & 15, g = lane >> 4;
  const int c = t.c, side = t.side, M = t.M, N = t.N, Nc = t.Nc, m0 = t.m0, n0 = t.n0;
  const int colb = n0 + WN * wn + l16;
  if (EPI == EPI_STORE) {
    float* Cm = a.Cm + c * a.c_cs + side * a.c_ss;
    // the chunk's weight (1 without weights: the product is exact), read once
    // into a scalar register
    const float sc = a.cscale ? wave_uniform(a.cscale[c]) : 1.0f;
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + WMR * wm + 16 * i + 4 * g + r;
        if (m < M) {
#pragma unroll
          for (int j = 0; j < JN; ++j) {
            const int n = colb + 16 * j;
            if (n < N) Cm[(int64_t)m * a.ldc + n] = acc[i][j][r] * sc;
          }
        }
      }
    return;
  }

  // column tiles past the batch's last column and tiles that meet the masked
  // diagonal need per-element checks
  const bool masked = (n0 + BN > N) || (m0 < n0 + BN && n0 < m0 + TM);
  if (EPI == EPI_LOSS_BITS) {
    if (masked) bits_rows<BN, true, TM>(a, t, acc, red, rowv);
    else bits_rows<BN, false, TM>(a, t, acc, red, rowv);
  } else {
    if (masked) value_rows<BN, EPI, true, TM>(a, t, acc, red, rowv);
    else value_rows<BN, EPI, false, TM>(a, t, acc, red, rowv);
  }
  __syncthreads();
  if (tid < TM && m0 + tid < M) {
    const int ml = tid;
    float v0, v1;
    if (EPI == EPI_LOSS || EPI == EPI_LOSS_BITS) {
      v0 = red[0][ml][0] + red[1][ml][0];
      v1 = red[0][ml][1] + red[1][ml][1];
    } else {
      const float ma = red[0][ml][0], mb = red[1][ml][0];
      const float mx = fmaxf(ma, mb);
      v0 = mx;
      v1 = (mx == -INFINITY) ? 0.0f
                             : (ma == -INFINITY ? 0.0f : red[0][ml][1] * expf(ma - mx)) +
                                   (mb == -INFINITY ? 0.0f : red[1][ml][1] * expf(mb - mx));
    }
    float* rp = a.rowpart + (((int64_t)(c * 2 + side) * a.C + m0 + ml) * a.nct + t.tn) * 2;
    rp[0] = v0;
    rp[1] = v1;
  }
}


// One 128 x BN output tile of A . B with bf16 operands.
template <int BN, int AMODE, int EPI>
__device__ __forceinline__ void gemm_bf16_tile(const GemmArgsH& a, int tiles_n, int tiles_m, int nwg, int id,
                                               SmemH<BN>& sm) {
  constexpr int WN = BN / 2;
  constexpr int JN = WN / 16;
  using TA = TileH<BM, AMODE>;
  using TB = TileH<BN, GA_KC>;
  auto& As = sm.As;
  auto& Bs = sm.Bs;
  TileGeo t;
  if (!tile_geo<BN, EPI>(a, tiles_n, tiles_m, nwg, id, t)) return;
  if (EPI != EPI_STORE) load_rowv<EPI>(a, t, sm.rowv);
  const int c = t.c, side = t.side, M = t.M, N = t.N, K = t.K, m0 = t.m0, n0 = t.n0;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = tid >> 6;
  const int wm = w >> 1, wn = w & 1;
  const int l16 = lane & 15, g = lane >> 4;

  const uint16_t* ra_s = a.A + c * a.a_cs + side * a.a_ss;
  const uint16_t* rb = a.B + c * a.b_cs + side * a.b_ss;

  v4f acc[4][JN];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};

  u32x4 pa[TA::LOADS], pb[TB::LOADS];
  const int nk = (K + BK - 1) / BK;
  TA::load(pa, ra_s, a.lda, m0, M, 0, K, tid);
  TB::load(pb, rb, a.ldb, n0, N, 0, K, tid);
  TA::store(As[0], pa, tid, m0, 0, K);
  TB::store(Bs[0], pb, tid, n0, 0, K);
  __syncthreads();

  // fragment offsets: row 16 i + l16 of the wave's block, group g (the
  // swizzle repeats every 16 rows)
  const int fa0 = swz(64 * wm + l16, g), fb0 = swz(WN * wn + l16, g);
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) {
      TA::load(pa, ra_s, a.lda, m0, M, (kt + 1) * BK, K, tid);
      TB::load(pb, rb, a.ldb, n0, N, (kt + 1) * BK, K, tid);
    }
    const uint16_t* as = As[buf];
    v8bf af[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) af[i] = *(const v8bf*)(as + fa0 + 16 * i * BK);
    v8bf bf[JN];
#pragma unroll
    for (int j = 0; j < JN; ++j) bf[j] = *(const v8bf*)(Bs[buf] + fb0 + 16 * j * BK);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
    if (kt + 1 < nk) {
      const int nbuf = buf ^ 1;
      TA::store(As[nbuf], pa, tid, m0, (kt + 1) * BK, K);
      TB::store(Bs[nbuf], pb, tid, n0, (kt + 1) * BK, K);
    }
    __syncthreads();
  }

  tile_epilogue<BN, EPI>(a, t, acc, sm.red, sm.rowv);
}

template <int BN, int AMODE, int EPI>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmArgsH a, int tiles_n, int tiles_m) {
  __shared__ __align__(16) SmemH<BN> sm;
  gemm_bf16_tile<BN, AMODE, EPI>(a, tiles_n, tiles_m, gridDim.x, blockIdx.x, sm);
}

// two independent products in one launch (dQ and dN of a step): workgroups
// [0, nwg0) take the first, the rest the second, so that the long-k tiles of
// the first start first and the short ones of the second fill in behind them
template <int BN, int AM0, int AM1>
__global__ __launch_bounds__(256) void gemm_bf16_pair_kernel(GemmArgsH a0, int tn0, int tm0, int nwg0,
                                                             GemmArgsH a1, int tn1, int tm1) {
  __shared__ __align__(16) SmemH<BN> sm;
  const int id = blockIdx.x;
  if (id < nwg0) gemm_bf16_tile<BN, AM0, EPI_STORE>(a0, tn0, tm0, nwg0, id, sm);
  else gemm_bf16_tile<BN, AM1, EPI_STORE>(a1, tn1, tm1, (int)gridDim.x - nwg0, id - nwg0, sm);
}

// fp32 rows [rows][ld_src] (columns [d, ld_src) zero) of Q and of N -> bf16
// rows [rows][ld_dst] (columns up to kp) and the transposed copy [kp][ld_T]
// (rows [rows, ld_T) zero), both operands in one launch (blockIdx.z < nz0:
// the first).  64 x 64 tiles: 16-byte loads, rounded once, eight bytes per
// thread to the row-major copy and into an LDS tile, then eight consecutive
// rows of one column per 16-byte store of the transposed copy.  ld_src is a
// multiple of 4, ld_dst of 4, ld_T of 8.
struct Bf16T {
  const float* src;
  int64_t src_bs;
  int rows, ld_src;
  uint16_t* dst;
  int64_t dst_bs;
  int ld_dst;
  uint16_t* dstT;
  int64_t dstT_bs;
  int ld_T;
};

__global__ __launch_bounds__(256) void to_bf16_t_kernel(Bf16T o0, Bf16T o1, int nz0, int kp) {
  __shared__ uint16_t tile[64][72];
  const bool first = (int)blockIdx.z < nz0;
  const Bf16T& o = first ? o0 : o1;
  const int b = first ? blockIdx.z : blockIdx.z - nz0;
  const int r0 = blockIdx.y * 64, k0 = blockIdx.x * 64;
  if (r0 >= o.ld_T) return;
  const float* s = o.src + (int64_t)b * o.src_bs;
  uint16_t* dr = o.dst + (int64_t)b * o.dst_bs;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int it = threadIdx.x + 256 * j;
    const int rr = it >> 4, k4 = 4 * (it & 15);
    const int r = r0 + rr, k = k0 + k4;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (r < o.rows && k < o.ld_src) v = *(const float4*)(s + (int64_t)r * o.ld_src + k);
    const uint32_t lo = f2_to_bf16x2(v.x, v.y), hi = f2_to_bf16x2(v.z, v.w);
    *(uint2*)&tile[rr][k4] = make_uint2(lo, hi);
    if (r < o.rows && k < kp) *(uint2*)(dr + (int64_t)r * o.ld_dst + k) = make_uint2(lo, hi);
  }
  __syncthreads();
  uint16_t* dT = o.dstT + (int64_t)b * o.dstT_bs;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int it = threadIdx.x + 256 * j;
    const int kk = it >> 3, r8 = 8 * (it & 7);
    const int k = k0 + kk, r = r0 + r8;
    if (k >= kp || r >= o.ld_T) continue;
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = (uint32_t)tile[r8 + 2 * i][kk] | ((uint32_t)tile[r8 + 2 * i + 1][kk] << 16);
    *(u32x4*)(dT + (int64_t)k * o.ld_T + r) = (u32x4){w[0], w[1], w[2], w[3]};
  }
}

// softmax row pass in bf16 mode: raw fp32 scores -> dS = softmax (masked),
// written as bf16 rows
__global__ __launch_bounds__(256) void softmax_rows_bf16_kernel(StepGeom g, const float* S, const float* rowpart,
                                                                const float* pos, uint16_t* dsh, int ldh) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int z = blockIdx.y;
  const int c = z >> 1;
  const int Cc = chunk_edges(g, c);
  if (row >= Cc) return;
  const int Nc = Cc + g.U;
  const float p = pos[pos_index(g, c, z & 1, row)];
  const float* rp = rowpart + ((int64_t)z * g.C + row) * g.nct * 2;
  float Mx = p;
  for (int ct = 0; ct < g.nct; ++ct) Mx = fmaxf(Mx, rp[2 * ct]);
  float Z = expf(p - Mx);
  for (int ct = 0; ct < g.nct; ++ct) {
    const float mx = rp[2 * ct];
    if (mx > -INFINITY) Z += rp[2 * ct + 1] * expf(mx - Mx);
  }
  const float lse = Mx + logf(Z);
  const float* srow = S + ((int64_t)z * g.C + row) * g.Np;
  uint16_t* hrow = dsh + ((int64_t)z * g.C) * ldh + (int64_t)row * ldh;
  const int Nh = (Nc + 31) & ~31;
  for (int t = lane; t < Nh; t += 64) {
    float v = 0.0f;
    if (t < Nc && t != row) v = expf(srow[t] - lse);
    hrow[t] = f_to_bf16(v);
  }
}


template <int BN, int AMODE, int EPI>
void launch_t(const GemmArgsH& a, int tiles_n, int tiles_m, int batches, hipStream_t s) {
  const int64_t nwg = (int64_t)tiles_n * tiles_m * batches;
  gemm_bf16_kernel<BN, AMODE, EPI><<<(unsigned)nwg, 256, 0, s>>>(a, tiles_n, tiles_m);
}

int dim_max(int sel, int fixed, int C, int U) { return sel == DIM_CC ? C : (sel == DIM_NC ? C + U : fixed); }

}  // namespace

void launch_gemm_bf16(const GemmArgsH& a, int epi, int batches, hipStream_t s) {
  const int maxM = dim_max(a.mdim, a.Mfix, a.C, a.U);
  const int maxN = dim_max(a.ndim, a.Nfix, a.C, a.U);
  if (maxM <= 0 || maxN <= 0 || batches <= 0) return;
  const int tiles_m = (maxM + BM - 1) / BM;
  const int tiles_n = (maxN + 127) / 128;   // = nct (PBG_SCORE_BN columns per tile)
  if (epi == EPI_LOSS) launch_t<128, GA_KC, EPI_LOSS>(a, tiles_n, tiles_m, batches, s);
  else if (epi == EPI_LOSS_BITS) launch_t<128, GA_KC, EPI_LOSS_BITS>(a, tiles_n, tiles_m, batches, s);
  else if (epi == EPI_SOFTMAX_STATS) launch_t<128, GA_KC, EPI_SOFTMAX_STATS>(a, tiles_n, tiles_m, batches, s);
  else launch_t<128, GA_KC, EPI_STORE>(a, tiles_n, tiles_m, batches, s);
}

namespace {
template <int BN, int AM0, int AM1>
void launch_pair_t(const GemmArgsH& a0, const GemmArgsH& a1, int batches, hipStream_t s) {
  const int tn0 = (dim_max(a0.ndim, a0.Nfix, a0.C, a0.U) + BN - 1) / BN;
  const int tm0 = (dim_max(a0.mdim, a0.Mfix, a0.C, a0.U) + BM - 1) / BM;
  const int tn1 = (dim_max(a1.ndim, a1.Nfix, a1.C, a1.U) + BN - 1) / BN;
  const int tm1 = (dim_max(a1.mdim, a1.Mfix, a1.C, a1.U) + BM - 1) / BM;
  const int64_t nwg0 = (int64_t)tn0 * tm0 * batches, nwg1 = (int64_t)tn1 * tm1 * batches;
  gemm_bf16_pair_kernel<BN, AM0, AM1><<<(unsigned)(nwg0 + nwg1), 256, 0, s>>>(a0, tn0, tm0, (int)nwg0, a1,
                                                                                 tn1, tm1);
}

template <int BN>
void launch_pair_bn(const GemmArgsH& a0, const GemmArgsH& a1, int batches, hipStream_t s) {
  if (a0.amode == GA_BITS_ROW) launch_pair_t<BN, GA_BITS_ROW, GA_BITS_COL>(a0, a1, batches, s);
  else launch_pair_t<BN, GA_KC, GA_MC>(a0, a1, batches, s);
}
}  // namespace

void launch_gemm_bf16_pair(const GemmArgsH& a0, const GemmArgsH& a1, int batches, hipStream_t s) {
  const int maxN = std::max(dim_max(a0.ndim, a0.Nfix, a0.C, a0.U), dim_max(a1.ndim, a1.Nfix, a1.C, a1.U));
  if (maxN <= 0 || batches <= 0) return;
  if (maxN <= 64) launch_pair_bn<64>(a0, a1, batches, s);
  else launch_pair_bn<128>(a0, a1, batches, s);
}

void launch_to_bf16_t(const float* q, int64_t q_bs, int q_rows, uint16_t* qh, int64_t qh_bs, uint16_t* qT,
                      int64_t qT_bs, int q_ldT, const float* n, int64_t n_bs, int n_rows, uint16_t* nh,
                      int64_t nh_bs, uint16_t* nT, int64_t nT_bs, int n_ldT, int ld_src, int kp, int batches,
                      hipStream_t s) {
  if (batches <= 0 || kp <= 0) return;
  const Bf16T o0{q, q_bs, q_rows, ld_src, qh, qh_bs, kp, qT, qT_bs, q_ldT};
  const Bf16T o1{n, n_bs, n_rows, ld_src, nh, nh_bs, kp, nT, nT_bs, n_ldT};
  const int nq = q ? batches : 0;   // no Q: only N
  dim3 grid((kp + 63) / 64, (std::max(q ? q_ldT : 0, n_ldT) + 63) / 64, nq + batches);
  to_bf16_t_kernel<<<grid, 256, 0, s>>>(o0, o1, nq, kp);
}

void launch_softmax_rows_bf16(const StepGeom& g, const StepBufs& b, uint16_t* dsh, int ldh, hipStream_t s) {
  dim3 grid((g.C + 3) / 4, g.nchunks * 2);
  softmax_rows_bf16_kernel<<<grid, 256, 0, s>>>(g, b.ds, b.rowpart, b.pos, dsh, ldh);
}
