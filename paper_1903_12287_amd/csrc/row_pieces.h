// Pieces of one packed row, written by the wave that holds it.
#pragma once

#include "pieces.h"

template <int RQ>
__device__ __forceinline__ void row_pieces(const StepGeom& g, uint16_t* p, float* inv,
                                           const RowT<RQ>& r, bool cplx, int lane) {
  if (g.pieces == PIECES_UNIT) {
    pieces::store_row(r, 32768.0f, p, g.d, g.dh, cplx, lane);
    return;
  }
  const float top = pieces::row_absmax(r);
  const int e = pieces::scale_exponent(top);
  pieces::store_row(r, pieces::scale_of(e), p, g.d, g.dh, cplx, lane);
  if (lane == 0) *inv = top == 0.0f ? PIECES_ZERO_ROW : pieces::inverse_scale_of(e);
}

// row t of side `side` of nn
template <int RQ>
__device__ __forceinline__ void candidate_pieces(const StepGeom& g, const StepBufs& b, int c, int side, int t,
                                                 const RowT<RQ>& r, bool cplx, int lane) {
  if (g.pieces == PIECES_NONE) return;
  const int64_t o = (int64_t)(c * 2 + side) * g.N + t;
  row_pieces(g, b.pn + o * g.pld, b.pn_is + o, r, cplx, lane);
}

// row e of side `side` of qk
template <int RQ>
__device__ __forceinline__ void query_pieces(const StepGeom& g, const StepBufs& b, int c, int side, int e,
                                             const RowT<RQ>& r, bool cplx, int lane) {
  if (g.pieces == PIECES_NONE) return;
  const int64_t o = (int64_t)(c * 2 + side) * g.C + e;
  row_pieces(g, b.pq + o * g.pld, b.pq_is + o, r, cplx, lane);
}
