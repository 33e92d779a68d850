// search_direct.hip -- direct shifted non-local search kernels (Sec. 3.2):
// each thread scores candidates straight from the video tensors with
// bilinear reads (the in-place computation of Sec. 3.4), for any parameter
// combination.  k == 0 writes every candidate; k >= 1 keeps the top-k per
// query row in registers.  These kernels are the general path; the tiled
// kernels (search_mfma.hip, search_tile.hip) and the single-pixel ones
// (search_p1.hip) cover patches up to 7 x 7 and windows up to 15 x 15 at any
// query stride faster.  The choice of the route is here too.
#include "snls_internal.h"

namespace snls {

// Decoded query row (b, hd, t, h, w) of a flattened row index over
// (B, HD, T, nH, nW).
struct QueryPos {
  int b, hd, t, h, w;
};

SNLS_DEV QueryPos decode_row(long long row, const Geo& g) {
  QueryPos qp;
  int mw = (int)(row % g.nW);
  row /= g.nW;
  int mh = (int)(row % g.nH);
  row /= g.nH;
  qp.t = (int)(row % g.T);
  row /= g.T;
  qp.hd = (int)(row % g.HD);
  qp.b = (int)(row / g.HD);
  qp.h = mh * g.s0;
  qp.w = mw * g.s0;
  return qp;
}

// Window offset F of frame step dt at the query pixel (zero for dt == 0).
SNLS_DEV void read_shift(const float* __restrict__ flows, const Geo& g, const QueryPos& qp, int dt, float* fh,
                         float* fw) {
  if (dt == 0) {
    *fh = 0.f;
    *fw = 0.f;
    return;
  }
  long long base = (((long long)qp.b * g.T + qp.t) * g.nslot + flow_slot(dt, g.wt)) * 2;
  long long pix = (long long)qp.h * g.W + qp.w;
  *fh = flows[base * g.HW + pix];
  *fw = flows[(base + 1) * g.HW + pix];
}

// One thread per (query row, candidate): every candidate in id order.
__global__ void __launch_bounds__(256) search_full_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                          const float* __restrict__ flows, Geo g,
                                                          float* __restrict__ dists, float* __restrict__ inds) {
  long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= g.rows * g.ncand) return;
  int cid = (int)(gid % g.ncand);
  QueryPos qp = decode_row(gid / g.ncand, g);
  int dw = cid % g.ws;
  int dh = (cid / g.ws) % g.ws;
  int dt = cid / (g.ws * g.ws) - g.wt;
  float fh, fw;
  read_shift(flows, g, qp, dt, &fh, &fw);
  float disp_h = cand_disp(fh, g.s1, dh, g.r);
  float disp_w = cand_disp(fw, g.s1, dw, g.r);
  int t2 = qp.t + dt;
  bool ok = t2 >= 0 && t2 < g.T && centre_ok(qp.h, disp_h, g.H) && centre_ok(qp.w, disp_w, g.W);
  float d = ok ? score_candidate(q, k, g, qp.b, qp.hd, qp.t, qp.h, qp.w, t2, disp_h, disp_w) : from_score(-INFINITY, g.dist);
  dists[gid] = d;
  inds[3 * gid + 0] = (float)t2;
  inds[3 * gid + 1] = disp_h;
  inds[3 * gid + 2] = disp_w;
}

// Positions of every candidate (one wave per query row at a time, lanes over
// its candidates), and the scores that the tiled kernel leaves: the invalid ones
// of frames outside the clip, and those that came out infinite or NaN, which
// are summed directly (the tiles multiply q's zeros outside the frame with keys
// and add infinite sums tap by tap).
__global__ void __launch_bounds__(256) search_positions_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                               const float* __restrict__ flows, Geo g, float* dists,
                                                               float* __restrict__ inds) {
  const int lane = threadIdx.x & 63, ncell = g.ws * g.ws;
  const float inv_cell = 1.f / (float)ncell, inv_ws = 1.f / (float)g.ws;
  const long long step = (long long)gridDim.x * 4;
  for (long long row = (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); row < g.rows;
       row += step) {
    const QueryPos qp = decode_row(row, g);
    for (int cid = lane; cid < g.ncand; cid += 64) {
      // quotients of small integers: (a + 1/2) / b is never within rounding of an integer
      const int fi = (int)(((float)cid + 0.5f) * inv_cell), cell = cid - fi * ncell;
      const int dh = (int)(((float)cell + 0.5f) * inv_ws), dw = cell - dh * g.ws;
      const int dt = fi - g.wt, t2 = qp.t + dt;
      float fh, fw;
      read_shift(flows, g, qp, dt, &fh, &fw);
      const long long o = row * g.ncand + cid;
      const float disp_h = cand_disp(fh, g.s1, dh, g.r), disp_w = cand_disp(fw, g.s1, dw, g.r);
      if (t2 < 0 || t2 >= g.T) dists[o] = from_score(-INFINITY, g.dist);
      else if (!(fabsf(dists[o]) < INFINITY) && centre_ok(qp.h, disp_h, g.H) && centre_ok(qp.w, disp_w, g.W))
        dists[o] = score_candidate(q, k, g, qp.b, qp.hd, qp.t, qp.h, qp.w, t2, disp_h, disp_w);
      inds[3 * o] = (float)t2;
      inds[3 * o + 1] = disp_h;
      inds[3 * o + 2] = disp_w;
    }
  }
}

// One thread per query row: all candidates, top-k kept in registers.
template <int KMAX>
__global__ void __launch_bounds__(128) search_topk_direct_kernel(const float* __restrict__ q,
                                                                 const float* __restrict__ k,
                                                                 const float* __restrict__ flows, Geo g,
                                                                 float* __restrict__ dists,
                                                                 float* __restrict__ inds) {
  long long row = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= g.rows) return;
  QueryPos qp = decode_row(row, g);
  TopList<KMAX> lst;
  lst.init(g.k);
  for (int dt = -g.wt; dt <= g.wt; ++dt) {
    int t2 = qp.t + dt;
    if (t2 < 0 || t2 >= g.T) continue;  // frame outside the clip: never selected ahead of a valid one
    float fh, fw;
    read_shift(flows, g, qp, dt, &fh, &fw);
    for (int dh = 0; dh < g.ws; ++dh) {
      float disp_h = cand_disp(fh, g.s1, dh, g.r);
      bool okh = centre_ok(qp.h, disp_h, g.H);
      for (int dw = 0; dw < g.ws; ++dw) {
        float disp_w = cand_disp(fw, g.s1, dw, g.r);
        int cid = ((dt + g.wt) * g.ws + dh) * g.ws + dw;
        float sc = -INFINITY;
        if (okh && centre_ok(qp.w, disp_w, g.W)) sc = to_score(score_candidate(q, k, g, qp.b, qp.hd, qp.t, qp.h, qp.w, t2, disp_h, disp_w), g.dist);
        lst.push(sc, cid);
      }
    }
  }
  // Rows with fewer than k valid candidates are completed with the invalid
  // candidates of smallest id (frames outside the clip included), matching
  // a full sort of all candidates.
  for (int dt = -g.wt; dt <= g.wt; ++dt) {
    int t2 = qp.t + dt;
    if (t2 >= 0 && t2 < g.T) continue;
    for (int c = 0; c < g.ws * g.ws; ++c) lst.push(-INFINITY, (dt + g.wt) * g.ws * g.ws + c);
  }
  float* drow = dists + row * g.k;
  float* irow = inds + row * g.k * 3;
  const int first = KMAX - g.k;  // slot of the best entry
#pragma unroll
  for (int e = 0; e < KMAX; ++e) {
    if (e >= first) {
      const int i = e - first;
      int cid = min(max(lst.id[e], 0), g.ncand - 1);  // every candidate was ranked: ids are real
      int dw = cid % g.ws;
      int dh = (cid / g.ws) % g.ws;
      int dt = cid / (g.ws * g.ws) - g.wt;
      float fh, fw;
      read_shift(flows, g, qp, dt, &fh, &fw);
      drow[i] = from_score(lst.s[e], g.dist);
      irow[3 * i + 0] = (float)(qp.t + dt);
      irow[3 * i + 1] = cand_disp(fh, g.s1, dh, g.r);
      irow[3 * i + 2] = cand_disp(fw, g.s1, dw, g.r);
    }
  }
}

snls_status launch_search_full(const float* q, const float* k, const float* flows, const Geo& g, float* dists,
                               float* inds, hipStream_t s) {
  long long total = g.rows * g.ncand;
  if (total == 0) return SNLS_OK;
  // Inner products inside the tiled kernel's domain: its scores straight into
  // the output rows (no workspace), then the positions (96 x 96, 32 channels,
  // P = 3, Ws = 5: 1.77 ms on search_full_kernel).  The squared L2 distance
  // would need its norm terms' workspace, and window quotients in floats are
  // exact below 2^20 candidates.
  Geo gt = g;
  gt.k = 1;
  if (g.dist == SNLS_DIST_PROD && tile_supported(gt) && g.ncand < (1 << 20) &&
      (long long)g.nW * g.nH * g.B * g.HD * g.T <= 0x7fffffffLL) {
    const snls_status st = launch_tile_scores(q, k, flows, gt, dists, g.ncand, s);
    if (st != SNLS_OK) return st;
    const long long blk = (g.rows + 3) / 4;
    hipLaunchKernelGGL(search_positions_kernel, dim3((unsigned)(blk < 8192 ? blk : 8192)), dim3(256), 0, s, q, k,
                       flows, g, dists, inds);
    return hipGetLastError() == hipSuccess ? SNLS_OK : SNLS_ERR_HIP;
  }
  long long blocks = (total + 255) / 256;
  hipLaunchKernelGGL(search_full_kernel, dim3((unsigned)blocks), dim3(256), 0, s, q, k, flows, g, dists, inds);
  return hipGetLastError() == hipSuccess ? SNLS_OK : SNLS_ERR_HIP;
}

snls_status launch_search_topk_direct(const float* q, const float* k, const float* flows, const Geo& g,
                                      float* dists, float* inds, hipStream_t s) {
  if (g.rows == 0) return SNLS_OK;
  unsigned blocks = (unsigned)((g.rows + 127) / 128);
  if (g.k <= 16)
    hipLaunchKernelGGL(search_topk_direct_kernel<16>, dim3(blocks), dim3(128), 0, s, q, k, flows, g, dists, inds);
  else if (g.k <= 32)
    hipLaunchKernelGGL(search_topk_direct_kernel<32>, dim3(blocks), dim3(128), 0, s, q, k, flows, g, dists, inds);
  else if (g.k <= 64)
    hipLaunchKernelGGL(search_topk_direct_kernel<64>, dim3(blocks), dim3(128), 0, s, q, k, flows, g, dists, inds);
  else
    hipLaunchKernelGGL(search_topk_direct_kernel<128>, dim3(blocks), dim3(128), 0, s, q, k, flows, g, dists, inds);
  return hipGetLastError() == hipSuccess ? SNLS_OK : SNLS_ERR_HIP;
}

SearchRoute search_route(const Geo& g, size_t have) {
  // The matrix cores, where the workspace has room for their operands: a
  // search with the scores' part alone, or none for single pixels, takes the
  // route without them.
  const bool matrix = tile_supported(g) && mfma_supported(g) && have >= tile_ws_bytes(g);
  // Single-pixel patches have no overlap for the tiles to share, but the
  // matrix cores still pay where the head has 32 channels or more and every
  // pixel is a query (k <= 16: the 16-lane top-k).  Fused kernel against the
  // tiled route, S_Q = 1, Ws = 9, k = 10, T = 5, smooth motion: 320x320 with 16
  // channels 1.23 and 1.25 ms, with 32 channels 1.84 and 1.30 ms, 256x256 with 64
  // channels 2.01 and 1.21 ms; 4 heads of 8 channels 0.22 and 0.31 ms.  Offsets
  // that neighbouring queries do not share cost the tiles more: 256x256, T = 3,
  // 32 channels, offsets of +-30 at random 2.99 and 1.59 ms, of +-100 3.38 and
  // 8.7 ms.  The fused
  // per-query kernel (k <= 32) takes the other single-pixel searches and needs
  // no score workspace; the scored single-pixel route only at a query stride
  // above 1.
  if (g.ps == 1 && g.s0 == 1 && g.Ch >= 32 && g.k <= 16 && matrix) return SearchRoute::Tile;
  if (g.ps == 1 && p1_fused(g)) return SearchRoute::P1Fused;
  if (g.ps == 1 && g.s0 > 1 && p1_supported(g)) return SearchRoute::P1Scored;
  if (tile_supported(g)) return matrix ? SearchRoute::Tile : SearchRoute::TileVector;
  if (p1_supported(g)) return p1_fused(g) ? SearchRoute::P1Fused : SearchRoute::P1Scored;
  return SearchRoute::Direct;
}

snls_status launch_search_topk(const float* q, const float* k, const float* flows, const Geo& g, float* dists,
                               float* inds, void* ws, size_t have, hipStream_t s) {
  const SearchRoute route = search_route(g, have);
  switch (route) {
    case SearchRoute::P1Fused: return launch_search_p1_topk(q, k, flows, g, dists, inds, s);
    case SearchRoute::P1Scored: return launch_search_p1(q, k, flows, g, dists, inds, static_cast<float*>(ws), s);
    case SearchRoute::Tile:
    case SearchRoute::TileVector:
      return launch_search_tile(q, k, flows, g, dists, inds, static_cast<float*>(ws), route == SearchRoute::Tile, s);
    default: return launch_search_topk_direct(q, k, flows, g, dists, inds, s);
  }
}

}  // namespace snls
