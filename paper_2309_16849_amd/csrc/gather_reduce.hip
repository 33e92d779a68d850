// gather_reduce.hip -- the code example's aggregation path (App. B): the
// gather with the caller's weights that keeps the k neighbours apart,
//     S[b,hd,l,t,f,y,x] = 1/cnt(y,x) * sum over the query patches covering
//                         (y,x) of w_l * v~_l(f, (y,x) + disp_l)
// (Sec. 3.2 "Aggregation" restricted to the l-th neighbours), and the
// reduction over the neighbours that follows it, a convolution with a
// (Cout, C, k, 1, 1) kernel at stride (k, 1, 1):
//     out[b,t,o,y,x] = sum over hd, f, l of proj[o, hd*F' + f, l] * S[b,hd,l,t,f,y,x].
//
// The reduction is a dense contraction per pixel (k * C inputs, Cout
// outputs), done on the matrix cores: per 8 x 8 pixel tile and per (head,
// neighbour rank), a (64 pixels x F') by (F' x Cout) product with
// v_mfma_f32_16x16x4f32, fp32 in and out; each of the 4 waves owns 16 pixels
// and all Cout columns.  The fused entry point gathers S for the tile into
// LDS and multiplies it straight away, so the k-fold stacked tensor never
// goes to memory.
//
// Gather: the tile's covering queries' records (weight, frame, integer
// offset, fractions) of as many ranks as fit are staged in LDS together; thread
// (pixel, slot) walks the queries covering its pixel, two at a time, and reads
// the four taps of each from a channels-last copy of v (4 consecutive channels
// per 16-byte load).  The four slots of a pixel are channel groups, or for
// heads of 4 or 8 channels also 4 or 2 ranks side by side.  Bound by the taps'
// latency: one rank's records staged at a time, one query's taps in flight and
// half the slots idle at 8 channels had taken 575 us on the code example (5 x
// 128 x 128, 2 x 8 channels, P = 3, k = 10), 197 us now.  Heads of 33 to 48
// channels have three blocks of their own: with four, a quarter of the reads in
// flight idle, 5 x 60 x 90, P = 3, k = 10 took 287 us at 36 channels and 306 at
// 48, now 221 and 241 (260 and 282 with one query's taps in flight).
// A neighbour whose weight is 0, whose frame is not an integer in [0, T) or
// whose offset is not finite (magnitude kFarDisp or more) adds nothing.
#include "snls_internal.h"

namespace snls {

namespace gr {
constexpr int TS = 8;             // 8 x 8 pixel tile
constexpr int NP = TS * TS;       // pixels per tile
constexpr int NT = 256;           // threads: 64 pixels x 4 slots
constexpr int FMAX = 64;          // channels per head
constexpr int RMAX = 256;         // covering queries of a tile
constexpr int RCAP = 1024;        // staged records (at least 4 ranks)
constexpr int OMAX = 128;         // output channels (8 blocks of 16)
constexpr int SP = NP + 4;        // LDS pitch of a channel row of S (pixels)
// ranks side by side for Ch channels per head, and the 16-row blocks their channels fill
inline __host__ __device__ int ranks(int Ch) { return Ch <= 4 ? 4 : Ch <= 8 ? 2 : 1; }
inline __host__ __device__ int blocks(int Ch) { return (Ch + 15) / 16; }
}  // namespace gr

// Covering-query range of the tile along one axis: grid positions m with
// m*S in [y0 - lo - P + 1, y0 + TS - 1 - lo], clipped to [0, n).
SNLS_DEV void cover_range(int y0, int S, int n, int lo, int P, int* m0, int* m1) {
  const int a = y0 - lo - P + 1, bnd = y0 + gr::TS - 1 - lo;
  *m0 = a <= 0 ? 0 : (a + S - 1) / S;
  *m1 = bnd < 0 ? -1 : min(bnd / S, n - 1);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct GrRecords {
  float4 w[gr::RCAP];  // weight (0: adds nothing), row and column fraction, frame (as bits)
  int2 n[gr::RCAP];    // integer offset
};

// NB blocks of 16 contraction rows (channels of the ranks in hand), NO blocks
// of 16 output channels.
template <int NB, int NO>
struct GrSmem {
  alignas(16) float S[16 * NB][gr::SP];            // gathered channels x pixels
  alignas(16) float Pm[16 * NO][16 * NB + 1];      // kernel slice [o][channel] of the ranks in hand
};

// The tile's covering queries: grid rows mh0 .., columns mw0 ...
struct GrCover {
  int mh0, mh1, mw0, mw1, nmw, nq;
};
SNLS_DEV GrCover gr_cover(const Geo& g, int y0, int x0) {
  GrCover c;
  cover_range(y0, g.s0, g.nH, g.lo, g.ps, &c.mh0, &c.mh1);
  cover_range(x0, g.s0, g.nW, g.lo, g.ps, &c.mw0, &c.mw1);
  c.nmw = max(c.mw1 - c.mw0 + 1, 0);
  c.nq = max(c.mh1 - c.mh0 + 1, 0) * c.nmw;
  return c;
}

// Records of ranks l0 .. l0 + nl - 1 (weight 0 from rank k on), rank after rank.
SNLS_DEV void gr_stage(GrRecords& rs, const float* __restrict__ weights, const float* __restrict__ inds, const Geo& g,
                       const GrCover& cv, int b, int t, int hd, int l0, int nl) {
  for (int e = threadIdx.x; e < cv.nq * nl; e += gr::NT) {
    const int j = e / nl, lr = e - j * nl, l = l0 + lr;  // consecutive threads: consecutive ranks of a row
    const int mh = cv.mh0 + j / cv.nmw, mw = cv.mw0 + j % cv.nmw;
    const long long row = ((((long long)b * g.HD + hd) * g.T + t) * g.nH + mh) * g.nW + mw;
    float4 r = make_float4(0.f, 0.f, 0.f, __int_as_float(0));
    int2 n = make_int2(0, 0);
    if (l < g.k) {
      const float w = weights[row * g.k + l];
      const float* ind = inds + (row * g.k + l) * 3;
      const float tf = ind[0], dh = ind[1], dw = ind[2];
      if (w != 0.f && tf >= 0.f && tf < (float)g.T && tf == floorf(tf) && fabsf(dh) < kFarDisp && fabsf(dw) < kFarDisp) {
        split_disp(dh, &n.x, &r.y);
        split_disp(dw, &n.y, &r.z);
        r.x = w;
        r.w = __int_as_float((int)tf);
      }
    }
    rs.w[lr * cv.nq + j] = r;
    rs.n[lr * cv.nq + j] = n;
  }
}

// Gather of one rank (records rw, rn) for pixel (y, x): channels 4 (cg + 4 i)
// .. + 3 of the head, i < NB; cnt: the number of covering queries.
template <int NB>
SNLS_DEV void gr_gather(const float4* rw, const int2* rn, const float* __restrict__ vcl, const Geo& g,
                        const GrCover& cv, int b, int hd, int cg, int y, int x, float4 (&acc)[NB], int* cnt) {
#pragma unroll
  for (int i = 0; i < NB; ++i) acc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  *cnt = 0;
  if (y >= g.H || x >= g.W) return;
  const int a = y - g.lo - g.ps + 1, c = x - g.lo - g.ps + 1;
  const int a0 = max(a <= 0 ? 0 : (a + g.s0 - 1) / g.s0, cv.mh0), a1 = min((y - g.lo) / g.s0, cv.mh1);
  const int c0 = max(c <= 0 ? 0 : (c + g.s0 - 1) / g.s0, cv.mw0), c1 = min((x - g.lo) / g.s0, cv.mw1);
  *cnt = max(a1 - a0 + 1, 0) * max(c1 - c0 + 1, 0);
  const long long fstride = g.HW * g.C;  // floats per frame of the channels-last copy
  // (a slot past the head's channels reads the first group's; its sums are not kept)
  const float* vb = vcl + (long long)b * g.T * fstride + (long long)hd * g.Ch + (4 * cg < g.Ch ? 4 * cg : 0);
  typedef float f4 __attribute__((ext_vector_type(4)));
  for (int mh = a0; mh <= a1; ++mh) {
    for (int mw = c0; mw <= c1; mw += 2) {
      const int j = (mh - cv.mh0) * cv.nmw + (mw - cv.mw0);
      f4 tv[2][4][NB];
      float tw[2][4];
      bool tok[2][4];
      // unconditional 16-byte reads (a tap that adds nothing reads the frame's
      // first record and is replaced by 0), all of both queries in flight
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const bool on = u == 0 || mw + 1 <= c1;
        const float4 r = rw[on ? j + u : j];
        const int2 n = rn[on ? j + u : j];
        const float w = on ? r.x : 0.f;
        const int Y = y + n.x, X = x + n.y;
        const float* f0 = vb + (long long)__float_as_int(r.w) * fstride;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int YY = Y + (e >> 1), XX = X + (e & 1);
          tw[u][e] = w * ((e >> 1) ? r.y : 1.f - r.y) * ((e & 1) ? r.z : 1.f - r.z);
          tok[u][e] = YY >= 0 && YY < g.H && XX >= 0 && XX < g.W && tw[u][e] != 0.f;
          const float* q = tok[u][e] ? f0 + ((long long)YY * g.W + XX) * g.C : vb;
#pragma unroll
          for (int i = 0; i < NB; ++i) tv[u][e][i] = *reinterpret_cast<const f4*>(q + (4 * (cg + 4 * i) < g.Ch ? 16 * i : 0));
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const f4 v = tv[u][e][i];
            const float wt = tw[u][e];
            const bool ok = tok[u][e];
            sum.x = fmaf(wt, ok ? v.x : 0.f, sum.x);
            sum.y = fmaf(wt, ok ? v.y : 0.f, sum.y);
            sum.z = fmaf(wt, ok ? v.z : 0.f, sum.z);
            sum.w = fmaf(wt, ok ? v.w : 0.f, sum.w);
          }
          acc[i].x += sum.x;
          acc[i].y += sum.y;
          acc[i].z += sum.z;
          acc[i].w += sum.w;
        }
    }
  }
}

// ---- standalone gather: S to the stacked tensor (B, HD, k, T, F', H, W) ----

template <int NB, int RK>
__global__ void __launch_bounds__(gr::NT) gather_stacked_tile_kernel(const float* __restrict__ vcl,
                                                                     const float* __restrict__ weights,
                                                                     const float* __restrict__ inds, Geo g,
                                                                     int tiles_x, int tiles_y,
                                                                     float* __restrict__ stacked) {
  using namespace gr;
  __shared__ GrRecords rs;
  const int tile = (int)(blockIdx.x % (unsigned)(tiles_x * tiles_y));
  const int bt = (int)(blockIdx.x / (unsigned)(tiles_x * tiles_y));
  const int b = bt / g.T, t = bt % g.T;
  const int y0 = (tile / tiles_x) * TS, x0 = (tile % tiles_x) * TS;
  const int tid = threadIdx.x, p = tid % NP, slot = tid / NP;
  const int y = y0 + p / TS, x = x0 + p % TS;
  const GrCover cv = gr_cover(g, y0, x0);
  const int rk = RK > 1 ? slot / (4 / RK) : 0, cg = RK > 1 ? slot % (4 / RK) : slot;
  const int kc = min((g.k + RK - 1) / RK * RK, RCAP / max(cv.nq, 1) / RK * RK);  // ranks staged at a time
  for (int hd = 0; hd < g.HD; ++hd)
    for (int l0 = 0; l0 < g.k; l0 += kc) {
      __syncthreads();  // the previous records are no longer read
      gr_stage(rs, weights, inds, g, cv, b, t, hd, l0, kc);
      __syncthreads();
      for (int l = l0 + rk; l < min(l0 + kc, g.k); l += RK) {
        float4 acc[NB];
        int cnt;
        gr_gather<NB>(rs.w + (l - l0) * cv.nq, rs.n + (l - l0) * cv.nq, vcl, g, cv, b, hd, cg, y, x, acc, &cnt);
        if (y < g.H && x < g.W) {
          const float inv = cnt > 0 ? 1.f / (float)cnt : 0.f;
          float* ob = stacked + ((((long long)b * g.HD + hd) * g.k + l) * g.T + t) * g.Ch * g.HW + (long long)y * g.W + x;
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            const int c = 4 * (cg + 4 * i);
            if (c >= g.Ch) break;
            const float a[4] = {acc[i].x, acc[i].y, acc[i].z, acc[i].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) ob[(long long)(c + e) * g.HW] = cnt > 0 ? a[e] * inv : 0.f;
          }
        }
      }
    }
}

// ---- reduction over the neighbours on the matrix cores ----
//
// For the tile's 64 pixels, out[p][o] += sum_f S[f][p] * Pm[o][f] for one
// (head, rank): wave w takes pixels 16w .. 16w+15 (A rows) and every block of
// 16 output channels (B columns); v_mfma_f32_16x16x4f32 takes A[i][kk] from
// lane i + 16 kk, B[kk][j] from lane j + 16 kk and leaves D[4 gq + r][j] in
// register r of lane j + 16 gq.
template <int NB, int NO>
SNLS_DEV void gr_mfma(const GrSmem<NB, NO>& sm, int F, int nob, f32x4 (&accv)[NO]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i = lane & 15, kk = lane >> 4;
  for (int f0 = 0; f0 < F; f0 += 4) {
    const float a = sm.S[f0 + kk][16 * wv + i];
#pragma unroll
    for (int ob = 0; ob < NO; ++ob) {
      if (ob < nob) {
        const float bv = sm.Pm[16 * ob + i][f0 + kk];
        accv[ob] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bv, accv[ob], 0, 0, 0);
      }
    }
  }
}

// Kernel slices of head hd, ranks l .. l + nr - 1: Pm[o][r*Ch + f] =
// proj[o, hd*F' + f, l + r] for the nob blocks of 16 output channels (0 past
// Cout and past rank k).
template <int NB, int NO>
SNLS_DEV void gr_stage_proj(GrSmem<NB, NO>& sm, const float* __restrict__ proj, const Geo& g, int cout, int nob,
                            int hd, int l, int nr) {
  const int F = nr * g.Ch;
  for (int e = threadIdx.x; e < 16 * nob * F; e += gr::NT) {
    const int o = e / F, c = e - o * F, r = c / g.Ch, f = c - r * g.Ch;
    sm.Pm[o][c] = o < cout && l + r < g.k ? proj[((long long)o * g.C + (long long)hd * g.Ch + f) * g.k + l + r] : 0.f;
  }
}

// out (B, T, Cout, H, W) from the accumulators of the tile.
template <int NO>
SNLS_DEV void gr_store(const f32x4 (&accv)[NO], int nob, const Geo& g, int cout, int b, int t, int y0,
                       int x0, int tw, float* __restrict__ out) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int j = lane & 15, gq = lane >> 4;
#pragma unroll
  for (int ob = 0; ob < NO; ++ob) {
    if (ob >= nob) break;
    const int o = 16 * ob + j;
    const float vals[4] = {accv[ob][0], accv[ob][1], accv[ob][2], accv[ob][3]};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int p = 16 * wv + 4 * gq + r;
      const int y = y0 + p / tw, x = x0 + p % tw;
      if (o < cout && y < g.H && x < g.W)
        out[(((long long)b * g.T + t) * cout + o) * g.HW + (long long)y * g.W + x] = vals[r];
    }
  }
}

// Fused gather + reduction: the stacked tensor stays on chip.  NB, NO: blocks
// of 16 contraction rows and output channels; RK ranks side by side.
template <int NB, int NO, int RK>
__global__ void __launch_bounds__(gr::NT) gather_reduce_kernel(const float* __restrict__ vcl,
                                                               const float* __restrict__ weights,
                                                               const float* __restrict__ inds,
                                                               const float* __restrict__ proj, Geo g, int cout,
                                                               int tiles_x, int tiles_y, float* __restrict__ out) {
  using namespace gr;
  __shared__ GrRecords rs;
  __shared__ GrSmem<NB, NO> sm;
  const int tile = (int)(blockIdx.x % (unsigned)(tiles_x * tiles_y));
  const int bt = (int)(blockIdx.x / (unsigned)(tiles_x * tiles_y));
  const int b = bt / g.T, t = bt % g.T;
  const int y0 = (tile / tiles_x) * TS, x0 = (tile % tiles_x) * TS;
  const int tid = threadIdx.x, p = tid % NP, slot = tid / NP;
  const int y = y0 + p / TS, x = x0 + p % TS;
  const int nob = (cout + 15) / 16;
  const GrCover cv = gr_cover(g, y0, x0);
  const int rk = RK > 1 ? slot / (4 / RK) : 0, cg = RK > 1 ? slot % (4 / RK) : slot;
  const int kc = min((g.k + RK - 1) / RK * RK, RCAP / max(cv.nq, 1) / RK * RK);  // ranks staged at a time
  f32x4 accv[NO];
#pragma unroll
  for (int ob = 0; ob < NO; ++ob) accv[ob] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int hd = 0; hd < g.HD; ++hd)
    for (int l0 = 0; l0 < g.k; l0 += kc) {
      // (the barrier before the last product: the previous records are no longer read)
      gr_stage(rs, weights, inds, g, cv, b, t, hd, l0, kc);
      __syncthreads();
      for (int l = l0; l < min(l0 + kc, g.k); l += RK) {
        float4 acc[NB];
        int cnt;
        const int ro = (l + rk - l0) * cv.nq;
        gr_gather<NB>(rs.w + ro, rs.n + ro, vcl, g, cv, b, hd, cg, y, x, acc, &cnt);
        const float inv = cnt > 0 ? 1.f / (float)cnt : 0.f;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          const int c = 4 * (cg + 4 * i);
          if (c >= g.Ch) break;
          const float a[4] = {acc[i].x, acc[i].y, acc[i].z, acc[i].w};
#pragma unroll
          for (int e = 0; e < 4; ++e) sm.S[rk * g.Ch + c + e][p] = a[e] * inv;
        }
        gr_stage_proj(sm, proj, g, cout, nob, hd, l, RK);
        __syncthreads();
        gr_mfma(sm, RK * g.Ch, nob, accv);
        __syncthreads();  // S and Pm are rewritten for the next ranks
      }
    }
  gr_store(accv, nob, g, cout, b, t, y0, x0, TS, out);
}

// Reduction of a stacked tensor from memory: a tile is 64 consecutive
// pixels of one row, so the stack's channel rows are read coalesced.
__global__ void __launch_bounds__(gr::NT) stacked_reduce_kernel(const float* __restrict__ stacked,
                                                                const float* __restrict__ proj, Geo g, int cout,
                                                                int tiles_x, int tiles_y, float* __restrict__ out) {
  using namespace gr;
  __shared__ GrSmem<FMAX / 16, OMAX / 16> sm;
  const int tile = (int)(blockIdx.x % (unsigned)(tiles_x * tiles_y));
  const int bt = (int)(blockIdx.x / (unsigned)(tiles_x * tiles_y));
  const int b = bt / g.T, t = bt % g.T;
  const int y0 = tile / tiles_x, x0 = (tile % tiles_x) * NP;
  const int nob = (cout + 15) / 16;
  f32x4 accv[OMAX / 16];
#pragma unroll
  for (int ob = 0; ob < OMAX / 16; ++ob) accv[ob] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int hd = 0; hd < g.HD; ++hd)
    for (int l = 0; l < g.k; ++l) {
      const float* sb = stacked + ((((long long)b * g.HD + hd) * g.k + l) * g.T + t) * g.Ch * g.HW + (long long)y0 * g.W;
      for (int e = threadIdx.x; e < g.Ch * NP; e += NT) {
        const int f = e / NP, p = e % NP;
        const int x = x0 + p;
        sm.S[f][p] = x < g.W ? sb[(long long)f * g.HW + x] : 0.f;
      }
      gr_stage_proj(sm, proj, g, cout, nob, hd, l, 1);
      __syncthreads();
      gr_mfma(sm, g.Ch, nob, accv);
      __syncthreads();
    }
  gr_store(accv, nob, g, cout, b, t, y0, x0, NP, out);
}

// The tiled kernels: channels of a head a multiple of 4 and at most 64, at
// most 256 covering queries per 8 x 8 tile, 32-bit frame offsets.
bool gather_tile_supported(const Geo& g) {
  const int nq = ((gr::TS + g.ps - 2) / g.s0 + 1);
  return g.Ch % 4 == 0 && g.Ch <= gr::FMAX && g.C % 4 == 0 && nq * nq <= gr::RMAX && g.k >= 1;
}

bool reduce_supported(const Geo& g, int cout) {
  return g.Ch % 4 == 0 && g.Ch <= gr::FMAX && cout >= 1 && cout <= gr::OMAX && g.k >= 1;
}

size_t gather_ws_bytes(const Geo& g) {
  return gather_tile_supported(g) ? (size_t)g.B * g.T * g.C * g.HW * sizeof(float) : 0;
}

static long long gr_tiles(const Geo& g, int* tx, int* ty) {
  *tx = (g.W + gr::TS - 1) / gr::TS;
  *ty = (g.H + gr::TS - 1) / gr::TS;
  return (long long)*tx * *ty * g.B * g.T;
}

snls_status launch_gather_stacked(const float* v, const float* weights, const float* inds, const Geo& g,
                                  float* stacked, void* ws, hipStream_t s) {
  if (g.rows == 0) return SNLS_OK;
  if (!gather_tile_supported(g)) return launch_gather_stacked_plain(v, weights, inds, g, stacked, s);
  float* vcl = static_cast<float*>(ws);
  snls_status st = launch_to_channels_last(v, g, vcl, s);
  if (st != SNLS_OK) return st;
  int tx, ty;
  const long long nwg = gr_tiles(g, &tx, &ty);
  if (nwg > 0x7fffffffLL) return SNLS_ERR_UNSUPPORTED;
#define SNLS_GS(NB, RK)                                                                                            \
  hipLaunchKernelGGL((gather_stacked_tile_kernel<NB, RK>), dim3((unsigned)nwg), dim3(gr::NT), 0, s, vcl, weights, \
                     inds, g, tx, ty, stacked)
  if (gr::ranks(g.Ch) == 4) SNLS_GS(1, 4);
  else if (gr::ranks(g.Ch) == 2) SNLS_GS(1, 2);
  else if (gr::blocks(g.Ch) == 1) SNLS_GS(1, 1);
  else if (gr::blocks(g.Ch) == 2) SNLS_GS(2, 1);
  else if (gr::blocks(g.Ch) == 3) SNLS_GS(3, 1);
  else SNLS_GS(4, 1);
#undef SNLS_GS
  return hipGetLastError() == hipSuccess ? SNLS_OK : SNLS_ERR_HIP;
}

snls_status launch_stacked_reduce(const float* stacked, const float* proj, const Geo& g, int cout, float* out,
                                  hipStream_t s) {
  const int tx = (g.W + gr::NP - 1) / gr::NP, ty = g.H;  // row strips of 64 pixels
  const long long nwg = (long long)tx * ty * g.B * g.T;
  if (nwg == 0) return SNLS_OK;
  if (nwg > 0x7fffffffLL) return SNLS_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(stacked_reduce_kernel, dim3((unsigned)nwg), dim3(gr::NT), 0, s, stacked, proj, g, cout, tx, ty,
                     out);
  return hipGetLastError() == hipSuccess ? SNLS_OK : SNLS_ERR_HIP;
}

snls_status launch_gather_reduce(const float* v, const float* weights, const float* inds, const float* proj,
                                 const Geo& g, int cout, float* out, void* ws, hipStream_t s) {
  int tx, ty;
  const long long nwg = gr_tiles(g, &tx, &ty);
  if (nwg == 0) return SNLS_OK;
  if (nwg > 0x7fffffffLL) return SNLS_ERR_UNSUPPORTED;
  float* vcl = static_cast<float*>(ws);
  snls_status st = launch_to_channels_last(v, g, vcl, s);
  if (st != SNLS_OK) return st;
#define SNLS_GR(NB, RK)                                                                                               \
  do {                                                                                                              \
    if (cout <= 64)                                                                                                 \
      hipLaunchKernelGGL((gather_reduce_kernel<NB, 4, RK>), dim3((unsigned)nwg), dim3(gr::NT), 0, s, vcl, weights,  \
                         inds, proj, g, cout, tx, ty, out);                                                         \
    else                                                                                                            \
      hipLaunchKernelGGL((gather_reduce_kernel<NB, 8, RK>), dim3((unsigned)nwg), dim3(gr::NT), 0, s, vcl, weights,  \
                         inds, proj, g, cout, tx, ty, out);                                                         \
  } while (0)
  if (gr::ranks(g.Ch) == 4) SNLS_GR(1, 4);
  else if (gr::ranks(g.Ch) == 2) SNLS_GR(1, 2);
  else if (gr::blocks(g.Ch) == 1) SNLS_GR(1, 1);
  else if (gr::blocks(g.Ch) == 2) SNLS_GR(2, 1);
  else if (gr::blocks(g.Ch) == 3) SNLS_GR(3, 1);
  else SNLS_GR(4, 1);
#undef SNLS_GR
  return hipGetLastError() == hipSuccess ? SNLS_OK : SNLS_ERR_HIP;
}

}  // namespace snls
