// search_mfma.hip -- scores of every candidate on the matrix cores for the
// tiled search route (Sec. 3.2; inner products, any S_Q, S_K <= 1, P <= 7).
//
// Same decomposition as search_tile.hip: a candidate's bilinear score is a
// 4-tap combination of box sums B_D(j) = sum_p c_D(j + p) of the pixel
// correlations c_D(x) = <q(x), K(x + D)>, D over the union of the integer
// shifts that the tile's windows read.  Here the contraction over the head's
// channels runs on the matrix cores.
//
// Precision.  A fp32 value is the sum of three bf16 numbers, each the nearest
// to what the ones before leave (8 significant bits and a sign each, fp32's
// exponents: no scale, whatever the range of an image or its channels).  Six of
// the nine partial products are formed (v_mfma_f32_16x16x32_bf16, fp32
// accumulation, the small ones first); the three left out are below 2^-25 of
// the product and of either sign.  With the 4-tap pass in 64 bits (one
// rounding) the scores' error against 64-bit sums is below that of the fp32
// vector-unit kernel: 64x64 noise with 16 channels, P = 3: 4.4e-8 against
// 4.7e-8; 96x96 with 32 channels, P = 3: 4.0e-8 against 4.7e-8, for channels of
// one size as for channels 2^24 apart.  Two fp16 parts of values scaled by image
// (four products) held 22 to 24 bits and lost channels below 2^-16 of the
// image's largest value (9.7e-7 at 2^24); they took a third less matrix-core
// time and key traffic (480x854, P = 7, 64 channels: 11.4 ms for the call, now
// 15.1).
//
// Work split (one workgroup = one query tile of one (b, head, t), looping over
// the frames of the window; 12 waves for heads up to 32 channels, else 8):
//  * the tile's halo of q -- hr rows of 16 pixels, tile rows (16 - P) / S_Q + 1
//    queries wide -- sits in LDS in split form, up to 64 channels of it; wider
//    heads go through in groups of 64, each group's sums added to the tables;
//  * a wave owns up to two (three: 8 waves and P < 5) consecutive shift rows
//    D_h at a time.  It streams the key rows straight from memory into
//    registers (matrix operand A: 16 key columns x the channels, 2 or 3 column
//    blocks), one key row at a time; key row Y pairs with halo row y = Y - D_h
//    for each of its shift rows, so one load serves them all, and the next
//    row's load is in flight while the current one's sums are formed.  No
//    workgroup barrier inside a round of shift rows;
//  * the 16 x 48 products (x, X) of a (halo row, shift row) go through the
//    wave's own LDS block, whose diagonals X - x = D_w the lanes read back:
//    lane = (shift column, part of the tile's columns; 3 parts of 21 lanes
//    for unions up to 21 shift columns, else 2 of 32, swept 32 columns at a
//    time).  The horizontal box sums are formed in registers, the vertical ones
//    as a running tree over the halo rows (each row adds once: v, v + v', ... as
//    in search_tile.hip), and every finished box sum goes to its query's window
//    table in LDS;
//  * the 4-tap pass writes the scores of the frame to the workspace rows.
//
// Measured (480x854, T = 5, 64 channels, P = 7, Ws = 9, the whole search): 15.1 ms
// against 21.3 ms with the scores on the vector units.  A step of a wave of two
// shift rows takes about 4,300 cycles: 820 to issue the vector instructions, 790
// of matrix cores, the rest waits, at 2 waves per SIMD -- without the key loads
// (stale operands) the call takes 3.2 ms less, without the third parts 3.9.
#include <math.h>
#include <type_traits>

#include "snls_internal.h"

namespace snls {

namespace mf {
// Waves per workgroup and shift rows per wave: 12 waves (3 per SIMD, 168
// VGPRs each) of up to 2 rows for records of one chunk; 8 (2 per SIMD, 256
// VGPRs) where two chunks' operands are held (480x854, 64 channels, P = 7: 15.1
// ms for the call, with 12 waves 22.3), of up to 3 rows for P < 5 (256x256, P =
// 3: 0.62 and 0.64 ms) and 2 above, whose vertical sums take more registers
// (480x854, P = 7: 3 rows 15.7 ms; P = 5 at S_Q = 2: 2.5 and 2.2 ms).
constexpr int waves(int CG) { return CG == 1 ? 12 : 8; }
constexpr int rows_per_wave(int PS, int CG) { return CG > 1 && PS < 5 ? 3 : 2; }
constexpr int HC = 16;           // halo columns = columns of operand B
constexpr int UW3 = 21;          // shift columns with three column parts (one per lane of a part)
constexpr int UW2 = 32;          // ... with two (16 + 32 - 1 <= 48 key columns): wider unions are swept 32 at a time
constexpr int UMAX = 16383;      // shift rows or columns of a union: a query's first one, relative to the union's, has 16 bits
constexpr int DP = 52;           // pitch of a product row in LDS (4 DP = 16 mod 64: the writes' banks)
constexpr int DBUF = HC * DP;    // floats per wave
constexpr int LDS_BYTES = 160 * 1024;
constexpr int PARTS = 3;         // bf16 parts of a value
constexpr int CHUNK = PARTS * 64;  // bytes of a pixel's 32 channels

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
}  // namespace mf

// Geometry of the split copies and of the tiles.
struct MfGeo {
  int nc32;     // 32-channel chunks of a pixel record (three parts of 64 bytes each)
  int rec;      // bytes of a pixel record
  int tqh, tqw; // queries per tile
  int hr;       // halo rows
  int tiles_x, tiles_y;
  int qpitch;   // bytes of a pixel's record (one or two chunks) in LDS
  int o_d, o_tab, o_qi, o_ql, o_fl, o_dump, o_uni;  // LDS offsets (bytes)
  int wp, win;  // window table pitch and size of a query
};

// Channels of a split record: 32, or a multiple of 64.
static int mf_chunks(const Geo& g) { return g.Ch <= 32 ? 1 : 2 * ((g.Ch + 63) / 64); }

// ---- split copies ----

// The three bf16 parts of a value, which sum to it: each the nearest bf16 to
// what the parts before leave (8 + 8 + 8 significant bits; values below 2^-110
// lose their last bits to the denormal range).  A value that bf16 would round
// to infinity starts from the largest finite one; the parts of an infinity or
// a NaN after the first are 0.
SNLS_DEV void mf_parts(float v, __bf16 (&p)[mf::PARTS]) {
  const bool fin = fabsf(v) < INFINITY;
  p[0] = (__bf16)(fin ? fminf(fmaxf(v, -0x1.fep127f), 0x1.fep127f) : v);
  const float r = fin ? v - (float)p[0] : 0.f;
  p[1] = (__bf16)r;
  p[2] = (__bf16)(r - (float)p[1]);
}

// One workgroup = 64 pixels of one (b, t, head): channels x pixels through
// LDS, 64 channels at a time, then 8 channels per thread are split and written
// as three 16-byte pieces.
__global__ void __launch_bounds__(256) mf_split_kernel(const float* __restrict__ x, Geo g, int nc32,
                                                       unsigned char* __restrict__ xs) {
  using namespace mf;
  __shared__ float tile[64][65];
  const long long slab = blockIdx.y;  // (b*T + t)*HD + hd
  const int hd = (int)(slab % g.HD);
  const long long p0 = (long long)blockIdx.x * 64;
  const float* src = x + ((slab / g.HD) * g.C + (long long)hd * g.Ch) * g.HW;
  const int px = threadIdx.x & 63, qt = threadIdx.x >> 6;
  const bool pin = p0 + px < g.HW;
  const int rec = nc32 * CHUNK;
  // row y of the plane: 16-byte pieces (8 channels of one part) of its pixels,
  // piece after piece: [32-channel chunk][part][4 pieces][W]
  const int p = (int)p0 + px;
  const int y = p / g.W;
  unsigned char* dst = xs + slab * g.HW * rec + ((long long)y * g.W * rec + (long long)(p - y * g.W) * 16);
  const long long pst = (long long)g.W * 16;  // bytes from piece to piece
  const int nch = nc32 * 32;                  // channels with padding
  for (int c0 = 0; c0 < nch; c0 += 64) {
    if (c0) __syncthreads();
    for (int i = qt; i < 64; i += 4) {
      const int c = c0 + i;
      tile[i][px] = (c < g.Ch && pin) ? src[(long long)c * g.HW + p0 + px] : 0.f;
    }
    __syncthreads();
    // piece pc (channels 8 pc ..) of pixel px: consecutive threads write
    // consecutive 16 bytes
    for (int pc = qt; pc < min(nch - c0, 64) / 8; pc += 4) {
      if (!pin) continue;
      bf8 part[PARTS];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        __bf16 e[PARTS];
        mf_parts(tile[8 * pc + i][px], e);
#pragma unroll
        for (int n = 0; n < PARTS; ++n) part[n][i] = e[n];
      }
      unsigned char* o = dst + ((c0 / 32 + pc / 4) * (4 * PARTS) + (pc & 3)) * pst;
#pragma unroll
      for (int n = 0; n < PARTS; ++n) *reinterpret_cast<bf8*>(o + 4 * n * pst) = part[n];
    }
  }
}

// Box sums of width P of L values in registers (N = L - P + 1 results), the
// same tree as search_tile.hip's: 4 a + 2 b + c.
template <int P, int N>
SNLS_DEV void mf_box(const float (&v)[N + P - 1], float (&o)[N]) {
  constexpr int L = N + P - 1;
  if constexpr (P == 1) {
#pragma unroll
    for (int x = 0; x < N; ++x) o[x] = v[x];
  } else {
    float b2[L - 1];
#pragma unroll
    for (int x = 0; x < L - 1; ++x) b2[x] = v[x] + v[x + 1];
    if constexpr ((P & 4) != 0) {
#pragma unroll
      for (int x = 0; x < N; ++x) {
        float r = b2[x] + b2[x + 2];
        if constexpr ((P & 2) != 0) r += b2[x + 4];
        if constexpr ((P & 1) != 0) r += v[x + P - 1];
        o[x] = r;
      }
    } else {
#pragma unroll
      for (int x = 0; x < N; ++x) {
        float r = b2[x];
        if constexpr ((P & 1) != 0) r += v[x + P - 1];
        o[x] = r;
      }
    }
  }
}

// Running vertical box sum: push the value of row y, get the sum of rows
// y-P+1 .. y (meaningful from the P-th push on).  State: the last value, the
// last pair sums and quad sums that later results read.  PH = y mod 3: the
// quad sums of P = 7 sit in a ring of three, so they need not be moved.
template <int P>
struct RunBox {
  float v1;        // v(y-1)
  float b2a, b2b;  // b2(y-2), b2(y-3)  (b2(i) = v(i) + v(i+1))
  float b4[3];     // quad sums b4(i) = b2(i) + b2(i+2): P = 7: b4(y-4 .. y-6); P = 5, 6: b4[0] = b4(y-4), b4[1] = b4(y-5)
  SNLS_DEV void clear() { v1 = b2a = b2b = b4[0] = b4[1] = b4[2] = 0.f; }
  template <int PH>
  SNLS_DEV float push(float v) {
    if constexpr (P == 1) {
      return v;
    } else {
      const float b2 = v1 + v;  // b2(y-1)
      float r;
      if constexpr (P == 2) {
        r = b2;
      } else if constexpr (P == 3) {
        r = b2a + v;  // b2(y-2) + v(y)
        b2a = b2;
      } else {
        const float q4 = b2b + b2;  // b4(y-3)
        if constexpr (P == 4) r = q4;
        if constexpr (P == 5) {
          r = b4[0] + v;  // b4(y-4) + v(y)
          b4[0] = q4;
        }
        if constexpr (P == 6) {
          r = b4[1] + b2;  // b4(y-5) + b2(y-1)
          b4[1] = b4[0];
          b4[0] = q4;
        }
        if constexpr (P == 7) {
          r = b4[PH] + b2a + v;  // b4(y-6) + b2(y-2) + v(y)
          b4[PH] = q4;
        }
        b2b = b2a;
        b2a = b2;
      }
      v1 = v;
      return r;
    }
  }
};

// What the waves of a workgroup need of one frame step (uniform values).
struct MfFrame {
  const unsigned char* kplane;  // split key plane of the frame
  int W, rec, plane_bytes;      // frame width; bytes of a pixel record and of a plane
  int row0;                     // frame row of (halo row 0, the wave's first shift row)
  int H, hr, qpitch;
  int dr0, dc0;                 // the wave's first shift row and column less the union's
  int col0, ncol;               // frame column of product column 0; product columns that the union needs
  int s0, tqw, wp;
  int gi;                       // channel group (CG chunks) in the q halo
};

// The box sums of ND consecutive shift rows for the whole tile, NB blocks of
// 16 key columns, NPART column parts (see the head of the file).  Step s
// reads key row s + row0 and pairs it with halo rows s, s - 1, ...; halo rows
// outside [0, hr) (the first and last ND - 1 steps) are computed from a
// clamped row: they enter only sums that are never written, and the loop has
// no branches.  ADD: the sums are added to those of the frame's earlier channel
// groups (a read and a select per sum: 5 to 15% of a whole call where a run-time
// flag made every call pay for them).
template <int PS, int CG, bool S1, int ND, int NB, int NPART, bool ADD>
SNLS_DEV void mf_stream(const MfFrame& f, const unsigned char* qlds, float* dbuf, const int2* qi, float* tab,
                        float* dump0) {
  using namespace mf;
  constexpr int NX = HC - PS + 1;                // patch origins per halo row
  constexpr int NXP = (NX + NPART - 1) / NPART;  // ... of a part (neighbouring parts may share some)
  constexpr int NV = NXP + PS - 1;               // products a lane reads per row
  constexpr int LW = NPART == 3 ? UW3 : UW2;     // lanes of a part
  constexpr bool LATE = PS == 7 && CG == 1;  // the keys' third parts are not in flight during the sums
  constexpr bool INTER = CG > 1;             // the products of all rows side by side
  constexpr unsigned OOB = 0x80000000u;
  const int lane = threadIdx.x & 63;
  const int lj = lane & 15, lg = lane >> 4;
  const int part = min(lane / LW, NPART - 1);
  const int le = lane - part * LW;               // shift column (lane 63 of three parts: column 21, never read)
  const int xh = min(part * NXP, NX - NXP);      // first patch origin of this part
  [[maybe_unused]] const int xdup = part * NXP - xh;  // its first ones that the part before has too
  const __amdgpu_buffer_rsrc_t k_rs =
      __builtin_amdgcn_make_buffer_rsrc((void*)f.kplane, (short)0, f.plane_bytes, 0x00020000);
  unsigned voff[NB];  // byte offsets of this lane's key columns (outside the frame or the union: reads 0)
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const int gx = f.col0 + 16 * n + lj;
    const bool in = gx >= 0 && gx < f.W && 16 * n + lj < f.ncol;
    voff[n] = in ? (unsigned)((lg * f.W + gx) * 16) : OOB;
  }
  bf8 kk[PARTS][NB][CG];
  // parts e0 .. e1 - 1 of operand A of step s; rows outside the frame read 0
  // (a scalar offset of the whole plane puts every lane past its end)
  auto load_k = [&](int s, int e0, int e1) {
    const int gy = f.row0 + s;
    const bool in = gy >= 0 && gy < f.H;
    const int part4 = f.W * 64;  // bytes of one part's pieces of a chunk
    const int so = in ? gy * f.W * f.rec + f.gi * CG * PARTS * part4 : f.plane_bytes;
#pragma unroll
    for (int e = e0; e < e1; ++e)
#pragma unroll
      for (int c = 0; c < CG; ++c)
#pragma unroll
        for (int n = 0; n < NB; ++n)
          kk[e][n][c] = __builtin_bit_cast(
              bf8, __builtin_amdgcn_raw_buffer_load_b128(k_rs, voff[n], in ? so + (c * PARTS + e) * part4 : so, 0));
  };
  RunBox<PS> st[ND][NXP];
#pragma unroll
  for (int i = 0; i < ND; ++i)
#pragma unroll
    for (int x = 0; x < NXP; ++x) st[i][x].clear();
  float* const dw = dbuf + lj * DP + 4 * lg;             // this lane's products
  const float* const dr = dbuf + xh * (DP + 1) + le;     // ... and its diagonal
  float* const dump = dump0 + lane;                      // box sums that no query reads go here
  // strided queries: query column of each patch origin (0 where it is none, bit x of xok clear)
  int jx[NXP];
  unsigned xok = 0;
#pragma unroll
  for (int x = 0; x < NXP; ++x) {
    const int j = (xh + x) / f.s0;
    const bool ok = j * f.s0 == xh + x;
    jx[x] = ok ? j : 0;
    xok |= (ok ? 1u : 0u) << x;
  }
  const unsigned char* const ap0 = qlds + lj * f.qpitch + lg * 16;
  const int qrow = HC * f.qpitch;
  const int nstep = f.hr + ND - 1;
  load_k(0, 0, LATE ? 2 : PARTS);
  auto step = [&](int s, auto phase) {
    constexpr int PH = decltype(phase)::value;
    f32x4 acc[ND][NB];
#pragma unroll
    for (int i = 0; i < ND; ++i)
#pragma unroll
      for (int n = 0; n < NB; ++n) acc[i][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    // The large products last: the others' roundings are small.  The next
    // step's keys are in flight during this step's sums; where 168 registers
    // cannot hold them (P = 7 with 12 waves) their third parts are loaded behind
    // the first products (128x128, 32 channels: 0.54 -> 0.50 ms).  With 8 waves
    // the products of all rows go side by side (480x854, P = 7: 16.0 -> 15.1 ms),
    // their operand B held one part at a time.
    auto mul = [&](int i, int ek, const bf8(&qq)[CG]) {
#pragma unroll
      for (int c = 0; c < CG; ++c)
#pragma unroll
        for (int n = 0; n < NB; ++n)
          acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk[ek][n][c], qq[c], acc[i][n], 0, 0, 0);
    };
    auto load_q = [&](int i, int e, bf8(&qq)[CG]) {  // operand B: part e of row i
      const unsigned char* ap = ap0 + min(max(s - i, 0), f.hr - 1) * qrow + e * 64;
#pragma unroll
      for (int c = 0; c < CG; ++c) qq[c] = *reinterpret_cast<const bf8*>(ap + c * CHUNK);
    };
    if constexpr (LATE) load_k(s, 2, 3);
    if constexpr (INTER) {
      bf8 qq[ND][CG];
      auto take = [&](int e) {
#pragma unroll
        for (int i = 0; i < ND; ++i) load_q(i, e, qq[i]);
      };
      auto mul_all = [&](int ek) {
#pragma unroll
        for (int i = 0; i < ND; ++i) mul(i, ek, qq[i]);
      };
      take(2);
      mul_all(0);
      take(1);
      mul_all(1);
      mul_all(0);
      take(0);
      mul_all(1);
      mul_all(2);
      mul_all(0);
    } else {
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        bf8 q0[CG], q1[CG], q2[CG];
        load_q(i, 2, q2);
        load_q(i, 1, q1);
        load_q(i, 0, q0);
        mul(i, 0, q2);
        mul(i, 1, q1);
        mul(i, 1, q0);
        mul(i, 0, q1);
        if constexpr (!LATE) {
          mul(i, 2, q0);
          mul(i, 0, q0);
        }
      }
      if constexpr (LATE) {
#pragma unroll
        for (int i = 0; i < ND; ++i) {
          bf8 q0[CG];
          load_q(i, 0, q0);
          mul(i, 2, q0);
          mul(i, 0, q0);
        }
      }
    }
    load_k(s + 1, 0, LATE ? 2 : PARTS);  // in flight during the sums below
    // The products of shift row i + 1 enter the wave's LDS block right behind
    // row i's reads (a wave's LDS accesses complete in order), so that they
    // are there when row i's sums are done.
    auto put_products = [&](int i) {
      // row x = lj, columns X = 16 n + 4 lg ..
#pragma unroll
      for (int n = 0; n < NB; ++n) *reinterpret_cast<f32x4*>(dw + 16 * n) = acc[i][n];
      wave_lds_sync();
    };
    put_products(0);
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      float v[NV];
#pragma unroll
      for (int x = 0; x < NV; ++x) v[x] = dr[x * (DP + 1)];
      wave_lds_sync();
      const int yq = s - i - (PS - 1);  // patch origin row of the sums this step finishes
      const bool live = yq >= 0 && yq <= f.hr - PS && (S1 || yq % f.s0 == 0);
      // the queries of that row: first shifts and table base (any row when
      // there is none: nothing is written then)
      const int jr = live ? (S1 ? yq : yq / f.s0) * f.tqw : 0;
      int2 w[NXP];
#pragma unroll
      for (int x = 0; x < NXP; ++x) w[x] = qi[jr + (S1 ? xh + x : jx[x])];
      if (i + 1 < ND) put_products(i + 1);
      float hb[NXP];
      mf_box<PS, NXP>(v, hb);
#pragma unroll
      for (int x = 0; x < NXP; ++x) hb[x] = st[i][x].template push<PH>(hb[x]);
      // the finished box sums to their queries' tables: entry (shift row less
      // the query's first, the same for columns) where it lies in the table
      if (live) {
        const int lc = f.dc0 + le, cell = (f.dr0 + i) * f.wp + lc;
#pragma unroll
        for (int x = 0; x < NXP; ++x) {
          const unsigned u = (unsigned)(f.dr0 + i - (w[x].x >> 16)), c = (unsigned)(lc - (int)(short)w[x].x);
          bool ok = max(u, c) < (unsigned)f.wp;
          if (!S1) ok = ok && ((xok >> x) & 1);
          if (ADD) ok = ok && x >= xdup;
          float* const at = ok ? tab + (w[x].y + cell) : dump;
          if constexpr (ADD) *at += hb[x];
          else *at = hb[x];
        }
      }
    }
  };
  if constexpr (PS == 7) {
    for (int s = 0; s < nstep; s += 3) {
      step(s, std::integral_constant<int, 0>{});
      if (s + 1 >= nstep) break;
      step(s + 1, std::integral_constant<int, 1>{});
      if (s + 2 >= nstep) break;
      step(s + 2, std::integral_constant<int, 2>{});
    }
  } else {
    for (int s = 0; s < nstep; ++s) step(s, std::integral_constant<int, 0>{});
  }
}

// Whether a frame's union is swept (in `rounds` passes of every wave over the
// tile's halo, 2,400 cycles a halo row) or its candidates are scored one by
// one (1,400 to 4,000 cycles a thread, patch pixel and channel: every read is
// a cache line of its own).  256x256, T = 3, Ws = 9, swept / one by one: a
// motion edge of 24 columns with P = 7 and 64 channels 0.80 / 126 ms, offsets
// of +-50 with P = 1 and 32 channels 2.8 / 8.1 ms, of +-100 8.4 / 8.7 ms.
SNLS_DEV bool mf_sweeps_pay(const Geo& g, const MfGeo& mg, int rounds, int nt) {
  const float sweep = 2400.f * (float)mg.hr * (float)rounds;
  const float direct = 2000.f * (float)((mg.tqh * mg.tqw * g.ws * g.ws + nt - 1) / nt) * (float)(g.ps * g.ps * g.Ch);
  return sweep < direct;
}

// What mf_redo needs of a frame step (in LDS).
struct MfRedo {
  const float *q, *k;                     // the videos
  const unsigned char *qplane, *kplane;   // split planes of the query and key frames
  const float2* ff;                       // the tile's offsets of the frame step
  float* scores;                          // at the frame step's first candidate
  int* infs;                              // last frame step (from 1) with an infinity in its reach
  long long qchan, kchan;                 // first channel plane of the query and key frames
  long long HW, rowb;
  int H, W, Ch, nH, nW, ws, r;
  float s1;
  int pitch, s0, tqw, qn, my0, mx0, hr, rec, npc, dmin_h, dmin_w, UH, UW, step;
};

// Scores that are infinite or NaN.  The products of an infinity's parts mix
// signs and zeros: with one in reach these scores are formed again from q and
// k.  Without, a NaN comes from a NaN -- of the patch, or, for patches that
// stick out of the frame, from keys that only q's zeros there meet: only those
// are formed again.  A function of its own, called by the whole workgroup:
// inlined, its values took registers from the frame loop (271x483, P = 5, two
// heads of 24 channels: 1.54 ms inlined, 1.47 called, 1.43 without).
template <int PS, int NT>
__device__ __noinline__ void mf_redo(const MfRedo* __restrict__ a) {
  using namespace mf;
  constexpr int LO = -(PS / 2);
  const int tid = threadIdx.x, lane = tid & 63;
  const int H = a->H, W = a->W, ws = a->ws, s0 = a->s0, tqw = a->tqw;
  bool infs = false;
  auto look = [&](const unsigned char* plane, int y0, int ny, int x0, int nx) {
    const int n = ny * nx * a->npc;
    for (int e = tid; e < n; e += NT) {
      const int pc = e / (ny * nx), p = e - pc * (ny * nx);
      const int gy = y0 + p / nx, gx = x0 + p % nx;
      if (gy < 0 || gy >= H || gx < 0 || gx >= W) continue;
      const u32x4 v = *reinterpret_cast<const u32x4*>(
          plane + (long long)gy * W * a->rec + ((long long)((pc >> 2) * (4 * PARTS) + (pc & 3)) * W + gx) * 16);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        infs = infs || (v[i] & 0x7fffu) == 0x7f80u || (v[i] & 0x7fff0000u) == 0x7f800000u;
    }
  };
  const int Y0 = a->my0 * s0 + LO, X0 = a->mx0 * s0 + LO;
  look(a->qplane, Y0, a->hr, X0, HC);
  look(a->kplane, Y0 + a->dmin_h, a->hr + a->UH - 1, X0 + a->dmin_w, HC + a->UW - 1);
  if (infs) *a->infs = a->step;
  __syncthreads();
  infs = *a->infs == a->step;
  const int ncell = ws * ws, nterm = PS * PS * a->Ch, ncand = a->qn * ncell;
  const float* const qbase = a->q + a->qchan * a->HW;
  const float* const kbase = a->k + a->kchan * a->HW;
  // a lane finds a candidate, the wave forms its score
  for (int e0 = tid - lane; e0 < ncand; e0 += NT) {
    const int e = e0 + lane;
    const int j = e / ncell, cell = e - j * ncell;
    const int mh = a->my0 + j / tqw, mw = a->mx0 + j % tqw;
    const int h = mh * s0, w = mw * s0;
    float dh = 0.f, dw = 0.f;
    float* at = nullptr;
    bool todo = e < ncand && mh < a->nH && mw < a->nW;
    if (todo) {
      dh = cand_disp(a->ff[j].x, a->s1, cell / ws, a->r);
      dw = cand_disp(a->ff[j].y, a->s1, cell % ws, a->r);
      at = a->scores + ((a->rowb + mh) * a->nW + mw) * a->pitch + cell;
      const bool out = h + LO < 0 || h + LO + PS > H || w + LO < 0 || w + LO + PS > W;
      todo = (infs || out) && centre_ok(h, dh, H) && centre_ok(w, dw, W) && !(fabsf(*at) < INFINITY);
    }
    unsigned long long m = __ballot(todo);
    while (m) {
      const int src = __ffsll((long long)m) - 1;
      m &= m - 1;
      const int ch = __shfl(h, src), cw = __shfl(w, src);
      int nh, nw;
      float ah, aw;
      split_disp(__shfl(dh, src), &nh, &ah);
      split_disp(__shfl(dw, src), &nw, &aw);
      float sum = 0.f;
      for (int i0 = 0; i0 < nterm; i0 += 64) {
        const int i = i0 + lane, c = i / (PS * PS), pp = i - c * (PS * PS);
        const int y = ch + LO + pp / PS, x = cw + LO + pp % PS;
        if (i < nterm && y >= 0 && y < H && x >= 0 && x < W)
          sum = fmaf(qbase[c * a->HW + (long long)y * W + x],
                     bilinear_plane(kbase + c * a->HW, H, W, y + nh, x + nw, ah, aw), sum);
        if (__any(sum != sum)) break;
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
      if (lane == src) *at = sum == sum ? sum : -INFINITY;
    }
  }
}

// CG: 32-channel chunks of a record multiplied per load (1 or 2).  S1: query stride 1.
template <int PS, int CG, bool S1>
__global__ void __launch_bounds__(mf::waves(CG) * 64, mf::waves(CG) / 4) search_mfma_scores_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const unsigned char* __restrict__ qs,
    const unsigned char* __restrict__ ks, const float* __restrict__ flows, Geo g, MfGeo mg, float* __restrict__ scores,
    int pitch) {
  using namespace mf;
  constexpr int LO = -(PS / 2);
  constexpr int NW = waves(CG), NT = NW * 64, NDW = rows_per_wave(PS, CG);
  __shared__ __attribute__((aligned(16))) unsigned char smem[LDS_BYTES];
  unsigned char* const qlds = smem;
  float* const tab = reinterpret_cast<float*>(smem + mg.o_tab);
  float2* const fl = reinterpret_cast<float2*>(smem + mg.o_fl);  // offsets: [frame of the window][query]
  // two buffers (this frame's and the next one's):
  // a query's first shift row (high half) and column less the union's, table base less their entry
  int2* const qi = reinterpret_cast<int2*>(smem + mg.o_qi);
  int2* const ql = reinterpret_cast<int2*>(smem + mg.o_ql);  // a query's first shift row and column
  float* const dump = reinterpret_cast<float*>(smem + mg.o_dump);
  // min N_h, max N_h, min N_w, max N_w of each frame; the last frame step (from 1) with an infinite or NaN
  // score, and with an infinity in its reach
  int* const uni = reinterpret_cast<int*>(smem + mg.o_uni);
  int* const nonfin = uni + 4 * (2 * g.wt + 1);
  MfRedo* const redo = reinterpret_cast<MfRedo*>(nonfin + 4);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* const dbuf = reinterpret_cast<float*>(smem + mg.o_d) + wave * DBUF;

  // XCD-aware order: each XCD takes a contiguous run of tiles; the query
  // frames, heads and batch entries of one tile are consecutive workgroups
  // (they share key frames in the XCD's L2).
  const long long nwg = (long long)gridDim.x;
  const long long xcd = blockIdx.x % 8, xq = nwg / 8, xrem = nwg % 8;
  const long long wg = xcd * xq + (xcd < xrem ? xcd : xrem) + blockIdx.x / 8;
  const int nimg = g.B * g.HD * g.T;
  const int img = (int)(wg % nimg);
  const int trem = (int)(wg / nimg);
  const int ty = trem / mg.tiles_x, tx = trem % mg.tiles_x;
  const int t = img % g.T;
  const int hd = (img / g.T) % g.HD;
  const int b = img / (g.T * g.HD);
  const int s0 = S1 ? 1 : g.s0, tqh = mg.tqh, tqw = mg.tqw, qn = tqh * tqw, hr = mg.hr;
  const int my0 = ty * tqh, mx0 = tx * tqw;  // tile origin (query grid)
  const int y0 = my0 * s0, x0 = mx0 * s0;    // tile origin (pixels)
  const int Y0 = y0 + LO, X0 = x0 + LO;      // halo origin
  const int ws = g.ws, r = g.r, wp = mg.wp, win = mg.win, rec = mg.rec;
  constexpr unsigned OOB = 0x80000000u;  // buffer offset past any extent: reads 0
  const unsigned plane_bytes = (unsigned)(g.HW * rec);
  const int dt0 = max(-g.wt, -t), dt1 = min(g.wt, g.T - 1 - t);  // frames inside the clip
  const int nfr = dt1 - dt0 + 1;

  auto slab = [&](int tt) { return ((long long)b * g.T + tt) * g.HD + hd; };

  // ---- the halo of q (split records), the tile's offsets ----
  if (tid < 2) nonfin[tid] = 0;
  for (int e = tid; e < nfr * qn; e += NT) {
    const int fi = e / qn, j = e - fi * qn, dt = dt0 + fi;
    const int h = y0 + s0 * (j / tqw), w = x0 + s0 * (j % tqw);
    float2 F = make_float2(0.f, 0.f);
    if (dt != 0 && h < g.H && w < g.W) {
      const long long base = (((long long)b * g.T + t) * g.nslot + flow_slot(dt, g.wt)) * 2;
      const long long pix = (long long)h * g.W + w;
      F = make_float2(flows[base * g.HW + pix], flows[(base + 1) * g.HW + pix]);
    }
    fl[e] = F;
  }
  // the halo's records of channel group gi
  const int npix = hr * HC, ngrp = CG > 1 ? mg.nc32 / CG : 1;
  const __amdgpu_buffer_rsrc_t q_rs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(qs + slab(t) * g.HW * rec), (short)0, (int)plane_bytes, 0x00020000);
  auto load_halo = [&](int gi) {
    const int n = npix * (CG * 4 * PARTS);
    for (int e0 = tid; e0 < n; e0 += 4 * NT) {  // four loads in flight
      u32x4 v[4];
      int at[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = e0 + i * NT;
        const int pc = e / npix, p = e - pc * npix;
        const int gy = Y0 + p / HC, gx = X0 + p % HC;
        const bool in = e < n && gy >= 0 && gy < g.H && gx >= 0 && gx < g.W;
        at[i] = p * mg.qpitch + pc * 16;
        v[i] = __builtin_amdgcn_raw_buffer_load_b128(
            q_rs, in ? (unsigned)(gy * g.W * rec + ((gi * CG * 4 * PARTS + pc) * g.W + gx) * 16) : OOB, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (e0 + i * NT < n) *reinterpret_cast<u32x4*>(qlds + at[i]) = v[i];
    }
  };
  int held = 0;  // the channel group in the halo
  load_halo(0);
  __syncthreads();
  // a query's first integer shifts of a frame, and its last ones + 1.
  // Offsets that are not finite or absurdly large count as zero here; their
  // candidates fail the exact validity test below.
  auto lo_of = [&](float F) { return (int)floorf(cand_disp(fabsf(F) < kFarDisp ? F : 0.f, g.s1, 0, r)); };
  auto hi_of = [&](float F) { return (int)floorf(cand_disp(fabsf(F) < kFarDisp ? F : 0.f, g.s1, ws - 1, r)) + 1; };
  // unions of the frames' shifts: one wave per frame
  for (int fi = wave; fi < nfr; fi += NW) {
    int a0 = INT_MAX, a1 = INT_MIN, a2 = INT_MAX, a3 = INT_MIN;
    for (int j = lane; j < qn; j += 64) {
      if (y0 + s0 * (j / tqw) < g.H && x0 + s0 * (j % tqw) < g.W) {
        const float2 F = fl[fi * qn + j];
        a0 = min(a0, lo_of(F.x));
        a1 = max(a1, hi_of(F.x));
        a2 = min(a2, lo_of(F.y));
        a3 = max(a3, hi_of(F.y));
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      a0 = min(a0, __shfl_xor(a0, off));
      a1 = max(a1, __shfl_xor(a1, off));
      a2 = min(a2, __shfl_xor(a2, off));
      a3 = max(a3, __shfl_xor(a3, off));
    }
    if (lane == 0) {
      uni[4 * fi] = a0;
      uni[4 * fi + 1] = a1;
      uni[4 * fi + 2] = a2;
      uni[4 * fi + 3] = a3;
    }
  }
  __syncthreads();
  // the union, clipped to the shifts that a valid cell can read: its centre
  // lies in the frame, so its taps lie in rows [-h, H - h] of a query at row h
  const int h_last = min(y0 + (tqh - 1) * s0, (g.nH - 1) * s0);
  const int w_last = min(x0 + (tqw - 1) * s0, (g.nW - 1) * s0);
  auto union_of = [&](int fi, int& u0, int& u1, int& u2, int& u3) {
    u0 = max(__builtin_amdgcn_readfirstlane(uni[4 * fi]), -h_last);
    u1 = min(__builtin_amdgcn_readfirstlane(uni[4 * fi + 1]), g.H - y0);
    u2 = max(__builtin_amdgcn_readfirstlane(uni[4 * fi + 2]), -w_last);
    u3 = min(__builtin_amdgcn_readfirstlane(uni[4 * fi + 3]), g.W - x0);
  };
  auto set_queries = [&](int fi) {
    int u0, u1, u2, u3;
    union_of(fi, u0, u1, u2, u3);
    for (int j = tid; j < qn; j += NT) {
      const float2 F = fl[fi * qn + j];
      const int lh = lo_of(F.x), lw = lo_of(F.y);
      // relative to the union (at most UMAX rows and columns, else the tables
      // are not used); a window that far from it reads none of it
      const int rh = min(max(lh - u0, -16384), 16383), rw = min(max(lw - u2, -16384), 16383);
      qi[(fi & 1) * qn + j] = make_int2((rh << 16) | (rw & 0xffff), j * win - rh * wp - rw);
      ql[(fi & 1) * qn + j] = make_int2(lh, lw);
    }
  };
  set_queries(0);
  __syncthreads();

  const long long rowb = (((long long)b * g.HD + hd) * g.T + t) * g.nH;
  for (int fi = 0; fi < nfr; ++fi) {
    const int dt = dt0 + fi, t2 = t + dt;
    const int cbase = (dt + g.wt) * ws * ws;
    int dmin_h, dmax_h, dmin_w, dmax_w;
    union_of(fi, dmin_h, dmax_h, dmin_w, dmax_w);
    const int UH = dmax_h - dmin_h + 1, UW = dmax_w - dmin_w + 1;
    const bool none = UH <= 0 || UW <= 0;  // every cell of the frame is invalid
    const float2* const ff = fl + fi * qn;
    // shift rows of a round, spread over the waves: up to NDW each, one each
    // for unions that need the two-part lane layout
    const int per = NW * (UW <= UW3 ? NDW : 1);
    const int nsweep = UW <= UW3 ? 1 : (UW + UW2 - 1) / UW2;  // column sweeps
    const int nround = (UH + per - 1) / per;
    const bool tabled = none || (UW <= UMAX && UH <= UMAX && mf_sweeps_pay(g, mg, ngrp * nsweep * nround, NT));
    if (tabled) {
      // No barrier inside a round: a wave without shift rows goes on.
      for (int go = 0; go < (none ? 0 : ngrp); ++go) {
      // channel groups upwards and downwards in turn: a frame begins with the one that is there
      const int gi = (fi & 1) ? ngrp - 1 - go : go;
      if (gi != held) {
        __syncthreads();  // the halo is no longer read
        load_halo(gi);
        held = gi;
        __syncthreads();
      }
      for (int it = 0; it < nsweep * nround; ++it) {
        const int cc0 = it / nround * UW2, rr0 = (it - it / nround * nround) * per;
        const int nr = min(per, UH - rr0);
        const int nd = nr / NW + (wave < nr % NW ? 1 : 0);
        MfFrame f;
        f.kplane = ks + slab(t2) * g.HW * rec;
        f.W = g.W;
        f.H = g.H;
        f.rec = rec;
        f.plane_bytes = (int)plane_bytes;
        f.dr0 = rr0 + wave * (nr / NW) + min(wave, nr % NW);
        f.dc0 = cc0;
        f.row0 = Y0 + dmin_h + f.dr0;
        f.hr = hr;
        f.gi = gi;
        f.qpitch = mg.qpitch;
        f.col0 = X0 + dmin_w + cc0;
        f.ncol = HC - 1 + UW - cc0;
        f.s0 = s0;
        f.tqw = tqw;
        f.wp = wp;
        const int2* const qif = qi + (fi & 1) * qn;
        auto stream = [&](auto nd_, auto nb_, auto npart_) {
          constexpr int ND = decltype(nd_)::value, NB = decltype(nb_)::value, NPART = decltype(npart_)::value;
          if (CG > 1 && go > 0) mf_stream<PS, CG, S1, ND, NB, NPART, (CG > 1)>(f, qlds, dbuf, qif, tab, dump);
          else mf_stream<PS, CG, S1, ND, NB, NPART, false>(f, qlds, dbuf, qif, tab, dump);
        };
        constexpr std::integral_constant<int, 1> i1{};
        constexpr std::integral_constant<int, 2> i2{};
        constexpr std::integral_constant<int, 3> i3{};
        constexpr std::integral_constant<int, NDW> iw{};
        if (UW <= 17) {  // 16 + UW - 1 key columns in two blocks
          if (nd == 1) stream(i1, i2, i3);
          else if (nd == 2) stream(i2, i2, i3);
          else if (nd == 3 && NDW == 3) stream(iw, i2, i3);
        } else if (UW <= UW3) {
          if (nd == 1) stream(i1, i3, i3);
          else if (nd == 2) stream(i2, i3, i3);
          else if (nd == 3 && NDW == 3) stream(iw, i3, i3);
        } else if (nd == 1) {
          stream(i1, i3, i2);
        }
      }
      }
      __syncthreads();
      if (fi + 1 < nfr) set_queries(fi + 1);
      // ---- 4-tap combination and exact validity: one thread per window
      // column, so that a store's lanes write runs of ws scores ----
      bool bad = false;
      for (int e = tid; e < qn * ws; e += NT) {
        const int j = e / ws, dw = e - j * ws;
        const int jh = j / tqw;
        const int mh = my0 + jh, mw = mx0 + j - jh * tqw;
        if (mh >= g.nH || mw >= g.nW) continue;
        const int h = mh * s0, w = mw * s0;
        float* srow = scores + ((rowb + mh) * g.nW + mw) * pitch + cbase + dw;
        const int2 lo = ql[(fi & 1) * qn + j];
        const float2 F = ff[j];
        const float disp_w = cand_disp(F.y, g.s1, dw, r);
        const bool okw = centre_ok(w, disp_w, g.W);
        const float fl_w = floorf(disp_w), aw = disp_w - fl_w;
        // table reads only matter for valid cells (row 0 / column 0 otherwise)
        const float* const cp = tab + j * win + (okw ? (int)fl_w - lo.y : 0);
        for (int dh = 0; dh < ws; ++dh) {
          const float disp_h = cand_disp(F.x, g.s1, dh, r);
          const bool ok = okw && centre_ok(h, disp_h, g.H);
          const float fl_h = floorf(disp_h), ah = disp_h - fl_h;
          const float* const r0p = cp + (ok ? (int)fl_h - lo.x : 0) * wp;
          // in 64 bits: one rounding per score instead of nine
          const double t0 = r0p[0], b0 = r0p[wp];
          const double top = fma((double)aw, (double)r0p[1], (1.0 - aw) * t0);
          const double bot = fma((double)aw, (double)r0p[wp + 1], (1.0 - aw) * b0);
          const float dv = (float)fma((double)ah, bot, (1.0 - ah) * top);
          srow[dh * ws] = ok && dv == dv ? dv : -INFINITY;  // NaN scores as invalid
          bad = bad || (ok && !(fabsf(dv) < INFINITY));
        }
      }
      if (bad) nonfin[0] = fi + 1;
    } else if (fi + 1 < nfr) {
      set_queries(fi + 1);
    }
    if (!tabled) {  // the frame's candidates one by one
      // (inner products for both distances, as the top-k pass expects)
      Geo gp = g;
      gp.dist = SNLS_DIST_PROD;
      for (int e = tid; e < qn * ws; e += NT) {
        const int j = e / ws, dh = e % ws;
        const int mh = my0 + j / tqw, mw = mx0 + j % tqw;
        if (mh >= g.nH || mw >= g.nW) continue;
        const int h = mh * s0, w = mw * s0;
        const float2 F = ff[j];
        const float disp_h = cand_disp(F.x, g.s1, dh, r);
        const bool okh = centre_ok(h, disp_h, g.H);
        for (int dw = 0; dw < ws; ++dw) {
          const float disp_w = cand_disp(F.y, g.s1, dw, r);
          float d = -INFINITY;
          if (okh && centre_ok(w, disp_w, g.W)) d = score_candidate(q, k, gp, b, hd, t, h, w, t2, disp_h, disp_w);
          scores[((rowb + mh) * g.nW + mw) * pitch + cbase + dh * ws + dw] = d;
        }
      }
    }
    __syncthreads();  // the tables are free, the next frame's queries set, the frame's scores written
    if (tabled && nonfin[0] == fi + 1) {
      if (tid == 0)
        *redo = MfRedo{q, k, qs + slab(t) * g.HW * rec, ks + slab(t2) * g.HW * rec, ff, scores + cbase, nonfin + 1,
                       ((long long)b * g.T + t) * g.C + (long long)hd * g.Ch, ((long long)b * g.T + t2) * g.C + (long long)hd * g.Ch,
                       g.HW, rowb, g.H, g.W, g.Ch, g.nH, g.nW, ws, r, g.s1, pitch, s0, tqw, qn, my0, mx0, hr, rec,
                       mg.nc32 * 4, dmin_h, dmin_w, UH, UW, fi + 1};
      __syncthreads();
      mf_redo<PS, NT>(redo);
    }
  }
}

// Tile geometry for tqh query rows; false when the LDS of one CU cannot hold it.
static bool mf_geo(const Geo& g, int tqh, MfGeo* m) {
  m->nc32 = mf_chunks(g);
  m->rec = m->nc32 * mf::CHUNK;
  m->tqw = (mf::HC - g.ps) / g.s0 + 1;
  m->tqh = tqh;
  m->hr = (tqh - 1) * g.s0 + g.ps;
  m->tiles_x = (g.nW + m->tqw - 1) / m->tqw;
  m->tiles_y = (g.nH + tqh - 1) / tqh;
  m->qpitch = (m->nc32 > 1 ? 2 : 1) * mf::CHUNK + 16;  // an odd number of 16-byte slots: consecutive pixels on different banks
  m->wp = g.ws + 2;
  m->win = m->wp * m->wp;
  const long long qn = (long long)m->tqh * m->tqw;
  long long o = (long long)m->hr * mf::HC * m->qpitch;
  m->o_d = (int)o;
  o += (long long)mf::waves(m->nc32 > 1 ? 2 : 1) * mf::DBUF * 4;
  m->o_qi = (int)o;
  o += 2 * qn * 8;
  m->o_ql = (int)o;
  o += 2 * qn * 8;
  m->o_fl = (int)o;
  o += (2 * g.wt + 1) * qn * 8;
  m->o_dump = (int)o;
  o += 64 * 4;
  m->o_uni = (int)o;
  o += (2 * g.wt + 1) * 16 + 16 + (sizeof(MfRedo) + 15) / 16 * 16;
  m->o_tab = (int)o;
  o += qn * m->win * 4;
  return o <= mf::LDS_BYTES;
}

// Query rows per tile: the tallest tile has the smallest halo overhead, but
// the workgroups (one per CU at a time) should fill the 256 CUs evenly: the
// height with the least (waves of workgroups) x (halo rows + a fixed part).
static bool mf_tile(const Geo& g, MfGeo* best) {
  double bc = 0;
  bool any = false;
  for (int tqh = 1; tqh <= 16; ++tqh) {
    MfGeo m;
    if (!mf_geo(g, tqh, &m) || (tqh > 1 && m.hr > 17)) break;
    const double nwg = (double)m.tiles_x * m.tiles_y * g.B * g.HD * g.T;
    const double cost = ceil(nwg / 256.0) * (m.hr + 4);
    if (!any || cost <= bc) {
      bc = cost;
      *best = m;
      any = true;
    }
  }
  return any;
}

// Heads of 8 channels or more: fewer would be padded to 32 (the contraction is
// then mostly zeros; 2 x 4-channel heads keep the vector-unit kernel).  At P = 7
// and S_Q > 1, where most of the box sums are not a query's, 16 or more (160x160,
// T = 5, Ws = 9, S_Q = 2: 8 channels 0.64 ms here, 0.52 on the vector units, 12
// channels 0.65 and 0.57; at S_Q = 1 8 channels 0.67 and 0.64, with Ws = 5 at
// half-pixel steps 0.43 and 0.61).
bool mfma_supported(const Geo& g) {
  if (!tile_supported(g) || g.Ch < (g.ps == 7 && g.s0 > 1 ? 16 : 8)) return false;
  // 32-bit byte offsets inside one frame's split plane
  if ((long long)mf_chunks(g) * mf::CHUNK * g.HW >= (1LL << 31)) return false;
  MfGeo m;
  if (!mf_tile(g, &m)) return false;
  return (long long)g.B * g.T * g.HD <= 65535 &&
         (long long)m.tiles_x * m.tiles_y * g.B * g.HD * g.T <= 0x7fffffffLL;
}

// Split copy of a video.
static size_t mf_plane_bytes(const Geo& g) {
  return ((size_t)g.B * g.T * g.HD * (size_t)g.HW * mf_chunks(g) * mf::CHUNK + 255) & ~(size_t)255;
}

// Split copies of q and k.
size_t mfma_ws_bytes(const Geo& g) { return 2 * mf_plane_bytes(g); }

snls_status launch_mfma_scores(const float* q, const float* k, const float* flows, const Geo& g, float* scores,
                               int pitch, void* ws, hipStream_t s) {
  MfGeo m;
  if (!mf_tile(g, &m)) return SNLS_ERR_UNSUPPORTED;
  const long long nwg = (long long)m.tiles_x * m.tiles_y * g.B * g.HD * g.T;
  if (nwg == 0) return SNLS_OK;
  const unsigned nslab = (unsigned)(g.B * g.T * g.HD), nblk = (unsigned)((g.HW + 63) / 64);
  unsigned char* const ks = static_cast<unsigned char*>(ws);
  unsigned char* const qs = q == k ? ks : ks + mf_plane_bytes(g);  // one video matched with itself: one copy serves both
  hipLaunchKernelGGL(mf_split_kernel, dim3(nblk, nslab), dim3(256), 0, s, k, g, m.nc32, ks);
  if (q != k) hipLaunchKernelGGL(mf_split_kernel, dim3(nblk, nslab), dim3(256), 0, s, q, g, m.nc32, qs);
  const dim3 grid((unsigned)nwg), block(mf::waves(m.nc32 > 1 ? 2 : 1) * 64);
  switch (4 * g.ps + (m.nc32 > 1 ? 2 : 0) + (g.s0 == 1 ? 1 : 0)) {
#define SNLS_MF_LAUNCH(P, C, S)                                                                                    \
  hipLaunchKernelGGL((search_mfma_scores_kernel<P, C, S>), grid, block, 0, s, q, k, qs, ks, flows, g, m, scores, \
                     pitch);                                                                                       \
  break
#define SNLS_MF_CASE(P)                         \
  case 4 * P: SNLS_MF_LAUNCH(P, 1, false);      \
  case 4 * P + 1: SNLS_MF_LAUNCH(P, 1, true);   \
  case 4 * P + 2: SNLS_MF_LAUNCH(P, 2, false);  \
  case 4 * P + 3: SNLS_MF_LAUNCH(P, 2, true);
    SNLS_MF_CASE(1)
    SNLS_MF_CASE(2)
    SNLS_MF_CASE(3)
    SNLS_MF_CASE(4)
    SNLS_MF_CASE(5)
    SNLS_MF_CASE(6)
    SNLS_MF_CASE(7)
#undef SNLS_MF_CASE
#undef SNLS_MF_LAUNCH
    default:
      return SNLS_ERR_UNSUPPORTED;
  }
  return hipGetLastError() == hipSuccess ? SNLS_OK : SNLS_ERR_HIP;
}

}  // namespace snls
