// Integrated fixed-point quantized convolution on gfx950 (MI355X) for every
// filter size and stride, from input windows resident in LDS: byte-per-code
// input and 2-bit NHWC packed input with c_in a multiple of 16, and 2-bit input of
// either layout with c_in a multiple of 64.
//
// The integer part of Eq. (1), a = W_b (x) X_q, is an implicit GEMM
// D[co][pixel] = sum_k W[co][k] * X[pixel][k] on v_mfma_i32_32x32x32_i8. What
// bounds it on these layers is not the matrix cores but how often operands
// cross the L2: a tile that gathers its pixels tap by tap reads every input
// byte kh*kw times. So:
//  - A tile's output pixels are a run of bn consecutive (n, oy, ox). The input
//    rows they touch, with the padding as zero codes (win columns a row), are
//    its window: loaded once into LDS for a chunk of channels by LDS-DMA, read
//    by every tap at a per-lane base plus a wave-uniform offset, with no
//    bounds check in the main loop. Chunks of u 16-channel units (all of
//    them where they fit) rotate through nbuf buffers, the next ones loading
//    while one is used.
//  - Weights stream through a ring of D stages of SK = S*WK K64 steps, one
//    barrier a stage. K runs over (chunk, tap, unit): the row-major weight
//    blob's 16-byte units are gathered in that order by the DMA's per-lane
//    addresses, four lanes to a row, so the blob needs no layout of its own
//    (with c_in % 64 == 0 on 2-bit codes it is in fragment order, 1 KB spans).
//  - Small layers (a few hundred pixels, K in the thousands) leave most CUs
//    idle on wide tiles: tiles down to 32 x 32 exist with WK = 4 or 8 wave
//    groups splitting the K64 steps of a stage, their sums added in LDS by
//    all the waves, each finishing its share of the tile's outputs.
//  - LDS cells are swizzled on the DMA's source side (weights by row, windows
//    by pixel, as far as the cells per pixel are a power of two), so the
//    16-byte fragment reads of 16 neighbouring rows or pixels fall on
//    distinct banks.
// Waits count exactly the loads a wave has issued after the ones it needs.
//
// Measured against the general kernel (ifq_conv.hip), which gathered every
// tap from L2 on 128 x 128 tiles: byte codes at 4 bits, batch 32, 13x13x384 ->
// 384 74.0 -> 14.6-17.6 us, 27x27x96 -> 256 5x5 67.9 -> 30 us; 2-bit byte codes,
// batch 8, 7x7x512 -> 512 57.7 -> 7.9 us, 56x56x64 -> 64 9.9 -> 7.0 us; 2-bit
// packed 27x27x96 -> 256 5x5, batch 32, 35.4 -> 26.3 us. A stage of 64 x 128
// x 256 takes about 1400 clocks against 512 of MFMAs per SIMD: barrier skew
// and the fragment reads' latency after it, then the address unit (16 KB of
// weights are 256 clocks there). The prologue (tables, first window, records)
// is 2-3 us of every launch.
#include <hip/hip_runtime.h>

#include "ifq_epilogue.h"
#include "ifq_internal.h"
#include "ifq_mfma_common.h"

namespace ifq {
namespace {

enum WinIn {
  kWinI8 = 0,   // byte codes: a cell is 16 bytes, one unit of 16 channels
  kWinU2 = 1,   // 2-bit packed codes: a cell is 4 bytes, one unit
  kWinF = 2,    // 2-bit codes, c_in % 64 == 0, weights in MFMA fragment order
};              // (mfma_layout): a cell is 16 bytes, 64 channels, a K64 step of a tap

struct WinGeom {
  int32_t u;          // cells per window pixel and chunk
  int32_t nch;        // chunks (the last one may hold fewer units)
  int32_t nbuf;       // window buffers
  int32_t nks;        // K64 steps per chunk (the last one padded with zeros)
  int32_t nkk;        // nch * nks
  int32_t win;        // window columns
  int32_t rimg;       // window rows of a whole image
  int32_t wcells;     // cells per buffer, a multiple of 64
  int32_t one;        // 1x1 filter: the window's pixels are the tile's own
  int32_t sh, msk;    // window swizzle: cell c of pixel q at c ^ ((q >> sh) & msk)
  int32_t ring_off, win_off, tab_off;   // LDS offsets past the epilogue's parameters
  int32_t ktab_off;
  int32_t red_off, out_off;             // after the main loop: K-group sums, output tile
  int32_t bn;
  FastDiv div_u, div_win, div_rimg, div_nks, div_kw;
};

// One LDS-DMA load of 4 bytes per lane (16 in dma16).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma4(const void* src, uint32_t dst) {
  const uint32_t d = __builtin_amdgcn_readfirstlane(dst);
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off"
               :: "s"(d), "v"(src) : "memory", "m0");
}
#pragma clang diagnostic pop

// Waits until at most n (wave-uniform) of this wave's loads are outstanding.
__device__ __forceinline__ void wait_vmcnt_le(int n) {
#define IFQ_W(k) case k: wait_vmcnt<k>(); break;
  switch (n < 31 ? n : 31) {
    IFQ_W(0) IFQ_W(1) IFQ_W(2) IFQ_W(3) IFQ_W(4) IFQ_W(5) IFQ_W(6) IFQ_W(7)
    IFQ_W(8) IFQ_W(9) IFQ_W(10) IFQ_W(11) IFQ_W(12) IFQ_W(13) IFQ_W(14) IFQ_W(15)
    IFQ_W(16) IFQ_W(17) IFQ_W(18) IFQ_W(19) IFQ_W(20) IFQ_W(21) IFQ_W(22) IFQ_W(23)
    IFQ_W(24) IFQ_W(25) IFQ_W(26) IFQ_W(27) IFQ_W(28) IFQ_W(29) IFQ_W(30)
    default: wait_vmcnt<31>(); break;
  }
#undef IFQ_W
}

// ---- Epilogue parameters ---------------------------------------------------
// A record {s, T_1 .. T_nq} of rec = 2^b entries is kept in LDS as {flip, heap
// of T'}: T' = T for s = +1; for s = -1, -a > T is the negation of
// a > -T - 1, so T' = -T - 1 in reversed order and the code is the count of
// T' below a, xor nq. Node 1 of the heap is the middle threshold, children
// 2i and 2i + 1: a sum's count is b steps node = 2 node + [a > T'(node)]
// (count = node - 2^b) instead of nq compares. That needs the thresholds
// ascending, as every fold writes them; unsorted is set where a record's are
// not, and sort_heaps then redoes the records (the count of thresholds below
// a sum needs no order).
__device__ __forceinline__ int heap_node(int i, int bits) {   // place of rank i = 1 .. nq
  const int z = __ffs(i) - 1;
  return (i >> (z + 1)) + (1 << (bits - 1 - z));
}

__device__ __forceinline__ const int32_t* heap_src(const ConvLaunch& a, int co0, int bm, int* n) {
  const int per = a.join_kind == IFQ_JOIN_IDENTITY ? 4 : 1;   // records per channel
  *n = (a.cout - co0 < bm ? a.cout - co0 : bm) * per * a.rec;
  return (a.join_kind == IFQ_JOIN_IDENTITY ? a.table : a.thr) + (int64_t)co0 * per * a.rec;
}

template <int NT>
__device__ __forceinline__ void stage_heaps(const ConvLaunch& a, uint8_t* lds, int co0, int bm,
                                            int32_t* unsorted) {
  if (a.out_mode == 0) return;
  if (a.join_kind == IFQ_JOIN_CONV) {
    stage_epilogue(a, lds, co0, bm);
    return;
  }
  int n;
  const int32_t* src = heap_src(a, co0, bm, &n);
  int32_t* dst = reinterpret_cast<int32_t*>(lds);
  const int bits = 31 - __clz(a.rec);
  constexpr int U = 4;                     // every load of U entries in flight
  for (int i0 = threadIdx.x; i0 < n; i0 += U * NT) {
    int t[U], before[U], sg[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int i = i0 + k * NT < n ? i0 + k * NT : 0;
      const int e = i & (a.rec - 1);
      t[k] = src[i];
      before[k] = src[e > 1 ? i - 1 : i];
      sg[k] = src[i - e];
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int i = i0 + k * NT;
      const int e = i & (a.rec - 1);
      if (i >= n) continue;
      const bool flip = sg[k] < 0;
      if (e == 0)
        dst[i] = flip ? a.nq : 0;
      else
        dst[i - e + heap_node(flip ? a.rec - e : e, bits)] = flip ? -t[k] - 1 : t[k];
      if (e && t[k] < before[k]) *unsorted = 1;
    }
  }
}

__device__ __forceinline__ void sort_heaps(const ConvLaunch& a, uint8_t* lds, int co0, int bm) {
  int n;
  const int32_t* src = heap_src(a, co0, bm, &n);
  int32_t* dst = reinterpret_cast<int32_t*>(lds);
  const int bits = 31 - __clz(a.rec);
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int e = i & (a.rec - 1);
    if (e == 0) continue;
    const int32_t* r = src + (i - e);
    int rank = 1;
    for (int j = 1; j < a.rec; ++j) rank += r[j] < r[e] || (r[j] == r[e] && j < e) ? 1 : 0;
    const bool flip = r[0] < 0;
    dst[i - e + heap_node(flip ? a.rec - rank : rank, bits)] = flip ? -r[e] - 1 : r[e];
  }
}

__host__ __device__ inline int win_param_bytes(const ConvLaunch& a, int bm) {
  if (a.out_mode == 0) return 0;
  if (a.join_kind == IFQ_JOIN_CONV) return kJoinCoefOff + bm * 24;
  return bm * a.rec * (a.join_kind == IFQ_JOIN_IDENTITY ? 16 : 4);
}

// Bytes of a pixel's row of the output tile: 16 more than its codes, so that
// the 32 pixels a wave stores at once fall on 8 banks and not on one.
__host__ __device__ inline int win_orow(const ConvLaunch& a, int bm) {
  return (a.out_mode == 2 ? bm / 4 : bm) + 16;
}

// Codes of sum v from the staged record t; LV: log2 of the record length
// where fixed, else 0.
template <int LV>
__device__ __forceinline__ int heap_code(const int32_t* t, int v, int bits, int nq) {
  if constexpr (LV == 2) {
    const int4 r = *reinterpret_cast<const int4*>(t);
    return ((v > r.y) + (v > r.z) + (v > r.w)) ^ r.x;
  } else {
    int node = 1;
    if constexpr (LV > 0) {
#pragma unroll
      for (int l = 0; l < LV; ++l) node = 2 * node + (v > t[node] ? 1 : 0);
    } else {
      for (int l = 0; l < bits; ++l) node = 2 * node + (v > t[node] ? 1 : 0);
    }
    return (node & nq) ^ t[0];
  }
}

// What a quad (four consecutive output channels co .. co+3 of pixel p) needs
// from memory: the shortcut codes of an identity join (in d[0]) or the
// downsample's sums of a conv join.
template <int MODE>
__device__ __forceinline__ void quad_in(const ConvLaunch& a, int co, int p, int (&d)[4]) {
  if constexpr (MODE == kEpiTab) {
    d[0] = (int)shortcut_codes(a, p, co);
  } else if constexpr (MODE == kEpiJoinConv) {
    const int32_t* s = reinterpret_cast<const int32_t*>(a.shortcut) + (int64_t)p * a.cout + co;
    if ((a.cout & 3) == 0) {
      const int4 s4 = *reinterpret_cast<const int4*>(s);
      d[0] = s4.x; d[1] = s4.y; d[2] = s4.z; d[3] = s4.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) d[i] = co + i < a.cout ? s[i] : 0;
    }
  }
}

// The quad's sums v (local channel cl, local pixel pl): codes into the LDS
// output tile, or the sums straight to memory.
template <int MODE, int LV>
__device__ __forceinline__ void quad_out(const ConvLaunch& a, const uint8_t* lds, const int (&v)[4],
                                         const int (&d)[4], int cl, int co, int pl, int p,
                                         uint8_t* otile, int orow) {
  if constexpr (MODE == kEpiI32) {
    int32_t* y = reinterpret_cast<int32_t*>(a.y) + (int64_t)p * a.cout + co;
    if ((a.cout & 3) == 0) {
      *reinterpret_cast<int4*>(y) = int4{v[0], v[1], v[2], v[3]};
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (co + i < a.cout) y[i] = v[i];
    }
    return;
  }
  const int bits = 31 - __clz(a.rec);
  int code[4];
  if constexpr (MODE == kEpiThr) {
    const int32_t* prm = reinterpret_cast<const int32_t*>(lds) + cl * (LV ? 1 << LV : a.rec);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      code[i] = heap_code<LV>(prm + i * (LV ? 1 << LV : a.rec), v[i], bits, a.nq);
  } else if constexpr (MODE == kEpiTab) {
    const int32_t* prm = reinterpret_cast<const int32_t*>(lds) + cl * 4 * a.rec;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      code[i] = heap_code<LV>(prm + (4 * i + ((d[0] >> (2 * i)) & 3)) * a.rec, v[i], bits, a.nq);
  } else {
    const double* qt = reinterpret_cast<const double*>(lds);
    const double* c = reinterpret_cast<const double*>(lds + kJoinCoefOff) + 3 * cl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double z = fma(c[3 * i], (double)v[i], fma(c[3 * i + 1], (double)d[i], c[3 * i + 2]));
      int n = 0;
      for (int q = 0; q < a.nq; ++q) n += z > qt[q];
      code[i] = n;
    }
  }
  if (a.out_mode == 2)
    otile[pl * orow + (cl >> 2)] =
        (uint8_t)(code[0] | (code[1] << 2) | (code[2] << 4) | (code[3] << 6));
  else
    *reinterpret_cast<uint32_t*>(otile + pl * orow + cl) =
        (uint32_t)code[0] | ((uint32_t)code[1] << 8) | ((uint32_t)code[2] << 16) |
        ((uint32_t)code[3] << 24);
}

// ---- The kernel ------------------------------------------------------------
template <int IN, int WM, int WN, int WK, int FM, int FN, int S, int D>
__global__ __launch_bounds__(64 * WM * WN * WK) void conv_win(ConvLaunch a, WinGeom g) {
  constexpr int NWG = WM * WN;                  // waves per K group
  constexpr int NW = NWG * WK;
  constexpr int BM = 32 * FM * WM;
  constexpr int BN = 32 * FN * WN;
  constexpr int SK = S * WK;                    // K64 steps per stage
  constexpr int A_STEP = BM * 64;
  constexpr int STAGE = SK * A_STEP;
  constexpr int CA1 = BM / 16;                  // 1 KB chunks (16 rows) per step
  constexpr int C = SK * CA1;
  static_assert(C % NW == 0, "equal loads per wave");
  constexpr int CPW = C / NW;
  constexpr int CB = IN == kWinU2 ? 4 : 16;     // bytes per window cell
  constexpr bool FR = IN == kWinF;
  constexpr int E = FR ? 1 : 4;                 // cells of a K64 step
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NWG;
  const int wig = wave - kg * NWG;
  const int wm = wig % WM;
  const int wn = wig / WM;
  const int h = lane >> 5;
  const int l32 = lane & 31;
  const int p0 = blockIdx.x * g.bn;
  const int co0 = blockIdx.y * BM;
  const int npx = a.m - p0 < g.bn ? a.m - p0 : g.bn;   // pixels of the tile
  const int cgt = a.cin >> (FR ? 6 : 4);        // cells of an input pixel
  const bool b64 = FR && a.in_layout == IFQ_LAYOUT_U2_BLOCK64;
  const int hw = a.h * a.w;
  const int ntaps = a.kh * a.kw;
  const int nst = (g.nkk + SK - 1) / SK;
  const int howo = a.ho * a.wo;
  const int pitch = g.u * CB;
  const uint32_t lds0 = lds_addr(lds);
  const uint32_t ring0 = lds0 + g.ring_off, win0 = lds0 + g.win_off;
  int32_t* wtab = reinterpret_cast<int32_t*>(lds + g.tab_off);
  int2* ktab_b = reinterpret_cast<int2*>(lds + g.ktab_off);
  int32_t* ktab_a = reinterpret_cast<int32_t*>(ktab_b + nst * SK * E);
  int32_t* unsorted = reinterpret_cast<int32_t*>(lds + g.ring_off - 16);   // past the parameters
  const uint8_t* zero_src = reinterpret_cast<const uint8_t*>(&g_zero_cell);

  // the tile's window: rows of the first image from oyf on, then whole
  // images (of the last one only the rows its pixels need)
  const int nf = fdiv(p0, a.div_howo);
  const int oyf = fdiv(p0 - nf * howo, a.div_wo);
  const int pl_ = p0 + npx - 1;
  const int nl = fdiv(pl_, a.div_howo);
  const int oyl = fdiv(pl_ - nl * howo, a.div_wo);
  const int r0 = (a.ho - 1 - oyf) * a.stride + a.kh;
  const int wrows = nf == nl ? (oyl - oyf) * a.stride + a.kh
                             : r0 + (nl - nf - 1) * g.rimg + oyl * a.stride + a.kh;
  const int wpx = g.one ? npx : wrows * g.win;
  const int ncw = (wpx * g.u + 63) / 64;        // DMA chunks of one window buffer

  // window pixel -> first cell of input pixel (n*h + iy)*w + ix, or -1 for
  // padding (and for one entry past the window)
  // (the upper half of the threads; the lower half does the K table)
  constexpr int NT2 = 32 * NW;
  for (int q = tid - NT2; q < wpx; q += NT2) {
    if (q < 0) break;
    int img, iy, ix;
    if (g.one) {
      const int p = p0 + q;
      img = fdiv(p, a.div_howo);
      const int rem = p - img * howo;
      const int oy = fdiv(rem, a.div_wo);
      iy = oy * a.stride - a.pad;
      ix = (rem - oy * a.wo) * a.stride - a.pad;
    } else {
      const int wr = fdiv(q, g.div_win);
      ix = q - wr * g.win - a.pad;
      if (nf == nl || wr < r0) {
        img = nf;
        iy = oyf * a.stride - a.pad + wr;
      } else {
        const int t = wr - r0;
        const int i = fdiv(t, g.div_rimg);
        img = nf + 1 + i;
        iy = t - i * g.rimg - a.pad;
      }
    }
    const bool ok = (unsigned)iy < (unsigned)a.h && (unsigned)ix < (unsigned)a.w;
    const int px = iy * a.w + ix;
    wtab[q] = !ok ? -1 : b64 ? img * cgt * hw + px : (img * hw + px) * cgt;
  }
  if (tid == NT2) wtab[wpx] = -1;

  // cell E*kk + j of the K order -> its byte in a weight row, or in a row
  // block's fragments (-1: padding of K, zero weights), its window's byte
  // offset (buffer, tap) and tap offset in pixels | cell in the pixel << 16
  // for the swizzle
  for (int i = tid; tid < NT2 && i < nst * SK * E; i += NT2) {
    int kk = i / E;
    const bool past = kk >= g.nkk;
    if (past) kk = g.nkk - 1;
    const int ch = fdiv(kk, g.div_nks);
    const int un = E * (kk - ch * g.nks) + (i & (E - 1));
    const int tap = fdiv(un, g.div_u);
    const int cu = un - tap * g.u;
    const bool ok = !past && tap < ntaps && ch * g.u + cu < cgt;
    const int c = ok ? cu : 0;
    const int r = fdiv(tap, g.div_kw);
    const int off = ok ? r * g.win + (tap - r * a.kw) : 0;
    ktab_a[i] = !ok ? -1 : FR ? ((ch * g.u + c) * ntaps + tap) * 2048 : (tap * cgt + ch * g.u + c) * 16;
    ktab_b[i] = int2{off * pitch + (ch % g.nbuf) * g.wcells * CB, off | (c << 16)};
  }
  if (tid == 0) *unsorted = 0;

  // the lane's output pixels as window pixels (those past the tile read the
  // last one's; their sums are never stored)
  int pb[FN];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    int pl = wn * 32 * FN + fn * 32 + l32;
    pl = pl < npx ? pl : npx - 1;
    if (g.one) {
      pb[fn] = pl;
    } else {
      const int p = p0 + pl;
      const int img = fdiv(p, a.div_howo);
      const int rem = p - img * howo;
      const int oy = fdiv(rem, a.div_wo);
      const int ox = rem - oy * a.wo;
      const int row = img == nf ? (oy - oyf) * a.stride
                                : r0 + (img - nf - 1) * g.rimg + oy * a.stride;
      pb[fn] = row * g.win + ox * a.stride;
    }
  }
  __syncthreads();

  // Loads chunk ch's window into buffer ch % nbuf, four loads' table reads at
  // a time; returns this wave's count of loads.
  auto issue_win = [&](int ch) {
    const uint32_t wb = win0 + (uint32_t)((ch % g.nbuf) * g.wcells * CB);
    const int cstr = b64 ? hw : 1;               // cells between a pixel's channel blocks
    const uint8_t* xc = a.x + (int64_t)ch * g.u * cstr * CB;
    int cnt = 0;
    for (int i0 = wave; i0 < ncw; i0 += 4 * NW) {
      int cell[4], c[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int ci = (i0 + k * NW) * 64 + lane;
        const int q = fdiv(ci, g.div_u);
        cell[k] = wtab[q < wpx ? q : wpx];
        c[k] = (ci - q * g.u) ^ ((q >> g.sh) & g.msk);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int i = i0 + k * NW;
        if (i >= ncw) break;
        const bool none = cell[k] < 0 || ch * g.u + c[k] >= cgt;
        const uint8_t* src = none ? zero_src : xc + (uint32_t)(cell[k] + c[k] * cstr) * CB;
        if constexpr (CB == 16) dma16(src, wb + (uint32_t)i * 1024);
        else dma4(src, wb + (uint32_t)i * 256);
        ++cnt;
      }
    }
    return cnt;
  };

  // The wave's weight loads: 1 KB chunk wave + NW*i of a stage is 16 rows of
  // one K64 step, four lanes to a row, slot j of row r holding unit
  // j ^ ((r >> 2) & 3); in fragment order a K32 half of 32 rows as it is.
  // Rows are fixed; the unit's byte comes from the table, read a stage ahead.
  int arow[CPW], aent[CPW], anext[CPW];
  const int azero = (int)a.wzero + lane * 16;
#pragma unroll
  for (int i = 0; i < CPW; ++i) {
    const int c = wave + NW * i;
    const int s_ = c / CA1;
    const int rg = c - s_ * CA1;
    if constexpr (FR) {
      const int rb = (co0 >> 5) + (rg >> 1);
      arow[i] = rb * 32 < a.cout_pad ? (rb * 2 * a.nk + (rg & 1)) * 1024 + lane * 16 : -1;
      aent[i] = s_;
    } else {
      const int row = rg * 16 + (lane >> 2);
      arow[i] = co0 + rg * 16 < a.cout_pad ? (co0 + row) * a.kpad : -1;
      aent[i] = s_ * 4 + ((lane & 3) ^ ((row >> 2) & 3));
    }
    anext[i] = ktab_a[aent[i]];
  }
  // Weight chunk i of stage st into ring slot st % D (stages in order).
  auto issue_a = [&](int st, int i) {
    const uint32_t slot = ring0 + (uint32_t)((st % D) * STAGE);
    const int nx = st + 1 < nst ? (st + 1) * SK * E : 0;
    const int off = (anext[i] | arow[i]) < 0 ? azero : arow[i] + anext[i];
    dma16s(a.wgt, (uint32_t)off, slot + (uint32_t)(wave + NW * i) * 1024);
    anext[i] = ktab_a[nx + aent[i]];
  };

  v16i acc[FM][FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = v16i{0};

  // the lane's weight fragments of K32 step t (units 2t + h): row l32 of each
  // block; in fragment order 1 KB a block and K32 step
  constexpr int ABLK = FR ? 2048 : 32 * 64;      // bytes between 32-row blocks
  int aoff[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
    aoff[t] = wm * FM * ABLK + (FR ? t * 1024 + lane * 16
                                   : l32 * 64 + (((2 * t + h) ^ ((l32 >> 2) & 3)) << 4));

  int pbp[FN];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) pbp[fn] = __umul24(pb[fn], pitch) + g.win_off;
  // the window offsets of a wave's K32 steps of a stage (of its K64 steps
  // where a cell holds both halves)
  constexpr int NT = FR ? 1 : 2;
  const int2* kb = ktab_b + kg * S * E + (FR ? 0 : h);
  int2 bnext[S][NT];
#pragma unroll
  for (int s_ = 0; s_ < S; ++s_)
#pragma unroll
    for (int t = 0; t < NT; ++t) bnext[s_][t] = kb[s_ * E + 2 * t];

  // One stage. The weight loads of stage st + D - 1 are issued between the
  // MFMA groups: the eight waves' loads queue at the CU's one address unit
  // (16 clocks each at least), and a wave that issued them first would stand
  // there with its matrix core idle.
  constexpr int NSUB = 2 * S;                    // K32 steps of a wave and stage
  auto compute = [&](int st) {
    const uint8_t* as = lds + g.ring_off + (st % D) * STAGE + kg * S * A_STEP;
    const bool more = st + D - 1 < nst;
    v4i af[NSUB][FM], bf[NSUB][FN];
    uint32_t braw[NSUB][FN];
    const int nx = st + 1 < nst ? (st + 1) * SK * E : 0;
    // fragments of K32 step j; a step's table entries are refilled for the
    // next stage once its last half has used them
    auto load = [&](int j) {
      const int s_ = j >> 1, t = j & 1;
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
        af[j][fm] = *reinterpret_cast<const v4i*>(as + s_ * A_STEP + aoff[t] + fm * ABLK);
      if (!FR || t == 0) {
        const int2 e = bnext[s_][FR ? 0 : t];
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
          const int sw = ((pb[fn] + (e.y & 0xFFFF)) >> g.sh) & g.msk;
          const uint8_t* src = lds + pbp[fn] + e.x + ((e.y >> 16) ^ sw) * CB;
          if constexpr (IN == kWinI8) {
            bf[j][fn] = *reinterpret_cast<const v4i*>(src);
          } else if constexpr (FR) {
            const v2i r = *reinterpret_cast<const v2i*>(src + 8 * h);
            braw[j][fn] = (uint32_t)r.x;
            braw[j + 1][fn] = (uint32_t)r.y;
          } else {
            braw[j][fn] = *reinterpret_cast<const uint32_t*>(src);
          }
        }
      }
      if (t == 1) {
#pragma unroll
        for (int q = 0; q < NT; ++q) bnext[s_][q] = kb[nx + s_ * E + 2 * q];
      }
    };
    load(0);
    load(1);
#pragma unroll
    for (int j = 0; j < NSUB; ++j) {
      if (j > 0 && j + 1 < NSUB) load(j + 1);
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        if constexpr (IN != kWinI8) bf[j][fn] = unpack2(braw[j][fn]);
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
          acc[fm][fn] =
              __builtin_amdgcn_mfma_i32_32x32x32_i8(af[j][fm], bf[j][fn], acc[fm][fn], 0, 0, 0);
      }
      if (more) {
#pragma unroll
        for (int i = 0; i < CPW; ++i)
          if (i * NSUB / CPW == j) issue_a(st + D - 1, i);
      }
    }
  };

  issue_win(0);
  int nwin = 1;                                  // windows issued
  const int pre = nst < D - 1 ? nst : D - 1;
  for (int st = 0; st < pre; ++st)
#pragma unroll
    for (int i = 0; i < CPW; ++i) issue_a(st, i);
  // in flight beside the loop's first stages; the compiler's own wait for
  // these loads also waits for the prologue's
  stage_heaps<64 * NW>(a, lds, co0, BM, unsorted);
  int hist[D - 2];                               // window loads of the last iterations
#pragma unroll
  for (int i = 0; i < D - 2; ++i) hist[i] = 0;
  for (int st = 0; st < nst; ++st) {
    int after = (nst - 1 - st < D - 2 ? nst - 1 - st : D - 2) * CPW;
#pragma unroll
    for (int i = 0; i < D - 2; ++i) after += hist[i];
    if (after == (D - 2) * CPW) wait_vmcnt<(D - 2) * CPW>();
    else wait_vmcnt_le(after);
    __syncthreads();                             // stage st landed; slot st-1 free
#pragma unroll
    for (int i = D - 3; i > 0; --i) hist[i] = hist[i - 1];
    hist[0] = 0;
    // one more window where its buffer's last chunk is done
    if (nwin < g.nch && (nwin < g.nbuf || st * SK >= (nwin - g.nbuf + 1) * g.nks)) {
      hist[0] = issue_win(nwin);
      ++nwin;
    }
    compute(st);
  }
  wait_vmcnt<0>();
  __syncthreads();
  if (*unsorted) {
    sort_heaps(a, lds, co0, BM);
    __syncthreads();
  }

  // ---- epilogue: quads of four consecutive channels of one pixel ----
  // Accumulator block (fm, fn) is four quads per lane; quad lb = (fm*FN +
  // fn)*4 + j of a wave. The WK waves with the same tile part share out its
  // quads: each keeps those it owns, hands the others over in LDS and adds
  // what the others hand to it.
  constexpr int NBL = FM * FN * 4;
  constexpr int NOWN = (NBL + WK - 1) / WK;
  const int orow = win_orow(a, BM);
  uint8_t* otile = lds + g.out_off;
  int own[NOWN][4];
  if constexpr (WK == 1) {
#pragma unroll
    for (int lb = 0; lb < NBL; ++lb)
#pragma unroll
      for (int i = 0; i < 4; ++i) own[lb][i] = acc[lb / (4 * FN)][(lb / 4) % FN][4 * (lb & 3) + i];
  } else {
    uint8_t* red = lds + g.red_off + wig * NBL * 1024 + lane * 16;
    constexpr int KSTR = NWG * NBL * 1024;       // one K group's sums
#pragma unroll
    for (int lb = 0; lb < NBL; ++lb) {
      const v16i& b = acc[lb / (4 * FN)][(lb / 4) % FN];
      const v4i q = v4i{b[4 * (lb & 3)], b[4 * (lb & 3) + 1], b[4 * (lb & 3) + 2],
                        b[4 * (lb & 3) + 3]};
      if (lb % WK == kg) {
#pragma unroll
        for (int i = 0; i < 4; ++i) own[lb / WK][i] = q[i];
      } else {
        *reinterpret_cast<v4i*>(red + kg * KSTR + lb * 1024) = q;
      }
    }
    __syncthreads();
    if (NBL % WK == 0 || kg < NBL) {
#pragma unroll
      for (int o = 0; o < NOWN; ++o)
#pragma unroll
        for (int k = 1; k < WK; ++k) {
          const int src = (kg + k) % WK;
          const v4i q = *reinterpret_cast<const v4i*>(red + src * KSTR + (o * WK + kg) * 1024);
#pragma unroll
          for (int i = 0; i < 4; ++i) own[o][i] += q[i];
        }
    }
  }
  auto finish = [&](auto mode, auto lv) {
    constexpr int MODE = decltype(mode)::value;
    constexpr int LV = decltype(lv)::value;
    constexpr int NB = NOWN < 4 ? NOWN : 4;      // quads in flight
#pragma unroll
    for (int o0 = 0; o0 < NOWN; o0 += NB) {
      int d[NB][4];
      int cl[NB], pl[NB];
      bool ok[NB];
#pragma unroll
      for (int o = 0; o < NB; ++o) {
        const int lb = WK == 1 ? o0 + o : (o0 + o) * WK + kg;
        const int f = lb >> 2;
        cl[o] = (wm * FM + f / FN) * 32 + 8 * (lb & 3) + 4 * h;
        pl[o] = (wn * FN + f % FN) * 32 + l32;
        ok[o] = lb < NBL && co0 + cl[o] < a.cout && pl[o] < npx;
        if (ok[o]) quad_in<MODE>(a, co0 + cl[o], p0 + pl[o], d[o]);
      }
#pragma unroll
      for (int o = 0; o < NB; ++o) {
        if (!ok[o]) continue;
        if (a.acc_dump) {
          int32_t* dump = a.acc_dump + (int64_t)(p0 + pl[o]) * a.cout + co0 + cl[o];
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (co0 + cl[o] + i < a.cout) dump[i] = own[o0 + o][i];
        }
        quad_out<MODE, LV>(a, lds, own[o0 + o], d[o], cl[o], co0 + cl[o], pl[o], p0 + pl[o], otile,
                           orow);
      }
    }
  };
#define IFQ_C(k) std::integral_constant<int, k>{}
  if (a.out_mode == 0) {
    finish(IFQ_C(kEpiI32), IFQ_C(0));
    return;
  }
  if (a.join_kind == IFQ_JOIN_CONV) {
    finish(IFQ_C(kEpiJoinConv), IFQ_C(0));
  } else if (a.join_kind == IFQ_JOIN_IDENTITY) {
    if (a.rec == 4) finish(IFQ_C(kEpiTab), IFQ_C(2)); else finish(IFQ_C(kEpiTab), IFQ_C(0));
  } else if (a.rec == 4) {
    finish(IFQ_C(kEpiThr), IFQ_C(2));
  } else if (a.rec == 8) {
    finish(IFQ_C(kEpiThr), IFQ_C(3));
  } else if (a.rec == 16) {
    finish(IFQ_C(kEpiThr), IFQ_C(4));
  } else {
    finish(IFQ_C(kEpiThr), IFQ_C(0));
  }
#undef IFQ_C
  __syncthreads();
  copy_out_tile(a, otile, orow, co0, BM, p0, npx);
}

// ---- Variants and planning --------------------------------------------------
struct WinVariant {
  int wm, wn, wk, fm, fn, s, d;
  const char* name[3];
};
#define IFQ_WV(wm, wn, wk, fm, fn, s, d)                                        \
  {wm, wn, wk, fm, fn, s, d,                                                     \
   {"conv_win<0, " #wm ", " #wn ", " #wk ", " #fm ", " #fn ", " #s ", " #d ">",  \
    "conv_win<1, " #wm ", " #wn ", " #wk ", " #fm ", " #fn ", " #s ", " #d ">",  \
    "conv_win<2, " #wm ", " #wn ", " #wk ", " #fm ", " #fn ", " #s ", " #d ">"}}
const WinVariant kWin[] = {
    IFQ_WV(2, 4, 1, 2, 2, 2, 3),   // 128 x 256, K split 1
    IFQ_WV(2, 2, 2, 2, 1, 2, 3),   // 128 x 64, K split 2
    IFQ_WV(1, 4, 2, 2, 2, 2, 3),   // 64 x 256, K split 2
    IFQ_WV(1, 4, 2, 2, 1, 2, 3),   // 64 x 128, K split 2
    IFQ_WV(1, 4, 2, 1, 2, 2, 3),   // 32 x 256, K split 2
    IFQ_WV(1, 2, 4, 2, 1, 1, 3),   // 64 x 64, K split 4
    IFQ_WV(1, 2, 4, 1, 1, 2, 3),   // 32 x 64, K split 4
    IFQ_WV(1, 2, 4, 1, 1, 1, 4),   // 32 x 64, K split 4
    IFQ_WV(1, 1, 8, 1, 1, 1, 3),   // 32 x 32, K split 8
};
constexpr int kNumWin = sizeof(kWin) / sizeof(kWin[0]);
constexpr int kWinLds = 160 * 1024;

int win_in(const ConvLaunch& a) {
  return a.in_layout == IFQ_LAYOUT_I8_NHWC ? kWinI8 : a.cin % 64 ? kWinU2 : kWinF;
}

struct WinPlan {
  int variant;
  int lds_bytes;
  WinGeom g;
  double t_us;      // ranks the variants
  double est_us;    // the chosen one's time, to weigh it against another kernel
};

// Predicted time of a plan, to compare with another kernel's: tiles of bm x bnmax
// outputs on the busiest CU, one, two or three at once where LDS holds them (two
// cost 1.36, three 1.75 of one); per tile a fixed part and an epilogue by kind,
// window loads, weight stages (barrier and latency, matrix cores) and K-group sums;
// int32 sums the time of their bytes, which are the layer's largest stream. Fitted
// to the variants that t_us picks, on 5366 layers in fragment order (1x1 to 5x5,
// every output and join; 5.1% rms) and 2000 byte and packed ones (7.2%).
// t_us is 15 to 30% off on filters of one tap or a few, which it was not fitted to,
// but ranks the variants a little better than this does (1.0% behind the best one on
// average against 1.2%, 1.1 against 1.5 on byte codes).
double win_estimate(const ConvLaunch& a, const WinVariant& V, const WinGeom& g, int64_t tiles,
                    int64_t lds, bool fr) {
  struct Kind {
    double tile, epi;       // us a tile, us per 512 of its outputs
  };
  // codes of up to 2 bits, sums, identity join, wider codes, those with the join,
  // conv join
  static const Kind kF[] = {{1.784, 0.076}, {1.158, 0}, {1.969, 0.127},
                            {1.808, 0.129}, {2.356, 0.314}, {2.563, 0.328}};
  static const Kind kR[] = {{1.748, 0.085}, {1.181, 0}, {1.992, 0.143},
                            {1.833, 0.127}, {2.535, 0.335}, {2.527, 0.321}};
  const bool id = a.join_kind == IFQ_JOIN_IDENTITY;
  const int kind = a.join_kind == IFQ_JOIN_CONV ? 5
                   : a.out_mode == 0            ? 1
                   : a.rec <= 4                 ? (id ? 2 : 0)
                                                : (id ? 4 : 3);
  const Kind& k = fr ? kF[kind] : kR[kind];
  const int bm = 32 * V.fm * V.wm, bnmax = 32 * V.fn * V.wn, sk = V.s * V.wk;
  const int nst = (g.nkk + sk - 1) / sk;
  const double outs = (double)bm * bnmax;
  const int rows = (a.cout + 31) / 32 * 32 < bm ? (a.cout + 31) / 32 * 32 : bm;
  const double loads = (double)g.nch * g.wcells / 64 / 8;
  const double mfma = outs * sk / 64 / 2150, red = (V.wk - 1) * outs * 4 / 200 / 2150;
  const double one = k.tile + k.epi * rows * g.bn / 512 +
                     (fr ? 0.090 * loads + nst * (0.337 + 1.536 * mfma) + 2.956 * red
                         : 0.118 * loads + nst * (0.240 + 1.551 * mfma) + 4.592 * red);
  static const double share[] = {0, 1, 1.36, 1.75};
  const int64_t per_cu = (tiles + kPlanCUs - 1) / kPlanCUs;
  const int occ = kWinLds / lds < 3 ? (int)(kWinLds / lds) : 3;
  const double rounds = (double)(per_cu / occ) * share[occ] + share[per_cu % occ];
  const double sums = a.out_mode == 0 ? 4.0 * a.m * a.cout / kSumBytesPerUs : 0;
  return (fr ? 2.199 : 2.128) + rounds * one + 1.15 * sums;
}

// Most window rows any tile of bn consecutive output pixels needs: the output
// rows it can touch, stride input rows each, and the filter's overhang once
// per image.
int64_t win_rows_bound(const ConvLaunch& a, int64_t bn) {
  const int64_t howo = (int64_t)a.ho * a.wo;
  int64_t rows = (bn - 1 + a.wo - 1) / a.wo + 1, imgs = (bn - 1 + howo - 1) / howo + 1;
  if (bn % howo == 0) {
    rows = bn / a.wo;
    imgs = bn / howo;
  }
  if (rows > (int64_t)a.n * a.ho) rows = (int64_t)a.n * a.ho;
  if (imgs > a.n) imgs = a.n;
  const int64_t over = a.kh > a.stride ? a.kh - a.stride : 0;
  return rows * a.stride + imgs * over;
}

// Fits variant v: the chunk width and buffers that hold the windows in LDS.
bool fit_win(const ConvLaunch& a, int v, WinPlan* out) {
  const WinVariant& V = kWin[v];
  const int bm = 32 * V.fm * V.wm, bnmax = 32 * V.fn * V.wn, sk = V.s * V.wk;
  const bool fr = win_in(a) == kWinF;
  const int cb = win_in(a) == kWinU2 ? 4 : 16, e = fr ? 1 : 4;
  const int64_t nco = (a.cout + bm - 1) / bm;
  const int64_t nb_min = (a.m + bnmax - 1) / bnmax;
  const int64_t rounds = (nco * nb_min + kPlanCUs - 1) / kPlanCUs;
  int64_t nb = rounds * kPlanCUs / nco;
  if (nb < nb_min) nb = nb_min;
  int64_t bn = ((a.m + nb - 1) / nb + 31) / 32 * 32;
  if (bn > bnmax) bn = bnmax;
  const int cgt = a.cin / (fr ? 64 : 16), ntaps = a.kh * a.kw;   // cells per pixel, taps
  const bool one = ntaps == 1;
  const int64_t wincols = one ? 1 : (int64_t)(a.wo - 1) * a.stride + a.kw;
  const int64_t wpx = one ? bn : win_rows_bound(a, bn) * wincols;
  if (wpx * cgt >= (1 << 23) || wpx >= (1 << 15)) return false;   // table fields
  const int prm = (win_param_bytes(a, bm) + 16 + 1023) / 1024 * 1024;
  const int ring = V.d * sk * bm * 64;
  const int64_t tab = (wpx * 4 + 4 + 1023) / 1024 * 1024;
  const int64_t red = V.wk > 1 ? (int64_t)V.wk * bm * bnmax * 4 : 0;
  const int64_t otile = a.out_mode == 0 ? 0 : (int64_t)bnmax * win_orow(a, bm);
  if (prm + red + otile > kWinLds || (int64_t)a.cout_pad * a.kpad >= ((int64_t)1 << 30)) return false;
  // the narrowest chunk whose K64 steps keep the ring busy while the next
  // window loads and pad K by at most 4% (16%, then 60%, where no such chunk
  // fits), or all channels at once; chunks of whole 64-byte spans of the
  // weight rows where c_in allows it
  const int kPad[] = {104, 116, 160};
  for (int pass = 0; pass < 3 * cgt; ++pass) {
    const int u = pass % cgt + 1;
    if (!fr && cgt % 4 == 0 && u % 4) continue;
    const int nch = (cgt + u - 1) / u;
    const int nks = (ntaps * u + e - 1) / e;
    if (nch > 1 && (nks < V.d * sk ||
                    (int64_t)100 * e * nks * nch > (int64_t)kPad[pass / cgt] * ntaps * cgt))
      continue;
    const int64_t wcells = (wpx * u + 63) / 64 * 64;
    const int64_t ktab = ((int64_t)(nch * nks + sk - 1) / sk * sk * 12 * e + 1023) / 1024 * 1024;
    const int64_t room = kWinLds - prm - ring - tab - ktab;
    const int64_t fitb = room / (wcells * cb);
    if (fitb < (nch > 1 ? 2 : 1)) continue;
    WinGeom& g = out->g;
    std::memset(&g, 0, sizeof(g));
    g.u = u;
    g.nch = nch;
    g.nbuf = (int)(nch <= 2 ? nch : (fitb < 3 ? 2 : 3));
    g.nks = nks;
    g.nkk = nch * nks;
    g.win = (int)wincols;
    g.rimg = (a.ho - 1) * a.stride + a.kh;
    g.wcells = (int)wcells;
    g.one = one;
    // bank swizzle over the low bits of the unit: neighbouring pixels pass
    // over the 64 banks, 16 lanes of 16 bytes or 32 of 4 at a time (16-byte
    // reads measured 4 clocks a wave so, 8 with a swizzle over 8 lanes)
    const int lg = cb == 16 ? 4 : 5;
    int z = 0;
    while (z < lg && u % (2 << z) == 0) ++z;
    g.msk = (1 << z) - 1;
    g.sh = lg - z;
    g.ring_off = prm;
    g.win_off = prm + ring;
    g.tab_off = (int)(g.win_off + g.nbuf * wcells * cb);
    g.ktab_off = (int)(g.tab_off + tab);
    g.red_off = prm;
    g.out_off = (int)(prm + red);
    g.bn = (int)bn;
    g.div_u = make_fastdiv(u);
    g.div_win = make_fastdiv(g.win);
    g.div_rimg = make_fastdiv(g.rimg);
    g.div_nks = make_fastdiv(nks);
    g.div_kw = make_fastdiv(a.kw);
    out->variant = v;
    int64_t total = g.ktab_off + ktab;
    if (prm + red + otile > total) total = prm + red + otile;
    out->lds_bytes = (int)total;
    // predicted time to rank the variants by, in clocks of a tile: prologue and window loads, stages
    // (barrier and latency, matrix cores, weights through the address unit),
    // K-group sums, epilogue; two tiles on a CU at once where LDS holds two
    // cost 1.28 (1.36) of one. Fitted to 620 measured (layer, variant) times
    // over 65 byte and 2-bit layers, and to 390 over 45 in fragment order (9%
    // rms both; the choice is 2% slower than the best one).
    const int64_t tiles = nco * ((a.m + bn - 1) / bn);
    const int64_t per_cu = (tiles + kPlanCUs - 1) / kPlanCUs;
    const int nst = (g.nkk + sk - 1) / sk;
    const double loads = (double)(nch * wcells) / 64 / 8;
    const double outs = (double)bm * bnmax;
    const double red = (V.wk - 1) * outs * 4 / 200;
    double one_clk, pair, t0;
    if (fr) {
      const double epi = a.out_mode == 0 ? 215 : a.join_kind ? 221 : 118;
      one_clk = 2360 + 943 * loads + nst * (497 + 1.07 * outs * sk / 64 + 0.65 * bm * sk) +
                6.76 * red + epi * outs / 512;
      pair = 1.36;
      t0 = 2.35;
    } else {
      const double lv = a.rec == 8 || a.rec == 16 ? 3.0 : a.rec == 2 ? 1.5 : 1.0;
      one_clk = 4650 + 276 * loads + nst * (506 + 1.06 * outs * sk / 64 + 0.62 * bm * sk) +
                3.26 * red + 85 * lv * outs / 512;
      pair = 1.28;
      t0 = 1.5;
    }
    out->t_us = t0 + (2 * total <= kWinLds ? (per_cu / 2) * pair + per_cu % 2 : per_cu) * one_clk / 2150;
    out->est_us = win_estimate(a, V, g, tiles, total, fr);
    return true;
  }
  return false;
}

bool plan_win(const ConvLaunch& a, WinPlan* out) {
  bool found = false;
  for (int v = 0; v < kNumWin; ++v) {
    WinPlan p;
    if (fit_win(a, v, &p) && (!found || p.t_us < out->t_us)) {
      *out = p;
      found = true;
    }
  }
  return found;
}

PlanCache<WinPlan> g_win_plans;

bool choose_win(const ConvLaunch& a, WinPlan* out) { return g_win_plans.get(a, out, plan_win); }

template <int IN>
hipError_t launch_in(const ConvLaunch& a, const WinPlan& p, hipStream_t stream) {
  auto go = [&](auto kern) {
    const WinVariant& V = kWin[p.variant];
    const int bm = 32 * V.fm * V.wm;
    const dim3 grid((a.m + p.g.bn - 1) / p.g.bn, (a.cout + bm - 1) / bm);
    hipLaunchKernelGGL(kern, grid, dim3(64 * V.wm * V.wn * V.wk), p.lds_bytes, stream, a, p.g);
    return hipGetLastError();
  };
  switch (p.variant) {
    case 0: return go(conv_win<IN, 2, 4, 1, 2, 2, 2, 3>);
    case 1: return go(conv_win<IN, 2, 2, 2, 2, 1, 2, 3>);
    case 2: return go(conv_win<IN, 1, 4, 2, 2, 2, 2, 3>);
    case 3: return go(conv_win<IN, 1, 4, 2, 2, 1, 2, 3>);
    case 4: return go(conv_win<IN, 1, 4, 2, 1, 2, 2, 3>);
    case 5: return go(conv_win<IN, 1, 2, 4, 2, 1, 1, 3>);
    case 6: return go(conv_win<IN, 1, 2, 4, 1, 1, 2, 3>);
    case 7: return go(conv_win<IN, 1, 2, 4, 1, 1, 1, 4>);
    default: return go(conv_win<IN, 1, 1, 8, 1, 1, 1, 3>);
  }
}

}  // namespace

// Byte codes below 8 bits and 2-bit NHWC codes in the row-major weight layout,
// c_in a multiple of 16, the input aligned for the DMA's cells.
bool win_eligible(const ConvLaunch& a, double* t_us) {
  if (a.cin % 16 || a.m <= 0 || a.pool_k || a.join_kind == IFQ_JOIN_CONV_FUSED) return false;
  if (a.in_layout == IFQ_LAYOUT_I8_NHWC) {
    if (a.in_bits == 8 || ((uintptr_t)a.x & 15)) return false;
  } else if (a.in_layout != IFQ_LAYOUT_U2_NHWC_PACKED || a.cin % 64 == 0 ||
             ((uintptr_t)a.x & 3)) {
    return false;   // c_in % 64 == 0: the MFMA dispatcher's choice (plan_win_us)
  }
  WinPlan p;
  if (!choose_win(a, &p)) return false;
  *t_us = p.est_us;
  return true;
}

bool plan_win_us(const ConvLaunch& a, double* t_us) {
  WinPlan p;
  if (a.m <= 0 || a.pool_k || a.join_kind == IFQ_JOIN_CONV_FUSED || a.f4 || !choose_win(a, &p))
    return false;
  *t_us = p.est_us;
  return true;
}

const char* conv_win_name(const ConvLaunch& a) {
  WinPlan p;
  return choose_win(a, &p) ? kWin[p.variant].name[win_in(a)] : "";
}

hipError_t launch_conv_win(const ConvLaunch& a, hipStream_t stream) {
  WinPlan p;
  if (!choose_win(a, &p)) return hipErrorNotSupported;
  switch (win_in(a)) {
    case kWinI8: return launch_in<kWinI8>(a, p, stream);
    case kWinU2: return launch_in<kWinU2>(a, p, stream);
    default: return launch_in<kWinF>(a, p, stream);
  }
}

}  // namespace ifq
