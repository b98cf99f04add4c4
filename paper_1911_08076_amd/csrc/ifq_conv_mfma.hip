// Fast path of the integrated fixed-point quantized convolution on gfx950
// (MI355X): 2-bit input codes with c_in a multiple of 64, in the BLOCK64 or
// the NHWC packed layout. The tiled kernel (conv_mfma), which the next paragraphs
// are about, the one for fully connected layers (conv_fc, further down), and the
// choice among them and the other kernels of the fast path (plan_choice).
//
// The integer part of Eq. (1), a = W_b (x) X_q, is an implicit GEMM
// D[co][pixel] = sum_k W[co][k] * X[pixel][k] on v_mfma_i32_32x32x32_i8:
// A (rows = output channels) is the +-1 weight matrix in fragment order, B
// (columns = output pixels) the input codes of one filter tap and 64 channels
// per K64 step, unpacked from 2 bits to int8 in registers right before the
// MFMA. K runs over K64 steps kk = g*kh*kw + (r*kw + s) (G = c_in/64
// channel blocks g, filter taps (r, s) fastest).
//
// A workgroup of WM x WN x WK waves computes a tile of 32*FM*WM output
// channels x up to 32*FN*WN pixels (bn, chosen per layer on the host); the
// WK wave groups split the K64 steps and their sums are added in LDS at the
// end. Operands reach LDS through the LDS-DMA form of the global load (one
// wave instruction moves 64 x 16 bytes, lane i's bytes landing at base +
// 16*i, no staging registers): a weight chunk is 1 KB of fragments, a code
// chunk the 16-byte cells of 64 consecutive output pixels for one tap and
// 64 channels, which in the BLOCK64 layout is one contiguous 1 KB span for a
// stride-1 conv. A ring of D stages of S K64 steps per wave group keeps the
// loads of the next D-1 stages in flight while one computes; every wave
// issues the same number of loads per stage and waits for its part of a
// stage with an explicit vmcnt that leaves younger stages in flight.
// Out-of-range operands are read from blocks of zeros, so the main loop has
// no branch around a load.
//
// Accumulator layout (32x32 MFMA): lane l = 32*h + j holds, for register v,
// row 8*(v/4) + 4*h + v%4 and column j; each lane therefore holds groups of
// four consecutive output channels of one pixel, and the fused epilogue of
// ifq_epilogue.h turns them into codes with integer compares (Eq. 7/8) or the
// residual join without cross-lane traffic.
#include <hip/hip_runtime.h>

#include "ifq_epilogue.h"
#include "ifq_internal.h"
#include "ifq_mfma_common.h"

namespace ifq {
namespace {

template <int WM, int WN, int WK, int FM, int FN, int S, int D>
__global__ __launch_bounds__(64 * WM * WN * WK) void conv_mfma(ConvLaunch a) {
  constexpr int NWG = WM * WN;                  // waves per K group
  constexpr int NW = NWG * WK;
  constexpr int BM = 32 * FM * WM;
  constexpr int BN = 32 * FN * WN;
  constexpr int BNL = (BN + 63) / 64 * 64;      // pixels loaded per K64 step
  constexpr int A_STEP = BM * 64;               // BM/32 row blocks x 2 K32 x 1 KB
  constexpr int B_STEP = BNL * 16;
  constexpr int STEP = A_STEP + B_STEP;
  constexpr int SK = S * WK;                    // K64 steps per stage
  constexpr int STAGE = SK * STEP;
  constexpr int CA1 = BM / 16, CB1 = BNL / 64;  // 1 KB chunks per K64 step
  constexpr int C = SK * (CA1 + CB1);
  static_assert(C % NW == 0, "equal loads per wave");
  constexpr int CPW = C / NW;
  static_assert((D - 2) * CPW <= 63, "vmcnt range");
  constexpr int EPI_BYTES = epilogue_param_bytes(BM);  // per-channel parameters
  constexpr int OUT_BYTES = BN * BM;            // byte-per-code output tile
  constexpr int RED_BYTES = (WK / 2) * NWG * FM * FN * 4096;
  constexpr int LDS0 = D * STAGE > RED_BYTES ? D * STAGE : RED_BYTES;
  constexpr int LDS_BYTES = LDS0 > EPI_BYTES + OUT_BYTES ? LDS0 : EPI_BYTES + OUT_BYTES;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS");

  __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS_BYTES];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NWG;                    // K group
  const int wig = wave - kg * NWG;              // wave in group
  const int wm = wig % WM;
  const int wn = wig / WM;
  const int h = lane >> 5;
  const int l32 = lane & 31;
  const int bn = a.bn;
  const int p0 = blockIdx.x * bn;
  const int co0 = blockIdx.y * BM;
  const int G = a.cin >> 6;
  const int nk = a.nk;
  const int nk32 = 2 * nk;
  const int nst = (nk + SK - 1) / SK;
  const int rbw = co0 >> 5;                     // first row block
  const int nrb = a.cout_pad >> 5;
  const int howo = a.ho * a.wo;
  const uint8_t* wbase = reinterpret_cast<const uint8_t*>(a.wgt) + lane * 16;
  const uint8_t* zero_src = reinterpret_cast<const uint8_t*>(&g_zero_cell);
  const uint32_t lds0 = lds_addr(lds);

  // input strides in 16-byte cells: n, channel block, row, column
  int sN, sG, sH, sW;
  if (a.in_layout == IFQ_LAYOUT_U2_BLOCK64) {
    sW = 1; sH = a.w; sG = a.h * a.w; sN = G * sG;
  } else {
    sG = 1; sW = G; sH = a.w * G; sN = a.h * sH;
  }

  // The loads of wave w are chunks c = w + NW*i of a stage; for code chunks
  // the lane's pixel is fixed across stages, so its position is computed once.
  int px_base[CPW], px_iy0[CPW], px_ix0[CPW];
  bool px_ok[CPW];
#pragma unroll
  for (int i = 0; i < CPW; ++i) {
    const int c = wave + NW * i;
    const int cb = (c % (CA1 + CB1)) - CA1;     // code chunk index in the step
    px_ok[i] = false;
    px_base[i] = px_iy0[i] = px_ix0[i] = 0;
    if (cb >= 0) {
      const int pl = cb * 64 + lane;
      const int p = p0 + pl;
      if (pl < bn && p < a.m) {
        const int nimg = fdiv(p, a.div_howo);
        const int rem = p - nimg * howo;
        const int oy = fdiv(rem, a.div_wo);
        const int ox = rem - oy * a.wo;
        px_ok[i] = true;
        px_iy0[i] = oy * a.stride - a.pad;
        px_ix0[i] = ox * a.stride - a.pad;
        px_base[i] = nimg * sN + px_iy0[i] * sH + px_ix0[i] * sW;
      }
    }
  }

  // Filter tap (r, s) and channel block g of K64 step kk, kept incrementally
  // (taps fastest): kpos is the position of the first step of the next stage
  // to issue.
  struct KPos {
    int g, s, r;
  };
  auto adv1 = [&](KPos& q) {
    q.s += 1;
    const bool ws = q.s == a.kw;
    q.s = ws ? 0 : q.s;
    q.r += ws ? 1 : 0;
    const bool wr = q.r == a.kh;
    q.r = wr ? 0 : q.r;
    q.g += wr ? 1 : 0;
  };
  KPos kpos{0, 0, 0};

  // Issue the loads of stage st into ring slot st % D (stages are issued in
  // order). Chunk c covers K64 step kk = st*SK + c / (CA1 + CB1) of the
  // stage; within the step the first CA1 chunks are weights (row block, K32
  // half), the rest codes.
  auto issue = [&](int st) {
    const uint32_t slot = lds0 + (uint32_t)((st % D) * STAGE);
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
      const int c = wave + NW * i;
      const int s_ = c / (CA1 + CB1);
      const int local = c - s_ * (CA1 + CB1);
      const int kk = st * SK + s_;
      const uint32_t dst = slot + (uint32_t)(s_ * STEP + local * 1024);
      if (local < CA1) {
        const int rb = local >> 1, t = local & 1;
        const bool ok = kk < nk && rbw + rb < nrb;
        const int64_t off = ok ? ((int64_t)(rbw + rb) * nk32 + 2 * kk + t) * 1024 : a.wzero;
        dma16(wbase + off, dst);
      } else {
        KPos q = kpos;
        for (int u = 0; u < s_; ++u) adv1(q);
        const int g = q.g, r = q.r, s = q.s;
        const int iy = px_iy0[i] + r;
        const int ix = px_ix0[i] + s;
        const bool ok = kk < nk && px_ok[i] && (unsigned)iy < (unsigned)a.h &&
                        (unsigned)ix < (unsigned)a.w;
        const uint8_t* src =
            ok ? a.x + (int64_t)(px_base[i] + g * sG + r * sH + s * sW) * 16 : zero_src;
        dma16(src, dst);
      }
    }
#pragma unroll
    for (int u = 0; u < SK; ++u) adv1(kpos);
  };

  v16i acc[FM][FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = v16i{0};

  // K64 steps beyond nk multiply zero weight fragments: no branch here.
  auto compute = [&](int st) {
    const uint8_t* sb = lds + (st % D) * STAGE + kg * S * STEP;
#pragma unroll
    for (int s_ = 0; s_ < S; ++s_) {
      const uint8_t* as = sb + s_ * STEP;
      const uint8_t* bs = as + A_STEP;
      v2i braw[FN];
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
        braw[fn] = *reinterpret_cast<const v2i*>(
            bs + (wn * 32 * FN + fn * 32 + l32) * 16 + 8 * h);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        v4i af[FM];
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
          af[fm] = *reinterpret_cast<const v4i*>(as + ((wm * FM + fm) * 2 + t) * 1024 +
                                                 lane * 16);
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
          const v4i bf = unpack2((uint32_t)braw[fn][t]);
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
            acc[fm][fn] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[fm], bf, acc[fm][fn],
                                                                0, 0, 0);
        }
      }
    }
  };

  const int pre = nst < D - 1 ? nst : D - 1;
  for (int st = 0; st < pre; ++st) issue(st);
  for (int st = 0; st < nst; ++st) {
    const int issued_after = nst - 1 - st;      // stages issued after st, capped
    wait_ahead<D - 2, CPW>(issued_after < D - 2 ? issued_after : D - 2);
    __syncthreads();                            // every wave's part landed; slot st-1 free
    if (st + D - 1 < nst) issue(st + D - 1);
    compute(st);
  }
  wait_vmcnt<0>();
  __syncthreads();

  // K groups: sums of groups half..2*half-1 are added into groups 0..half-1
  if constexpr (WK > 1) {
#pragma unroll
    for (int half = WK / 2; half >= 1; half /= 2) {
      if (kg >= half && kg < 2 * half) {
        uint8_t* dst = lds + (((kg - half) * NWG + wig) * FM * FN) * 4096;
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int fn = 0; fn < FN; ++fn)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              *reinterpret_cast<v4i*>(dst + (fm * FN + fn) * 4096 + j * 1024 + lane * 16) =
                  v4i{acc[fm][fn][4 * j], acc[fm][fn][4 * j + 1], acc[fm][fn][4 * j + 2],
                      acc[fm][fn][4 * j + 3]};
      }
      __syncthreads();
      if (kg < half) {
        const uint8_t* src = lds + ((kg * NWG + wig) * FM * FN) * 4096;
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int fn = 0; fn < FN; ++fn)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const v4i v = *reinterpret_cast<const v4i*>(src + (fm * FN + fn) * 4096 +
                                                          j * 1024 + lane * 16);
              acc[fm][fn][4 * j] += v.x;
              acc[fm][fn][4 * j + 1] += v.y;
              acc[fm][fn][4 * j + 2] += v.z;
              acc[fm][fn][4 * j + 3] += v.w;
            }
      }
      __syncthreads();
    }
  }

  stage_epilogue(a, lds, co0, BM);
  __syncthreads();
  const int orow = a.out_mode == 2 ? BM / 4 : BM;
  uint8_t* otile = lds + EPI_BYTES;
  if (kg == 0) {
    const bool fast = (a.cout & 31) == 0 && (a.out_mode == 0 || a.rec == 4);
    if (fast) {
      int32_t* y32 = reinterpret_cast<int32_t*>(a.y);
      if (a.acc_dump)
        epilogue32<kE32I32, FM, FN>(a, lds, acc, wm, wn, h, l32, co0, p0, bn, otile, orow,
                                    a.acc_dump);
      if (a.out_mode == 0)
        epilogue32<kE32I32, FM, FN>(a, lds, acc, wm, wn, h, l32, co0, p0, bn, otile, orow, y32);
      else if (a.join_kind == IFQ_JOIN_IDENTITY)
        epilogue32<kE32Tab4, FM, FN>(a, lds, acc, wm, wn, h, l32, co0, p0, bn, otile, orow, y32);
      else if (a.join_kind == IFQ_JOIN_CONV)
        epilogue32<kE32Conv, FM, FN>(a, lds, acc, wm, wn, h, l32, co0, p0, bn, otile, orow, y32);
      else
        epilogue32<kE32Thr4, FM, FN>(a, lds, acc, wm, wn, h, l32, co0, p0, bn, otile, orow, y32);
    } else {
      epilogue_lane<FM * 4, FN>(
          a, lds, [&](int g, int fn, int i) { return acc[g >> 2][fn][4 * (g & 3) + i]; },
          [&](int g) { return co0 + (wm * FM + (g >> 2)) * 32 + 8 * (g & 3) + 4 * h; }, co0,
          p0,
          [&](int fn) {
            const int pl = wn * 32 * FN + fn * 32 + l32;
            return (pl < bn && p0 + pl < a.m) ? pl : -1;
          },
          otile, orow);
    }
  }
  __syncthreads();
  const int npx = a.m - p0 < bn ? a.m - p0 : bn;
  copy_out_tile(a, otile, orow, co0, BM, p0, npx);
}

// Fully connected layers: one filter window covering the whole image (kh == h,
// kw == w, no padding), so a layer is a product of n pixels with a weight
// matrix that is read once. AlexNet's first one is 38 MB of weights for 32
// images: HBM bounds it, and what it needs is many bytes in flight from every
// CU. A workgroup takes 16 output channels (256 workgroups for 4096) and 16*NB
// images; its eight waves split the groups of four K64 steps, each loading
// weight fragments and codes straight into registers, two batches of U groups
// ahead of the MFMAs (v_mfma_i32_16x16x64_i8), with no LDS and no barrier
// until the sums are added. Lane 16*q + r takes step q of a group for weight
// row and image r, so one 16-byte load holds its codes for all four of the
// group's MFMAs, the m-th of which contracts unit m of the four steps.
// Measured at batch 32, calls in a row: 6x6x256 -> 4096 on the 64 x 128 tiles above
// 43.0 us, here 9.5 us (4.0 TB/s of weights); 1x1x4096 -> 4096 23.6 and 5.9 us, -> 1000
// sums 21.5 and 4.5 us.
struct FcGeom {
  int32_t sn, sg, st;    // cells between images, channel blocks, taps
  FastDiv div_taps;
};

template <int NB>
__global__ __launch_bounds__(512) void conv_fc(ConvLaunch a, FcGeom g) {
  constexpr int NW = 8, U = 3;
  constexpr int SUMS = NW * NB * 1024;
  __shared__ __attribute__((aligned(16))) uint8_t lds[SUMS + 1024];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, r = lane & 15;
  const int co0 = blockIdx.x * 16, p0 = blockIdx.y * 16 * NB;
  const int ntaps = a.kh * a.kw;
  const int ng = (a.nk + 3) / 4;
  const int s0 = wave * ng / NW, s1 = (wave + 1) * ng / NW;   // this wave's groups

  // the tile's threshold records, in flight beside the main loop's loads
  const int nthr = (a.cout - co0 < 16 ? a.cout - co0 : 16) * a.rec;
  const int32_t trec = a.out_mode && tid < nthr ? a.thr[(int64_t)co0 * a.rec + tid] : 0;

  const uint8_t* wl = reinterpret_cast<const uint8_t*>(a.wgt) +
                      (int64_t)(co0 >> 5) * 2 * a.nk * 1024 + ((co0 & 16) + r) * 16;
  const uint8_t* xl[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int p = p0 + 16 * b + r < a.m ? p0 + 16 * b + r : a.m - 1;
    xl[b] = a.x + (int64_t)p * g.sn * 16;
  }
  v4i acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = v4i{0, 0, 0, 0};

  struct Batch {
    v4i w[U][4];
    v4i x[U][NB];
  };
  // steps past the last read the last one again, with zero codes
  auto load = [&](Batch& t, int s) {
#pragma unroll
    for (int j = 0; j < U; ++j) {
      if (s + j >= s1) break;
      const int k = 4 * (s + j) + q;
      const int kk = k < a.nk ? k : a.nk - 1;
      const int cb = fdiv(kk, g.div_taps);
      const int64_t cell = (int64_t)cb * g.sg + (int64_t)(kk - cb * ntaps) * g.st;
#pragma unroll
      for (int m = 0; m < 4; ++m)
        t.w[j][m] = *reinterpret_cast<const v4i*>(wl + (int64_t)kk * 2048 + (m & 1) * 1024 +
                                                  (m >> 1) * 512);
#pragma unroll
      for (int b = 0; b < NB; ++b) t.x[j][b] = *reinterpret_cast<const v4i*>(xl[b] + cell * 16);
    }
  };
  auto compute = [&](const Batch& t, int s) {
#pragma unroll
    for (int j = 0; j < U; ++j) {
      if (s + j >= s1) break;
      const uint32_t in = 4 * (s + j) + q < a.nk ? ~0u : 0u;
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
              t.w[j][m], unpack2((uint32_t)t.x[j][b][m] & in), acc[b], 0, 0, 0);
    }
  };
  Batch t0, t1;
  load(t0, s0);
  load(t1, s0 + U);
  __builtin_amdgcn_sched_barrier(0);   // every load before the first MFMA
  for (int s = s0; s < s1; s += 2 * U) {
    compute(t0, s);
    load(t0, s + 2 * U);
    compute(t1, s + U);
    load(t1, s + 3 * U);
  }

  // lane: channels 4q .. 4q+3 of image r of each block
#pragma unroll
  for (int b = 0; b < NB; ++b)
    *reinterpret_cast<v4i*>(lds + (wave * NB + b) * 1024 + lane * 16) = acc[b];
  int32_t* rec = reinterpret_cast<int32_t*>(lds + SUMS);
  if (tid < 256) rec[tid] = trec;
  __syncthreads();
  if (tid >= 64 * NB) return;
  v4i v = v4i{0, 0, 0, 0};
#pragma unroll
  for (int w = 0; w < NW; ++w)
    v += *reinterpret_cast<const v4i*>(lds + (w * NB + wave) * 1024 + lane * 16);
  const int p = p0 + 16 * wave + r, co = co0 + 4 * q;
  if (p >= a.m) return;
  const int64_t e = (int64_t)p * a.cout + co;
  uint32_t code[4] = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (co + i >= a.cout) continue;
    if (a.acc_dump) a.acc_dump[e + i] = v[i];
    if (a.out_mode == 0) {
      reinterpret_cast<int32_t*>(a.y)[e + i] = v[i];
      continue;
    }
    const int32_t* t = rec + (4 * q + i) * a.rec;
    const int sv = sgn(v[i], t[0]);
    for (int k = 1; k <= a.nq; ++k) code[i] += sv > t[k];
  }
  uint8_t* y8 = reinterpret_cast<uint8_t*>(a.y);
  if (a.out_mode == 2) {          // c_out % 4 == 0
    if (co < a.cout)
      y8[a.out_layout == IFQ_LAYOUT_U2_BLOCK64 ? block64_byte(p, co, 1, a.div_howo, a.cout)
                                               : e >> 2] =
          (uint8_t)(code[0] | code[1] << 2 | code[2] << 4 | code[3] << 6);
  } else if (a.out_mode == 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (co + i < a.cout) y8[e + i] = (uint8_t)code[i];
  }
}

// Up to 64 images: beyond, the weights are read again for each 64 and the
// tiles of the other kernels reuse them better.
bool fc_eligible(const ConvLaunch& a) {
  return a.kh == a.h && a.kw == a.w && a.pad == 0 && a.ho * a.wo == 1 && a.m > 0 && a.m <= 64 &&
         a.join_kind == IFQ_JOIN_NONE && !a.pool_k && !a.f4;
}

int fc_blocks(const ConvLaunch& a) { return a.m <= 16 ? 1 : a.m <= 32 ? 2 : 4; }

const char* fc_name(const ConvLaunch& a) {
  const int nb = fc_blocks(a);
  return nb == 1 ? "conv_fc<1>" : nb == 2 ? "conv_fc<2>" : "conv_fc<4>";
}

hipError_t launch_fc(const ConvLaunch& a, hipStream_t stream) {
  FcGeom g;
  const int hw = a.h * a.w, G = a.cin / 64;
  const bool blk = a.in_layout == IFQ_LAYOUT_U2_BLOCK64;
  g.sn = hw * G;
  g.sg = blk ? hw : 1;
  g.st = blk ? 1 : G;
  g.div_taps = make_fastdiv(a.kh * a.kw);
  const int nb = fc_blocks(a);
  const dim3 grid((a.cout + 15) / 16, (a.m + 16 * nb - 1) / (16 * nb));
  switch (nb) {
    case 1: hipLaunchKernelGGL((conv_fc<1>), grid, dim3(512), 0, stream, a, g); break;
    case 2: hipLaunchKernelGGL((conv_fc<2>), grid, dim3(512), 0, stream, a, g); break;
    default: hipLaunchKernelGGL((conv_fc<4>), grid, dim3(512), 0, stream, a, g); break;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Variants and per-layer planning
// ---------------------------------------------------------------------------
// Times (us) of the busiest CU's tiles, one at a time: of a launch, a tile, a stage
// of s*wk K64 steps, a coded (not int32) tile, and of 512 of its outputs by
// epilogue: 2-bit thresholds, identity join on 2-bit codes, per threshold other
// codes without and with that join, conv join.
struct Variant {
  int wm, wn, wk, fm, fn, s;
  double t0, tile, stage, coded;
  double thr, join, wide, wide_join, conv;
  const char* name;
};

// Index order must match the switch in launch_conv_mfma. Fitted to 5366 layers, each
// timed on every tile (1x1 to 5x5, both layouts, every output and join): 2-bit codes
// 5-8% rms (13% on the first tile), int32 sums 5-8%, the joins 5-15%, wider codes
// 8-30%, which this kernel is never the fastest on.
const Variant kVariants[] = {
    {2, 4, 1, 2, 4, 1, 2.837, 1.291, 0.845, 5.376, 0.024, 0.118, 0.140, 0.127, 1.198,
     "conv_mfma<2, 4, 1, 2, 4, 1, 6>"},    // 128 x 512
    {2, 4, 1, 2, 2, 2, 2.534, 1.274, 0.981, 2.939, 0.027, 0.103, 0.096, 0.111, 0.743,
     "conv_mfma<2, 4, 1, 2, 2, 2, 4>"},    // 128 x 256
    {1, 8, 1, 2, 2, 2, 2.400, 1.285, 1.055, 2.892, 0.027, 0.096, 0.077, 0.083, 0.839,
     "conv_mfma<1, 8, 1, 2, 2, 2, 4>"},    //  64 x 512
    {2, 4, 1, 1, 2, 2, 1.872, 1.223, 0.778, 1.997, 0.016, 0.080, 0.078, 0.086, 0.557,
     "conv_mfma<2, 4, 1, 1, 2, 2, 6>"},    //  64 x 256
    {2, 2, 2, 2, 2, 2, 2.180, 2.645, 1.190, 2.826, 0.028, 0.137, 0.147, 0.173, 0.861,
     "conv_mfma<2, 2, 2, 2, 2, 2, 3>"},    // 128 x 128, K split 2
    {2, 1, 4, 1, 4, 1, 1.791, 3.722, 0.851, 2.438, 0.041, 0.211, 0.186, 0.238, 1.182,
     "conv_mfma<2, 1, 4, 1, 4, 1, 6>"},    //  64 x 128, K split 4
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);
constexpr int kNumCUs = 256;

struct Plan {
  int variant;
  int bn;        // pixels per workgroup
  int blocks_m;  // workgroups along pixels
  double t_us;   // predicted time
};

double tiled_us(const ConvLaunch& a, const Variant& V, int64_t bn, int64_t tiles) {
  const int64_t per_cu = (tiles + kNumCUs - 1) / kNumCUs;
  const int sk = V.s * V.wk, bm = 32 * V.fm * V.wm;
  const int rows = (a.cout + 31) / 32 * 32 < bm ? (a.cout + 31) / 32 * 32 : bm;
  const bool id = a.join_kind == IFQ_JOIN_IDENTITY;
  const double per512 = a.join_kind == IFQ_JOIN_CONV ? V.conv
                        : a.out_mode == 0            ? 0
                        : a.rec == 4                 ? (id ? V.join : V.thr)
                                                     : (id ? V.wide_join : V.wide) * a.nq;
  const double one = V.tile + V.stage * ((a.nk + sk - 1) / sk) + (a.out_mode ? V.coded : 0) +
                     per512 * rows * (double)bn / 512;
  const double sums = a.out_mode == 0 ? 4.0 * a.m * a.cout / kSumBytesPerUs : 0;
  return V.t0 + (double)per_cu * one + 0.8 * sums;
}

// For each variant take the fewest rounds of one workgroup per CU that fit
// the layer and spread the pixels evenly over the workgroups of those rounds
// (in multiples of 32); the variant predicted fastest runs.
Plan plan_mfma(const ConvLaunch& a) {
  Plan best{0, 0, 0, 0.0};
  double best_t = 1e30;
  for (int v = 0; v < kNumVariants; ++v) {
    const Variant& V = kVariants[v];
    const int bm = 32 * V.fm * V.wm;
    const int bnmax = 32 * V.fn * V.wn;
    const int64_t nco = (a.cout + bm - 1) / bm;
    const int64_t nb_min = (a.m + bnmax - 1) / bnmax;
    const int64_t rounds = (nco * nb_min + kNumCUs - 1) / kNumCUs;
    int64_t nb = rounds * kNumCUs / nco;
    if (nb < nb_min) nb = nb_min;
    int64_t bn = (a.m + nb - 1) / nb;
    bn = (bn + 31) / 32 * 32;
    if (bn > bnmax) bn = bnmax;
    const int64_t blocks = nco * ((a.m + bn - 1) / bn);
    const double t = tiled_us(a, V, bn, blocks);
    if (t < best_t - 1e-9) {
      best_t = t;
      best = Plan{v, (int)bn, (int)((a.m + bn - 1) / bn), t};
    }
  }
  return best;
}

template <int WM, int WN, int WK, int FM, int FN, int S, int D>
hipError_t launch_variant(ConvLaunch a, const Plan& pl, hipStream_t stream) {
  a.bn = pl.bn;
  dim3 grid(pl.blocks_m, (a.cout + 32 * FM * WM - 1) / (32 * FM * WM));
  hipLaunchKernelGGL((conv_mfma<WM, WN, WK, FM, FN, S, D>), grid,
                     dim3(64 * WM * WN * WK), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

bool mfma_eligible(const ConvLaunch& a) {
  return a.in_bits == 2 && a.cin % 64 == 0 &&
         (a.in_layout == IFQ_LAYOUT_U2_NHWC_PACKED || a.in_layout == IFQ_LAYOUT_U2_BLOCK64);
}

// The dispatcher's choice among the kernels on the MFMA fast path for one layer, and
// their plans, kept by layer geometry.
namespace {

struct MfmaChoice {
  int kind;   // 0 register-blocked (reg3), 1 windowed 3x3, 2 tiled, 3 windowed, 4 fully
              // connected, -1 none
  HaloPlan hp;
  Reg3Plan rp;
  Plan pl;
};

// The windowed 3x3 kernel's prediction is a fit to the threshold epilogue with 2-bit
// codes at one tile a CU; beside other kernels its time by epilogue, fitted to 1002
// layers that the register-blocked kernels do not take (5% rms on the joins with
// identity, 7 to 10% on 2-bit codes and sums, 15 to 18% on the others).
double halo_weigh(const ConvLaunch& a, double t_us) {
  if (a.join_kind == IFQ_JOIN_CONV) return 1.12 * t_us + 6.4;
  if (a.out_mode == 0) return t_us - 0.5;
  if (a.rec != 4) return 1.13 * t_us + 10.9;
  return a.join_kind == IFQ_JOIN_IDENTITY ? 0.95 * t_us + 4.6 : 0.98 * t_us + 2.0;
}

// The kernel predicted fastest, each by a fit to its own measured times, among
//  - the register-blocked ones (3x3 on BLOCK64 codes, 2-bit codes out), or where they
//    do not take such a layer in one piece the windowed 3x3 one,
//  - the tiled one,
//  - conv_win; but not on layers of 64 channels that the register-blocked kernels
//    take: their K is one stage deep and the prediction too rough for what could be
//    gained (3.5% on average over 313 layers, 49 of them more than 3% slower;
//    28x28x64 -> 64 at batch 1: 4.9 us, conv_win 5.2).
// Beside every kernel and tile, each timed on 6664 layers, the choice is 1.5% behind
// the fastest on average where the register-blocked kernels do not take the layer and
// 1.3% where they do. In us on one card:
//  - few stages on many pixels stay on the tiled kernel: 1x1 28x28x128 -> 512 at batch
//    16 8.0, conv_win 9.1; 56x56x64 -> 256 at batch 8 8.0, 9.2; 69x67x64 -> 320 sums
//    at batch 2 6.7, 9.3;
//  - deeper K goes to conv_win, which does not gather its input tap by tap: 5x5
//    27x27x128 -> 256 at batch 4 18.9, 10.5; and where the register-blocked tiles leave
//    CUs idle its small tiles, K split over the waves: 13x13x512 -> 512 at batch 1
//    11.1, 8.3, 14x14x256 -> 512 strided at batch 2 8.3, 6.4, 7x7x512 -> 512 with an
//    identity join at batch 16 12.3, 9.8; not where they fill them: 28x28x128 -> 128
//    with the join at batch 8 7.4, 7.7;
//  - windows too wide for the register-blocked kernels: strided 64x80x448 -> 448 with
//    the join, batch 10, on the windowed 3x3 kernel 35.3, conv_win 43.7, tiled 43.3.
MfmaChoice plan_choice(const ConvLaunch& a) {
  MfmaChoice c{};
  if (fc_eligible(a)) {
    c.kind = 4;
    return c;
  }
  const bool halo = plan_halo(a, &c.hp);
  const bool r3 = plan_reg3(a, -1, &c.rp);
  if (a.join_kind == IFQ_JOIN_CONV_FUSED) {
    c.kind = r3 ? 0 : (halo ? 1 : -1);
    return c;
  }
  c.pl = plan_mfma(a);
  c.kind = 2;
  double t = c.pl.t_us, tw = 0;
  const bool win = plan_win_us(a, &tw);
  if (r3 && c.rp.weigh_us <= t) {
    c.kind = 0;
    t = c.rp.weigh_us;
  }
  // (a plan that splits K across workgroups needs a workspace and is the register-blocked
  // kernels' only one on its layer)
  const bool split = r3 && !c.rp.persistent && c.rp.w2.ksplit > 1;
  if (halo && (!r3 || split) && halo_weigh(a, c.hp.t_us) < t) {
    c.kind = 1;
    t = halo_weigh(a, c.hp.t_us);
  }
  if (win && tw < t && !(r3 && a.cin < 128)) c.kind = 3;
  return c;
}

PlanCache<MfmaChoice> g_choice;

MfmaChoice choose_mfma(const ConvLaunch& a) {
  MfmaChoice c;
  g_choice.get(a, &c, [](const ConvLaunch& l, MfmaChoice* o) {
    *o = plan_choice(l);
    return true;
  });
  return c;
}

}  // namespace

// The fast path picks the kernel with the lowest predicted time (plan_choice);
// a fully connected layer runs on conv_fc. A fused downsample join runs on
// the register-blocked kernel wherever it takes the layer (faster on every
// downsampling block of the ResNet-18-shaped stack as measured), else on the
// windowed kernel (the host checks fused_supported before launching one).
const char* conv_mfma_name(const ConvLaunch& a) {
  const MfmaChoice c = choose_mfma(a);
  if (c.kind == 0) return reg3_name(c.rp, a);
  if (c.kind == 1) return conv_halo_name(c.hp, a);
  if (c.kind == 3) return conv_win_name(a);
  if (c.kind == 4) return fc_name(a);
  if (c.kind < 0) return "";
  return kVariants[c.pl.variant].name;
}

// The workspace of the kernel launch_conv_mfma picks (the same choice).
int64_t conv_mfma_workspace_bytes(const ConvLaunch& a) {
  const MfmaChoice c = choose_mfma(a);
  if (c.kind != 0 || c.rp.persistent) return 0;
  return w2_split_bytes(a, c.rp.w2);
}

// A fused pool the windowed 3x3 kernel covers: conv_w2 where its prediction is below
// the windowed kernel's by the margin that the pooling itself takes of its lead (its
// prediction is of the unpooled layer, 11% below the pooled one's time). Over 905 int8
// layers timed on both the choice is 0.4% behind the faster one on average and 10% at
// most; with the bound at 0.85 or 0.95 of it 0.9% and 22%, 0.5% and 10%. Over 521 fp4
// layers conv_w2 is never more than 5% slower. us: 28x28x512 -> 512 at batch 2 20.8 on
// the windowed kernel, 12.2 on conv_w2; 28x36x448 -> 256 at batch 9 25.8, 33.0.
namespace {

bool pool_on_w2(const ConvLaunch& a, const HaloPlan& hp, Reg3Plan* rp) {
  return plan_reg3(a, -1, rp) && !rp->persistent && rp->t_us < 0.9 * hp.t_us;
}

}  // namespace

const char* conv_pool_name(const ConvLaunch& a, const HaloPlan& hp) {
  Reg3Plan rp;
  return pool_on_w2(a, hp, &rp) ? conv_w2_name(rp.w2, a) : conv_halo_name(hp, a);
}

hipError_t launch_conv_pool(const ConvLaunch& a, const HaloPlan& hp, hipStream_t stream) {
  Reg3Plan rp;
  return pool_on_w2(a, hp, &rp) ? launch_conv_w2(a, rp.w2, stream)
                                : launch_conv_halo(a, hp, stream);
}

hipError_t launch_conv_mfma(const ConvLaunch& a, hipStream_t stream) {
  const MfmaChoice c = choose_mfma(a);
  if (c.kind == 0) return launch_reg3(a, c.rp, stream);
  if (c.kind == 1) return launch_conv_halo(a, c.hp, stream);
  if (c.kind == 3) return launch_conv_win(a, stream);
  if (c.kind == 4) return launch_fc(a, stream);
  if (c.kind < 0) return hipErrorNotSupported;
  const Plan& pl = c.pl;
  switch (pl.variant) {
    case 0: return launch_variant<2, 4, 1, 2, 4, 1, 6>(a, pl, stream);
    case 1: return launch_variant<2, 4, 1, 2, 2, 2, 4>(a, pl, stream);
    case 2: return launch_variant<1, 8, 1, 2, 2, 2, 4>(a, pl, stream);
    case 3: return launch_variant<2, 4, 1, 1, 2, 2, 6>(a, pl, stream);
    case 4: return launch_variant<2, 2, 2, 2, 2, 2, 3>(a, pl, stream);
    default: return launch_variant<2, 1, 4, 1, 4, 1, 6>(a, pl, stream);
  }
}

}  // namespace ifq
