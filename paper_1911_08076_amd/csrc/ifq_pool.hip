// Integer max-pool on codes (Eq. 4 applied to the quantizer output) and
// conversion between the code layouts.
//
// Both stream HBM, and on the networks' tensors (0.1 to 16 MB) latency decides:
// a thread owns a vector of V bytes of one output pixel (V = 16, 4 or 1, the
// widest that divides the bytes per pixel) and has every load of its window
// in flight before the first compare; indexes are 32-bit with divisions by
// multiplication. Before, each position's loads waited for the last compare
// behind 64-bit divisions: 3x3/2 on 64x55x55x96 2-bit codes 7.0 -> 3.9 us for calls in
// a row (1.5 TB/s), on 32x13x13x256 6.9 -> 4.0, of which the kernel 5.9 -> 2.2.
#include <hip/hip_runtime.h>

#include "ifq_internal.h"

namespace ifq {
namespace {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t fdivu(uint32_t n, FastDiv d) {
  return (__umulhi(n, d.mul) + n) >> d.shift;
}

struct PoolGeom {
  FastDiv div_nv, div_wo, div_ho;   // vectors per pixel, output columns, rows
  int32_t total;                    // vectors in all
  int32_t cb;                       // bytes per pixel
};

// Running maximum over words of codes. Bytes: even and odd bytes as 16-bit
// halves. 2-bit fields: h collects the high bits, and in a second pass l the
// low bits of the fields whose high bit equals the maximum's.
template <bool U2>
__device__ __forceinline__ uint32_t window_max(const uint32_t* v, int n, int stride) {
  if constexpr (U2) {
    uint32_t hi = 0, lo = 0;
    for (int i = 0; i < n; ++i) hi |= v[i * stride];
    hi &= 0xAAAAAAAAu;
    for (int i = 0; i < n; ++i) {
      const uint32_t t = v[i * stride];
      lo |= t & ~((hi ^ t) >> 1);
    }
    return hi | (lo & 0x55555555u);
  } else {
    u16x2 e = {0, 0}, o = {0, 0};
    for (int i = 0; i < n; ++i) {
      const uint32_t t = v[i * stride];
      e = __builtin_elementwise_max(e, __builtin_bit_cast(u16x2, t & 0x00FF00FFu));
      o = __builtin_elementwise_max(o, __builtin_bit_cast(u16x2, t & 0xFF00FF00u));
    }
    return __builtin_bit_cast(uint32_t, e) | __builtin_bit_cast(uint32_t, o);
  }
}

template <int V>
__device__ __forceinline__ void load_vec(const uint8_t* p, uint32_t* v) {
  if constexpr (V == 16) {
    const uint4 q = *reinterpret_cast<const uint4*>(p);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
  } else if constexpr (V == 4) {
    v[0] = *reinterpret_cast<const uint32_t*>(p);
  } else {
    v[0] = *p;
  }
}

// K: the window where fixed (every load of it in flight at once), 0: any, a
// row of up to four positions at a time. Positions past the bottom or right
// edge (SAME mode) read the edge, which the window holds already.
template <int V, bool U2, int K>
__global__ void maxpool_codes(PoolLaunch a, PoolGeom g) {
  constexpr int W = V == 16 ? 4 : 1;
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (uint32_t)g.total) return;
  const uint32_t pix = fdivu(t, g.div_nv);
  const uint32_t chunk = t - pix * (uint32_t)(g.cb / V);
  const uint32_t row = fdivu(pix, g.div_wo);
  const int px = (int)(pix - row * a.wo);
  const uint32_t img = fdivu(row, g.div_ho);
  const int py = (int)(row - img * a.ho);
  const uint8_t* x = a.x + (int64_t)img * a.h * a.w * g.cb + chunk * V;
  uint32_t m[W];
  if constexpr (K > 0) {
    uint32_t v[K * K * W];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const int iy = py * a.stride + i < a.h ? py * a.stride + i : a.h - 1;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const int ix = px * a.stride + j < a.w ? px * a.stride + j : a.w - 1;
        load_vec<V>(x + (int64_t)(iy * a.w + ix) * g.cb, v + (i * K + j) * W);
      }
    }
#pragma unroll
    for (int w = 0; w < W; ++w) m[w] = window_max<U2>(v + w, K * K, W);
  } else {
#pragma unroll
    for (int w = 0; w < W; ++w) m[w] = 0;
    for (int i = 0; i < a.k && py * a.stride + i < a.h; ++i)
      for (int j0 = 0; j0 < a.k && px * a.stride + j0 < a.w; j0 += 4) {
        uint32_t v[5 * W];
        const int jn = a.k - j0 < 4 ? a.k - j0 : 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int jx = px * a.stride + j0 + (j < jn ? j : 0);
          load_vec<V>(x + (int64_t)((py * a.stride + i) * a.w + (jx < a.w ? jx : a.w - 1)) * g.cb,
                      v + j * W);
        }
#pragma unroll
        for (int w = 0; w < W; ++w) {
          v[4 * W + w] = m[w];
          m[w] = window_max<U2>(v + w, 5, W);
        }
      }
  }
  uint8_t* dst = a.y + (int64_t)t * V;
  if constexpr (V == 16) *reinterpret_cast<uint4*>(dst) = make_uint4(m[0], m[1], m[2], m[3]);
  else if constexpr (V == 4) *reinterpret_cast<uint32_t*>(dst) = m[0];
  else *dst = (uint8_t)m[0];
}

template <bool U2>
hipError_t launch_pool_mode(const PoolLaunch& a, int cb, hipStream_t stream) {
  auto go = [&](auto kern, int v) {
    PoolGeom g;
    g.cb = cb;
    g.total = a.n * a.ho * a.wo * (cb / v);
    g.div_nv = make_fastdiv(cb / v);
    g.div_wo = make_fastdiv(a.wo);
    g.div_ho = make_fastdiv(a.ho);
    // small tensors: one wave a workgroup, spread over the CUs
    const int nt = g.total <= 64 * 1024 ? 64 : 256;
    hipLaunchKernelGGL(kern, dim3((unsigned)((g.total + (int64_t)nt - 1) / nt)), dim3(nt), 0,
                       stream, a, g);
    return hipGetLastError();
  };
#define IFQ_POOL(V)                                         \
  (a.k == 2 ? go(maxpool_codes<V, U2, 2>, V)                \
            : a.k == 3 ? go(maxpool_codes<V, U2, 3>, V) : go(maxpool_codes<V, U2, 0>, V))
  if (cb % 16 == 0) return IFQ_POOL(16);
  if (cb % 4 == 0) return IFQ_POOL(4);
  return IFQ_POOL(1);
#undef IFQ_POOL
}

// Byte offset of the four codes of channel group cg (channels 4cg..4cg+3)
// of pixel p in a 2-bit code tensor: NHWC packed, or BLOCK64 cells.
__device__ __forceinline__ int64_t u2_offset(int32_t layout, int64_t p, int64_t cg,
                                             int64_t hw, int32_t c) {
  if (layout == IFQ_LAYOUT_U2_NHWC_PACKED) return p * (c >> 2) + cg;
  const int64_t nimg = p / hw;
  return ((nimg * (c >> 6) + (cg >> 4)) * hw + (p - nimg * hw)) * 16 + (cg & 15);
}

// One thread per group of four codes: reads them in the source layout and
// writes them in the destination layout (byte per code or 2-bit).
__global__ __launch_bounds__(256) void convert_codes(const uint8_t* src, uint8_t* dst,
                                                     int64_t groups, int64_t hw,
                                                     int32_t c, int32_t sl, int32_t dl) {
  const int64_t cgs = c >> 2;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < groups;
       g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t p = g / cgs, cg = g - p * cgs;
    uint32_t codes;  // byte i = code of channel 4cg + i
    if (sl == IFQ_LAYOUT_I8_NHWC) {
      codes = *reinterpret_cast<const uint32_t*>(src + 4 * g) & 0x03030303u;
    } else {
      const uint32_t b = src[u2_offset(sl, p, cg, hw, c)];
      codes = (b & 3u) | ((b & 0x0Cu) << 6) | ((b & 0x30u) << 12) | ((b & 0xC0u) << 18);
    }
    if (dl == IFQ_LAYOUT_I8_NHWC) {
      *reinterpret_cast<uint32_t*>(dst + 4 * g) = codes;
    } else {
      dst[u2_offset(dl, p, cg, hw, c)] =
          (uint8_t)((codes & 3u) | ((codes >> 6) & 0x0Cu) | ((codes >> 12) & 0x30u) |
                    ((codes >> 18) & 0xC0u));
    }
  }
}

// Sixteen codes, one a byte (a 16-byte vector) <-> packed two bits each (a word).
__device__ __forceinline__ uint32_t pack16(v4u v) {
  auto byte = [](uint32_t w) {      // c0 | c1 << 2 | c2 << 4 | c3 << 6 of a word's low bits
    w &= 0x03030303u;
    w |= w >> 6;
    return (w | w >> 12) & 0xFFu;
  };
  return byte(v.x) | byte(v.y) << 8 | byte(v.z) << 16 | byte(v.w) << 24;
}
__device__ __forceinline__ v4u unpack16(uint32_t u) {
  auto word = [](uint32_t b) {
    b = (b | b << 12) & 0x000F000Fu;
    return (b | b << 6) & 0x03030303u;
  };
  return v4u{word(u & 0xFFu), word((u >> 8) & 0xFFu), word((u >> 16) & 0xFFu),
                    word(u >> 24)};
}

// Conversions by units of 16 channels. convert_codes moves four at a time,
// one byte of a 2-bit layout per thread: 9.4 us for 64x56x56x64 bytes to
// BLOCK64 (16 MB, 1.7 TB/s), here 4.3 us (3.7 TB/s) for calls in a row;
// 16x224x224x64 31 -> 10.5 us (6.1 TB/s). A thread has four units' loads in flight,
// or one where four would leave CUs idle. Units run in
// the order of the BLOCK64 side where there is one (unit 4*cell + j, so that
// side is one contiguous stream and the other 64-byte spans), else in memory
// order, where byte and packed NHWC tensors are both plain streams of units.
// CELLS: 16-byte cells of 64 channels between the two 2-bit layouts instead.
struct UnitGeom {
  int32_t total;              // units (or cells)
  int32_t hw, G;              // pixels per image, channel blocks of 64
  FastDiv div_hw, div_g;
};

template <int SL, int DL, int U>
__global__ __launch_bounds__(256) void convert_units(const uint8_t* src, uint8_t* dst,
                                                     UnitGeom g) {
  constexpr bool CELLS = SL != IFQ_LAYOUT_I8_NHWC && DL != IFQ_LAYOUT_I8_NHWC;
  constexpr bool BLK = SL == IFQ_LAYOUT_U2_BLOCK64 || DL == IFQ_LAYOUT_U2_BLOCK64;
  const uint32_t t0 = blockIdx.x * (256 * U) + threadIdx.x;
  v4u v[U];
  uint32_t so[U], po[U];
#pragma unroll
  for (int k = 0; k < U; ++k) {
    const uint32_t t = t0 + 256 * k < (uint32_t)g.total ? t0 + 256 * k : g.total - 1;
    uint32_t nhwc = t;        // the unit's (cell's) place in the NHWC tensor
    if constexpr (BLK) {
      const uint32_t cell = CELLS ? t : t >> 2;
      const uint32_t nb = fdivu(cell, g.div_hw), p = cell - nb * g.hw;
      const uint32_t n = fdivu(nb, g.div_g), b = nb - n * g.G;
      nhwc = (n * g.hw + p) * g.G + b;
      if constexpr (!CELLS) nhwc = nhwc * 4 + (t & 3);
    }
    so[k] = SL == IFQ_LAYOUT_U2_BLOCK64 ? t : nhwc;
    po[k] = DL == IFQ_LAYOUT_U2_BLOCK64 ? t : nhwc;
  }
#pragma unroll
  for (int k = 0; k < U; ++k) {
    if constexpr (CELLS || SL == IFQ_LAYOUT_I8_NHWC)
      v[k] = reinterpret_cast<const v4u*>(src)[so[k]];
    else
      v[k].x = reinterpret_cast<const uint32_t*>(src)[so[k]];
  }
#pragma unroll
  for (int k = 0; k < U; ++k) {
    if (t0 + 256 * k >= (uint32_t)g.total) continue;
    if constexpr (CELLS) reinterpret_cast<v4u*>(dst)[po[k]] = v[k];
    else if constexpr (SL == IFQ_LAYOUT_I8_NHWC)
      reinterpret_cast<uint32_t*>(dst)[po[k]] = pack16(v[k]);
    else reinterpret_cast<v4u*>(dst)[po[k]] = unpack16(v[k].x);
  }
}

}  // namespace

hipError_t launch_pool(const PoolLaunch& a, hipStream_t stream) {
  if ((int64_t)a.n * a.ho * a.wo == 0) return hipSuccess;
  if (a.layout == IFQ_LAYOUT_U2_NHWC_PACKED)
    return launch_pool_mode<true>(a, a.c / 4, stream);
  return launch_pool_mode<false>(a, a.c, stream);
}

hipError_t launch_convert(int64_t n, int64_t hw, int32_t c, int32_t src_layout,
                          int32_t dst_layout, const void* src, void* dst,
                          hipStream_t stream) {
  const int64_t groups = n * hw * (c / 4);
  if (groups == 0) return hipSuccess;
  // by units where the tensor is whole units on both sides, aligned for them
  // (16 bytes, 4 for the packed side of a byte tensor), and indexes fit
  const bool s8 = src_layout == IFQ_LAYOUT_I8_NHWC, d8 = dst_layout == IFQ_LAYOUT_I8_NHWC;
  const bool blk = src_layout == IFQ_LAYOUT_U2_BLOCK64 || dst_layout == IFQ_LAYOUT_U2_BLOCK64;
  const int64_t per = !s8 && !d8 ? 16 : 4;          // groups per unit or cell
  const uintptr_t off = ((uintptr_t)src & (s8 || !d8 ? 15 : 3)) |
                        ((uintptr_t)dst & (d8 || !s8 ? 15 : 3));
  if (src_layout != dst_layout && groups % per == 0 && groups / per < ((int64_t)1 << 30) &&
      off == 0) {
    UnitGeom g;
    g.total = (int32_t)(groups / per);
    g.hw = blk ? (int32_t)hw : 1;
    g.G = blk ? c / 64 : 1;
    g.div_hw = make_fastdiv(g.hw);
    g.div_g = make_fastdiv(g.G);
    auto go = [&](auto k1, auto k4) {
      // one unit a thread up to eight workgroups a CU
      const int per_wg = g.total <= 8 * kPlanCUs * 256 ? 256 : 1024;
      hipLaunchKernelGGL(per_wg == 256 ? k1 : k4, dim3((g.total + per_wg - 1) / per_wg), dim3(256),
                         0, stream, reinterpret_cast<const uint8_t*>(src),
                         reinterpret_cast<uint8_t*>(dst), g);
      return hipGetLastError();
    };
    constexpr int I = IFQ_LAYOUT_I8_NHWC, N = IFQ_LAYOUT_U2_NHWC_PACKED, B = IFQ_LAYOUT_U2_BLOCK64;
#define IFQ_CONVERT(s, d) \
  if (src_layout == s && dst_layout == d) return go(convert_units<s, d, 1>, convert_units<s, d, 4>);
    IFQ_CONVERT(I, N)
    IFQ_CONVERT(I, B)
    IFQ_CONVERT(N, I)
    IFQ_CONVERT(B, I)
    IFQ_CONVERT(N, B)
    IFQ_CONVERT(B, N)
#undef IFQ_CONVERT
  }
  int64_t blocks = (groups + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(convert_codes, dim3((unsigned)blocks), dim3(256), 0, stream,
                     reinterpret_cast<const uint8_t*>(src), reinterpret_cast<uint8_t*>(dst),
                     groups, hw, c, src_layout, dst_layout);
  return hipGetLastError();
}

}  // namespace ifq
