// Block quantisation of a shard's weight rows to INT8 / INT4 (paper Sec.
// 2.2 precision heterogeneity, Sec. 4.2.2 importance-aware mixed
// precision, Sec. 4.3.1 precision scaling): the format the decode kernel
// reads through vt_layer_decode_q.
//
// Per row, blocks of 32 consecutive columns (the last may be partial; its
// missing columns count as zero). Block scale s = fp16(absmax / Q) (fp32
// division, round to nearest even; Q = 127 or 7); codes c = clamp(rint(w /
// s), -Q, Q) with w and s as fp32 and the division in fp32 (ties to even);
// s = 0 gives c = 0. INT8 codes are bytes in column order; INT4 codes are
// nibbles c + 8, 8 columns per 4 bytes: column 8g + i (i < 4) in the low
// nibble of byte 4g + i, column 8g + 4 + i in its high nibble.
#include <hip/hip_runtime.h>

#include "device.hpp"
#include "internal.hpp"

namespace vt {
namespace wq {

constexpr int QT = 256;          // threads per workgroup
constexpr int QU = 4;            // 8-column chunks per thread
constexpr int QCH = QT * QU;     // chunks per workgroup

// The 8 codes of a chunk, as documented: fp32 division, ties to even, clamp.
// Any scale (zero, subnormal, infinite) and any value (NaN included).
__device__ __forceinline__ void codes_general(const float (&v)[8], float s, float qm, int (&c)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e)
    c[e] = s > 0.f ? static_cast<int>(fminf(fmaxf(__builtin_rintf(__fdiv_rn(v[e], s)), -qm), qm)) : 0;
}

// Byte 0 of a, b, c and d as one word.
__device__ __forceinline__ uint32_t low_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const uint32_t lo = __builtin_amdgcn_perm(b, a, 0x0c0c0400), hi = __builtin_amdgcn_perm(d, c, 0x04000c0c);
  return lo | hi;
}

// A lane quantises chunks of 8 columns (one 16-byte load each, a wave's loads
// contiguous); the 4 lanes of a quad hold one block of 32 and agree on its
// absmax by quad swaps. A workgroup takes ``rpw`` whole rows of ``cpr``
// chunks, or QCH chunks of one longer row (``segs`` workgroups per row).
//
// The codes are bound by VALU work, not by memory, if every value takes an
// IEEE division (one block per thread and 32 divisions: 196 us and 0.96 TB/s
// for the seven matrices of a 7B 30% shard). With r = 1 / s correctly rounded
// the quotient is q0 = v r, then q0 + (v - q0 s) r, which rounds to the same
// fp32 value as the division for every pair of fp16 numbers whose quotient is
// below 128 (a host test goes through all mantissa pairs), and adding 1.5 * 2^23 rounds it to the
// integer in the sum's low bits, ties to even: four instructions per value, and the
// seven matrices take 55 us (3.4 TB/s, the seven launches included). A normal
// finite fp16 scale keeps |q| below Q + 1/2, so that sum needs no clamp. A wave
// in which any lane has another scale (a NaN or infinity in its block, a block of
// zeros, no chunk at all past a row's end) takes codes_general as a whole: the
// same codes, at matrices with 30% of their blocks zero 1.3-1.7 times the time (8192 x
// 8192 to INT8: 36.5 us dense, 48.7 pruned; 139 with divisions throughout).
template <int PREC>
__global__ void __launch_bounds__(QT) quantize_kernel(const uint16_t* __restrict__ w, int64_t ld, int rows,
                                                      int cols, uint8_t* __restrict__ codes, int64_t ld_codes,
                                                      uint16_t* __restrict__ scales, int64_t ld_scales, int cpr,
                                                      int rpw, int segs, uint32_t magic) {
  constexpr float qm = PREC == VT_W_INT8 ? 127.f : 7.f;
  const int64_t r0 = segs > 1 ? blockIdx.x / segs : static_cast<int64_t>(blockIdx.x) * rpw;
  const int c0 = segs > 1 ? static_cast<int>(blockIdx.x % segs) * QCH : 0;
  const int nrow = static_cast<int>(min(static_cast<int64_t>(rpw), rows - r0));
  int row[QU], ch[QU];
  u32x4 raw[QU];
#pragma unroll
  for (int u = 0; u < QU; ++u) {
    const int n = u * QT + static_cast<int>(threadIdx.x);
    // n / cpr for n < 1024 (magic = ceil(2^20 / cpr), exact as n cpr < 2^20)
    const int dr = segs > 1 ? 0 : static_cast<int>((static_cast<uint32_t>(n) * magic) >> 20);
    row[u] = dr;
    ch[u] = segs > 1 ? c0 + n : n - dr * cpr;
    if (dr >= nrow || ch[u] >= cpr) row[u] = -1;
    raw[u] = u32x4{0u, 0u, 0u, 0u};
    const int left = cols - ch[u] * 8;
    if (row[u] >= 0 && left > 0) {
      const uint16_t* src = w + (r0 + dr) * ld + ch[u] * 8;
      if (left >= 8) {
        raw[u] = load_stream(src);
      } else {
        uint16_t h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = e < left ? src[e] : 0;
        raw[u] = pack8(h);
      }
    }
  }
#pragma unroll
  for (int u = 0; u < QU; ++u) {
    // absmax on the magnitudes' bits: ordered like the values, NaN above all
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    u16x2 m = __builtin_bit_cast(u16x2, raw[u].x & 0x7FFF7FFFu);
    m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, raw[u].y & 0x7FFF7FFFu));
    m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, raw[u].z & 0x7FFF7FFFu));
    m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, raw[u].w & 0x7FFF7FFFu));
    int mb = max(static_cast<int>(m.x), static_cast<int>(m.y));
    mb = max(mb, __builtin_amdgcn_update_dpp(0, mb, 0xB1, 0xF, 0xF, false));  // lane ^ 1
    mb = max(mb, __builtin_amdgcn_update_dpp(0, mb, 0x4E, 0xF, 0xF, false));  // lane ^ 2
    float v[8];
    unpack8(raw[u], v);
    uint16_t s16 = f2h(__fdiv_rn(h2f(static_cast<uint16_t>(mb)), qm));
    float s = h2f(s16);
    const bool plain = mb < 0x7C00 && s16 >= 0x0400;
    uint32_t t[8];
    if (__builtin_amdgcn_ballot_w64(!plain) == 0) {
      const float r = __fdiv_rn(1.0f, s);
      constexpr float bias = PREC == VT_W_INT8 ? 12582912.f : 12582920.f;  // 1.5 * 2^23 (+ 8)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float q0 = v[e] * r;
        t[e] = __builtin_bit_cast(uint32_t, fmaf(fmaf(-q0, s, v[e]), r, q0) + bias);
      }
    } else {
      if (mb > 0x7C00) {
        // a NaN in the block: the absmax is that of its other values
        float a = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) a = fmaxf(a, fabsf(v[e]));
        a = fmaxf(a, dpp_f<0xB1>(0.f, a));
        a = fmaxf(a, dpp_f<0x4E>(0.f, a));
        s16 = f2h(__fdiv_rn(a, qm));
        s = h2f(s16);
      }
      int c[8];
      codes_general(v, s, qm, c);
#pragma unroll
      for (int e = 0; e < 8; ++e) t[e] = static_cast<uint32_t>(PREC == VT_W_INT8 ? c[e] : c[e] + 8);
    }
    if (row[u] < 0) continue;
    const int64_t rr = r0 + row[u];
    if (ch[u] % 4 == 0) scales[rr * ld_scales + ch[u] / 4] = s16;
    if (PREC == VT_W_INT8) {
      const uint64_t lo = low_bytes(t[0], t[1], t[2], t[3]), hi = low_bytes(t[4], t[5], t[6], t[7]);
      *reinterpret_cast<uint64_t*>(codes + rr * ld_codes + ch[u] * 8) = lo | (hi << 32);
    } else {
      *reinterpret_cast<uint32_t*>(codes + rr * ld_codes + ch[u] * 4) =
          low_bytes(t[0] | (t[4] << 4), t[1] | (t[5] << 4), t[2] | (t[6] << 4), t[3] | (t[7] << 4));
    }
  }
}

}  // namespace wq
}  // namespace vt

using namespace vt;

extern "C" vt_status vt_quantize_rows(const void* w, int64_t ld, int32_t rows, int32_t cols, int32_t prec,
                                      void* codes, int64_t ld_codes, void* scales, int64_t ld_scales,
                                      void* stream) {
  clear_error();
  if (prec != VT_W_INT8 && prec != VT_W_INT4)
    return fail(VT_ERR_ARG, "precision %d is neither VT_W_INT8 nor VT_W_INT4", prec);
  if (rows < 0 || cols < 1) return fail(VT_ERR_ARG, "rows %d / cols %d invalid", rows, cols);
  if (rows == 0) return VT_OK;
  if (!w || !codes || !scales) return fail(VT_ERR_ARG, "null buffer");
  if (!aligned16(w) || !aligned16(codes)) return fail(VT_ERR_ALIGN, "weights or codes not 16-byte aligned");
  if (reinterpret_cast<uintptr_t>(scales) % 2) return fail(VT_ERR_ALIGN, "scales not 2-byte aligned");
  const int64_t nb = (cols + 31) / 32;
  const int64_t need = nb * (prec == VT_W_INT8 ? 32 : 16);
  if (ld < cols || ld % 8) return fail(VT_ERR_ARG, "ld %lld must be a multiple of 8 and >= cols %d",
                                       static_cast<long long>(ld), cols);
  if (ld_codes < need || ld_codes % 16)
    return fail(VT_ERR_ARG, "ld_codes %lld must be a multiple of 16 and >= %lld",
                static_cast<long long>(ld_codes), static_cast<long long>(need));
  if (ld_scales < nb)
    return fail(VT_ERR_ARG, "ld_scales %lld < %lld blocks", static_cast<long long>(ld_scales),
                static_cast<long long>(nb));
  const int64_t items = static_cast<int64_t>(rows) * nb;
  if (items > (int64_t(1) << 31) - wq::QT) return fail(VT_ERR_UNSUPPORTED, "%lld blocks", static_cast<long long>(items));
  // workgroups of whole rows, or several to a row of more than QCH chunks
  const int cpr = static_cast<int>(nb) * 4;
  const int segs = (cpr + wq::QCH - 1) / wq::QCH, rpw = segs > 1 ? 1 : wq::QCH / cpr;
  const int64_t grid = segs > 1 ? static_cast<int64_t>(rows) * segs : (static_cast<int64_t>(rows) + rpw - 1) / rpw;
  const uint32_t magic = ((1u << 20) + cpr - 1) / cpr;
  auto* kernel = prec == VT_W_INT8 ? wq::quantize_kernel<VT_W_INT8> : wq::quantize_kernel<VT_W_INT4>;
  hipLaunchKernelGGL(kernel, dim3(static_cast<uint32_t>(grid)), dim3(wq::QT), 0, static_cast<hipStream_t>(stream),
                     static_cast<const uint16_t*>(w), ld, rows, cols, static_cast<uint8_t*>(codes), ld_codes,
                     static_cast<uint16_t*>(scales), ld_scales, cpr, rpw, segs, magic);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? VT_OK : fail(VT_ERR_HIP, "quantize launch: %s", hipGetErrorString(e));
}
