// Elastic re-partition (paper Sec. 4.3.1): when the partition changes, a
// device gathers its new shard's weights out of the layer's full weights
// and takes over the KV heads its new shard owns. Shards are allocated
// separately (Sec. 4.3.1, Overhead Mitigation), so a new shard is packed
// into new buffers on a second stream while decode continues on the old
// ones. Pure data movement: every value is copied bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "internal.hpp"

namespace vt {
namespace rp {

constexpr int CT = 256;  // threads per workgroup, one 16-byte chunk each

// The 16 bytes that start 2 * sh bytes into lo (sh in 0..7), continued by hi.
__device__ __forceinline__ u32x4 shifted(u32x4 lo, u32x4 hi, int sh) {
  const int w = sh >> 1;
  uint32_t x[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const uint32_t v[4] = {i < 4 ? lo[i] : hi[i - 4], i < 3 ? lo[i + 1] : hi[i - 3], i < 2 ? lo[i + 2] : hi[i - 2],
                           i < 1 ? lo[i + 3] : hi[i - 1]};
    x[i] = w == 0 ? v[0] : (w == 1 ? v[1] : (w == 2 ? v[2] : v[3]));
  }
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = sh & 1 ? (x[i] >> 16) | (x[i + 1] << 16) : x[i];
  return r;
}

// dst[r][c] = src[r][c0 + c] for c < cols and 0 for cols <= c < dcols
// (fp16, strides in elements; dst rows and dcols in whole 8-element chunks
// of 16 bytes). A workgroup takes ``rpw`` whole rows of ``nch`` chunks (x counts
// such groups), or CT chunks of every gridDim.y-th longer row (x counts a row's
// segments). ALIGNED: c0 is a multiple of 8 and a whole chunk is one 16-byte
// load; else a chunk comes from the two aligned chunks it lies across, shifted
// together (5120 x 8294 of a Wd: 35 us; 47 us with eight 2-byte loads per
// chunk). Chunks at the end of the row's cols, past which nothing is read, go
// element by element.
// One chunk per thread: with four, a small copy had too few waves to hide its one
// round trip (KV heads of 3 x 2048 x 128: 5.2 us against 4.2 for one, 8 x 16 x 128: 4.7
// against 3.8).
// STREAM: 1 stores past the caches, 2 loads past them as well.
template <bool ALIGNED, int STREAM>
__global__ void __launch_bounds__(CT) copy2d_kernel(const uint16_t* __restrict__ src, int64_t lds, int64_t c0,
                                                    uint16_t* __restrict__ dst, int64_t ldd, int rows, int cols,
                                                    int nch, int rpw, uint32_t magic) {
  const int sh = ALIGNED ? 0 : static_cast<int>(c0 % 8);
  const int n = static_cast<int>(threadIdx.x);
  int64_t r = blockIdx.y;
  int ch = static_cast<int>(blockIdx.x) * CT + n;
  if (rpw > 0) {
    // n / nch for n < 256 (magic = ceil(2^16 / nch), exact as n nch < 2^16)
    const int dr = static_cast<int>((static_cast<uint32_t>(n) * magic) >> 16);
    r = static_cast<int64_t>(blockIdx.x) * rpw + dr;
    ch = n - dr * nch;
    if (dr >= rpw) return;
  }
  if (ch >= nch) return;
  const int c = ch * 8;
  for (; r < rows; r += gridDim.y) {
    const uint16_t* s = src + r * lds + c0 + c;
    u32x4 v;
    if (c + (ALIGNED ? 8 : 16 - sh) <= cols) {
      if (ALIGNED) v = STREAM == 2 ? load_stream(s) : load16(s);
      else v = shifted(load16(s - sh), load16(s - sh + 8), sh);
    } else {
      uint16_t h[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) h[e] = c + e < cols ? s[e] : 0;
      v = pack8(h);
    }
    u32x4* d = reinterpret_cast<u32x4*>(dst + r * ldd + c);
    if (STREAM) __builtin_nontemporal_store(v, d);
    else *d = v;
    if (rpw > 0) return;
  }
}

// Bytes from which a copy stores past the caches, and loads past them as well. What is
// copied is not read again soon, but a small copy's target stays in the last-level
// cache and is cheaper to write there. Layer shards packed over four rotated
// sets of buffers, plain / stores / both: matrices of 1-6 MB (hidden 1032) 19.1 / 20.8
// / 20.8 us; 9 MB 35.3 / 27.4 / 29.4; KV heads of 67 MB 49.2 / 47.6 / 46.0 (one set: 41.8 / 41.6
// / 44.6); 57 MB 105.9 / 98.0 / 95.7; 290 MB 296.8 / 274.5 / 267.0.
constexpr int64_t kStoreStream = int64_t(4) << 20, kLoadStream = int64_t(72) << 20;

static vt_status copy2d(const uint16_t* src, int64_t lds, int64_t c0, uint16_t* dst, int64_t ldd, int rows, int cols,
                        int dcols, hipStream_t s) {
  if (rows <= 0 || dcols <= 0) return VT_OK;
  const int nch = dcols / 8, rpw = nch > CT ? 0 : CT / nch;
  const dim3 grid(static_cast<uint32_t>(rpw > 0 ? (static_cast<int64_t>(rows) + rpw - 1) / rpw : (nch + CT - 1) / CT),
                  rpw > 0 ? 1 : std::min(rows, 65535));
  const uint32_t magic = ((1u << 16) + nch - 1) / nch;
  const int64_t bytes = static_cast<int64_t>(rows) * dcols * 2;
  auto pick = [&](auto* plain, auto* store, auto* both) {
    return bytes >= kLoadStream ? both : (bytes >= kStoreStream ? store : plain);
  };
  auto* kernel = c0 % 8 == 0 ? pick(copy2d_kernel<true, 0>, copy2d_kernel<true, 1>, copy2d_kernel<true, 2>)
                             : pick(copy2d_kernel<false, 0>, copy2d_kernel<false, 1>, copy2d_kernel<false, 1>);
  hipLaunchKernelGGL(kernel, grid, dim3(CT), 0, s, src, lds, c0, dst, ldd, rows, cols, nch, rpw, magic);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? VT_OK : fail(VT_ERR_HIP, "copy launch: %s", hipGetErrorString(e));
}

}  // namespace rp
}  // namespace vt

using namespace vt;

namespace {

// A matrix argument: rows x row length (elements) at stride ld.
vt_status check_mat(const void* p, int64_t ld, int64_t rowlen, int64_t rows, const char* what) {
  if (rows == 0 || rowlen == 0) return VT_OK;
  if (!p) return fail(VT_ERR_ARG, "%s is NULL", what);
  if (!aligned16(p)) return fail(VT_ERR_ALIGN, "%s is not 16-byte aligned", what);
  if (ld < rowlen || ld % 8)
    return fail(VT_ERR_ARG, "ld of %s (%lld) must be a multiple of 8 and >= %lld", what,
                static_cast<long long>(ld), static_cast<long long>(rowlen));
  return VT_OK;
}

}  // namespace

extern "C" vt_status vt_shard_pack(const vt_shard_spec* spec, const vt_layer_weights* full,
                                   const vt_layer_weights* out, void* stream) {
  clear_error();
  if (!spec || !full || !out) return fail(VT_ERR_ARG, "null argument");
  const vt_layer_dims& D = spec->dims;
  const vt_shard_info& in = spec->info;
  const int64_t H = D.hidden, d = D.head_dim, F = D.ffn;
  const int64_t nqd = static_cast<int64_t>(D.n_heads) * d, nkd = static_cast<int64_t>(D.n_kv_heads) * d;
  const int64_t qd = static_cast<int64_t>(in.n_q_heads) * d, kd = static_cast<int64_t>(in.n_kv_heads) * d;
  const int64_t q0 = static_cast<int64_t>(in.q_head_begin) * d, k0 = static_cast<int64_t>(in.kv_head_begin) * d;
  const int64_t nc = in.n_cols, c0 = in.col_begin;
  const int64_t ncp = (nc + 7) / 8 * 8;  // the shard's Wd rows: n_cols rounded up to 8, zero past n_cols
  vt_status st;
  struct M {
    const void* p;
    int64_t ld, rowlen, rows;
    const char* what;
  };
  const M checks[] = {
      {full->g_attn, H, H, 1, "full g_attn"}, {full->g_ffn, H, H, 1, "full g_ffn"},
      {full->wq, full->ld_q, H, nqd, "full wq"}, {full->wk, full->ld_k, H, nkd, "full wk"},
      {full->wv, full->ld_v, H, nkd, "full wv"}, {full->wo, full->ld_o, nqd, H, "full wo"},
      {full->wg, full->ld_g, H, F, "full wg"},   {full->wu, full->ld_u, H, F, "full wu"},
      {full->wd, full->ld_d, F, H, "full wd"},   {out->g_attn, H, H, 1, "g_attn"},
      {out->g_ffn, H, H, 1, "g_ffn"},            {out->wq, out->ld_q, H, qd, "wq"},
      {out->wk, out->ld_k, H, kd, "wk"},         {out->wv, out->ld_v, H, kd, "wv"},
      {out->wo, out->ld_o, qd, H, "wo"},         {out->wg, out->ld_g, H, nc, "wg"},
      {out->wu, out->ld_u, H, nc, "wu"},         {out->wd, out->ld_d, ncp, H, "wd"},
  };
  for (const M& m : checks)
    if ((st = check_mat(m.p, m.ld, m.rowlen, m.rows, m.what)) != VT_OK) return st;
  for (const M& m : checks)
    if (m.rows * m.ld * 2 >= (int64_t(1) << 40))
      return fail(VT_ERR_UNSUPPORTED, "%s is implausibly large", m.what);
  hipStream_t s = static_cast<hipStream_t>(stream);
  auto h = [](const void* p) { return static_cast<const uint16_t*>(p); };
  auto o = [](const void* p) { return static_cast<uint16_t*>(const_cast<void*>(p)); };
  if ((st = rp::copy2d(h(full->g_attn), H, 0, o(out->g_attn), H, 1, H, H, s)) != VT_OK) return st;
  if ((st = rp::copy2d(h(full->g_ffn), H, 0, o(out->g_ffn), H, 1, H, H, s)) != VT_OK) return st;
  if (qd > 0) {
    if ((st = rp::copy2d(h(full->wq) + q0 * full->ld_q, full->ld_q, 0, o(out->wq), out->ld_q, qd, H, H, s)) != VT_OK)
      return st;
    if ((st = rp::copy2d(h(full->wk) + k0 * full->ld_k, full->ld_k, 0, o(out->wk), out->ld_k, kd, H, H, s)) != VT_OK)
      return st;
    if ((st = rp::copy2d(h(full->wv) + k0 * full->ld_v, full->ld_v, 0, o(out->wv), out->ld_v, kd, H, H, s)) != VT_OK)
      return st;
    // Wo: the shard's columns; its rows are whole 8-element chunks since qd is
    if ((st = rp::copy2d(h(full->wo), full->ld_o, q0, o(out->wo), out->ld_o, H, qd, qd, s)) != VT_OK) return st;
  }
  if (nc > 0) {
    if ((st = rp::copy2d(h(full->wg) + c0 * full->ld_g, full->ld_g, 0, o(out->wg), out->ld_g, nc, H, H, s)) != VT_OK)
      return st;
    if ((st = rp::copy2d(h(full->wu) + c0 * full->ld_u, full->ld_u, 0, o(out->wu), out->ld_u, nc, H, H, s)) != VT_OK)
      return st;
    if ((st = rp::copy2d(h(full->wd), full->ld_d, c0, o(out->wd), out->ld_d, H, nc, ncp, s)) != VT_OK) return st;
  }
  return VT_OK;
}

extern "C" vt_status vt_kv_copy_heads(const vt_kv_view* src, int32_t src_head0, const vt_kv_view* dst,
                                      int32_t dst_head0, int32_t n_heads, int32_t n_pos, void* stream) {
  clear_error();
  if (!src || !dst) return fail(VT_ERR_ARG, "null KV view");
  if (n_heads < 0 || n_pos < 0) return fail(VT_ERR_ARG, "n_heads %d / n_pos %d < 0", n_heads, n_pos);
  if (n_heads == 0 || n_pos == 0) return VT_OK;
  if (src->head_dim != dst->head_dim || (src->head_dim != 64 && src->head_dim != 128))
    return fail(VT_ERR_ARG, "head_dim %d vs %d", src->head_dim, dst->head_dim);
  if (src_head0 < 0 || dst_head0 < 0 || src_head0 + static_cast<int64_t>(n_heads) > src->n_kv_heads ||
      dst_head0 + static_cast<int64_t>(n_heads) > dst->n_kv_heads)
    return fail(VT_ERR_ARG, "head range outside a cache (%d+%d of %d, %d+%d of %d)", src_head0, n_heads,
                src->n_kv_heads, dst_head0, n_heads, dst->n_kv_heads);
  if (n_pos > src->capacity || n_pos > dst->capacity)
    return fail(VT_ERR_ARG, "n_pos %d exceeds a capacity (%d, %d)", n_pos, src->capacity, dst->capacity);
  if (!src->k || !src->v || !dst->k || !dst->v) return fail(VT_ERR_ARG, "null cache buffer");
  if (!aligned16(src->k) || !aligned16(src->v) || !aligned16(dst->k) || !aligned16(dst->v))
    return fail(VT_ERR_ALIGN, "cache buffers must be 16-byte aligned");
  const int64_t d = src->head_dim;
  const int64_t lds = static_cast<int64_t>(src->capacity) * d, ldd = static_cast<int64_t>(dst->capacity) * d;
  const int cols = static_cast<int>(n_pos * d);
  hipStream_t s = static_cast<hipStream_t>(stream);
  vt_status st;
  const uint16_t* sk = static_cast<const uint16_t*>(src->k) + src_head0 * lds;
  const uint16_t* sv = static_cast<const uint16_t*>(src->v) + src_head0 * lds;
  uint16_t* dk = static_cast<uint16_t*>(dst->k) + dst_head0 * ldd;
  uint16_t* dv = static_cast<uint16_t*>(dst->v) + dst_head0 * ldd;
  if ((st = rp::copy2d(sk, lds, 0, dk, ldd, n_heads, cols, cols, s)) != VT_OK) return st;
  return rp::copy2d(sv, lds, 0, dv, ldd, n_heads, cols, cols, s);
}
