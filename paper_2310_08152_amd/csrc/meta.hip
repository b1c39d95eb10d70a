// Span metadata, tied position ids, rotary embedding and decode-step commit.
//
// Span metadata follows Section 3.1 (sentinel tokens around a span; <CL>
// visible only to itself; enclosed tokens hidden from tokens after the <CR>)
// and the position tie of Section 3.1 "Input Transformation".
#include <math.h>

#include <cmath>
#include <cstring>
#include <vector>

#include "sckv_common.h"

namespace sckv {

// ---------------------------------------------------------------------------
// vu[t] and tied positions: one thread per token.  The spans being sorted and
// disjoint, the search for the last <CL> at or before t also gives the number
// of sentinels before t, hence the number of normal tokens: no scan over the
// tokens (one workgroup per sequence that scanned them took 20 us at 4096
// tokens and 162 us at 32000; this takes 5-6 us at either).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void span_meta_kernel(const int32_t* __restrict__ spans,
                                                        const int32_t* __restrict__ nspan,
                                                        int32_t b, int32_t s_max, int32_t L_meta,
                                                        int32_t* __restrict__ vu,
                                                        int32_t* __restrict__ pos) {
  const int t = (int)((int64_t)blockIdx.x * 256 + threadIdx.x);
  if (t >= L_meta) return;
  for (int s = blockIdx.y; s < b; s += gridDim.y) {
    const int32_t* cl = spans + (int64_t)s * s_max;
    const int32_t* cr = spans + (int64_t)b * s_max + (int64_t)s * s_max;
    // last span whose <CL> is at or before t
    int lo = 0, hi = nspan[s];  // answer in [lo-1, hi-1]
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (cl[mid] <= t) lo = mid + 1; else hi = mid;
    }
    const int k = lo - 1;
    int v = SCKV_INF_VU, sentinels = 0;  // sentinels in [0, t)
    bool normal = true;
    if (k >= 0) {
      const int c = cl[k], r = cr[k];
      if (t == c) {
        v = t;  // <CL>
        normal = false;
      } else if (t < r) {
        v = r;  // enclosed token
      } else if (t == r) {
        normal = false;  // <CR>
      }
      sentinels = 2 * k + (c < t) + (r < t);
    }
    vu[(int64_t)s * L_meta + t] = v;
    if (pos != nullptr) {
      const int before = t - sentinels;  // normal tokens in [0, t)
      pos[(int64_t)s * L_meta + t] = normal ? before : (before > 0 ? before - 1 : 0);
    }
  }
}

// ---------------------------------------------------------------------------
// rotary embedding, rotate-half form: pair (i, i + d/2) turns by
// pos * theta^(-2i/d).  A thread owns one 16-byte piece of the first half of
// one token's rows (and the matching piece of the second half) in a group of
// hpt heads: it takes the piece's angles once and applies them to the
// token's row in each head of the group, so the group shares the sines and
// cosines.
// ---------------------------------------------------------------------------
struct InvFreq {
  double w[64];
};
// heads per thread of a rotation: two halves the angle work and keeps
// enough threads in flight (measured faster than 4..32 on 16x32x4096x80)
constexpr int ROPE_HPT = 2;

// row0 (nullable): per sequence, the row of y that receives row 0 of x; a
// sequence whose rows would leave [0, y_rows) (row0 < 0 included) is not
// written and sets SCKV_STATUS_CAP.
template <typename T, int D>
__device__ __forceinline__ void rope_body(const T* x, T* y, int32_t b, int32_t H, int32_t n,
                                          int64_t xs, int64_t ys,
                                          const int32_t* __restrict__ pos, int32_t L_meta,
                                          int32_t tok0, const InvFreq& inv, int rotate,
                                          int32_t hpt, const int32_t* __restrict__ row0,
                                          int32_t y_rows, int32_t* status) {
  constexpr int E = Piece<T>::E;
  constexpr int HALF = D / 2;
  constexpr int PPH = HALF / E;  // pieces per half row
  static_assert(HALF % E == 0, "half row must be whole pieces");
  const double two_pi = 6.283185307179586476925286766559;
  const int g = blockIdx.x * blockDim.x + threadIdx.x;  // (token, piece) of a sequence
  const int t = g / PPH;
  const int p = g - t * PPH;
  if (t >= n) return;
  // the piece's inverse frequencies, picked from the argument table
  double w[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    w[e] = 0.0;
#pragma unroll
    for (int pp = 0; pp < PPH; ++pp) w[e] = p == pp ? inv.w[pp * E + e] : w[e];
  }
  const int n_hg = (H + hpt - 1) / hpt;
  for (int sg = blockIdx.y; sg < b * n_hg; sg += gridDim.y) {
    const int s = sg / n_hg;
    const int h0 = (sg - s * n_hg) * hpt;
    const int h1 = min(h0 + hpt, H);
    int64_t drow = t;
    if (row0) {
      const int r0 = row0[s];
      if (r0 < 0 || (int64_t)r0 + n > y_rows) {
        if (status && g == 0 && h0 == 0) atomicOr(status, SCKV_STATUS_CAP);
        continue;
      }
      drow += r0;
    }
    float cs[E], sn[E];
    if (rotate) {
      const double ps = (double)pos[(int64_t)s * L_meta + tok0 + t];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        double ang = ps * w[e];
        ang -= two_pi * rint(ang / two_pi);
        sincosf((float)ang, &sn[e], &cs[e]);
      }
    }
    const T* src = x + (int64_t)s * H * xs + (int64_t)t * D + p * E;
    T* dst = y + (int64_t)s * H * ys + drow * D + p * E;
#pragma unroll 4
    for (int h = h0; h < h1; ++h) {
      u32x4 a = ld16(src + h * xs), c = ld16(src + h * xs + HALF);
      if (rotate) {
        float fa[E], fc[E];
        Piece<T>::unpack(a, fa);
        Piece<T>::unpack(c, fc);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const float x1 = fa[e], x2 = fc[e];
          // the fused forms are written out: which product of a pair stays
          // unrounded is then the same in this file's kernels (the decode
          // step, which turns one key, leaves it to the compiler)
          fa[e] = fmaf(x1, cs[e], -(x2 * sn[e]));
          fc[e] = fmaf(x2, cs[e], x1 * sn[e]);
        }
        a = Piece<T>::pack(fa);
        c = Piece<T>::pack(fc);
      }
      st16(dst + h * ys, a);
      st16(dst + h * ys + HALF, c);
    }
  }
}

template <typename T, int D>
__global__ __launch_bounds__(256) void rope_kernel(const T* x, T* y,
                                                   int32_t b, int32_t H, int32_t n, int64_t xs,
                                                   int64_t ys, const int32_t* __restrict__ pos,
                                                   int32_t L_meta, int32_t tok0, InvFreq inv,
                                                   int rotate, int32_t hpt,
                                                   const int32_t* __restrict__ row0,
                                                   int32_t y_rows, int32_t* status) {
  rope_body<T, D>(x, y, b, H, n, xs, ys, pos, L_meta, tok0, inv, rotate, hpt, row0, y_rows, status);
}

// One layer's block of a long prompt in one launch: grid.z picks the keys
// (rotated, into the cache), the values (copied, into the cache) or the
// queries (rotated).  A block's rows are few (4 sequences of 512 tokens, 32
// heads of 80: 10.5 MB a tensor) and three launches spent 9.5 us each, most
// of it starting and draining.
template <typename T>
struct RopeBlock {
  const T* x[3];
  T* y[3];
  int64_t xs[3], ys[3];
};
template <typename T, int D>
__global__ __launch_bounds__(256) void rope_block_kernel(RopeBlock<T> rb, int32_t b, int32_t H,
                                                         int32_t n, const int32_t* __restrict__ pos,
                                                         int32_t L_meta, int32_t tok0, InvFreq inv,
                                                         int rotate, int32_t hpt,
                                                         const int32_t* __restrict__ row0,
                                                         int32_t L_cap, int32_t* status) {
  const int z = blockIdx.z;
  rope_body<T, D>(z == 0 ? rb.x[0] : z == 1 ? rb.x[1] : rb.x[2],
                  z == 0 ? rb.y[0] : z == 1 ? rb.y[1] : rb.y[2], b, H, n,
                  z == 0 ? rb.xs[0] : z == 1 ? rb.xs[1] : rb.xs[2],
                  z == 0 ? rb.ys[0] : z == 1 ? rb.ys[1] : rb.ys[2], pos, L_meta, tok0, inv,
                  z == 1 ? 0 : rotate, hpt, z == 2 ? nullptr : row0, L_cap, status);
}

// ---------------------------------------------------------------------------
// bookkeeping of a whole prompt's rows: one thread per row
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void start_kernel(int32_t* __restrict__ kv_len,
                                                    int32_t* __restrict__ tok_idx,
                                                    int32_t* __restrict__ pos_ids,
                                                    int32_t* __restrict__ cur_tok,
                                                    const int32_t* __restrict__ pos,
                                                    int32_t L_meta, int32_t n, int32_t b,
                                                    int32_t L_cap) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  for (int s = blockIdx.y; s < b; s += gridDim.y) {
    tok_idx[(int64_t)s * L_cap + i] = i;
    pos_ids[(int64_t)s * L_cap + i] = pos[(int64_t)s * L_meta + i];
    if (i == 0) {
      kv_len[s] = n;
      cur_tok[s] = n;
    }
  }
}

// ---------------------------------------------------------------------------
// decode-step commit: one thread per sequence
// ---------------------------------------------------------------------------
__global__ void commit_kernel(int32_t* __restrict__ kv_len, int32_t* __restrict__ tok_idx,
                              int32_t* __restrict__ pos_ids, int32_t* __restrict__ cur_tok,
                              const int32_t* __restrict__ vu, const int32_t* __restrict__ pos,
                              int32_t L_meta, int32_t b, int32_t L_cap, int32_t* status) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= b) return;
  const int t = cur_tok[s];
  const int n = kv_len[s];  // loaded along with t: a round trip less where it is used
  if (t < 0 || t >= L_meta) {
    if (status) atomicOr(status, SCKV_STATUS_TOKEN);
  } else if (vu[(int64_t)s * L_meta + t] != t) {
    if (n < 0 || n >= L_cap) {
      if (status) atomicOr(status, SCKV_STATUS_CAP);
    } else {
      tok_idx[(int64_t)s * L_cap + n] = t;
      pos_ids[(int64_t)s * L_cap + n] = pos[(int64_t)s * L_meta + t];
      kv_len[s] = n + 1;
    }
  }
  cur_tok[s] = t + 1;
}

// ---------------------------------------------------------------------------
// block append bookkeeping: one workgroup per sequence
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void extend_kernel(int32_t* __restrict__ kv_len,
                                                     int32_t* __restrict__ tok_idx,
                                                     int32_t* __restrict__ pos_ids,
                                                     int32_t* __restrict__ row0_out,
                                                     const int32_t* __restrict__ pos,
                                                     int32_t L_meta, int32_t tok0, int32_t n,
                                                     int32_t L_cap, int32_t* status) {
  const int s = blockIdx.x;
  const int r0 = kv_len[s];
  const bool ok = r0 >= 0 && (int64_t)r0 + n <= L_cap;
  if (ok) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      tok_idx[(int64_t)s * L_cap + r0 + i] = tok0 + i;
      pos_ids[(int64_t)s * L_cap + r0 + i] = pos[(int64_t)s * L_meta + tok0 + i];
    }
  }
  __syncthreads();  // every thread has read kv_len[s]
  if (threadIdx.x == 0) {
    row0_out[s] = ok ? r0 : -1;
    if (ok) kv_len[s] = r0 + n;
    else if (status) atomicOr(status, SCKV_STATUS_CAP);
  }
}

}  // namespace sckv

using namespace sckv;

extern "C" int sckv_span_meta(const int32_t* cl_host, const int32_t* cr_host,
                              const int32_t* n_host, int32_t s_max, int32_t b, int32_t L_meta,
                              int32_t* spans_dev, int32_t* vu, int32_t* pos, hipStream_t stream) {
  clear_error();
  if (!cl_host || !cr_host || !n_host || !spans_dev || !vu)
    return fail(SCKV_EINVAL, "sckv_span_meta: null pointer");
  if (b <= 0 || s_max <= 0 || L_meta <= 0)
    return fail(SCKV_EINVAL, "sckv_span_meta: b, s_max and L_meta must be positive");
  for (int s = 0; s < b; ++s) {
    const int n = n_host[s];
    if (n < 0 || n > s_max)
      return fail(SCKV_ESPAN, "sckv_span_meta: span count of sequence " + std::to_string(s) +
                                  " outside [0, s_max]");
    for (int k = 0; k < n; ++k) {
      const int32_t c = cl_host[(int64_t)s * s_max + k], r = cr_host[(int64_t)s * s_max + k];
      if (c < 0 || c >= L_meta || r <= c)
        return fail(SCKV_ESPAN, "sckv_span_meta: sequence " + std::to_string(s) + " span " +
                                    std::to_string(k) + " needs 0 <= cl < L_meta and cl < cr");
      if (k > 0 && c <= cr_host[(int64_t)s * s_max + k - 1])
        return fail(SCKV_ESPAN, "sckv_span_meta: sequence " + std::to_string(s) + " span " +
                                    std::to_string(k) + " overlaps or is out of order");
    }
  }
  // Pack [cl | cr | n] and copy it in one transfer.  The source is a
  // pageable host vector: the copy has consumed it when the call returns.
  std::vector<int32_t> packed((size_t)2 * b * s_max + b);
  std::memcpy(packed.data(), cl_host, (size_t)b * s_max * sizeof(int32_t));
  std::memcpy(packed.data() + (size_t)b * s_max, cr_host, (size_t)b * s_max * sizeof(int32_t));
  std::memcpy(packed.data() + (size_t)2 * b * s_max, n_host, (size_t)b * sizeof(int32_t));
  int rc = hip_check(hipMemcpyAsync(spans_dev, packed.data(), packed.size() * sizeof(int32_t),
                                    hipMemcpyHostToDevice, stream),
                     "sckv_span_meta: span upload");
  if (rc) return rc;
  const dim3 grid((unsigned)((L_meta + (int64_t)255) / 256), (unsigned)(b < 65535 ? b : 65535));
  span_meta_kernel<<<grid, 256, 0, stream>>>(spans_dev, spans_dev + (size_t)2 * b * s_max, b, s_max,
                                          L_meta, vu, pos);
  return hip_check(hipGetLastError(), "sckv_span_meta: launch");
}

template <typename T, int D>
static int launch_rope(const void* x, void* y, int32_t b, int32_t H, int32_t n, int64_t xs,
                       int64_t ys, const int32_t* pos, int32_t L_meta, int32_t tok0, float theta,
                       const int32_t* row0, int32_t y_rows, int32_t* status,
                       hipStream_t stream) {
  InvFreq inv;
  for (int i = 0; i < 64; ++i) inv.w[i] = 0.0;
  for (int i = 0; i < D / 2; ++i) inv.w[i] = std::pow((double)theta, -2.0 * i / D);
  constexpr int PPH = D / 2 / Piece<T>::E;
  const int64_t per_seq = (int64_t)n * PPH;
  if (per_seq > 0x7fffffffLL - 255) return fail(SCKV_EUNSUP, "rope_apply: too many rows");
  // heads per thread: a rotation shares its angles over ROPE_HPT heads; a
  // plain copy takes one head per thread
  const int rotate = theta > 0.f ? 1 : 0;
  const int hpt = rotate ? (H < ROPE_HPT ? H : ROPE_HPT) : 1;
  const int64_t groups = (int64_t)b * ((H + hpt - 1) / hpt);
  const dim3 grid((unsigned)((per_seq + 255) / 256), (unsigned)(groups < 65535 ? groups : 65535));
  rope_kernel<T, D><<<grid, 256, 0, stream>>>(
      static_cast<const T*>(x), static_cast<T*>(y), b, H, n, xs, ys, pos, L_meta, tok0, inv,
      rotate, hpt, row0, y_rows, status);
  return hip_check(hipGetLastError(), "rope_apply: launch");
}

template <typename T, int D>
static int launch_rope_block(const RopeBlock<T>& rb, int32_t b, int32_t H, int32_t n,
                             const int32_t* pos, int32_t L_meta, int32_t tok0, float theta,
                             const int32_t* row0, int32_t L_cap, int32_t* status,
                             hipStream_t stream) {
  InvFreq inv;
  for (int i = 0; i < 64; ++i) inv.w[i] = 0.0;
  for (int i = 0; i < D / 2; ++i) inv.w[i] = std::pow((double)theta, -2.0 * i / D);
  const int64_t per_seq = (int64_t)n * (D / 2 / Piece<T>::E);
  if (per_seq > 0x7fffffffLL - 255) return fail(SCKV_EUNSUP, "rope_block: too many rows");
  const int rotate = theta > 0.f ? 1 : 0;
  const int hpt = rotate ? (H < ROPE_HPT ? H : ROPE_HPT) : 1;
  const int64_t groups = (int64_t)b * ((H + hpt - 1) / hpt);
  const dim3 grid((unsigned)((per_seq + 255) / 256), (unsigned)(groups < 65535 ? groups : 65535), 3);
  rope_block_kernel<T, D><<<grid, 256, 0, stream>>>(rb, b, H, n, pos, L_meta, tok0, inv, rotate,
                                                    hpt, row0, L_cap, status);
  return hip_check(hipGetLastError(), "rope_block: launch");
}

static int rope_checks(const std::string& w, const void* x, const void* y, int32_t b, int32_t H,
                       int32_t n, int64_t x_stride_bh, int64_t y_stride_bh, int32_t d_head,
                       sckv_dtype dt, const int32_t* pos, int32_t L_meta, int32_t tok0,
                       float theta, bool at, int32_t y_rows) {
  if (!x || !y) return fail(SCKV_EINVAL, w + ": null pointer");
  if (!valid_dtype(dt)) return fail(SCKV_EINVAL, w + ": unknown dtype");
  if (!supported_d(d_head)) return fail(SCKV_EUNSUP, w + ": d_head must be 64 or 80");
  if (b <= 0 || H <= 0 || n < 0) return fail(SCKV_EINVAL, w + ": bad sizes");
  if (x_stride_bh < (int64_t)n * d_head)
    return fail(SCKV_EINVAL, w + ": x slice stride smaller than n*d_head");
  if (at ? (y_rows < n || y_stride_bh < (int64_t)y_rows * d_head)
         : y_stride_bh < (int64_t)n * d_head)
    return fail(SCKV_EINVAL, w + ": y slice smaller than its rows");
  if (!(theta >= 0.f) || std::isinf(theta)) return fail(SCKV_EINVAL, w + ": theta must be finite and >= 0");
  if (theta > 0.f) {
    if (!pos) return fail(SCKV_EINVAL, w + ": null pos");
    if (tok0 < 0 || L_meta <= 0 || (int64_t)tok0 + n > L_meta)
      return fail(SCKV_EINVAL, w + ": rows [tok0, tok0+n) exceed L_meta");
  }
  if (!aligned16(x) || !aligned16(y) || (x_stride_bh * elem_bytes(dt)) % 16 ||
      (y_stride_bh * elem_bytes(dt)) % 16)
    return fail(SCKV_EINVAL, w + ": buffers and strides must be 16-byte aligned");
  return SCKV_OK;
}

static int rope_common(const char* who, const void* x, void* y, int32_t b, int32_t H, int32_t n,
                       int64_t x_stride_bh, int64_t y_stride_bh, int32_t d_head, sckv_dtype dt,
                       const int32_t* pos, int32_t L_meta, int32_t tok0, float theta,
                       const int32_t* row0, int32_t y_rows, int32_t* status, hipStream_t stream) {
  const int rc = rope_checks(who, x, y, b, H, n, x_stride_bh, y_stride_bh, d_head, dt, pos, L_meta,
                             tok0, theta, row0 != nullptr, y_rows);
  if (rc) return rc;
  if (n == 0) return SCKV_OK;
  if (dt == SCKV_BF16)
    return d_head == 64 ? launch_rope<uint16_t, 64>(x, y, b, H, n, x_stride_bh, y_stride_bh, pos, L_meta, tok0, theta, row0, y_rows, status, stream)
                        : launch_rope<uint16_t, 80>(x, y, b, H, n, x_stride_bh, y_stride_bh, pos, L_meta, tok0, theta, row0, y_rows, status, stream);
  return d_head == 64 ? launch_rope<float, 64>(x, y, b, H, n, x_stride_bh, y_stride_bh, pos, L_meta, tok0, theta, row0, y_rows, status, stream)
                      : launch_rope<float, 80>(x, y, b, H, n, x_stride_bh, y_stride_bh, pos, L_meta, tok0, theta, row0, y_rows, status, stream);
}

extern "C" int rope_apply(const void* x, void* y, int32_t b, int32_t H, int32_t n,
                          int64_t x_stride_bh, int64_t y_stride_bh, int32_t d_head, sckv_dtype dt,
                          const int32_t* pos, int32_t L_meta, int32_t tok0, float theta,
                          hipStream_t stream) {
  clear_error();
  return rope_common("rope_apply", x, y, b, H, n, x_stride_bh, y_stride_bh, d_head, dt, pos,
                     L_meta, tok0, theta, nullptr, 0, nullptr, stream);
}

extern "C" int rope_apply_at(const void* x, void* y, const int32_t* row0, int32_t y_rows,
                             int32_t b, int32_t H, int32_t n, int64_t x_stride_bh,
                             int64_t y_stride_bh, int32_t d_head, sckv_dtype dt,
                             const int32_t* pos, int32_t L_meta, int32_t tok0, float theta,
                             int32_t* status, hipStream_t stream) {
  clear_error();
  if (!row0) return fail(SCKV_EINVAL, "rope_apply_at: null row0");
  return rope_common("rope_apply_at", x, y, b, H, n, x_stride_bh, y_stride_bh, d_head, dt, pos,
                     L_meta, tok0, theta, row0, y_rows, status, stream);
}

template <typename T>
static int rope_block_typed(const void* q, const void* k, const void* v, void* qr, void* k_cache,
                            void* v_cache, const int32_t* row0, int32_t L_cap, int32_t b,
                            int32_t H, int32_t n, int64_t q_s, int64_t k_s, int64_t v_s,
                            int64_t qr_s, int64_t cache_s, int32_t d_head, const int32_t* pos,
                            int32_t L_meta, int32_t tok0, float theta, int32_t* status,
                            hipStream_t stream) {
  const RopeBlock<T> rb = {{static_cast<const T*>(k), static_cast<const T*>(v), static_cast<const T*>(q)},
                           {static_cast<T*>(k_cache), static_cast<T*>(v_cache), static_cast<T*>(qr)},
                           {k_s, v_s, q_s},
                           {cache_s, cache_s, qr_s}};
  return d_head == 64 ? launch_rope_block<T, 64>(rb, b, H, n, pos, L_meta, tok0, theta, row0, L_cap, status, stream)
                      : launch_rope_block<T, 80>(rb, b, H, n, pos, L_meta, tok0, theta, row0, L_cap, status, stream);
}

extern "C" int rope_block(const void* q, const void* k, const void* v, void* qr, void* k_cache,
                          void* v_cache, const int32_t* row0, int32_t L_cap, int32_t b, int32_t H,
                          int32_t n, int64_t q_stride_bh, int64_t k_stride_bh, int64_t v_stride_bh,
                          int64_t qr_stride_bh, int64_t cache_stride_bh, int32_t d_head,
                          sckv_dtype dt, const int32_t* pos, int32_t L_meta, int32_t tok0,
                          float theta, int32_t* status, hipStream_t stream) {
  clear_error();
  if (!row0) return fail(SCKV_EINVAL, "rope_block: null row0");
  int rc = rope_checks("rope_block", k, k_cache, b, H, n, k_stride_bh, cache_stride_bh, d_head, dt,
                       pos, L_meta, tok0, theta, true, L_cap);
  if (!rc)
    rc = rope_checks("rope_block", v, v_cache, b, H, n, v_stride_bh, cache_stride_bh, d_head, dt,
                     pos, L_meta, tok0, 0.f, true, L_cap);
  if (!rc)
    rc = rope_checks("rope_block", q, qr, b, H, n, q_stride_bh, qr_stride_bh, d_head, dt, pos,
                     L_meta, tok0, theta, false, 0);
  if (rc) return rc;
  if (n == 0) return SCKV_OK;
  return dt == SCKV_BF16
             ? rope_block_typed<uint16_t>(q, k, v, qr, k_cache, v_cache, row0, L_cap, b, H, n, q_stride_bh, k_stride_bh, v_stride_bh, qr_stride_bh, cache_stride_bh, d_head, pos, L_meta, tok0, theta, status, stream)
             : rope_block_typed<float>(q, k, v, qr, k_cache, v_cache, row0, L_cap, b, H, n, q_stride_bh, k_stride_bh, v_stride_bh, qr_stride_bh, cache_stride_bh, d_head, pos, L_meta, tok0, theta, status, stream);
}

extern "C" int kv_start(int32_t* kv_len, int32_t* tok_idx, int32_t* pos_ids, int32_t* cur_tok,
                        const int32_t* pos, int32_t L_meta, int32_t n, int32_t b, int32_t L_cap,
                        hipStream_t stream) {
  clear_error();
  if (!kv_len || !tok_idx || !pos_ids || !cur_tok || !pos)
    return fail(SCKV_EINVAL, "kv_start: null pointer");
  if (b <= 0 || L_cap <= 0 || L_meta <= 0 || n <= 0) return fail(SCKV_EINVAL, "kv_start: bad sizes");
  if (n > L_cap || n > L_meta) return fail(SCKV_EINVAL, "kv_start: n exceeds L_cap or L_meta");
  const dim3 grid((unsigned)((n + (int64_t)255) / 256), (unsigned)(b < 65535 ? b : 65535));
  start_kernel<<<grid, 256, 0, stream>>>(kv_len, tok_idx, pos_ids, cur_tok, pos, L_meta, n, b, L_cap);
  return hip_check(hipGetLastError(), "kv_start: launch");
}

extern "C" int kv_extend(int32_t* kv_len, int32_t* tok_idx, int32_t* pos_ids, int32_t* row0_out,
                         const int32_t* pos, int32_t L_meta, int32_t tok0, int32_t n, int32_t b,
                         int32_t L_cap, int32_t* status, hipStream_t stream) {
  clear_error();
  if (!kv_len || !tok_idx || !pos_ids || !row0_out || !pos)
    return fail(SCKV_EINVAL, "kv_extend: null pointer");
  if (b <= 0 || L_cap <= 0 || L_meta <= 0 || n < 0) return fail(SCKV_EINVAL, "kv_extend: bad sizes");
  if (tok0 < 0 || (int64_t)tok0 + n > L_meta)
    return fail(SCKV_EINVAL, "kv_extend: tokens [tok0, tok0+n) exceed L_meta");
  extend_kernel<<<b, 256, 0, stream>>>(kv_len, tok_idx, pos_ids, row0_out, pos, L_meta, tok0, n,
                                       L_cap, status);
  return hip_check(hipGetLastError(), "kv_extend: launch");
}

extern "C" int kv_commit(int32_t* kv_len, int32_t* tok_idx, int32_t* pos_ids, int32_t* cur_tok,
                         const int32_t* vu, const int32_t* pos, int32_t L_meta, int32_t b,
                         int32_t L_cap, int32_t* status, hipStream_t stream) {
  clear_error();
  if (!kv_len || !tok_idx || !pos_ids || !cur_tok || !vu || !pos)
    return fail(SCKV_EINVAL, "kv_commit: null pointer");
  if (b <= 0 || L_cap <= 0 || L_meta <= 0) return fail(SCKV_EINVAL, "kv_commit: bad sizes");
  commit_kernel<<<(b + 255) / 256, 256, 0, stream>>>(kv_len, tok_idx, pos_ids, cur_tok, vu, pos,
                                                     L_meta, b, L_cap, status);
  return hip_check(hipGetLastError(), "kv_commit: launch");
}
