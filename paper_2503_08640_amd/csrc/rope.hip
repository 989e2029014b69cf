// Rotary position tables and the encoding-time rotation of keys (Sec. 2.1: the pool is encoded
// with sequential position ids; Sec. 2.2: new in-order ids at query time).  Convention of the
// Llama models the paper runs: channel i pairs with channel i + D/2, angle = id * inv_freq[i].
#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "kernels.hpp"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct FreqArg {
  double f[64];
};

// table[n][i] = (cos, sin)(n * inv_freq[i]) rounded to fp32 from an fp64 evaluation: the angle
// reaches ~1e5 rad at the pool sizes in question, where an fp32 product would already be off
// by several 1e-3 rad.
__global__ void rope_table_kernel(FreqArg fr, int half_dim, int n_pos, float* table) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= static_cast<int64_t>(n_pos) * half_dim) return;
  const int n = static_cast<int>(idx / half_dim), i = static_cast<int>(idx % half_dim);
  const double ang = static_cast<double>(n) * fr.f[i];
  double s, c;
  sincos(ang, &s, &c);
  table[2 * idx] = static_cast<float>(c);
  table[2 * idx + 1] = static_cast<float>(s);
}

// One thread rotates 8 channel pairs (i .. i+7, partners at + D/2) of kHeads heads of one token: 16-byte accesses,
// and the table row, as long as a token's heads are few, is read once for all of them.  Bound by memory: rows of 32
// heads x 128 channels, 1900 tokens (31 MB) 19.1 -> 7.0 us, 8 heads 6.4 -> 5.3; 90k tokens x 8 heads (369 MB) 196 -> 74 us, 5.0 TB/s.
// Needs rows on 16-byte addresses (the kernel below takes every other tensor).
template <typename T>
struct Eight {
  typedef T type __attribute__((ext_vector_type(16 / sizeof(T))));
  static constexpr int kVecs = 8 * sizeof(T) / 16;
  type v[kVecs];
  __device__ float get(int i) const { return static_cast<float>(v[i / (8 / kVecs)][i % (8 / kVecs)]); }
  __device__ void set(int i, float x) { v[i / (8 / kVecs)][i % (8 / kVecs)] = static_cast<T>(x); }
  __device__ void load(const T* p) {
#pragma unroll
    for (int i = 0; i < kVecs; ++i) v[i] = reinterpret_cast<const type*>(p)[i];
  }
  __device__ void store(T* p) const {
#pragma unroll
    for (int i = 0; i < kVecs; ++i) reinterpret_cast<type*>(p)[i] = v[i];
  }
};

template <typename T, int kHeads>
__global__ __launch_bounds__(256) void rope_apply_rows_kernel(const T* x, int64_t x_tok, int64_t x_head, T* out, int64_t o_tok,
                                                              int64_t o_head, int n_tokens, int n_heads, int half_dim,
                                                              const int32_t* positions, int first_id, const float* table, int n_pos) {
  typedef float floatx4 __attribute__((ext_vector_type(4)));
  const unsigned parts = half_dim / 8, head_groups = (n_heads + kHeads - 1) / kHeads, per_token = parts * head_groups;
  const unsigned per_block = 256 / per_token > 0 ? 256 / per_token : 1;  // tokens of a workgroup
  // (a token with more than 256 parts takes several workgroups side by side: blockIdx.y)
  const unsigned in_token = blockIdx.y * 256 + threadIdx.x % (per_token < 256 ? per_token : 256);
  const int64_t tok = static_cast<int64_t>(blockIdx.x) * per_block + threadIdx.x / (per_token < 256 ? per_token : 256);
  if (threadIdx.x >= per_block * per_token || in_token >= per_token || tok >= n_tokens) return;
  const int part = in_token % parts, head0 = static_cast<int>(in_token / parts) * kHeads;
  int id = positions ? positions[tok] : first_id + static_cast<int>(tok);
  id = min(max(id, 0), n_pos - 1);
  const floatx4* cs = reinterpret_cast<const floatx4*>(table + (static_cast<int64_t>(id) * half_dim + 8 * part) * 2);
  floatx4 t[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) t[i] = cs[i];
  const T* xp = x + tok * x_tok + head0 * x_head + 8 * part;
  T* op = out + tok * o_tok + head0 * o_head + 8 * part;
  Eight<T> lo[kHeads], hi[kHeads];  // (heads past the last repeat it)
#pragma unroll
  for (int h = 0; h < kHeads; ++h) {
    const T* row = xp + min(h, n_heads - 1 - head0) * x_head;
    lo[h].load(row);
    hi[h].load(row + half_dim);
  }
#pragma unroll
  for (int h = 0; h < kHeads; ++h) {
    if (head0 + h >= n_heads) break;
    Eight<T> a, b;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float c = t[e / 2][2 * (e % 2)], s = t[e / 2][2 * (e % 2) + 1], u = lo[h].get(e), w = hi[h].get(e);
      a.set(e, u * c - w * s);
      b.set(e, w * c + u * s);
    }
    a.store(op + h * o_head);
    b.store(op + h * o_head + half_dim);
  }
}

// the same for tensors on any address, element by element: one thread, 8 channel pairs of one (token, head)
template <typename T>
__global__ void rope_apply_kernel(const T* x, int64_t x_tok, int64_t x_head, T* out, int64_t o_tok, int64_t o_head,
                                  int n_tokens, int n_heads, int half_dim, const int32_t* positions, int first_id,
                                  const float* table, int n_pos) {
  const int per_row = half_dim / 8;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= static_cast<int64_t>(n_tokens) * n_heads * per_row) return;
  const int part = static_cast<int>(idx % per_row);
  const int head = static_cast<int>((idx / per_row) % n_heads);
  const int tok = static_cast<int>(idx / (static_cast<int64_t>(per_row) * n_heads));
  int id = positions ? positions[tok] : first_id + tok;
  id = min(max(id, 0), n_pos - 1);
  const float* cs = table + (static_cast<int64_t>(id) * half_dim + 8 * part) * 2;
  const T* xp = x + tok * x_tok + head * x_head + 8 * part;
  T* op = out + tok * o_tok + head * o_head + 8 * part;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float a = static_cast<float>(xp[e]), b = static_cast<float>(xp[e + half_dim]);
    const float c = cs[2 * e], s = cs[2 * e + 1];
    op[e] = static_cast<T>(a * c - b * s);
    op[e + half_dim] = static_cast<T>(b * c + a * s);
  }
}

}  // namespace

hipError_t launch_rope_table(const double* inv_freq, int head_dim, int n_pos, float* table, hipStream_t stream) {
  FreqArg fr{};
  for (int i = 0; i < head_dim / 2; ++i) fr.f[i] = inv_freq[i];
  const int64_t n = static_cast<int64_t>(n_pos) * (head_dim / 2);
  if (n == 0) return hipSuccess;
  rope_table_kernel<<<static_cast<unsigned>((n + 255) / 256), 256, 0, stream>>>(fr, head_dim / 2, n_pos, table);
  return hipGetLastError();
}

hipError_t launch_rope_apply(const TensorView& x, const TensorView& out, int n_tokens, int n_heads, int head_dim,
                             bool bf16, const int32_t* positions, int first_id, const float* table, int n_pos,
                             hipStream_t stream) {
  const int64_t n = static_cast<int64_t>(n_tokens) * n_heads * (head_dim / 16);
  if (n == 0) return hipSuccess;
  const int es = bf16 ? 2 : 4;
  bool rows = reinterpret_cast<uintptr_t>(table) % 16 == 0;
  for (const TensorView* v : {&x, &out})
    rows = rows && reinterpret_cast<uintptr_t>(v->ptr) % 16 == 0 && v->stride_tok * es % 16 == 0 && v->stride_head * es % 16 == 0;
  // an output that overlaps the input other than row on row is read as it is written: element order stays as it was
  rows = rows && (x.ptr != out.ptr || (x.stride_tok == out.stride_tok && x.stride_head == out.stride_head));
  if (rows) {
    // four heads a thread once that leaves enough threads to fill the chip (about 64 k), else fewer
    int per_thread = 4;
    while (per_thread > 1 && n / per_thread < 65536) per_thread /= 2;
    const int per_token = head_dim / 16 * ((n_heads + per_thread - 1) / per_thread);
    const int per_block = std::max(1, 256 / per_token);
    const dim3 grid(static_cast<unsigned>((n_tokens + per_block - 1) / per_block), static_cast<unsigned>((per_token + 255) / 256));
    auto launch_as = [&](auto type, auto heads) {
      using T = decltype(type);
      rope_apply_rows_kernel<T, decltype(heads)::value><<<grid, 256, 0, stream>>>(
          static_cast<const T*>(x.ptr), x.stride_tok, x.stride_head, static_cast<T*>(const_cast<void*>(out.ptr)), out.stride_tok,
          out.stride_head, n_tokens, n_heads, head_dim / 2, positions, first_id, table, n_pos);
    };
    auto launch = [&](auto type) {
      if (per_thread == 4) launch_as(type, std::integral_constant<int, 4>{});
      else if (per_thread == 2) launch_as(type, std::integral_constant<int, 2>{});
      else launch_as(type, std::integral_constant<int, 1>{});
    };
    if (bf16) launch(__bf16{});
    else launch(float{});
    return hipGetLastError();
  }
  const unsigned grid = static_cast<unsigned>((n + 255) / 256);
  if (bf16)
    rope_apply_kernel<__bf16><<<grid, 256, 0, stream>>>(
        static_cast<const __bf16*>(x.ptr), x.stride_tok, x.stride_head,
        static_cast<__bf16*>(const_cast<void*>(out.ptr)), out.stride_tok, out.stride_head, n_tokens, n_heads,
        head_dim / 2, positions, first_id, table, n_pos);
  else
    rope_apply_kernel<float><<<grid, 256, 0, stream>>>(
        static_cast<const float*>(x.ptr), x.stride_tok, x.stride_head, static_cast<float*>(const_cast<void*>(out.ptr)),
        out.stride_tok, out.stride_head, n_tokens, n_heads, head_dim / 2, positions, first_id, table, n_pos);
  return hipGetLastError();
}
