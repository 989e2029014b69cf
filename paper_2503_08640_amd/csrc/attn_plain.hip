// fp32-arithmetic attention kernel on the fp32 matrix instructions: the DBSA_F32 dtype (any tile sizes,
// Sec. 2.1 / 2.2 semantics as documented in dbsa.h), and re-positioning (Sec. 2.2) for the bf16 shapes the
// bf16 matrix kernels do not re-position.  With a rotary table the row of Q is rotated at list_shift[e] +
// (its index inside the Q tile) before it meets the keys of list entry e (decode: dec_shift[e] +
// self_len - 1, own cache: self_len - 1), anew wherever that id changes along the list.
//
// A workgroup owns 16 rows (prefill: tokens of one query head; decode: the query heads of one KV head) and
// its W waves share the KEYS: wave w walks the blocks of 16 keys w % 4, w % 4 + 4, ... of every (W / 4)-th list
// entry, so that even one 16-token question over a few hundred keys occupies all SIMDs of a compute unit and a
// wave's serial chain is a few blocks long.  The waves' softmax states are merged in LDS at the end.  What bounds
// the small calls this dtype is used for is that chain of latencies, not bandwidth: K and V go straight from
// memory into operand registers (no LDS, no barrier) one block ahead of their use.
// Measured (2 heads x 64, 260-token pool, 16-token question): encoding 539 -> 6.8 us, prefill 86 -> 7.0 us, decode
// step 20 -> 6.6 us against one wave per (row, head) with a lane per key; 4 heads over 1400 tokens, all three calls:
// 3295 -> 56 us.  (Error against fp64 halves: shorter sums.)
//
// v_mfma_f32_16x16x4_f32 multiplies in any order of the contraction index as long as both operands agree, which
// lets every operand be loaded 16 bytes at a time: lane (n = lane % 16, g = lane / 16) holds channels
// 16 t + 4 g + e of its K row / Q row (product t, e), and for the second product channels 64 h + 4 n + c of the
// V rows 4 g + j; the scores S^T come out as keys 4 g + j of row n, which is the layout the second product reads.
#include <atomic>
#include <climits>

#include "kernels.hpp"
#include "mfma_common.hpp"

namespace {

using namespace dbsa_mfma;

constexpr int kRows = 16;            // rows of a workgroup, keys of a block
constexpr float kNoKey = -3.0e38f;   // below every finite score: "no key seen yet"

__device__ inline floatx4 load4(const float* p) { return *reinterpret_cast<const floatx4*>(p); }
__device__ inline floatx4 load4(const __bf16* p) {
  const bf16x4 x = *reinterpret_cast<const bf16x4*>(p);
  return floatx4{static_cast<float>(x[0]), static_cast<float>(x[1]), static_cast<float>(x[2]), static_cast<float>(x[3])};
}
__device__ inline void store4(float* p, floatx4 x) { *reinterpret_cast<floatx4*>(p) = x; }
__device__ inline void store4(__bf16* p, floatx4 x) { *reinterpret_cast<bf16x4*>(p) = __builtin_convertvector(x, bf16x4); }

// combine a value over the four lanes that share n = lane % 16
__device__ inline float quad_max(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return half_swap_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ inline float quad_sum(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return half_swap_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// 16 keys a wave attends to: rows row0 .. row0 + n - 1 of the pool or of the call's own K/V
struct KeyBlock {
  int row0, n;      // n == 0: the wave has no further block
  int shift;        // ROPE: rotation id of row 0
  bool self, causal;
};

template <typename T, int D, bool ROPE, bool DECODE, int W>
__global__ __launch_bounds__(64 * W) void attn_f32_kernel(AttnParams p, int chunks) {
  static_assert(W % 4 == 0, "four waves share a list entry");
  constexpr int kT = D / 16, kH = D / 64, kORow = D + 4;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float* lds_m = smem;                  // [W][16]
  float* lds_l = smem + W * kRows;      // [W][16]
  float* lds_o = smem + 2 * W * kRows;  // [W][16][D + 4]

  const int lane = threadIdx.x % 64, n = lane % 16, g = lane / 16;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / 64);
  const int r = p.n_q_heads / p.n_kv_heads;

  // ---- the 16 rows and the entries they attend to ----
  const int unit = static_cast<int>(blockIdx.x) / chunks, chunk = static_cast<int>(blockIdx.x) % chunks;
  int hk, q_start = 0, q_len, self_len = 0;
  int64_t e0, e1;
  const int32_t* ent;
  const int32_t* ids;
  if constexpr (DECODE) {  // unit = query
    hk = blockIdx.y;
    q_len = r;
    self_len = __builtin_amdgcn_readfirstlane(p.self_len[unit]);
    e0 = p.split_ptr[static_cast<int64_t>(unit) * (p.n_split + 1)];
    e1 = p.split_ptr[static_cast<int64_t>(unit) * (p.n_split + 1) + p.n_split];
    ent = p.dec_ent;
    ids = p.dec_shift;
  } else {  // unit = Q tile
    hk = static_cast<int>(blockIdx.y) / r;
    q_start = p.qtile_tab[unit * 4 + 0];
    q_len = p.qtile_tab[unit * 4 + 1];
    e0 = p.list_ptr[unit];
    e1 = p.list_ptr[unit + 1];
    ent = p.list_ent;
    ids = p.list_shift;
  }
  if (chunk * kRows >= q_len) return;
  const int row = chunk * kRows + min(n, q_len - 1 - chunk * kRows);  // rows past the last repeat it
  const int q_pos = q_start + row, q_hi = q_start + min(chunk * kRows + kRows, q_len) - 1;
  const int n_listed = static_cast<int>(e1 - e0), n_ent = n_listed + (DECODE ? 1 : 0);  // decode: the own cache comes last

  const T* kp = static_cast<const T*>(p.k_pool.ptr) + hk * p.k_pool.stride_head;
  const T* vp = static_cast<const T*>(p.v_pool.ptr) + hk * p.v_pool.stride_head;
  const T* ks = static_cast<const T*>(p.k_self.ptr) + hk * p.k_self.stride_head + (DECODE ? unit * p.stride_query : 0);
  const T* vs = static_cast<const T*>(p.v_self.ptr) + hk * p.v_self.stride_head + (DECODE ? unit * p.stride_query : 0);

  auto row_offset = [&](const TensorView& t, int i) {  // of row i of the workgroup
    return DECODE ? static_cast<int64_t>(unit) * t.stride_tok + static_cast<int64_t>(hk * r + i) * t.stride_head
                  : static_cast<int64_t>(q_start + i) * t.stride_tok + static_cast<int64_t>(blockIdx.y) * t.stride_head;
  };
  floatx4 q0[ROPE ? kT : 1], qf[kT];
  {
    const T* qp = static_cast<const T*>(p.q.ptr) + row_offset(p.q, row) + 4 * g;
#pragma unroll
    for (int t = 0; t < kT; ++t) {
      qf[t] = load4(qp + 16 * t);
      if constexpr (ROPE) q0[t] = qf[t];
    }
  }

  // ---- this wave's blocks ----
  int cur_e = wave / 4, cur_off = kRows * (wave % 4);
  auto next_block = [&]() {
    KeyBlock b{0, 0, 0, false, false};
    while (cur_e < n_ent) {
      int start = 0, len = self_len, kind = 2, id = 0;
      if (!DECODE || cur_e < n_listed) {
        const int w1 = ent[2 * (e0 + cur_e) + 1];
        start = ent[2 * (e0 + cur_e)];
        len = w1 & 0xFFFF;
        kind = w1 >> 16;
        if constexpr (ROPE) id = ids[e0 + cur_e];
      }
      const bool causal = !DECODE && (kind & 1);
      if (cur_off < len && (!causal || start + cur_off <= q_hi)) {
        b.row0 = start + cur_off;
        b.n = min(kRows, len - cur_off);
        b.shift = id;
        b.self = kind & 2;
        b.causal = causal;
        cur_off += 4 * kRows;
        break;
      }
      cur_e += W / 4;
      cur_off = kRows * (wave % 4);
    }
    return b;
  };
  struct Operands {
    floatx4 k[kT], v[4][kH];
  };
  auto load_block = [&](const KeyBlock& b, Operands& x) {
    const int64_t k_stride = b.self ? p.k_self.stride_tok : p.k_pool.stride_tok;
    const int64_t v_stride = b.self ? p.v_self.stride_tok : p.v_pool.stride_tok;
    const T* kr = (b.self ? ks : kp) + (b.row0 + min(n, b.n - 1)) * k_stride + 4 * g;  // keys past the last repeat it
#pragma unroll
    for (int t = 0; t < kT; ++t) x.k[t] = load4(kr + 16 * t);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const T* vr = (b.self ? vs : vp) + (b.row0 + min(4 * g + j, b.n - 1)) * v_stride + 4 * n;
#pragma unroll
      for (int h = 0; h < kH; ++h) x.v[j][h] = load4(vr + 64 * h);
    }
  };

  // ---- running softmax state: raw scores, their maximum, this lane's share of the sum, O^T ----
  float m = kNoKey, l = 0.f;
  floatx4 o[kH][4];
#pragma unroll
  for (int h = 0; h < kH; ++h)
#pragma unroll
    for (int c = 0; c < 4; ++c) o[h][c] = floatx4{0.f, 0.f, 0.f, 0.f};
  const float c2 = p.scale_log2e;
  int rotated_at = INT_MIN;

  auto attend = [&](const KeyBlock& b, Operands& x) {
    if constexpr (ROPE) {
      if (b.shift != rotated_at) {  // uniform over the wave
        rotated_at = b.shift;
        const int id = min(max(b.shift + (DECODE ? self_len - 1 : row), 0), p.rope_n_pos - 1);
        const float* cs = p.rope_table + static_cast<int64_t>(id) * D + 8 * g;
#pragma unroll
        for (int t = 0; t < kT / 2; ++t) {
          const floatx4 ab = load4(cs + 32 * t), cd = load4(cs + 32 * t + 4);  // (cos, sin) of four channel pairs
          const floatx4 c = {ab[0], ab[2], cd[0], cd[2]}, s = {ab[1], ab[3], cd[1], cd[3]};
          const floatx4 lo = q0[t], hi = q0[t + kT / 2];
          qf[t] = lo * c - hi * s;
          qf[t + kT / 2] = hi * c + lo * s;
        }
      }
    }
    floatx4 s = {0.f, 0.f, 0.f, 0.f}, s2 = s;  // two chains: half the latency
#pragma unroll
    for (int t = 0; t < kT; ++t) {
      s = __builtin_amdgcn_mfma_f32_16x16x4f32(x.k[t][0], qf[t][0], s, 0, 0, 0);
      s2 = __builtin_amdgcn_mfma_f32_16x16x4f32(x.k[t][1], qf[t][1], s2, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_16x16x4f32(x.k[t][2], qf[t][2], s, 0, 0, 0);
      s2 = __builtin_amdgcn_mfma_f32_16x16x4f32(x.k[t][3], qf[t][3], s2, 0, 0, 0);
    }
    s += s2;
    if (b.causal || b.n < kRows) {
      const int last = min(b.causal ? q_pos - b.row0 : kRows, b.n - 1);  // last key of the block the row sees
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s[j] = 4 * g + j <= last ? s[j] : -INFINITY;
        if (4 * g + j >= b.n)  // a value that no row sees must not meet its weight of zero (it may be infinite)
#pragma unroll
          for (int h = 0; h < kH; ++h) x.v[j][h] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
    }
    const float m_new = fmaxf(m, quad_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))));
    const float alpha = __builtin_amdgcn_exp2f((m - m_new) * c2);
    m = m_new;
    floatx4 w;
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = __builtin_amdgcn_exp2f((s[j] - m_new) * c2);
    l = fmaf(l, alpha, (w[0] + w[1]) + (w[2] + w[3]));
#pragma unroll
    for (int h = 0; h < kH; ++h)
#pragma unroll
      for (int c = 0; c < 4; ++c) o[h][c] *= alpha;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < kH; ++h)
#pragma unroll
        for (int c = 0; c < 4; ++c) o[h][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.v[j][h][c], w[j], o[h][c], 0, 0, 0);
  };

  Operands xa, xb;
  KeyBlock a = next_block();
  if (a.n) load_block(a, xa);
  while (a.n) {
    const KeyBlock b = next_block();
    if (b.n) load_block(b, xb);
    attend(a, xa);
    if (!b.n) break;
    a = next_block();
    if (a.n) load_block(a, xa);
    attend(b, xb);
  }

  // ---- merge the waves' states: o = sum_w o_w 2^((m_w - m*) c2) / sum_w l_w 2^((m_w - m*) c2) ----
  l = quad_sum(l);
  if (g == 0) {
    lds_m[wave * kRows + n] = m;
    lds_l[wave * kRows + n] = l;
  }
#pragma unroll
  for (int h = 0; h < kH; ++h)
#pragma unroll
    for (int j = 0; j < 4; ++j)  // channels 64 h + 4 (4 g + j) .. + 3
      store4(lds_o + (wave * kRows + n) * kORow + 64 * h + 16 * g + 4 * j, floatx4{o[h][0][j], o[h][1][j], o[h][2][j], o[h][3][j]});
  __syncthreads();
  for (int i = threadIdx.x; i < kRows * D / 4; i += 64 * W) {
    const int lr = i / (D / 4), d = 4 * (i % (D / 4)), out_row = chunk * kRows + lr;
    if (out_row >= q_len) continue;
    float m_star = lds_m[lr];
#pragma unroll
    for (int w = 1; w < W; ++w) m_star = fmaxf(m_star, lds_m[w * kRows + lr]);
    float l_star = 0.f;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float f = __builtin_amdgcn_exp2f((lds_m[w * kRows + lr] - m_star) * c2);
      l_star = fmaf(lds_l[w * kRows + lr], f, l_star);
      acc += load4(lds_o + (w * kRows + lr) * kORow + d) * f;
    }
    const float inv = 1.f / l_star;
    store4(static_cast<T*>(const_cast<void*>(p.o.ptr)) + row_offset(p.o, out_row) + d, acc * inv);
    if (!DECODE && p.lse && d == 0)
      p.lse[static_cast<int64_t>(blockIdx.y) * p.lse_stride + q_start + out_row] = m_star * p.scale + __logf(l_star);
  }
}

template <typename T, int D, bool ROPE, bool DECODE, int W>
hipError_t launch_waves(const AttnParams& p, dim3 grid, int chunks, hipStream_t stream) {
  constexpr int lds_bytes = W * kRows * (2 + D + 4) * static_cast<int>(sizeof(float));
  static std::atomic<bool> attr_set{false};  // setting it twice from two threads is harmless
  if (lds_bytes > 65536 && !attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_f32_kernel<T, D, ROPE, DECODE, W>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  attn_f32_kernel<T, D, ROPE, DECODE, W><<<grid, dim3(64 * W), lds_bytes, stream>>>(p, chunks);
  return hipGetLastError();
}

template <typename T, int D, bool DECODE>
hipError_t launch_rope_or_not(const AttnParams& p, dim3 grid, int chunks, int compute_units, hipStream_t stream) {
  // Four waves are one per SIMD.  While the launch leaves compute units without a second workgroup, eight waves
  // halve each wave's chain of blocks; with more workgroups than that the waves only queue up.
  const bool wide = static_cast<int64_t>(grid.x) * grid.y <= compute_units;
  if (p.rope_table)
    return wide ? launch_waves<T, D, true, DECODE, 8>(p, grid, chunks, stream)
                : launch_waves<T, D, true, DECODE, 4>(p, grid, chunks, stream);
  return wide ? launch_waves<T, D, false, DECODE, 8>(p, grid, chunks, stream)
              : launch_waves<T, D, false, DECODE, 4>(p, grid, chunks, stream);
}

template <bool DECODE>
hipError_t launch_typed(const AttnParams& p, int head_dim, bool bf16_storage, dim3 grid, int chunks, int compute_units,
                        hipStream_t stream) {
  if (head_dim == 64)
    return bf16_storage ? launch_rope_or_not<__bf16, 64, DECODE>(p, grid, chunks, compute_units, stream)
                        : launch_rope_or_not<float, 64, DECODE>(p, grid, chunks, compute_units, stream);
  return bf16_storage ? launch_rope_or_not<__bf16, 128, DECODE>(p, grid, chunks, compute_units, stream)
                      : launch_rope_or_not<float, 128, DECODE>(p, grid, chunks, compute_units, stream);
}

}  // namespace

hipError_t launch_prefill_plain(const AttnParams& p, int head_dim, bool bf16_storage, int compute_units, hipStream_t stream) {
  if (p.n_qtiles == 0) return hipSuccess;
  const int chunks = (p.largest_tile + kRows - 1) / kRows;
  return launch_typed<false>(p, head_dim, bf16_storage, dim3(p.n_qtiles * chunks, p.n_q_heads), chunks, compute_units, stream);
}

hipError_t launch_decode_plain(const AttnParams& p, int head_dim, bool bf16_storage, int compute_units, hipStream_t stream) {
  const int chunks = (p.n_q_heads / p.n_kv_heads + kRows - 1) / kRows;
  return launch_typed<true>(p, head_dim, bf16_storage, dim3(p.n_queries * chunks, p.n_kv_heads), chunks, compute_units, stream);
}
