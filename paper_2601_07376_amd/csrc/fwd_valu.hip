// Forward kernels for any mix of float32 / bfloat16 storage with a float32
// operand (Section 3.4, LoRA layer equation), on the float32 matrix-core
// instruction v_mfma_f32_16x16x4_f32: float32 products and sums, fixed
// summation order.
//
// Matrix core: lane l holds row l % 16 of the A operand and column l % 16 of the B
// operand at K index l / 16; the accumulator lane l holds rows 4 (l / 16) + v of
// column l % 16.  A lane loads four consecutive K values at K offset 4 (l / 16) of
// a 16-wide K step and feeds one of them to each of four instructions: any
// assignment of K values to instructions gives the same sum as long as both
// operands use it.
//
// What bounds them: latency.  With one thread per output and operands staged in
// LDS, a unit's sums were one chain of d_in fused multiply-adds and every row
// group of a short batch had a few busy waves; here eight waves share K.
// Whole float32 lora_apply calls, before and now: 64 rows 256 -> 256 rank 8 13.5
// and 11.4 us; 200 rows 1024 -> 1024 rank 16 45 and 16; 2000 rows 4096 -> 4096 rank 16
// 261 and 97, rank 128 1897 and 486.  The error against 64 bits fell from 1.0e-6 to
// 0.4e-6 (eight shorter sums instead of one chain of 4096).
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "lora_internal.h"

namespace lora {

namespace {

typedef f32x4 v4;

// Four consecutive values as float32 (16-byte aligned float32, 8-byte bfloat16).
template <bool BF16>
__device__ __forceinline__ v4 ld4(const void* p, int64_t i) {
  if (BF16) {
    const uint2 u = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(p) + i);
    return v4{bf16_to_f32(u.x & 0xffffu), bf16_to_f32(u.x >> 16), bf16_to_f32(u.y & 0xffffu),
              bf16_to_f32(u.y >> 16)};
  }
  return *reinterpret_cast<const v4*>(reinterpret_cast<const float*>(p) + i);
}
template <bool BF16>
__device__ __forceinline__ float ld(const void* p, int64_t i) {
  if (BF16) return bf16_to_f32(reinterpret_cast<const uint16_t*>(p)[i]);
  return reinterpret_cast<const float*>(p)[i];
}
// (not a template: the host pass cannot resolve the builtin inside one)
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

struct ValuArgs {
  const int32_t* hdr;
  const int4* rb;
  const int32_t* perm;
  const SlotMeta* meta;
  int32_t d_in, d_out;
  int32_t count_word, first_word;
  const void* X;
  int64_t ldx;
  float* H;
  int64_t ldh;
  void* Y;
  int64_t ldy;
  int32_t num_slots;
  int32_t n_rows;           // rows of the batch: the bound of every row id read from the plan
};

// Work unit: an entry's rows in groups of VG (one matrix-core tile).
constexpr int VG = 16;
constexpr int VGROUPS = RB_ROWS / VG;  // most row groups of an entry
constexpr int VW = 8;                  // waves of the shrink

// H[t, j] = sum_k X[t, k] A[j, k], ranks up to 16 NT: wave w takes the K steps
// w, w + 8, ..., two per batch, double buffered; the waves' sums meet in LDS.
template <bool XB, bool WB, int NT>
__global__ __launch_bounds__(VW * 64) void shrink_valu_kernel(ValuArgs p) {
  constexpr int U = NT <= 2 ? 2 : 1;
  __shared__ f32x4 s_red[VW * NT * 64];
  const int tid = threadIdx.x, lane = tid & 63, w = wave_id();
  const int n = lane & 15, kg = (lane >> 4) * 4;
  const int first = p.first_word >= 0 ? p.hdr[p.first_word] : 0;
  const int count = p.hdr[p.count_word] - first;
  for (int tile = blockIdx.x; tile < count * VGROUPS; tile += gridDim.x) {
    const int e = tile / VGROUPS, g = tile - e * VGROUPS;
    const int4 en = load_entry(p.rb, first + e);
    const int a = ck_slot(p.hdr, en.x, p.num_slots), rows = min(VG, en.z - g * VG), p0 = en.y + g * VG;
    if (rows <= 0) continue;
    const Slot m = load_slot(p.meta, a);
    const int r = m.rank;
    if (r <= 0) continue;
    const int64_t xo = (int64_t)ck_row(p.hdr, p.perm[p0 + min(n, rows - 1)], p.n_rows) * p.ldx;
    int64_t ao[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) ao[nt] = (int64_t)min(nt * 16 + n, r - 1) * p.d_in;
    struct Buf {
      v4 x[U], a[U][NT];
    };
    auto load = [&](Buf& b, int bt) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = (bt * VW * U + w * U + u) * 16 + kg, kk = min(k, p.d_in - 4);
        b.x[u] = ld4<XB>(p.X, xo + kk);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) b.a[u][nt] = ld4<WB>(m.A, ao[nt] + kk);
      }
    };
    f32x4 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mul = [&](const Buf& b, int bt) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool kv = (bt * VW * U + w * U + u) * 16 + kg < p.d_in;   // d_in is a multiple of 8
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int c = 0; c < 4; ++c)
            // (both operands zeroed: an infinity in the clamped values times 0 is not 0)
            acc[nt] = mfma_f32(kv ? b.x[u][c] : 0.0f, kv ? b.a[u][nt][c] : 0.0f, acc[nt]);
      }
    };
    const int nb = (p.d_in + VW * U * 16 - 1) / (VW * U * 16);
    Buf b0, b1;
    load(b0, 0);
    for (int bt = 0; bt < nb; bt += 2) {      // (batches past the end add zeros)
      load(b1, bt + 1);
      __builtin_amdgcn_sched_barrier(0);
      mul(b0, bt);
      load(b0, bt + 2);
      __builtin_amdgcn_sched_barrier(0);
      mul(b1, bt + 1);
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_nop 7");
      __builtin_amdgcn_sched_barrier(0);
    }
    mfma_fence();
    __syncthreads();                          // the previous unit's reads of s_red are done
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) s_red[(w * NT + nt) * 64 + lane] = acc[nt];
    __syncthreads();
    for (int q = tid; q < NT * 64; q += VW * 64) {
      f32x4 v[VW];
#pragma unroll
      for (int k = 0; k < VW; ++k) v[k] = s_red[k * NT * 64 + q];
      const f32x4 s = ((v[0] + v[4]) + (v[2] + v[6])) + ((v[1] + v[5]) + (v[3] + v[7]));
      const int j = (q >> 6) * 16 + (q & 15), i0 = ((q & 63) >> 4) * 4;
      if (j >= r) continue;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (i0 + k < rows)
          p.H[(int64_t)ck_row(p.hdr, p.perm[p0 + i0 + k], p.n_rows) * p.ldh + j] = s[k];
    }
  }
}

// Y[t, o] += s * sum_j H[t, j] B[o, j]; unit = (entry, 256 columns, row group), 64
// columns per wave.  B is the A operand, so a lane ends with four consecutive
// columns of one row.  NT: rank tiles of 16.
template <bool WB, bool YB, int NT>
__global__ __launch_bounds__(256) void expand_valu_kernel(ValuArgs p) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int n = lane & 15, g4 = (lane >> 4) * 4;
  const int first = p.first_word >= 0 ? p.hdr[p.first_word] : 0;
  const int count = p.hdr[p.count_word] - first;
  const int n_ot = (p.d_out + 255) / 256;
  for (int tile = blockIdx.x; tile < count * n_ot * VGROUPS; tile += gridDim.x) {
    const int g = tile % VGROUPS, eo = tile / VGROUPS;
    const int e = eo / n_ot, o0 = (eo - e * n_ot) * 256 + w * 64;
    const int4 en = load_entry(p.rb, first + e);
    const int a = ck_slot(p.hdr, en.x, p.num_slots), rows = min(VG, en.z - g * VG), p0 = en.y + g * VG;
    if (rows <= 0) continue;
    const Slot m = load_slot(p.meta, a);
    const int r = m.rank;
    const float s = m.scale;
    if (r <= 0) continue;
    const bool r4 = (r & 3) == 0;
    const int t = ck_row(p.hdr, p.perm[p0 + min(n, rows - 1)], p.n_rows);
    // Y of the lane's columns and the first B tile are requested together with H
    v4 y[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
      y[c] = ld4<YB>(p.Y, (int64_t)t * p.ldy + min(o0 + c * 16 + g4, p.d_out - 4));
    f32x4 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    // four values of a row from rank column j on, zero past the rank
    auto rank4 = [&](auto b16, const void* q, int64_t row, int j, bool vec) {
      constexpr bool B16 = decltype(b16)::value;
      v4 v;
      if (vec) {
        v = ld4<B16>(q, row + min(j, r - 4));
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = j < r ? v[c] : 0.0f;
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float x = ld<B16>(q, row + min(j + c, r - 1));
          v[c] = j + c < r ? x : 0.0f;
        }
      }
      return v;
    };
    v4 h[NT], b[NT][4];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int j = nt * 16 + g4;
      h[nt] = rank4(std::integral_constant<bool, false>{}, p.H, (int64_t)t * p.ldh, j, r4);
#pragma unroll
      for (int c = 0; c < 4; ++c)
        b[nt][c] = rank4(std::integral_constant<bool, WB>{}, m.B,
                         (int64_t)min(o0 + c * 16 + n, p.d_out - 1) * r, j, r4);
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[c] = mfma_f32(b[nt][c][k], h[nt][k], acc[c]);
    mfma_fence();
    if (n >= rows) continue;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int o = o0 + c * 16 + g4;
      if (o >= p.d_out) continue;             // d_out is a multiple of 8
      v4 v;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = fmaf(s, acc[c][k], y[c][k]);
      const int64_t yo = (int64_t)t * p.ldy + o;
      if (YB) *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(p.Y) + yo) =
          make_uint2(pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]));
      else *reinterpret_cast<v4*>(reinterpret_cast<float*>(p.Y) + yo) = v;
    }
  }
}

ValuArgs base_args(const OpLaunch& o) {
  ValuArgs a{};
  a.hdr = o.hdr;
  a.rb = o.rb;
  a.perm = o.perm;
  a.meta = o.meta;
  a.d_in = o.d_in;
  a.d_out = o.d_out;
  a.count_word = o.count_word;
  a.first_word = o.first_word;
  a.num_slots = o.num_slots;
  a.n_rows = o.n;
  return a;
}

}  // namespace

hipError_t launch_shrink_valu(const OpLaunch& o, const void* X, lora_dtype x_dtype,
                              int64_t ldx, lora_dtype w_dtype, float* H, int64_t ldh,
                              hipStream_t s) {
  ValuArgs a = base_args(o);
  a.X = X;
  a.ldx = ldx;
  a.H = H;
  a.ldh = ldh;
  const int grid = (int)std::max<long long>(1, std::min<long long>((long long)o.rb_ub * VGROUPS, 4096));
  const bool xb = x_dtype == LORA_BF16, wb = w_dtype == LORA_BF16;
  const int nt = (o.r_max + 15) / 16;
#define SV(NT)                                                                                         \
  do {                                                                                                 \
    const dim3 g(grid), b(VW * 64);                                                                    \
    if (xb && wb) hipLaunchKernelGGL((shrink_valu_kernel<true, true, NT>), g, b, 0, s, a);             \
    else if (xb) hipLaunchKernelGGL((shrink_valu_kernel<true, false, NT>), g, b, 0, s, a);             \
    else if (wb) hipLaunchKernelGGL((shrink_valu_kernel<false, true, NT>), g, b, 0, s, a);             \
    else hipLaunchKernelGGL((shrink_valu_kernel<false, false, NT>), g, b, 0, s, a);                    \
  } while (0)
  if (nt <= 1) SV(1);
  else if (nt <= 2) SV(2);
  else if (nt <= 4) SV(4);
  else SV(8);
#undef SV
  return hipGetLastError();
}

hipError_t launch_expand_valu(const OpLaunch& o, const float* H, int64_t ldh,
                              lora_dtype w_dtype, void* Y, lora_dtype y_dtype, int64_t ldy,
                              hipStream_t s) {
  ValuArgs a = base_args(o);
  a.H = const_cast<float*>(H);
  a.ldh = ldh;
  a.Y = Y;
  a.ldy = ldy;
  const long long tiles = (long long)o.rb_ub * ((o.d_out + 255) / 256) * VGROUPS;
  const int grid = (int)std::max<long long>(1, std::min<long long>(tiles, 8192));
  const bool wb = w_dtype == LORA_BF16, yb = y_dtype == LORA_BF16;
  const int nt = (o.r_max + 15) / 16;
#define EV(NT)                                                                                         \
  do {                                                                                                 \
    const dim3 g(grid), b(256);                                                                        \
    if (wb && yb) hipLaunchKernelGGL((expand_valu_kernel<true, true, NT>), g, b, 0, s, a);             \
    else if (wb) hipLaunchKernelGGL((expand_valu_kernel<true, false, NT>), g, b, 0, s, a);             \
    else if (yb) hipLaunchKernelGGL((expand_valu_kernel<false, true, NT>), g, b, 0, s, a);             \
    else hipLaunchKernelGGL((expand_valu_kernel<false, false, NT>), g, b, 0, s, a);                    \
  } while (0)
  if (nt <= 1) EV(1);
  else if (nt <= 2) EV(2);
  else if (nt <= 4) EV(4);
  else EV(8);
#undef EV
  return hipGetLastError();
}

}  // namespace lora
