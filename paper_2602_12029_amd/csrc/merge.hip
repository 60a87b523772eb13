// Log-sum-exp merge of partial attention states.
//
// For each (request, q head) the partial states (o_i, lse_i) of its prefix and suffix splits are
// combined as lse = log sum_i exp(lse_i), o = sum_i exp(lse_i - lse) o_i -- exact by softmax algebra
// over the concatenated cache [C_base ; own tokens] (Background Eq. 2).  One thread owns four
// consecutive head-dim elements of one row.
#include "device_common.h"
#include "launch.h"

namespace psdev {

// four columns of a row of the output, rounded to the queries' format
template <int QT>
__device__ __forceinline__ void store_row(void* out, int64_t row, int head_dim, int c4, f32x4 acc) {
  if constexpr (QT == PS_F32) {
    *reinterpret_cast<f32x4*>(static_cast<float*>(out) + row * head_dim + 4 * c4) = acc;
  } else {
    bf16x2 lo, hi;
    lo.x = (__bf16)acc.x; lo.y = (__bf16)acc.y; hi.x = (__bf16)acc.z; hi.y = (__bf16)acc.w;
    uint2 packed;
    packed.x = __builtin_bit_cast(uint32_t, lo);
    packed.y = __builtin_bit_cast(uint32_t, hi);
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(out) + row * head_dim + 4 * c4) = packed;
  }
}

// BATCH: partial states whose loads go out together, chosen by the most states a request of the launch has.
template <int QT, int BATCH>
__global__ __launch_bounds__(256) void merge_states_kernel(const int32_t* __restrict__ slot_base,
                                                           const int32_t* __restrict__ requests,
                                                           const float* __restrict__ ws_o,
                                                           const float* __restrict__ ws_lse, void* __restrict__ out,
                                                           float* __restrict__ out_lse, int num_rows, int num_q_heads,
                                                           int head_dim) {
  const int per_row = head_dim >> 2;
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t listed = gid / per_row;
  if (listed >= num_rows) return;
  const int c4 = int(gid % per_row);
  const int h = int(listed % num_q_heads);
  const int r = requests ? requests[listed / num_q_heads] : int(listed / num_q_heads);
  const int64_t row = int64_t(r) * num_q_heads + h;
  const int s0 = slot_base[r], s1 = slot_base[r + 1];
  const float neg_inf = -__builtin_inff();

  // Batches of up to BATCH partial states: their lse and o loads all go out before anything is used, so a row with
  // at most that many splits costs one memory round trip after slot_base instead of one for the maxima and one for the
  // values.  Across batches the running state (mx, total, acc) is rescaled like an online softmax; a single batch is
  // the plain two-pass formula.
  float mx = neg_inf, total = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int b0 = s0; b0 < s1; b0 += BATCH) {
    float lse[BATCH];
    f32x4 o[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      lse[i] = neg_inf;                    // a slot past the end has weight zero and is not read
      o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (b0 + i < s1) {
        const int64_t s = b0 + i;
        lse[i] = ws_lse[s * num_q_heads + h];
        // the states are read once: non-temporal
        o[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(ws_o + (s * num_q_heads + h) * head_dim + 4 * c4));
      }
    }
    float bm = mx;
#pragma unroll
    for (int i = 0; i < BATCH; ++i) bm = fmaxf(bm, lse[i]);
    if (bm == neg_inf) {                   // nothing but empty states so far, or not a number, which fmaxf passes by
#pragma unroll
      for (int i = 0; i < BATCH; ++i)
        if (lse[i] != lse[i]) mx = lse[i];
      if (mx != mx) {
        total = mx;
        acc = f32x4{mx, mx, mx, mx};
      }
      continue;
    }
    const float keep = (mx == neg_inf) ? 0.f : fast_exp2((mx - bm) * kLog2e);
    total *= keep;
    acc *= keep;
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      if (lse[i] != neg_inf) {             // an empty state has weight zero, whatever its o holds
        const float w = fast_exp2((lse[i] - bm) * kLog2e);
        total += w;
        acc += w * o[i];
      }
    }
    mx = bm;
  }
  if (mx != neg_inf) acc *= 1.f / total;
  store_row<QT>(out, row, head_dim, c4, acc);
  if (out_lse && c4 == 0) out_lse[row] = (mx != neg_inf) ? mx + __builtin_amdgcn_logf(total) * kLn2 : neg_inf;
}

// Rows of many partial states: a workgroup per row, HD / 4 threads to a state and 1024 / HD states at a time; the groups of threads
// meet in LDS.
template <int QT, int HD>
__global__ __launch_bounds__(256) void merge_many_kernel(const int32_t* __restrict__ slot_base, const int32_t* __restrict__ requests,
                                                         const float* __restrict__ ws_o, const float* __restrict__ ws_lse,
                                                         void* __restrict__ out, float* __restrict__ out_lse, int num_q_heads) {
  constexpr int kLanes = HD / 4, kGroups = 256 / kLanes, kBatch = 4;
  __shared__ f32x4 sm_acc[kGroups][kLanes];
  __shared__ float sm_mx[kGroups], sm_total[kGroups];
  const int listed = int(blockIdx.x / unsigned(num_q_heads)), h = int(blockIdx.x % unsigned(num_q_heads));
  const int r = requests ? requests[listed] : listed;
  const int s0 = slot_base[r], s1 = slot_base[r + 1];
  const int group = int(threadIdx.x) / kLanes, c4 = int(threadIdx.x) % kLanes;
  const float neg_inf = -__builtin_inff();
  float mx = neg_inf, total = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int b0 = s0 + group; b0 < s1; b0 += kBatch * kGroups) {
    float lse[kBatch];
    f32x4 o[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int64_t s = b0 + i * kGroups;
      lse[i] = neg_inf;
      o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (s < s1) {
        lse[i] = ws_lse[s * num_q_heads + h];
        o[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(ws_o + (s * num_q_heads + h) * HD + 4 * c4));
      }
    }
    float bm = mx;
#pragma unroll
    for (int i = 0; i < kBatch; ++i) bm = fmaxf(bm, lse[i]);
    if (bm == neg_inf) {                   // nothing but empty states so far, or not a number, which fmaxf passes by
#pragma unroll
      for (int i = 0; i < kBatch; ++i)
        if (lse[i] != lse[i]) mx = lse[i];
      if (mx != mx) {
        total = mx;
        acc = f32x4{mx, mx, mx, mx};
      }
      continue;
    }
    const float keep = (mx == neg_inf) ? 0.f : fast_exp2((mx - bm) * kLog2e);
    total *= keep;
    acc *= keep;
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      if (lse[i] != neg_inf) {             // an empty state has weight zero, whatever its o holds
        const float w = fast_exp2((lse[i] - bm) * kLog2e);
        total += w;
        acc += w * o[i];
      }
    }
    mx = bm;
  }
  sm_acc[group][c4] = acc;
  if (c4 == 0) {
    sm_mx[group] = mx;
    sm_total[group] = total;
  }
  __syncthreads();
  if (group != 0) return;
  float top = neg_inf;
#pragma unroll
  for (int g = 0; g < kGroups; ++g) top = fmaxf(top, sm_mx[g]);
  if (top == neg_inf) {
#pragma unroll
    for (int g = 0; g < kGroups; ++g)
      if (sm_mx[g] != neg_inf) top = sm_mx[g];   // not a number
  }
  float sum = 0.f;
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  if (top != neg_inf) {
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      if (sm_mx[g] != neg_inf) {
        const float w = fast_exp2((sm_mx[g] - top) * kLog2e);
        sum += w * sm_total[g];
        o += w * sm_acc[g][c4];
      }
    }
    o *= 1.f / sum;
  }
  store_row<QT>(out, int64_t(r) * num_q_heads + h, HD, c4, o);
  if (out_lse && c4 == 0) out_lse[int64_t(r) * num_q_heads + h] = (top != neg_inf) ? top + __builtin_amdgcn_logf(sum) * kLn2 : neg_inf;
}

int32_t launch_merge(const int32_t* slot_base, const int32_t* requests, const float* ws_o, const float* ws_lse, void* out,
                     float* out_lse, int num_requests, int max_states, const ps_geometry& g, hipStream_t st) {
  const int64_t rows = int64_t(num_requests) * g.num_q_heads;
  if (rows == 0) return PS_OK;
  if (g.head_dim % 4 != 0) return PS_ERR_UNSUPPORTED;
  const int64_t threads = rows * (g.head_dim / 4);
  const dim3 grid(unsigned((threads + 255) / 256)), block(256);
  // One round trip for up to 4 or 16 states: most batches have two to four a row; a lone session, cut into many chunks
  // to fill the chip, has a dozen (12 states, 128 rows: 4.57 us in rounds of four, 3.30 us in one).
#define PS_MANY(QT, HD)                                                                                                 \
  hipLaunchKernelGGL((merge_many_kernel<QT, HD>), dim3(unsigned(rows)), block, 0, st, slot_base, requests, ws_o, ws_lse, out, out_lse, g.num_q_heads)
  // Few rows of more than four states, and up to eight workgroups a compute unit of more than sixteen: a workgroup per row.  A thread
  // alone walks such a row's states in rounds of sixteen, and a launch of few rows has few threads (one thread / one workgroup for
  // a row's columns, us a step: 61 states, 96 rows of 64 20.5 / 15.9; 51, 160 of 64 21.0 / 17.1; 40, 112 17.0 / 14.3; 31, 192 22.6 / 20.5;
  // 23, 480 18.3 / 16.8; 17, 960 of 256 68.1 / 67.5; 8, 320 11.5 / 11.0; 7, 280 10.9 / 10.4; 5, 256 11.0 / 10.6; but 12, 592 of 256 62.2 /
  // 62.0; 12, 1344 23.0 / 23.4; 7, 3072 of 64 21.2 / 22.0; 7, 8576 36.0 / 37.1).
  const bool whole = g.head_dim == 64 || g.head_dim == 128 || g.head_dim == 256;
  if (whole && ((max_states > 4 && rows <= 512) || (max_states > 16 && rows <= 2048))) {
    if (g.q_dtype == PS_F32) {
      if (g.head_dim == 64) PS_MANY(PS_F32, 64); else if (g.head_dim == 128) PS_MANY(PS_F32, 128); else PS_MANY(PS_F32, 256);
    } else {
      if (g.head_dim == 64) PS_MANY(PS_BF16, 64); else if (g.head_dim == 128) PS_MANY(PS_BF16, 128); else PS_MANY(PS_BF16, 256);
    }
    return PS_OK;
  }
#undef PS_MANY
#define PS_MERGE(QT, BATCH)                                                                                            \
  hipLaunchKernelGGL((merge_states_kernel<QT, BATCH>), grid, block, 0, st, slot_base, requests, ws_o, ws_lse, out, out_lse, \
                     int(rows), g.num_q_heads, g.head_dim)
  if (g.q_dtype == PS_F32) {
    if (max_states <= 4) PS_MERGE(PS_F32, 4); else PS_MERGE(PS_F32, 16);
  } else {
    if (max_states <= 4) PS_MERGE(PS_BF16, 4); else PS_MERGE(PS_BF16, 16);
  }
#undef PS_MERGE
  return PS_OK;
}

}  // namespace psdev
