// Log-sum-exp merge of partial attention states.
//
// For each (request, q head) the partial states (o_i, lse_i) of its prefix and suffix splits are
// combined as lse = log sum_i exp(lse_i), o = sum_i exp(lse_i - lse) o_i -- exact by softmax algebra
// over the concatenated cache [C_base ; own tokens] (Background Eq. 2).  One thread owns four
// consecutive head-dim elements of one row.
#include "device_common.h"
#include "launch.h"

namespace psdev {

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
    if (bm == neg_inf) continue;           // nothing but empty states so far
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
  if (out_lse && c4 == 0) out_lse[row] = (mx != neg_inf) ? mx + __builtin_amdgcn_logf(total) * kLn2 : neg_inf;
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
