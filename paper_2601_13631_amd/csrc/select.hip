// select.hip -- standalone top-k ContiguousChunk selection (Sec. 4.4).
//
// Up to kRegKeys scores: one workgroup holds every key in registers (256
// threads with 4 or 8 consecutive scores each, then 512 with 8 and 1,024 with 8,
// 16 and 32) and runs the register-resident radix select of select_regs.h.
// Larger m: one 1,024-thread workgroup runs select_topk_block (select_block.h),
// which re-reads the scores in every pass.  Both produce the same set under the
// same total order (score descending, index ascending), ascending.
//
// One workgroup is bound by its rounds: each counts every key's digit (about 14
// VALU instructions a key) and meets at two barriers.  16,384 scores: 75 us with
// 256 threads and the keys in LDS, whose per-bin atomics nearly all collide (a
// layer's scores share their high bits), 26 us with 16 keys per thread in
// registers; 32,768: 192 -> 33 us; 100,000, where 1,024 threads re-read instead of
// 256: 749 -> 238 us.  (The same rounds on 32-bit windows of the keys, with the
// 64-bit ones behind for what they leave open, took 28 us, and 6.5 against 6.1 us
// at 1,024 scores.)

#include "select_regs.h"

namespace ckv {
namespace {

constexpr int64_t kRegKeys = 32 * 1024;  // 1024 threads, 32 keys each

template <int THREADS>
__global__ __launch_bounds__(THREADS) void select_kernel(const double* __restrict__ scores,
                                                         int64_t m, int64_t k,
                                                         int32_t* __restrict__ sel,
                                                         int32_t* __restrict__ sel_copy) {
  __shared__ SelShared sh;
  select_topk_block<THREADS>(scores, m, k, sel, sel_copy, sh);
}

template <int THREADS, int E>
__global__ __launch_bounds__(THREADS) void select_small_kernel(
    const double* __restrict__ scores, int m, int k, int32_t* __restrict__ sel,
    int32_t* __restrict__ sel_copy) {
  __shared__ RegSelShared<THREADS, E> sh;
  select_topk_regs<THREADS, E>(scores, m, k, sh, sel, sel_copy);
}

// One workgroup of THREADS threads with E keys each in registers.
template <int THREADS, int E>
void launch_small(const double* scores, int m, int k, int32_t* sel, int32_t* sel_copy,
                  hipStream_t st) {
  hipLaunchKernelGGL((select_small_kernel<THREADS, E>), dim3(1), dim3(THREADS), 0, st, scores, m,
                     k, sel, sel_copy);
}

}  // namespace

size_t select_ws_bytes(int64_t) { return 0; }

ckv_status launch_select(const double* scores, int64_t m, int64_t k, int32_t* sel, void*, size_t,
                         hipStream_t st, int32_t* sel_copy) {
  if (m <= kRegKeys) {
    // the fewest waves that hold the keys at up to 8 per thread: per round
    // every wave counts its digits and meets the others at two barriers, so
    // fewer, fuller waves finish a round sooner; past 8,192 keys all 16 waves
    // with as many keys per thread as it takes
    if (m <= 1024) launch_small<256, 4>(scores, (int)m, (int)k, sel, sel_copy, st);
    else if (m <= 2048) launch_small<256, 8>(scores, (int)m, (int)k, sel, sel_copy, st);
    else if (m <= 4096) launch_small<512, 8>(scores, (int)m, (int)k, sel, sel_copy, st);
    else if (m <= 8192) launch_small<1024, 8>(scores, (int)m, (int)k, sel, sel_copy, st);
    else if (m <= 16384) launch_small<1024, 16>(scores, (int)m, (int)k, sel, sel_copy, st);
    else launch_small<1024, 32>(scores, (int)m, (int)k, sel, sel_copy, st);
  } else {
    hipLaunchKernelGGL(select_kernel<1024>, dim3(1), dim3(1024), 0, st, scores, m, k, sel, sel_copy);
  }
  CKV_HIP(hipGetLastError());
  return CKV_OK;
}

}  // namespace ckv
