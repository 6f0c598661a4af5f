// Device-side pieces shared by the persistent group kernels (replica groups spread over several
// workgroups that exchange their spins through memory every iteration): the control block, the
// registration of workgroups with their XCDs, the group barrier, waits, and the widening of J.
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

#include "nmfa_device.h"
#include "nmfa_internal.h"

namespace nmfa {

// control block layout (uint32 words)
enum : int {
  CTL_REG = 0,        // [16] workgroups registered per XCD
  CTL_TOTAL = 16,     // workgroups registered
  CTL_ABORT = 17,     // barrier timeout
  CTL_MODE = 18,      // 1 = XCD-local exchange, 2 = device-scope fences (written by workgroup 0)
  CTL_BAR = 64,       // group barrier counters, one per 16 words
  CTL_WG = 64 + 16 * 256,  // per workgroup: group, row block, exchange mode (4 words each)
  CTL_WORDS = CTL_WG + 4 * GROUP_MAX_WGS,
};

// Cache policy of the spin loads: device scope (sc1), i.e. past the CU's L1, which may hold the lines
// of two iterations ago. (buffer_inv sc0 does not drop them: with 16 KB of spins per iteration,
// which two iterations' lines of fit the L1, loads without sc1 have read stale spins. The L1 would
// not serve these loads anyway, since a workgroup reads each line once per iteration: no cost.)
constexpr int AUX_SC1 = 16;

constexpr unsigned SPIN_LIMIT = 1u << 22;  // about a second of polling
// The workgroups of a launch wait longer for each other to start: other kernels' workgroups, each of which
// ends by itself, may hold CUs for as long as their runs take.
constexpr unsigned START_LIMIT = 16 * SPIN_LIMIT;

__device__ __forceinline__ unsigned ld_dev(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Widen 8 FP8 E4M3 values (two 32-bit words) to 8 BF16 (exact for every FP8 value).
__device__ __forceinline__ bf16x8 fp8x8_to_bf16x8(uint32_t lo, uint32_t hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, false);
  const bf16x2 p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, true);
  const bf16x2 p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, false);
  const bf16x2 p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, true);
  bf16x8 r;
  r[0] = p0[0]; r[1] = p0[1]; r[2] = p1[0]; r[3] = p1[1];
  r[4] = p2[0]; r[5] = p2[1]; r[6] = p3[0]; r[7] = p3[1];
  return r;
}

// Widen 8 FP4 E2M1 values (one 32-bit word, value 2b in the low nibble of byte b) to 8 BF16.
__device__ __forceinline__ bf16x8 fp4x8_to_bf16x8(uint32_t w) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, 1.0f, 0);
  const bf16x2 p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, 1.0f, 1);
  const bf16x2 p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, 1.0f, 2);
  const bf16x2 p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, 1.0f, 3);
  bf16x8 r;
  r[0] = p0[0]; r[1] = p0[1]; r[2] = p1[0]; r[3] = p1[1];
  r[4] = p2[0]; r[5] = p2[1]; r[6] = p3[0]; r[7] = p3[1];
  return r;
}

// Wait until at most N of this wave's vector-memory operations are outstanding (N <= 63: the
// counter's low four bits sit in bits 3:0 of the immediate, the high two in bits 15:14; LDS and
// export counters are not waited on).
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N <= 63, "vmcnt immediate");
  __builtin_amdgcn_s_waitcnt(0xF70 | (N & 15) | ((N >> 4) << 14));
}

// Wait until this wave's LDS reads (and scalar loads) are complete; vector-memory counters are
// left alone.
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// Workgroup barrier without the memory fence of __syncthreads (which would also wait for the
// chunks still in flight); the asm statements keep the compiler from moving LDS accesses across.
__device__ __forceinline__ void bare_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Where a workgroup sits: its replica group, its row block and the exchange mode.
struct XcdSlot {
  unsigned my_group;  // group index within this launch
  int rb;             // row block
  bool xcd_mode;      // spins exchanged through the XCD's L2 (no device-scope fences)
  bool aborted;
};

// Registration: every workgroup reports its XCD (HW_REG_XCC_ID); when each XCD holds a multiple
// of P workgroups, groups are formed inside XCDs, else by launch order with device-scope fences.
// Where all XCDs in use hold equally many, the group numbers go round the XCDs, so that groups
// beyond x.groups (a launch may hold more workgroups than its groups need, to give every XCD a
// multiple of P) are spread over the XCDs too; the workgroups of such a group leave at once.
// Thread 0 does the work; the result is broadcast through this workgroup's control words.
__device__ XcdSlot xcd_register(const XcdArgs& x, int tid) {
  unsigned* ctl = x.ctl;
  const unsigned P = (unsigned)x.P;
  if (tid == 0) {
    const unsigned xcc = __builtin_amdgcn_s_getreg((20) | (0 << 6) | (15 << 11)) & 0xfu;
    const unsigned slot = atomicAdd(&ctl[CTL_REG + xcc], 1u);
    __builtin_amdgcn_s_waitcnt(0);  // counted on its XCD before it is counted in the total
    atomicAdd(&ctl[CTL_TOTAL], 1u);
    unsigned spins = 0;
    while (ld_dev(&ctl[CTL_TOTAL]) < gridDim.x) {
      if (++spins > START_LIMIT) {
        atomicExch(&ctl[CTL_ABORT], 1u);
        break;
      }
    }
    // XCD-local exchange needs every XCD's workgroup count to be a multiple of P.
    unsigned base = 0, ok = 1, used = 0, rank = 0, most = 0, even = 1;
    for (unsigned k = 0; k < 16; ++k) {
      const unsigned cnt = ld_dev(&ctl[CTL_REG + k]);
      if (cnt % P) ok = 0;
      if (k < xcc) base += cnt;
      if (cnt == 0) continue;
      if (used && cnt != most) even = 0;
      most = cnt;
      ++used;
      if (k < xcc) ++rank;
    }
    unsigned* info = &ctl[CTL_WG + 4 * blockIdx.x];
    info[0] = !ok ? blockIdx.x / P : (even ? slot / P * used + rank : (base + slot) / P);
    info[1] = ok ? slot % P : blockIdx.x % P;
    info[2] = (ok && !x.force_fenced) ? 1u : 0u;
    if (blockIdx.x == 0) atomicMax(&ctl[CTL_MODE], (ok && !x.force_fenced) ? 1u : 2u);
    __builtin_amdgcn_s_waitcnt(0);
  }
  __syncthreads();
  XcdSlot r;
  r.my_group = __builtin_amdgcn_readfirstlane(ld_dev(&ctl[CTL_WG + 4 * blockIdx.x]));
  r.rb = (int)__builtin_amdgcn_readfirstlane(ld_dev(&ctl[CTL_WG + 4 * blockIdx.x + 1]));
  r.xcd_mode = ld_dev(&ctl[CTL_WG + 4 * blockIdx.x + 2]) != 0;
  r.aborted = ld_dev(&ctl[CTL_ABORT]) != 0;
  return r;
}

// Device-scope release (of stores that are complete) and acquire by one thread for its workgroup, each complete
// before it goes on. Written out: behind the write-back or the invalidation of a fence the compiler waits for
// nothing where it knows of no other memory operation in flight. The arrival then passes the write-back (with the
// L2 full of another kernel's dirty lines one run in twelve read old spins), as other waves' loads might pass the
// invalidation. (A fence with a wait behind it changes the schedule of the whole loop: 37.25 ms per headline
// anneal instead of 37.1.)
__device__ __forceinline__ void release_agent() {
  asm volatile("buffer_wbl2 sc1\n\ts_waitcnt vmcnt(0)" ::: "memory");
}
__device__ __forceinline__ void acquire_agent() {
  asm volatile("s_waitcnt vmcnt(0)\n\tbuffer_inv sc1\n\ts_waitcnt vmcnt(0)" ::: "memory");
}

// Group barrier after the new spins are stored, in two halves so that work which does not
// depend on the other workgroups can run in between. Arrive: this workgroup's stores are
// complete (and released to the device when the group spans XCDs); one thread adds to the
// group's counter.
__device__ __forceinline__ void xcd_group_arrive(unsigned* bar, bool xcd_mode, int tid) {
  __builtin_amdgcn_s_waitcnt(0);  // this wave's stores of the new spins are complete
  __syncthreads();
  if (tid == 0) {
    if (!xcd_mode) release_agent();
    __hip_atomic_fetch_add(bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Wait: one thread polls until all P workgroups have arrived for this epoch (bounded), then the
// other workgroups' spins are made visible. Returns whether the anneal was aborted (a wait timed
// out somewhere).
__device__ __forceinline__ bool xcd_group_wait(const XcdArgs& x, unsigned* bar, unsigned epoch, bool xcd_mode,
                                               int tid) {
  unsigned* ctl = x.ctl;
  if (tid == 0) {
    const unsigned target = (unsigned)x.P * epoch;
    unsigned spins = 0;
    while (ld_dev(bar) < target) {
      if (++spins > SPIN_LIMIT || ld_dev(&ctl[CTL_ABORT])) {
        atomicExch(&ctl[CTL_ABORT], 1u);
        break;
      }
    }
    if (!xcd_mode) acquire_agent();
  }
  __syncthreads();
  return ld_dev(&ctl[CTL_ABORT]) != 0;
}

// Wait of the register-J kernel, which keeps the round trips to L2 off its critical path: the
// caller polls the counter once ahead (seen, read while it draws the next noise), the polling
// thread reads the abort word only every 64 polls, and its decision reaches the other waves
// through an LDS word (abort_word) rather than a load of the control block by every thread.
// Every wave of the workgroup therefore sees the same decision.
__device__ __forceinline__ bool xrj_group_wait(const XcdArgs& x, unsigned* bar, unsigned epoch, bool xcd_mode,
                                               int tid, unsigned seen, unsigned* abort_word) {
  unsigned* ctl = x.ctl;
  if (tid == 0) {
    const unsigned target = (unsigned)x.P * epoch;
    unsigned ab = 0;
    if (seen < target) {
      unsigned spins = 0;
      while (ld_dev(bar) < target) {
        if ((++spins & 63u) == 0 && (spins > SPIN_LIMIT || ld_dev(&ctl[CTL_ABORT]))) {
          atomicExch(&ctl[CTL_ABORT], 1u);
          ab = 1;
          break;
        }
      }
    }
    if (!xcd_mode) acquire_agent();
    *abort_word = ab;
  }
  __syncthreads();
  return *abort_word != 0;
}

__device__ __forceinline__ bool xcd_group_barrier(const XcdArgs& x, unsigned* bar, unsigned epoch,
                                                  bool xcd_mode, int tid) {
  xcd_group_arrive(bar, xcd_mode, tid);
  return xcd_group_wait(x, bar, epoch, xcd_mode, tid);
}

// Raw J fragment of one lane for one k-step: 8 values as 16 (BF16), 8 (FP8) or 4 (FP4) bytes.
template <int JFMT> struct JRaw;
template <> struct JRaw<0> { typedef bf16x8 T; };
template <> struct JRaw<1> { typedef uint2 T; };
template <> struct JRaw<2> { typedef uint32_t T; };

template <int JFMT>
__device__ __forceinline__ bf16x8 widen(const typename JRaw<JFMT>::T& v);
template <> __device__ __forceinline__ bf16x8 widen<0>(const bf16x8& v) { return v; }
template <> __device__ __forceinline__ bf16x8 widen<1>(const uint2& v) { return fp8x8_to_bf16x8(v.x, v.y); }
template <> __device__ __forceinline__ bf16x8 widen<2>(const uint32_t& v) { return fp4x8_to_bf16x8(v); }

typedef float f32x16 __attribute__((ext_vector_type(16)));

template <class F, int... I>
__device__ __forceinline__ void static_for(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

}  // namespace nmfa
