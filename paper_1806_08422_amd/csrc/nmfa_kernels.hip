// NMFA hot-path kernels for gfx950.
//
// One iteration of Algorithm 1 (paper Sec. II) for every spin i and replica r:
//   Phi_i = (h_i + sum_j J_ij s_j) / sqrt(h_i^2 + sum_j J_ij^2) + N(0, sigma)
//   s^_i  = -tanh(Phi_i / T_t)
//   s_i  <- alpha s^_i + (1 - alpha) s_i          (after all s^ of the iteration are known)
// The contraction sum_j J_ij s_j over all replicas is the matrix product J . S and runs on
// MFMA; the normalisation, noise, Boltzmann factor and damped update are fused into the MFMA
// epilogue in registers. After the last iteration the sign readout s~_i = s_i/|s_i| and the
// energy of Eq. 1 are evaluated.
//
// Kernels:
//   anneal_small      persistent: one workgroup owns 16 replicas and all N <= 256 spins for the
//                     whole anneal. J and the master state live in registers, the operand copy
//                     of S is double-buffered in LDS; one barrier per iteration.
//   small_noise       the noise of small FP64 runs with few replicas, drawn ahead on the whole chip.
//   anneal_step_tiled, anneal_step_tiled_f
//                     one iteration for large N as a tiled matrix product through LDS with the fused
//                     epilogue: BF16 operands on 256 x 128 workgroup tiles where they fill the chip,
//                     and on 64 x 32 to 256 x 64; FP64 and FP32 on 128 x 64, 64 x 64 or 32 x 32.
//   anneal_sparse*    degree-d graphs with J in ELL rows (see their own comments).
//   readout_kernel    s~ = sign(s) (s = 0 reads +1).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "nmfa_device.h"
#include "nmfa_internal.h"
#include "nmfa_plan.h"

namespace nmfa {

// ------------------------------------------------------------------------------------------
// Shared epilogue: from the accumulated field of four consecutive rows of one replica to the
// updated master state. acc[v] = sum_j J_ij s_j for row i = row0 + v.
// ------------------------------------------------------------------------------------------
template <bool B>
struct StBool {
  static constexpr bool value = B;
};
template <int I>
struct StInt {
  static constexpr int value = I;
};

template <int P>
struct Epilogue;

template <>
struct Epilogue<PREC_FP64> {
  // sigma z, with the sign of the noise test hook
  template <int MODE = PHILOX_PLAIN>
  __device__ static __forceinline__ void noise(double z[4], const AnnealArgs& a, uint32_t q, uint32_t r, uint32_t t) {
#pragma clang fp contract(off)
    gauss4_f64(philox4x32_10<MODE>(q, r, t, 0u, a.key0, a.key1), z);
    const double sg = a.negate_noise ? -a.sigma : a.sigma;
#pragma unroll
    for (int v = 0; v < 4; ++v) z[v] = sg * z[v];
  }
  // the same for one half of the quad (z[0..1] of rows 2 half, 2 half + 1)
  __device__ static __forceinline__ void noise_half(double z[2], const AnnealArgs& a, uint32_t q, uint32_t r,
                                                    uint32_t t, int half) {
#pragma clang fp contract(off)
    const Philox4 w = philox4x32_10<PHILOX_LOOP>(q, r, t, 0u, a.key0, a.key1);
    gauss2_f64(half ? w.x2 : w.x0, half ? w.x3 : w.x1, z[0], z[1]);
    const double sg = a.negate_noise ? -a.sigma : a.sigma;
    z[0] = sg * z[0];
    z[1] = sg * z[1];
  }
  template <int NV>
  __device__ static __forceinline__ void update(const double* acc, const double* inv, const double* h, double* s,
                                                const double* z, const AnnealArgs& a, double coef_t) {
    // every operation rounded on its own (no contraction into FMAs), so that all kernels that
    // share this epilogue round alike, whatever the surrounding code lets the compiler fuse
#pragma clang fp contract(off)
    const double oma = 1.0 - a.alpha;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const double phi = (h[v] + acc[v]) * inv[v] + z[v];
      const double s_hat = -tanh(phi * coef_t);
      s[v] = a.alpha * s_hat + oma * s[v];
    }
  }
  template <int MODE = PHILOX_PLAIN>
  __device__ static __forceinline__ void apply(const double acc[4], const double inv[4], const double h[4],
                                               double s[4], const AnnealArgs& a, double coef_t, uint32_t q,
                                               uint32_t r, uint32_t t) {
    double z[4];
    noise<MODE>(z, a, q, r, t);
    update<4>(acc, inv, h, s, z, a, coef_t);
  }
};

template <int P>
struct EpilogueF32 {
  template <int MODE = PHILOX_PLAIN>
  __device__ static __forceinline__ void noise(float z[4], const AnnealArgs& a, uint32_t q, uint32_t r, uint32_t t) {
    const float sg = (float)a.sigma;
    sigma_gauss4_f32(philox4x32_10<MODE>(q, r, t, 0u, a.key0, a.key1), -2.0f * 0.6931471805599453f * sg * sg, z);
  }
  // sigma_gauss4_f32 for one half of the quad
  __device__ static __forceinline__ void noise_half(float z[2], const AnnealArgs& a, uint32_t q, uint32_t r, uint32_t t,
                                                    int half) {
    const float sg = (float)a.sigma;
    const Philox4 w = philox4x32_10<PHILOX_LOOP>(q, r, t, 0u, a.key0, a.key1);
    const float u0 = fmaf((float)(half ? w.x2 : w.x0), 0x1p-32f, 0x1p-33f);
    const float u1 = fmaf((float)(half ? w.x3 : w.x1), 0x1p-32f, 0x1p-33f);
    const float rho = __builtin_amdgcn_sqrtf(-2.0f * 0.6931471805599453f * sg * sg * __builtin_amdgcn_logf(u0));
    z[0] = rho * __builtin_amdgcn_cosf(u1);
    z[1] = rho * __builtin_amdgcn_sinf(u1);
  }
  template <int NV>
  __device__ static __forceinline__ void update(const float* acc, const float* inv, const float* hinv, float* s,
                                                const float* z, const AnnealArgs& a, float coef_t) {
    const float alpha = (float)a.alpha;
    const float oma = (float)(1.0 - a.alpha);
    const float sgn = a.negate_noise ? -1.0f : 1.0f;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const float x = fmaf(acc[v], inv[v], hinv[v]);
      const float phi = fmaf(z[v], sgn, x);  // x + z or x - z exactly rounded, in one instruction
      const float s_hat = neg_tanh_from_exp2_arg(phi * coef_t);
      s[v] = fmaf(alpha, s_hat, oma * s[v]);
    }
  }
  template <int MODE = PHILOX_PLAIN>
  __device__ static __forceinline__ void apply(const float acc[4], const float inv[4], const float hinv[4], float s[4],
                                               const AnnealArgs& a, float coef_t, uint32_t q, uint32_t r, uint32_t t) {
    float z[4];
    noise<MODE>(z, a, q, r, t);
    update<4>(acc, inv, hinv, s, z, a, coef_t);
  }
};
template <>
struct Epilogue<PREC_FP32> : EpilogueF32<PREC_FP32> {};
template <>
struct Epilogue<PREC_BF16> : EpilogueF32<PREC_BF16> {};

// ------------------------------------------------------------------------------------------
// anneal_small<P, J8, NK, SPLIT, PRE, LS>: see the file header. Wave w owns rows [16w, 16w+16) (FP64 with
// SPLIT > 1: SPLIT waves share a tile's rows, see small_split); grid = ceil(R / 16) workgroups,
// workgroup b owns replicas [16b, 16b+16) (LS > 1: 16 / LS of them, each in LS columns of the product
// whose lanes share the replica's rows; while a CU is free for every workgroup, see small_split). Each
// lane keeps its part of J in registers (NK reads of 16 bytes; J8: FP8 E4M3 in memory, widened to BF16).
// LDS: Ss[2][16][js] (op_t), js = padded row stride in elements. The iterations are unrolled by two, so
// that the buffers' addresses are constants. The body is shared with anneal_small_batched, where one
// launch carries replica blocks of many jobs (serving): a workgroup may then have more waves than its
// job has row tiles, and the extra waves only take part in the barriers. What bounds it: the vector
// instructions, about 120 per wave and iteration, most of them the noise (BF16, N = 100, R = 16384: 28
// waves per CU, 593 cycles per wave and iteration; five or seven waves per SIMD make no difference);
// FP32: the chain of 16x16x4 products (32 cycles each) beside it. Against J in LDS, a rolled k loop and
// buffer addresses multiplied out in every iteration, per iteration: BF16 N = 100, R = 16384 1.94 ->
// 1.73 us, N = 173, R = 64 1.09 -> 0.60, N = 256, R = 1024 1.55 -> 0.81; FP32 N = 112, R = 4096 1.43 ->
// 1.21; FP64 N = 20, R = 256 2.73 -> 0.88 (with the noise drawn ahead, PRE: launch_small_noise). FP32
// draws the noise after it has issued the products, a serial chain of 32 cycles each, which leaves the
// registers of their operands free as well: drawn before them, N = 48, R = 8192 took 0.86 us (0.81 with
// J in LDS) instead of 0.76, N = 80, R = 32768 7.2 (6.8) instead of 6.2, N = 112, R = 4096 1.31 (1.43)
// instead of 1.21.
// ------------------------------------------------------------------------------------------
template <int P, bool J8, int NK, int SPLIT = 1, bool PRE = false, int LS = 1>
__device__ __forceinline__ void anneal_small_body(const AnnealArgs& a, const int rblock) {
  static_assert(SPLIT == 1 || P == PREC_FP64, "split tiles are built for FP64");
  constexpr int SUB = SPLIT * LS, NV = 4 / SUB;  // rows of its quad that a lane updates
  constexpr int RPB = 16 / LS;                   // replicas of the workgroup
  using Tr = Traits<P>;
  using op_t = typename Tr::op_t;
  using acc_t = typename Tr::acc_t;
  using frag_t = typename Tr::frag_t;
  using acc4_t = typename Tr::acc4_t;
  constexpr int KW = Tr::KW;
  constexpr int EPC = 16 / (int)sizeof(op_t);  // elements per 16-byte read
  constexpr int VEC = EPC / KW;                // MFMA steps per 16-byte read

  extern __shared__ __align__(16) unsigned char smem[];
  const int N = a.N, Mp = a.Mp, Kp = a.Kp, js = a.lds_stride;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4;
  const int c = lane & 15;
  const int cr = c % RPB, r = rblock * RPB + cr;  // replica of this lane
  const int tile = wave / SPLIT, part = wave % SPLIT * LS + c / RPB;  // part of the quad's rows
  const bool act = tile < (Mp >> 4);  // this wave owns (its part of) a row tile of the job
  const int quad0 = tile * 16 + 4 * g;    // first of this lane's four rows (accumulator layout)
  const int row0 = quad0 + NV * part;     // first of the rows this wave updates
  const int arow = tile * 16 + Tr::a_row(c);  // row this lane supplies to the A operand
  const int Kq = Kp >> 2;

  {
    uint32_t* Sw = reinterpret_cast<uint32_t*>(smem);
    const int s_words = (2 * 16 * js * (int)sizeof(op_t)) / 4;
    for (int k = tid; k < s_words; k += blockDim.x) Sw[k] = 0u;
  }
  __syncthreads();
  if (!act) {  // spare wave of a batched launch: only the barriers
    for (int t = a.t_begin; t <= a.t_end; ++t) __syncthreads();
    return;
  }

  // ---- this lane's part of J, its constants and initial state -------------------------------
  uint4 jr[NK];
#pragma unroll
  for (int m = 0; m < NK; ++m) {
    const size_t off = (size_t)arow * Kp + g * Kq + m * EPC;
    if constexpr (J8) {
      const uint2 raw = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint8_t*>(a.J) + off);
      __bf16 w[8];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        w[k] = (__bf16)fp8e4m3_to_float(((k < 4 ? raw.x : raw.y) >> (8 * (k & 3))) & 0xffu);
      jr[m] = *reinterpret_cast<const uint4*>(w);
    } else {
      jr[m] = *reinterpret_cast<const uint4*>(reinterpret_cast<const op_t*>(a.J) + off);
    }
  }
  acc_t inv[NV], hv[NV], s[NV];
  const acc_t* inv_g = reinterpret_cast<const acc_t*>(a.inv_norm);
  const acc_t* h_g = reinterpret_cast<const acc_t*>(a.hterm);
  acc_t* state = reinterpret_cast<acc_t*>(a.state);
  const bool live_r = r < a.R;
  op_t* Sl = reinterpret_cast<op_t*>(smem) + (size_t)cr * js;  // this lane's replica, buffer 0
  const int sbuf = 16 * js;                                   // elements of one buffer
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    // rows beyond N: a field that no 1 / T, however large, turns into a NaN (0 x NaN would spread it)
    inv[v] = (row0 + v) < N ? inv_g[row0 + v] : (acc_t)1;
    hv[v] = (row0 + v) < N ? h_g[row0 + v] : (acc_t)1;
    const bool live = live_r && (row0 + v) < N;
    s[v] = (a.load_state && live) ? state[(size_t)r * N + row0 + v] : (acc_t)0;
    Sl[row0 + v] = (op_t)s[v];
  }
  const acc_t* coef = reinterpret_cast<const acc_t*>(a.coef);
  acc_t* traj = reinterpret_cast<acc_t*>(a.traj);
  const uint32_t q = (uint32_t)(quad0 >> 2);
  __syncthreads();

  auto draw = [&](acc_t* z, int t) {
    if constexpr (SUB == 1) {
      Epilogue<P>::template noise<PHILOX_LOOP>(z, a, q, (uint32_t)r, (uint32_t)t);
    } else {
      acc_t zz[2];
      Epilogue<P>::noise_half(zz, a, q, (uint32_t)r, (uint32_t)t, SUB == 2 ? part : part >> 1);
      if constexpr (SUB == 2) {
        z[0] = zz[0];
        z[1] = zz[1];
      } else {
        z[0] = (part & 1) ? zz[1] : zz[0];
      }
    }
  };
  // One iteration: read the operands of buffer CUR, draw the noise while they arrive, multiply, update,
  // write buffer 1 - CUR. Rows beyond N are updated too: the couplings to them are zero.
  // PRE: the noise comes from memory (launch_small_noise), read four iterations ahead
  static_assert(!PRE || P == PREC_FP64, "noise drawn ahead is built for FP64");
  constexpr int NPRE = 4;
  typedef acc_t zvec __attribute__((ext_vector_type(NV)));
  zvec zr[PRE ? NPRE : 1];
  const size_t zstep = (size_t)((a.R + 15) / 16) * (Mp >> 4) * 256;  // values per iteration
  const acc_t* zl = reinterpret_cast<const acc_t*>(a.z) + ((size_t)(rblock / LS) * (Mp >> 4) + tile) * 256 +
                    (16 * g + rblock % LS * RPB + cr) * 4 + NV * part;
  auto read_z = [&](int t) {
    return *reinterpret_cast<const zvec*>(zl + (size_t)((t < a.t_end ? t : a.t_end) - a.t_begin) * zstep);
  };
  auto step = [&](auto cur_c, auto slot_c, int t) {
    constexpr int CUR = decltype(cur_c)::value, SLOT = decltype(slot_c)::value;
    const acc_t coef_t = coef[t - 1];
    uint4 bv[NK];
    const op_t* Bc = Sl + (CUR ? sbuf : 0) + g * Kq;
#pragma unroll
    for (int m = 0; m < NK; ++m) bv[m] = *reinterpret_cast<const uint4*>(Bc + m * EPC);
    acc_t z[NV];
    if constexpr (PRE) {
      const zvec zt = zr[SLOT];
#pragma unroll
      for (int v = 0; v < NV; ++v) z[v] = zt[v];
      zr[SLOT] = read_z(t + NPRE);
    } else if constexpr (P != PREC_FP32) {
      draw(z, t);
    }
    acc4_t acc;
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = (acc_t)0;
#pragma unroll
    for (int m = 0; m < NK; ++m) {
      const frag_t* af = reinterpret_cast<const frag_t*>(&jr[m]);
      const frag_t* bf = reinterpret_cast<const frag_t*>(&bv[m]);
#pragma unroll
      for (int u = 0; u < VEC; ++u) acc = Tr::mfma(af[u], bf[u], acc);
    }
    if constexpr (P == PREC_FP32) {  // under the chain of products, whose operands' registers are free by then
      __builtin_amdgcn_sched_barrier(0);
      draw(z, t);
    }
    acc_t fld[NV];
    if constexpr (SUB == 1) {
#pragma unroll
      for (int v = 0; v < 4; ++v) fld[v] = acc[v];
    } else if constexpr (SUB == 2) {
      fld[0] = part ? acc[2] : acc[0];
      fld[1] = part ? acc[3] : acc[1];
    } else {
      fld[0] = (part & 2) ? ((part & 1) ? acc[3] : acc[2]) : ((part & 1) ? acc[1] : acc[0]);
    }
    Epilogue<P>::template update<NV>(fld, inv, hv, s, z, a, coef_t);
    op_t* Sn = Sl + (CUR ? 0 : sbuf) + row0;
#pragma unroll
    for (int v = 0; v < NV; ++v) Sn[v] = (op_t)s[v];
    const int k = t - a.t_begin;
    if (traj && k < a.record && live_r) {
#pragma unroll
      for (int v = 0; v < NV; ++v)
        if (row0 + v < N) traj[((size_t)k * a.R + r) * N + row0 + v] = s[v];
    }
    if constexpr (PRE) {  // a barrier that does not wait for the noise in flight
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0xC07F);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    } else {
      __syncthreads();
    }
  };
  int t = a.t_begin;
  if constexpr (PRE) {
#pragma unroll
    for (int k = 0; k < NPRE; ++k) zr[k] = read_z(t + k);
    for (; t + 3 <= a.t_end; t += 4) {
      step(StBool<false>{}, StInt<0>{}, t);
      step(StBool<true>{}, StInt<1>{}, t + 1);
      step(StBool<false>{}, StInt<2>{}, t + 2);
      step(StBool<true>{}, StInt<3>{}, t + 3);
    }
    if (t <= a.t_end) step(StBool<false>{}, StInt<0>{}, t);
    if (t + 1 <= a.t_end) step(StBool<true>{}, StInt<1>{}, t + 1);
    if (t + 2 <= a.t_end) step(StBool<false>{}, StInt<2>{}, t + 2);
  } else {
    for (; t < a.t_end; t += 2) {
      step(StBool<false>{}, StInt<0>{}, t);
      step(StBool<true>{}, StInt<0>{}, t + 1);
    }
    if (t == a.t_end) step(StBool<false>{}, StInt<0>{}, t);
  }

  // ---- final state and sign readout -------------------------------------------------------
  if (live_r) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (row0 + v < N) {
        state[(size_t)r * N + row0 + v] = s[v];
        if (a.spins) a.spins[(size_t)r * N + row0 + v] = (s[v] >= (acc_t)0) ? (int8_t)1 : (int8_t)-1;
      }
    }
  }
}

// 16-byte reads per lane group and operand row: a quarter of a row of Kp elements
template <int P>
__host__ __device__ constexpr int small_nk(int Kp) {
  return Kp * (int)sizeof(typename Traits<P>::op_t) / 64;
}

// Largest workgroup (Mp / 16 waves) and the waves per SIMD that the registers must leave room for (FP32, 6 reads:
// with 82 registers instead of 80 only two workgroups of six waves were on a CU, N = 96, R = 12000 4.0 us
// instead of 3.0)
template <int P>
constexpr int small_threads() {
  return P == PREC_FP64 ? 512 : (P == PREC_FP32 ? 768 : 1024);
}
template <int P>
constexpr int small_min_waves(int NK) {
  return P == PREC_FP64 ? 2 : (P == PREC_FP32 ? (NK == 6 ? 6 : 4) : (NK > 4 ? 4 : 5));
}

template <int P, bool J8, int NK, int SPLIT, bool PRE, int LS>
__global__ __launch_bounds__(small_threads<P>(), small_min_waves<P>(NK)) void anneal_small(AnnealArgs a) {
  anneal_small_body<P, J8, NK, SPLIT, PRE, LS>(a, (int)blockIdx.x);
}

// The noise of iterations t_begin .. t_end for anneal_small, the values it would draw itself: a wave per
// iteration, replica block and row tile, the four of a lane's quad side by side. Bound by the vector
// instructions, like the draws in the annealing kernel, but spread over the whole chip.
__global__ __launch_bounds__(256) void small_noise(AnnealArgs a, double* __restrict__ out, int blocks) {
  const int tiles = a.Mp >> 4, lane = threadIdx.x & 63;
  const unsigned w = blockIdx.x * 4u + (threadIdx.x >> 6);
  const unsigned per = (unsigned)(blocks * tiles), it = w / per, k = w - it * per;
  if (it > (unsigned)(a.t_end - a.t_begin)) return;
  const unsigned b = k / tiles, tile = k - b * tiles;
  double z[4];
  Epilogue<PREC_FP64>::noise(z, a, tile * 4 + (lane >> 4), b * 16 + (lane & 15), (uint32_t)a.t_begin + it);
  reinterpret_cast<double4*>(out)[(size_t)w * 64 + lane] = make_double4(z[0], z[1], z[2], z[3]);
}

// Calls f with the number of 16-byte reads as a compile-time constant. Kp is a multiple of 32 (BF16, at
// most 256) or 16 (FP32, at most 176; FP64, at most 112: what the path's limit on LDS admits).
template <int P, class F>
__host__ __device__ __forceinline__ bool small_dispatch(int nk, F&& f) {
  if constexpr (P == PREC_FP64) {
    switch (nk) {
      case 2: f(StInt<2>{}); return true;
      case 4: f(StInt<4>{}); return true;
      case 6: f(StInt<6>{}); return true;
      case 8: f(StInt<8>{}); return true;
      case 10: f(StInt<10>{}); return true;
      case 12: f(StInt<12>{}); return true;
      case 14: f(StInt<14>{}); return true;
    }
  } else {
    switch (nk) {
      case 1: f(StInt<1>{}); return true;
      case 2: f(StInt<2>{}); return true;
      case 3: f(StInt<3>{}); return true;
      case 4: f(StInt<4>{}); return true;
      case 5: f(StInt<5>{}); return true;
      case 6: f(StInt<6>{}); return true;
      case 7: f(StInt<7>{}); return true;
      case 8: f(StInt<8>{}); return true;
    }
    if constexpr (P == PREC_FP32) {
      switch (nk) {
        case 9: f(StInt<9>{}); return true;
        case 10: f(StInt<10>{}); return true;
        case 11: f(StInt<11>{}); return true;
      }
    }
  }
  return false;
}

// One launch for replica blocks of many jobs: tasks[b] = (job index, replica block). NKMAX: the most operand
// reads of any of the jobs, which sets the registers, so the workgroups that a CU holds. 16 requests of 4096
// replicas, ms with J in LDS (46 registers, 8 waves per SIMD whatever the size) / one kernel for all sizes (109 to
// 125 registers) / one per size: BF16, 2000 iterations, N = 80 14.0 / 15.0 / 12.8, N = 256 58 / 39 / 39; FP32, 4000
// iterations, N = 80 58 / 65 / 51, N = 100 81 / 85 / 73.
template <int P, bool J8, int NKMAX>
__global__ __launch_bounds__(small_threads<P>()) void anneal_small_batched(const AnnealArgs* __restrict__ jobs,
                                                             const int2* __restrict__ tasks) {
  const int2 tk = tasks[blockIdx.x];
  const AnnealArgs a = jobs[tk.x];
  small_dispatch<P>(small_nk<P>(a.Kp), [&](auto nk) {
    if constexpr (decltype(nk)::value <= NKMAX) anneal_small_body<P, J8, decltype(nk)::value>(a, tk.y);
  });
}

// ------------------------------------------------------------------------------------------
// Operand copy of a master state: S[r][i] = (op_t) state[r][i] for i < N, r < R; zero padding.
// ------------------------------------------------------------------------------------------
template <typename op_t, typename acc_t>
__global__ void pack_state_kernel(const acc_t* __restrict__ state, op_t* __restrict__ S, int N, int R,
                                  int Kp, int ld, int Rp, int zero) {
  const size_t total = (size_t)Rp * Kp;
  for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (size_t)gridDim.x * blockDim.x) {
    const int r = (int)(idx / Kp);
    const int i = (int)(idx - (size_t)r * Kp);
    acc_t v = 0;
    if (!zero && r < R && i < N) v = state[(size_t)r * N + i];
    S[(size_t)r * ld + i] = (op_t)v;
  }
}

// FP8 E4M3 operand copy (the FP8-spin precision), rounded as the annealing kernel's epilogue
// rounds (v_cvt_pk_fp8_f32: nearest even, saturating), so a resumed run continues bit-exactly.
__global__ void pack_state_fp8_kernel(const float* __restrict__ state, uint8_t* __restrict__ S, int N, int R, int Kp,
                                      int ld, int Rp, int zero) {
  const size_t total = (size_t)Rp * Kp;
  for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (size_t)gridDim.x * blockDim.x) {
    const int r = (int)(idx / Kp);
    const int i = (int)(idx - (size_t)r * Kp);
    float v = 0.0f;
    if (!zero && r < R && i < N) v = state[(size_t)r * N + i];
    S[(size_t)r * ld + i] = (uint8_t)(__builtin_amdgcn_cvt_pk_fp8_f32(v, 0.0f, 0, false) & 0xff);
  }
}

// ------------------------------------------------------------------------------------------
// Readout: s~ = +1 if s >= 0 (including -0.0), else -1.
// ------------------------------------------------------------------------------------------
template <typename acc_t>
__global__ void readout_kernel(const acc_t* __restrict__ state, int8_t* __restrict__ spins, size_t count) {
  for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < count;
       idx += (size_t)gridDim.x * blockDim.x)
    spins[idx] = (state[idx] >= (acc_t)0) ? (int8_t)1 : (int8_t)-1;
}

// ------------------------------------------------------------------------------------------
// anneal_sparse<P>: sparse couplings (degree-d graphs). J is stored row by row in ELL form, the
// nonzeros of row i in ascending column order padded to D entries with zero weights, so the
// field sum_j J_ij s_j is the dense sum with its exact zero terms left out (bit-identical up to
// the FMA contraction of each term). One workgroup owns RB replicas and all N spins for the whole
// anneal: the state of its replicas sits in LDS, double-buffered by iteration parity (layout
// [Nq][RB], replica fastest, so the threads of one spin gather consecutive words), and a
// workgroup barrier separates iterations. Thread tasks are (quad q of 4 consecutive spins,
// replica): one Philox call draws exactly the quad's noise, and the update is the shared
// Epilogue. FP64 precision runs in FP64; the other precisions run in FP32.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float fma_acc(float x, float y, float z) { return __builtin_fmaf(x, y, z); }
__device__ __forceinline__ double fma_acc(double x, double y, double z) { return __builtin_fma(x, y, z); }

template <int P>
__global__ __launch_bounds__(P == PREC_FP64 ? 512 : 1024) void anneal_sparse(AnnealArgs a,
                                                                             const int* __restrict__ ell_col,
                                                     const void* __restrict__ ell_val, int D, int RB) {
  using acc_t = typename Traits<P>::acc_t;
  extern __shared__ __align__(16) unsigned char smem_sp[];
  const int N = a.N, Nq = (N + 3) / 4;
  acc_t* buf0 = reinterpret_cast<acc_t*>(smem_sp);
  acc_t* buf1 = buf0 + (size_t)4 * Nq * RB;
  const acc_t* val = reinterpret_cast<const acc_t*>(ell_val);
  const acc_t* inv_g = reinterpret_cast<const acc_t*>(a.inv_norm);
  const acc_t* h_g = reinterpret_cast<const acc_t*>(a.hterm);
  const acc_t* coef = reinterpret_cast<const acc_t*>(a.coef);
  acc_t* state = reinterpret_cast<acc_t*>(a.state);
  acc_t* traj = reinterpret_cast<acc_t*>(a.traj);
  const int r0 = blockIdx.x * RB;
  const int slots = 4 * Nq * RB;
  for (int idx = threadIdx.x; idx < slots; idx += blockDim.x) {
    const int i = idx / RB, rr = idx - i * RB, r = r0 + rr;
    buf0[idx] = (a.load_state && r < a.R && i < N) ? state[(size_t)r * N + i] : (acc_t)0;
  }
  __syncthreads();
  int cur = 0;
  const int tasks = Nq * RB;
  for (int t = a.t_begin; t <= a.t_end; ++t) {
    const acc_t coef_t = coef[t - 1];
    const acc_t* sc = cur ? buf1 : buf0;
    acc_t* sn = cur ? buf0 : buf1;
    const int k_rec = t - a.t_begin;
    for (int task = threadIdx.x; task < tasks; task += blockDim.x) {
      const int q = task / RB, rr = task - q * RB, r = r0 + rr;
      acc_t acc[4], inv[4], hv[4], sv[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 4 * q + v;
        acc_t f = (acc_t)0;
        if (i < N) {
          const int* cl = ell_col + (size_t)i * D;
          const acc_t* vl = val + (size_t)i * D;
          for (int d = 0; d < D; ++d) f = fma_acc(vl[d], sc[cl[d] * RB + rr], f);
          inv[v] = inv_g[i];
          hv[v] = h_g[i];
        } else {
          inv[v] = (acc_t)0;
          hv[v] = (acc_t)0;
        }
        acc[v] = f;
        sv[v] = sc[i * RB + rr];
      }
      Epilogue<P>::apply(acc, inv, hv, sv, a, coef_t, (uint32_t)q, (uint32_t)r, (uint32_t)t);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 4 * q + v;
        sn[i * RB + rr] = (i < N) ? sv[v] : (acc_t)0;
        if (traj && k_rec < a.record && r < a.R && i < N) traj[((size_t)k_rec * a.R + r) * N + i] = sv[v];
      }
    }
    __syncthreads();
    cur ^= 1;
  }
  const acc_t* sf = cur ? buf1 : buf0;
  for (int idx = threadIdx.x; idx < slots; idx += blockDim.x) {
    const int i = idx / RB, rr = idx - i * RB, r = r0 + rr;
    if (r < a.R && i < N) {
      state[(size_t)r * N + i] = sf[idx];
      if (a.spins) a.spins[(size_t)r * N + i] = (sf[idx] >= (acc_t)0) ? (int8_t)1 : (int8_t)-1;
    }
  }
}

// ------------------------------------------------------------------------------------------
// anneal_sparse_rq<P, RB, DM, QP>: the sparse kernel with the couplings in registers. A thread
// owns the quads q = tid + k * blockDim.x (k < QP) for all RB replicas of its workgroup and for
// the whole anneal: its ELL rows (DM entries each, those beyond D zero-weight) are read from
// global memory once, the quads' own state stays in registers, and one neighbour read is one
// vector LDS load of that spin's RB replica values (layout [4 Nq][RB], replica fastest, as in
// anneal_sparse). Each replica's arithmetic (terms in ELL order, one FMA each, noise counters,
// epilogue) is that of anneal_sparse; a zero-weight term adds a signed zero to a sum that starts
// at +0 and so changes nothing. Both kernels therefore give bit-identical trajectories, whatever
// RB and whichever kernel the launcher picks.
// What bounds it: the vector instructions, about 108 per spin quad and replica at degree 3, of which
// the noise takes 60; hence nothing per read but the read (addresses in both buffers held in registers
// where there is room, iterations unrolled by two), no selects for padding spins or the noise's sign,
// and slots for the degree rather than the next power of two. Per iteration: N = 2000, R = 1024,
// degree 3 1.98 -> 1.71 us; degree 3, N = 2000, R = 100 0.93 -> 0.61 and N = 301, R = 64 0.73 -> 0.38;
// degree 6, N = 1000, R = 512 0.99 -> 0.85, N = 2000, R = 1024 2.8 -> 2.6; degree 8, N = 2000, R = 4096 11.0 -> 10.5;
// degree 10, N = 1537, R = 256 2.20 -> 1.22. Where two workgroups of 512 threads share a CU the registers must
// leave four waves per SIMD (128): with 129 or 130, degree 6, N = 2000, R = 4096 took 11.4 instead of 8.7 and
// degree 8 13.2; with one register spilled inside the loop, degree 8, N = 300, R = 64 1.20 instead of 0.62.
// ------------------------------------------------------------------------------------------
template <typename T, int RB>
struct alignas(sizeof(T) * RB) RepVec {
  T v[RB];
};

// Waves per SIMD that the registers must leave room for: four, two workgroups of 512 threads, wherever a register
// or two decide it and none is spilled for it.
template <int P, int RB, int DM, int QP>
constexpr int rq_min_waves() {
  return P != PREC_FP64 && QP == 1 && (RB <= 2 ? DM <= 6 : DM == 3) ? 4 : 2;
}

// Iterations unrolled by two, which takes registers: not where they would leave a SIMD fewer waves than the rolled
// loop (FP32, 8 or 10 slots, two or four replicas) nor where it gained nothing (FP64, 8 slots).
template <int P, int RB, int DM, int QP>
constexpr bool rq_unrolled() {
  return QP == 1 && (P == PREC_FP64 ? DM != 8 : RB == 1 || (DM != 8 && DM != 10));
}

template <int P, int RB, int DM, int QP, bool UNROLL = rq_unrolled<P, RB, DM, QP>()>
__global__ __launch_bounds__(512, (rq_min_waves<P, RB, DM, QP>())) void anneal_sparse_rq(
    AnnealArgs a, const int* __restrict__ ell_col, const void* __restrict__ ell_val, int D) {
  using acc_t = typename Traits<P>::acc_t;
  using V = RepVec<acc_t, RB>;
  extern __shared__ __align__(16) unsigned char smem_sp[];
  const int N = a.N, Nq = (N + 3) / 4;
  const int buf_bytes = 4 * Nq * (int)sizeof(V);
  // With few slots the neighbours' addresses in both buffers stay in registers, so that a read needs no
  // address arithmetic; otherwise the buffer's base is added at each read.
  constexpr bool TWO = DM * QP <= 4;
  const acc_t* val = reinterpret_cast<const acc_t*>(ell_val);
  const acc_t* inv_g = reinterpret_cast<const acc_t*>(a.inv_norm);
  const acc_t* h_g = reinterpret_cast<const acc_t*>(a.hterm);
  const acc_t* coef = reinterpret_cast<const acc_t*>(a.coef);
  acc_t* state = reinterpret_cast<acc_t*>(a.state);
  acc_t* traj = reinterpret_cast<acc_t*>(a.traj);
  const int r0 = blockIdx.x * RB;

  int off[TWO ? 2 : 1][QP][4][DM];  // byte offset of the neighbour's replica vector (in each buffer)
  acc_t w[QP][4][DM];
  acc_t inv[QP][4], hv[QP][4], s[QP][RB][4];
#pragma unroll
  for (int k = 0; k < QP; ++k) {
    const int q = threadIdx.x + k * blockDim.x;
    const bool own = q < Nq;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 4 * q + v;  // < 4 Nq = Mp when own: inv_g and h_g hold Mp entries
      const bool live = own && i < N;
      inv[k][v] = own ? inv_g[i] : (acc_t)0;
      hv[k][v] = own ? h_g[i] : (acc_t)0;
#pragma unroll
      for (int d = 0; d < DM; ++d) {
        const bool e = live && d < D;
        off[0][k][v][d] = e ? ell_col[(size_t)i * D + d] * (int)sizeof(V) : 0;
        if constexpr (TWO) {
          off[1][k][v][d] = off[0][k][v][d] + buf_bytes;
          asm volatile("" : "+v"(off[1][k][v][d]));  // a register of its own
        }
        w[k][v][d] = e ? val[(size_t)i * D + d] : (acc_t)0;
      }
#pragma unroll
      for (int rr = 0; rr < RB; ++rr) {
        const int r = r0 + rr;
        s[k][rr][v] = (a.load_state && live && r < a.R) ? state[(size_t)r * N + i] : (acc_t)0;
      }
    }
    if (own) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        V y;
#pragma unroll
        for (int rr = 0; rr < RB; ++rr) y.v[rr] = s[k][rr][v];
        *reinterpret_cast<V*>(smem_sp + (4 * q + v) * (int)sizeof(V)) = y;
      }
    }
  }
  __syncthreads();
  // one iteration: reads buffer CUR, writes the other. Spins beyond N are updated too: nothing reads them.
  auto step = [&](auto cur_c, int t) {
    const int cur = cur_c;  // a compile-time constant where the loop is unrolled twice
    const acc_t coef_t = coef[t - 1];
    const unsigned char* sc = smem_sp + (cur && !TWO ? buf_bytes : 0);
    unsigned char* sn = smem_sp + (cur ? 0 : buf_bytes);
    const int k_rec = t - a.t_begin;
#pragma unroll
    for (int k = 0; k < QP; ++k) {
      const int q = threadIdx.x + k * blockDim.x;
      if (q >= Nq) continue;
      acc_t acc[RB][4];
#pragma unroll
      for (int rr = 0; rr < RB; ++rr)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[rr][v] = (acc_t)0;
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int d = 0; d < DM; ++d) {
          const V x = *reinterpret_cast<const V*>(sc + off[TWO ? cur : 0][k][v][d]);
#pragma unroll
          for (int rr = 0; rr < RB; ++rr) acc[rr][v] = fma_acc(w[k][v][d], x.v[rr], acc[rr][v]);
        }
#pragma unroll
      for (int rr = 0; rr < RB; ++rr)
        Epilogue<P>::template apply<PHILOX_LOOP_R>(acc[rr], inv[k], hv[k], s[k][rr], a, coef_t, (uint32_t)q,
                                                   (uint32_t)(r0 + rr), (uint32_t)t);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        V y;
#pragma unroll
        for (int rr = 0; rr < RB; ++rr) y.v[rr] = s[k][rr][v];
        *reinterpret_cast<V*>(sn + (4 * q + v) * (int)sizeof(V)) = y;
      }
      if (traj && k_rec < a.record) {
#pragma unroll
        for (int rr = 0; rr < RB; ++rr) {
          const int r = r0 + rr;
          if (r >= a.R) continue;
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (4 * q + v < N) traj[((size_t)k_rec * a.R + r) * N + 4 * q + v] = s[k][rr][v];
        }
      }
    }
    __syncthreads();
  };
  if constexpr (UNROLL) {
    int t = a.t_begin;
    for (; t < a.t_end; t += 2) {
      step(std::integral_constant<int, 0>{}, t);
      step(std::integral_constant<int, 1>{}, t + 1);
    }
    if (t == a.t_end) step(std::integral_constant<int, 0>{}, t);
  } else {
    for (int t = a.t_begin; t <= a.t_end; ++t) step((t - a.t_begin) & 1, t);
  }
#pragma unroll
  for (int k = 0; k < QP; ++k) {
    const int q = threadIdx.x + k * blockDim.x;
    if (q >= Nq) continue;
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) {
      const int r = r0 + rr;
      if (r >= a.R) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 4 * q + v;
        if (i >= N) continue;
        state[(size_t)r * N + i] = s[k][rr][v];
        if (a.spins) a.spins[(size_t)r * N + i] = (s[k][rr][v] >= (acc_t)0) ? (int8_t)1 : (int8_t)-1;
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// Noise words / values for a range of spins (library utility and test hook for the stream).
// words: out[(k*n + i)] for replica r0 + k ... see nmfa.h.
// ------------------------------------------------------------------------------------------
__global__ void noise_words_kernel(uint32_t key0, uint32_t key1, uint32_t t, uint32_t r0, int nrep,
                                   int nq, uint32_t* out) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nrep * nq) return;
  const int k = idx / nq, q = idx - k * nq;
  const Philox4 w = philox4x32_10((uint32_t)q, r0 + (uint32_t)k, t, 0u, key0, key1);
  out[4 * (size_t)idx + 0] = w.x0;
  out[4 * (size_t)idx + 1] = w.x1;
  out[4 * (size_t)idx + 2] = w.x2;
  out[4 * (size_t)idx + 3] = w.x3;
}

__global__ void noise_values_kernel(uint32_t key0, uint32_t key1, uint32_t t, uint32_t r0, int nrep,
                                    int nq, int fp64, double* out) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nrep * nq) return;
  const int k = idx / nq, q = idx - k * nq;
  const Philox4 w = philox4x32_10((uint32_t)q, r0 + (uint32_t)k, t, 0u, key0, key1);
  if (fp64) {
    double z[4];
    gauss4_f64(w, z);
    for (int v = 0; v < 4; ++v) out[4 * (size_t)idx + v] = z[v];
  } else {
    float z[4];
    // sigma = 1: -2 ln 2 * 1
    sigma_gauss4_f32(w, -2.0f * 0.6931471805599453f, z);
    for (int v = 0; v < 4; ++v) out[4 * (size_t)idx + v] = (double)z[v];
  }
}

// ------------------------------------------------------------------------------------------
// Host-side launchers.
// ------------------------------------------------------------------------------------------
static int device_cus() {
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) == hipSuccess)
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  return cus;
}

template <int P, bool J8>
static hipError_t launch_small_t(const AnnealArgs& a, hipStream_t st) {
  const int waves = a.Mp / 16;
  const size_t lds = (size_t)2 * 16 * a.lds_stride * sizeof(typename Traits<P>::op_t);
  hipError_t e = hipErrorInvalidValue;
  const SmallSplit sp = small_split(P == PREC_FP64, waves, a.R, device_cus());
  const int split = sp.split, ls = sp.ls;
  small_dispatch<P>(small_nk<P>(a.Kp), [&](auto nk) {
    constexpr int NK = decltype(nk)::value;
    auto launch = [&](auto split_c, auto ls_c, auto pre_c) {
      constexpr int SP = decltype(split_c)::value, LS = decltype(ls_c)::value;
      hipLaunchKernelGGL((anneal_small<P, J8, NK, SP, decltype(pre_c)::value, LS>), dim3((a.R * LS + 15) / 16),
                         dim3(64 * SP * waves), lds, st, a);
      e = hipGetLastError();
    };
    auto with_ls = [&](auto split_c, auto pre_c) {
      constexpr int SP = decltype(split_c)::value;
      if constexpr (P == PREC_FP64 && SP == 1) {
        if (ls == 4) return launch(split_c, StInt<4>{}, pre_c);
      }
      if constexpr (SP <= 2) {
        if (ls == 2) return launch(split_c, StInt<2>{}, pre_c);
      }
      launch(split_c, StInt<1>{}, pre_c);
    };
    auto with_pre = [&](auto split_c) {
      if constexpr (P == PREC_FP64) {
        if (a.z) return with_ls(split_c, StBool<true>{});
      }
      with_ls(split_c, StBool<false>{});
    };
    if constexpr (P == PREC_FP64 && NK <= 4) {  // at most two tiles
      if (split == 4) return with_pre(StInt<4>{});
      if (split == 2) return with_pre(StInt<2>{});
    }
    with_pre(StInt<1>{});
  });
  return e;
}

// With few replica blocks the FP64 noise (libm log and sincos) is a third of the small-N kernel's time while
// most CUs are idle: another launch draws it on all of them, as many iterations ahead as 2 MB hold (a buffer
// of 4 MB costs a new context 0.35 ms to allocate, 2 MB 0.1). A pair of launches costs about 7.5 us and an
// iteration saves 0.4 us or more, hence at least 24 iterations per pair. ms per 1000 iterations without and
// with it: N = 16, R = 64 1.12, 0.58; N = 20, R = 256 (32 iterations per pair) 1.20, 0.88; N = 35, R = 217
// (24) 1.29, 1.12; N = 100, R = 64 (36) 3.79, 2.99. In FP32 and BF16 an iteration saves 0.13 to 0.17 us,
// which pays for the launches from 64 iterations per pair on, but hardly for the buffer: not built.
constexpr size_t NOISE_BYTES = (size_t)2 << 20;

size_t small_noise_bytes() { return NOISE_BYTES; }

int small_noise_iters(int prec, int Mp, int R, int iters) {
  if (prec != PREC_FP64) return 0;
  const size_t per = (size_t)((R + 15) / 16) * Mp * 16 * sizeof(double);
  const int n = (int)std::min(NOISE_BYTES / per, (size_t)iters);
  return n >= 24 ? n : 0;
}

hipError_t launch_small_noise(const AnnealArgs& a, void* z, hipStream_t st) {
  const int blocks = (a.R + 15) / 16;
  const size_t waves = (size_t)(a.t_end - a.t_begin + 1) * blocks * (a.Mp / 16);
  hipLaunchKernelGGL(small_noise, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, st, a, (double*)z, blocks);
  return hipGetLastError();
}

hipError_t launch_anneal_small(int prec, const AnnealArgs& a, hipStream_t st) {
  switch (prec) {
    case PREC_FP64: return launch_small_t<PREC_FP64, false>(a, st);
    case PREC_FP32: return launch_small_t<PREC_FP32, false>(a, st);
    case PREC_BF16: return launch_small_t<PREC_BF16, false>(a, st);
    case PREC_FP8J_BF16S: return launch_small_t<PREC_BF16, true>(a, st);
  }
  return hipErrorInvalidValue;
}

template <int P, bool J8>
static hipError_t launch_small_batched_t(const AnnealArgs* jobs, const int2* tasks, int n_tasks, int max_Mp,
                                         int max_Kp, size_t lds, hipStream_t st) {
  hipError_t e = hipErrorInvalidValue;
  small_dispatch<P>(small_nk<P>(max_Kp), [&](auto nk) {
    constexpr int NK = decltype(nk)::value;
    e = hipFuncSetAttribute((const void*)anneal_small_batched<P, J8, NK>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds);
    if (e != hipSuccess) return;
    hipLaunchKernelGGL((anneal_small_batched<P, J8, NK>), dim3(n_tasks), dim3(64 * (max_Mp / 16)), lds, st, jobs,
                       tasks);
    e = hipGetLastError();
  });
  return e;
}

hipError_t launch_anneal_small_batched(int prec, const AnnealArgs* jobs, const int2* tasks, int n_tasks, int max_Mp,
                                       int max_Kp, size_t lds, hipStream_t st) {
  switch (prec) {
    case PREC_FP64: return launch_small_batched_t<PREC_FP64, false>(jobs, tasks, n_tasks, max_Mp, max_Kp, lds, st);
    case PREC_FP32: return launch_small_batched_t<PREC_FP32, false>(jobs, tasks, n_tasks, max_Mp, max_Kp, lds, st);
    case PREC_BF16: return launch_small_batched_t<PREC_BF16, false>(jobs, tasks, n_tasks, max_Mp, max_Kp, lds, st);
    case PREC_FP8J_BF16S: return launch_small_batched_t<PREC_BF16, true>(jobs, tasks, n_tasks, max_Mp, max_Kp, lds, st);
  }
  return hipErrorInvalidValue;
}

// Decides whether an instance takes this path (the LDS that J and both spin buffers would need; J
// itself is held in registers).
size_t small_lds_bytes(int prec, int Mp, int stride) {
  const size_t es = (prec == PREC_FP64) ? 8 : (prec == PREC_FP32 ? 4 : 2);
  return ((size_t)Mp + 32) * stride * es;
}

size_t small_run_lds_bytes(int prec, int stride) {
  const size_t es = (prec == PREC_FP64) ? 8 : (prec == PREC_FP32 ? 4 : 2);
  return (size_t)2 * 16 * stride * es;
}

// ------------------------------------------------------------------------------------------
// anneal_step_tiled: one iteration for large N with BF16 operands (BF16 and FP8-J precisions),
// as a tiled matrix product with the fused epilogue. Workgroup (bx, by) owns rows [256 bx, +256)
// x replicas [128 by, +128) with eight waves (two per SIMD); wave w owns rows 64 (w / 2) .. +63
// and replicas 64 (w % 2) .. +63 (4 x 4 MFMA tiles of 16 x 16). J [Mp][Kp] and S_cur [Rp][Kp]
// (both k contiguous) stream through an LDS ring of 64-k blocks (256 rows of J and 128 replicas
// of S per stage) filled by direct-to-LDS loads: with BF16 J, 2 stages, one barrier per block and
// the next block issued at each barrier (a third stage measured 3.5% slower); with FP8 / FP4 J,
// 4 stages and one barrier per two blocks, the two blocks of a group with no branch between them
// so that the second block's fragment reads are scheduled under the first block's MFMAs (25.0 ->
// 23.9 ms; 4 stages of BF16 J do not fit in LDS). Unit u (8 k) of S row q sits at
// u ^ ((q >> 1) & 7) of its 128-byte row, so the 16 lanes a ds_read_b128 serves hit distinct bank
// groups. At N = 8192, R = 1024 this is one workgroup per CU, and a quarter fewer bytes per flop
// come from L2 than with 128 x 128 tiles (measured 28.7 against 36.4 ms per 200-iteration
// anneal). Needs Mp % 256 == 0 and S buffers of roundup(R, 128) rows (padding rows zero). Each
// wave loads its tile of the FP32 master state before the k loop, so that the epilogue does not
// wait for it (27.1 -> 25.0 ms).
// JFMT: format of J in memory and LDS, the narrowest that holds the couplings exactly (0 = BF16,
// 1 = FP8 E4M3, 2 = FP4 E2M1), widened to BF16 in registers: FP8 / FP4 rows of 64 / 32 bytes per
// block cut the J bytes each block moves into LDS to a half / a quarter (stages of 32 / 24 KB
// against 48; 29.3 -> 27.0 ms with FP4). Unit u (16 bytes) of J row q sits at u ^ f(q) with
// f = (q >> 1) & 7, (q >> 2) & 3, (q >> 3) & 1 for the three formats, so the 16 rows one fragment
// read spans hit distinct banks.
// ------------------------------------------------------------------------------------------
// Tile of a workgroup of the tiled kernels: row tile and replica tile. Workgroups are dispatched round robin
// over the eight XCDs; each XCD takes a contiguous eighth of the tiles, replica tiles within a row tile
// first, so that it reads about an eighth of J through its L2 whatever the number of row tiles is. (Plain
// two-dimensional grids do so only if that is a multiple of 8: FP64, N = 2000, R = 256, 63 row tiles, 57.0
// us per iteration against 53.7; BF16 J, N = 2100, R = 300, 33 row tiles, 18.0 against 15.3; FP4 J, N =
// 8192, R = 1024, 32 row tiles, 120.5 against 118.9.)
constexpr int TILE_XCDS = 8;
static dim3 tile_grid(int rows, int cols) { return dim3((rows * cols + TILE_XCDS - 1) / TILE_XCDS * TILE_XCDS); }
__device__ __forceinline__ bool tile_of(int rows, int cols, int& row, int& col) {
  const int tile = (int)(blockIdx.x % TILE_XCDS * (gridDim.x / TILE_XCDS) + blockIdx.x / TILE_XCDS);
  row = tile / cols;
  col = tile - row * cols;
  return row < rows;
}

constexpr int ST_M = 256;                 // rows per workgroup
constexpr int ST_R = 128;                 // replicas per workgroup
constexpr int ST_K = 64;                  // k per block
constexpr int ST_STAGES = 2;                // ring stages with one barrier per block (BF16 J)

template <int JFMT>
struct StFmt {
  static constexpr int JRB = JFMT == 0 ? 128 : (JFMT == 1 ? 64 : 32);  // bytes of a J row per block
  static constexpr int JT = ST_M * JRB;                               // bytes of the J tile
  static constexpr int STAGE = JT + ST_R * ST_K * 2;                  // J tile + S tile (128-byte rows)
  static constexpr int JB = JT / 1024;                                // 1 KB blocks of the J tile
  static constexpr int LPW = STAGE / 1024 / 8;                        // 1 KB loads per wave and block
  static constexpr int UPR = JRB / 16;                                // 16-byte units per J row
  // blocks per barrier: two where four stages fit in LDS (FP8 / FP4 J), else one
  static constexpr int G = JFMT == 0 ? 1 : 2;
  static constexpr int NS = G > 1 ? 2 * G : ST_STAGES;                // stages of the LDS ring
  __device__ static __forceinline__ int swz(int q) {
    return JFMT == 0 ? ((q >> 1) & 7) : (JFMT == 1 ? ((q >> 2) & 3) : ((q >> 3) & 1));
  }
};
static_assert(StFmt<0>::LPW * 8 * 1024 == StFmt<0>::STAGE && StFmt<1>::LPW * 8 * 1024 == StFmt<1>::STAGE &&
                  StFmt<2>::LPW * 8 * 1024 == StFmt<2>::STAGE,
              "every wave issues the same number of 1 KB loads per block");
static_assert(StFmt<0>::NS * StFmt<0>::STAGE <= 160 * 1024 && StFmt<1>::NS * StFmt<1>::STAGE <= 160 * 1024 &&
                  StFmt<2>::NS * StFmt<2>::STAGE <= 160 * 1024 && StFmt<1>::G <= 2 && StFmt<2>::G <= 2,
              "the ring fits in LDS; the first wait of the grouped loop covers up to two blocks per group");

// 8 FP8 E4M3 (two words) or 8 FP4 E2M1 values (one word; value 2b in the low nibble of byte b)
// widened to BF16 (exact for every value of either format)
__device__ __forceinline__ bf16x8 tiled_widen_fp8(uint2 v) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v.x, 1.0f, false);
  const bf16x2 p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v.x, 1.0f, true);
  const bf16x2 p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v.y, 1.0f, false);
  const bf16x2 p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v.y, 1.0f, true);
  return bf16x8{p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
}
__device__ __forceinline__ bf16x8 tiled_widen_fp4(uint32_t w) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, 1.0f, 0);
  const bf16x2 p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, 1.0f, 1);
  const bf16x2 p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, 1.0f, 2);
  const bf16x2 p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, 1.0f, 3);
  return bf16x8{p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
}

template <int NV>
__device__ __forceinline__ void step_wait_vm() {
  static_assert(NV >= 0 && NV <= 63, "vmcnt range");
  __builtin_amdgcn_s_waitcnt(0xF70 | (NV & 15) | ((NV >> 4) << 14));
}

// The body takes the kernel arguments by reference, which measured 2% faster than the same code in
// the kernel itself (the compiler then reads the arguments where they are used).
template <int JFMT>
__device__ __forceinline__ void step_tiled_body(const AnnealArgs& a, const __bf16* __restrict__ S_cur,
                                                __bf16* __restrict__ S_next, int t) {
  using F = StFmt<JFMT>;
  constexpr int NS = F::NS, G = F::G;
  constexpr int LPW = F::LPW, JB = F::JB, JRB = F::JRB, UPR = F::UPR;
  extern __shared__ __align__(16) unsigned char smem_st[];  // NS x (J tile, S tile)
  const int N = a.N, Kp = a.Kp;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g4 = lane >> 4, c = lane & 15;
  int m0, r0;
  if (!tile_of((N + ST_M - 1) / ST_M, (a.R + ST_R - 1) / ST_R, m0, r0)) return;
  m0 *= ST_M;
  r0 *= ST_R;
  const int wm = 64 * (wave >> 1), wr = 64 * (wave & 1);

  // direct-to-LDS loads: blocks 0 .. JB - 1 hold the J tile (1024 / JRB rows each), JB .. JB + 15
  // the S tile (eight 128-byte rows each); wave w issues blocks LPW w .. LPW w + LPW - 1. Lane l
  // fills position l % (units per row) of row (rows per block) b' + l / (units per row) (b' the
  // block within its tile) with the global unit the swizzle puts there.
  const size_t jrow = (size_t)Kp * JRB / ST_K;  // bytes of one J row in memory
  size_t goff[LPW];
#pragma unroll
  for (int u = 0; u < LPW; ++u) {
    const int b = LPW * wave + u;
    if (b < JB) {
      const int q = (1024 / JRB) * b + lane / UPR;
      const int unit = (lane % UPR) ^ F::swz(q);
      goff[u] = (size_t)(m0 + q) * jrow + unit * 16;
    } else {
      const int q = 8 * (b - JB) + (lane >> 3);
      const int unit = (lane & 7) ^ ((q >> 1) & 7);
      goff[u] = (size_t)(r0 + q) * Kp * 2 + unit * 16;
    }
  }
  const unsigned char* Jb = reinterpret_cast<const unsigned char*>(a.J);
  const unsigned char* Sb = reinterpret_cast<const unsigned char*>(S_cur);
  unsigned char* ring = smem_st;
  auto issue = [&](int kb, int stage) {
#pragma unroll
    for (int u = 0; u < LPW; ++u) {
      const int b = LPW * wave + u;
      __builtin_amdgcn_global_load_lds(
          reinterpret_cast<const uint32_t*>((b < JB ? Jb + (size_t)kb * JRB : Sb + (size_t)kb * ST_K * 2) + goff[u]),
          ring + stage * F::STAGE + b * 1024, 16, 0, 0);
    }
  };
  // fragment offsets within a 16-row tile: lane (c, g4) reads k octet o = 4 s + g4 of row c at k
  // step s (the swizzle of row q depends on q mod 16 only): S and BF16 J in unit o, FP8 J in half
  // o % 2 of unit o / 2, FP4 J in quarter o % 4 of unit o / 4
  int foff[2], joff[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int o = 4 * s + g4;
    foff[s] = c * 128 + ((o ^ ((c >> 1) & 7)) * 16);
    if (JFMT == 0) joff[s] = foff[s];
    else if (JFMT == 1) joff[s] = c * 64 + (((o >> 1) ^ F::swz(c)) * 16) + (o & 1) * 8;
    else joff[s] = c * 32 + (((o >> 2) ^ F::swz(c)) * 16) + (o & 3) * 4;
  }

  f32x4 acc[4][4];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[rt][ct][v] = 0.0f;

  const int nkb = (N + ST_K - 1) / ST_K;  // the blocks beyond N would add zeros
  // This wave's 64 x 64 master states are loaded before the k loop, so that their latency hides
  // under the matrix work rather than stalling the epilogue. They are issued ahead of the first
  // blocks, so the first block's wait also covers them. When the wave's tile lies inside N x R and
  // N % 4 == 0 (a wave-uniform test), a lane's four rows are one 16-byte load and store.
  float* state = reinterpret_cast<float*>(a.state);
  const bool full = (N & 3) == 0 && (reinterpret_cast<uintptr_t>(state) & 15) == 0 && m0 + wm + 64 <= N &&
                    r0 + wr + 64 <= a.R;
  float st[4][4][4];
  if (full) {
#pragma unroll
    for (int rt = 0; rt < 4; ++rt)
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        const float4 v4 = *reinterpret_cast<const float4*>(state + (size_t)(r0 + wr + 16 * ct + c) * N + m0 + wm +
                                                           16 * rt + 4 * g4);
        st[rt][ct][0] = v4.x;
        st[rt][ct][1] = v4.y;
        st[rt][ct][2] = v4.z;
        st[rt][ct][3] = v4.w;
      }
  } else {
#pragma unroll
    for (int rt = 0; rt < 4; ++rt)
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        const int row0 = m0 + wm + 16 * rt + 4 * g4;
        const int r = r0 + wr + 16 * ct + c;
#pragma unroll
        for (int v = 0; v < 4; ++v)
          st[rt][ct][v] = (r < a.R && row0 + v < N) ? state[(size_t)r * N + row0 + v] : 0.0f;
      }
  }

  // one 64-k block: both k steps' fragments are read up front, so that the second step's reads
  // land under the first step's MFMAs
  auto compute = [&](int stage) {
    const unsigned char* At = ring + stage * F::STAGE + wm * JRB;
    const unsigned char* Bt = ring + stage * F::STAGE + F::JT + wr * 128;
    bf16x8 af[2][4], bfr[2][4];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned char* ap = At + 16 * JRB * i + joff[s];
        if constexpr (JFMT == 0) af[s][i] = *reinterpret_cast<const bf16x8*>(ap);
        else if constexpr (JFMT == 1) af[s][i] = tiled_widen_fp8(*reinterpret_cast<const uint2*>(ap));
        else af[s][i] = tiled_widen_fp4(*reinterpret_cast<const uint32_t*>(ap));
        bfr[s][i] = *reinterpret_cast<const bf16x8*>(Bt + 2048 * i + foff[s]);
      }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int rt = 0; rt < 4; ++rt)
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
          acc[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[s][rt], bfr[s][ct], acc[rt][ct], 0, 0, 0);
  };

  if constexpr (G > 1) {
    // Groups of G blocks share one barrier, over a ring of 2G stages: the barrier at group kb
    // finds blocks kb .. kb + G - 1 landed and the previous group's stages read, and the next
    // group's blocks (issued at the previous barrier, or up front) have a whole group's work to
    // land. Two blocks per barrier measured 2% faster than one.
#pragma unroll
    for (int p = 0; p < NS; ++p)
      if (p < nkb) issue(p, p);
    int kb = 0;
    for (; kb + G <= nkb; kb += G) {
      if (kb == 0) {
        // blocks G .. 2G - 1 of the up-front issue may still be in flight
        const int ahead = nkb - G;
        if (ahead >= G) step_wait_vm<LPW * G>();
        else if (ahead == 1) step_wait_vm<LPW>();
        else step_wait_vm<0>();
      } else {
        step_wait_vm<0>();
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      if (kb > 0) {
#pragma unroll
        for (int j = 0; j < G; ++j)
          if (kb + G + j < nkb) issue(kb + G + j, (kb + G + j) % NS);
      }
      // a whole group with no branch between its blocks, so that the next block's fragment reads
      // can be scheduled under the current block's MFMAs
#pragma unroll
      for (int j = 0; j < G; ++j) compute((kb + j) % NS);
      // the reads of this group are complete before the next barrier frees its stages
      __builtin_amdgcn_s_waitcnt(0xC07F);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (kb < nkb) {
      // the last nkb % G blocks, issued at the previous barrier (or up front)
      step_wait_vm<0>();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < G - 1; ++j)
        if (kb + j < nkb) compute((kb + j) % NS);
    }
  } else {
    constexpr int LA = NS - 1;  // blocks issued ahead
    static_assert(LA >= 1 && LA <= 3, "the waits below cover up to two blocks in flight");
#pragma unroll
    for (int p = 0; p < LA; ++p)
      if (p < nkb) issue(p, p);
    for (int kb = 0; kb < nkb; ++kb) {
      // this wave's part of block kb has landed (the blocks after it may still be in flight)
      const int rem = nkb - 1 - kb;
      if (rem >= LA - 1) step_wait_vm<LPW * (LA - 1)>();
      else if (rem == 0) step_wait_vm<0>();
      else if (rem == 1) step_wait_vm<LPW>();
      else step_wait_vm<2 * LPW>();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();  // every wave's part landed; every wave is done with block kb - 1
      __builtin_amdgcn_sched_barrier(0);
      if (kb + LA < nkb) issue(kb + LA, (kb + LA) % NS);
      compute(kb % NS);
      // the reads of this block are complete before the next barrier frees its buffer
      __builtin_amdgcn_s_waitcnt(0xC07F);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- fused epilogue (the FP32 epilogue shared by every kernel) --------------------------------
  const float* inv_g = reinterpret_cast<const float*>(a.inv_norm);
  const float* h_g = reinterpret_cast<const float*>(a.hterm);
  float* traj = reinterpret_cast<float*>(a.traj);
  if (!(traj && t - a.t_begin < a.record)) traj = nullptr;
  else traj += (size_t)(t - a.t_begin) * a.R * N;
  const bool vec_traj = full && (reinterpret_cast<uintptr_t>(traj) & 15) == 0;
  const float coef_t = reinterpret_cast<const float*>(a.coef)[t - 1];
  // two copies of the epilogue, so that the bounds tests of a partial tile stay out of the full one
  auto epilogue = [&](auto full_c) {
    constexpr bool FULL = decltype(full_c)::value;
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
      const int row0 = m0 + wm + 16 * rt + 4 * g4;
      // inv_norm and hterm hold Mp entries (zero past N) and row0 is a multiple of 4
      const float4 inv4 = *reinterpret_cast<const float4*>(inv_g + row0);
      const float4 h4 = *reinterpret_cast<const float4*>(h_g + row0);
      const float inv[4] = {inv4.x, inv4.y, inv4.z, inv4.w};
      const float hv[4] = {h4.x, h4.y, h4.z, h4.w};
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        const int r = r0 + wr + 16 * ct + c;
        const bool live_r = FULL || r < a.R;
        float* sv = st[rt][ct];
        float fld[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) fld[v] = acc[rt][ct][v];
        Epilogue<PREC_BF16>::apply(fld, inv, hv, sv, a, coef_t, (uint32_t)(row0 >> 2), (uint32_t)r, (uint32_t)t);
        __bf16 outv[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (!FULL && (row0 + v >= N || !live_r)) sv[v] = 0.0f;
          outv[v] = (__bf16)sv[v];
        }
        *reinterpret_cast<uint2*>(S_next + (size_t)r * Kp + row0) = *reinterpret_cast<const uint2*>(outv);
        float* sp = state + (size_t)r * N + row0;
        float* tp = traj + (size_t)r * N + row0;
        if constexpr (FULL) {
          const float4 o4 = make_float4(sv[0], sv[1], sv[2], sv[3]);
          *reinterpret_cast<float4*>(sp) = o4;
          if (traj) {
            if (vec_traj) *reinterpret_cast<float4*>(tp) = o4;
            else
#pragma unroll
              for (int v = 0; v < 4; ++v) tp[v] = sv[v];
          }
        } else if (live_r) {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (row0 + v < N) {
              sp[v] = sv[v];
              if (traj) tp[v] = sv[v];
            }
        }
      }
    }
  };
  if (full) epilogue(StBool<true>{});
  else epilogue(StBool<false>{});
}

template <int JFMT>
__global__ __launch_bounds__(512, 1) void anneal_step_tiled(AnnealArgs a, const __bf16* __restrict__ S_cur,
                                                            __bf16* __restrict__ S_next, int t) {
  step_tiled_body<JFMT>(a, S_cur, S_next, t);
}

// ------------------------------------------------------------------------------------------
// anneal_step_tiled_f<P, JFMT, RT, CT, WM, WR, WPC>: one FP64 or FP32 iteration for large N, or a BF16
// one whose grid of 256 x 128 tiles would leave CUs idle, as a tiled matrix product with the fused
// epilogue. A workgroup of WM x WR waves owns 16 RT WM rows x 16 CT WR replicas, RT x CT accumulators of
// 16 x 16 per wave; WPC of them share a CU. J [Mp][Kp] and S_cur [Rp][Kp] (k contiguous) stream through
// an LDS ring of NS stages, 256 bytes of k per row of S and stage, filled by direct-to-LDS loads issued
// NS - 1 blocks ahead. The 16-byte unit u of tile row q is stored at u ^ (q & 15) of its 256-byte row, so
// the lanes one LDS cycle serves hit distinct bank groups (the A rows of a 16-row FP64 tile are permuted
// as that instruction's output needs, which keeps them distinct modulo 16; the 128- and 64-byte rows of
// FP8 and FP4 J take u ^ ((q >> 1) & 7) and u ^ ((q >> 2) & 3)). Which k a unit holds:
//   FP64  a block is 32 consecutive k, four 8-k windows of two MFMA steps; in window i, step s, lane
//         group g carries k = 8 i + 2 g + s, so unit 4 i + g holds both steps' operands.
//   FP32  lane group g owns the k range [g Kp/4, (g+1) Kp/4); a block is 16 consecutive k of each of
//         the four ranges, and in window i lane group g carries k = g Kp/4 + 16 kb + 4 i + s in
//         step s = 0..3: unit 4 g + i holds the four steps' operands.
//   BF16  a block is 128 consecutive k; in window i lane group g carries k = 32 i + 8 g .. + 7, unit
//         4 i + g (of FP8 / FP4 J half or a quarter of a unit, widened to BF16 in registers).
// Each wave loads its master states before the k loop, so that their latency hides under the
// matrix work. The order of each output's sum does not depend on the tile, so every tile size gives
// the same results bit for bit.
// What bounds it: the matrix cores (64 cycles per 16x16x4 FP64 instruction and SIMD, 32 in FP32),
// and beside them the block boundaries (about 330 cycles, and 50 per load that a wave issues),
// which a second wave per SIMD covers in part: hence eight waves per large tile, or two workgroups
// per CU. Where the tiles do not cover the chip, the serial k loop and the FP64 epilogue of one tile
// (32 x libm log, sincos and tanh per lane take 40 us) are the time, hence the smaller tiles
// (launch_step_f_pick). Measured per iteration, N = 2000, against the former kernels (FP64 always
// 128 x 64 with four waves; FP32 without LDS, operands straight from L2): FP64 R = 1024 226 -> 178
// us (46.0 TFLOP/s), R = 256 212 -> 55, R = 64 214 -> 34; FP32 R = 1024 270 -> 94 us, R = 256
// 107 -> 31, N = 777 R = 256 45 -> 12. Padding the operand rows to spread them over the L2 channels
// changed nothing, nor did reading three windows ahead instead of one, nor (64 x 32, FP4 J, one workgroup
// per CU: 0.37 us per block) a ring of 8 stages instead of 5; 3 stages take 0.58 us per block (BF16 J).
// The grid covers the N rows; rows of the last tile beyond N are written as zeros, and the columns of S
// past them, which the last block of k multiplies by zero couplings, are finite: the zeros they were
// allocated with, or what a group kernel kept there. (With rows and k padded to a multiple of 256, FP64,
// us per iteration: N = 120, R = 64 8.9 against 7.4; N = 300, R = 256 13.5, 10.7; N = 777, R = 256 21.9,
// 18.7; N = 1100, R = 200 33.4, 23.3. FP32, N = 1100, R = 200 19.7, 14.4.)
// Needs Mp % 256 == 0, Kp = Mp, and S buffers of roundup(R, 64) rows (padding rows finite).
// ------------------------------------------------------------------------------------------
template <int P, int JFMT, int RT, int CT, int WM, int WR, int WPC = 1>
struct SfTile {
  static constexpr int TM = 16 * RT * WM;               // rows per workgroup
  static constexpr int TR = 16 * CT * WR;               // replicas per workgroup
  static constexpr int W = WM * WR;                     // waves
  static constexpr int JRB = 256 >> JFMT;               // bytes of a J row per block
  static constexpr int JT = TM * JRB;                   // bytes of the J tile of one block
  static constexpr int JB = JT / 1024;                  // 1 KB loads of it
  static constexpr int STAGE = JT + TR * 256;           // J tile + S tile of one block
  static constexpr int LPW = STAGE / 1024 / W;          // 1 KB direct-to-LDS loads per wave and block
  static constexpr int NS_LDS = 160 * 1024 / WPC / STAGE, NS_MAX = STAGE > 24 * 1024 ? 4 : 5;
  static constexpr int NS = NS_LDS < NS_MAX ? NS_LDS : NS_MAX;  // stages of the ring
  static constexpr int BLK = P == PREC_FP64 ? 32 : (P == PREC_FP32 ? 64 : 128);  // k per block
  static constexpr int JADV = P == PREC_FP32 ? 64 : JRB;  // bytes from one block to the next in a row of J,
  static constexpr int SADV = P == PREC_FP32 ? 64 : 256;  // of S
  // where 16-byte unit u of tile row q of J is kept: u ^ swz(q)
  __device__ static __forceinline__ int swz(int q) {
    return JFMT == 0 ? (q & 15) : (JFMT == 1 ? ((q >> 1) & 7) : ((q >> 2) & 3));
  }
  static_assert(JFMT == 0 || P == PREC_BF16, "FP8 / FP4 couplings are widened to BF16");
  static_assert(LPW * 1024 * W == STAGE && NS >= 3, "whole loads per wave; the ring fits in LDS");
  static_assert((NS - 2) * LPW <= 63, "wait counts fit the vmcnt field");
};

template <int P, int JFMT, int RT, int CT, int WM, int WR, int WPC>
__device__ __forceinline__ void step_tiled_f_body(const AnnealArgs& a, const void* __restrict__ S_cur,
                                                  void* __restrict__ S_next_v, int t) {
  using Tr = Traits<P>;
  using T = SfTile<P, JFMT, RT, CT, WM, WR, WPC>;
  using op_t = typename Tr::op_t;
  using acc_t = typename Tr::acc_t;
  using acc4_t = typename Tr::acc4_t;
  using frag_t = typename Tr::frag_t;
  op_t* S_next = reinterpret_cast<op_t*>(S_next_v);
  constexpr int ES = sizeof(op_t), EPU = 16 / ES;  // element bytes; elements of a 16-byte unit
  constexpr int SPU = EPU / Tr::KW;                // MFMA steps per unit
  constexpr int LPW = T::LPW, NS = T::NS, LA = NS - 1, JRB = T::JRB, UPR = JRB / 16;
  typedef op_t unit_t __attribute__((ext_vector_type(EPU)));
  typedef uint32_t junit_t __attribute__((ext_vector_type(4 >> JFMT)));  // a unit's worth of J as stored
  extern __shared__ __align__(16) unsigned char smem_sf[];  // NS x (J tile, S tile)
  const int N = a.N, Kp = a.Kp;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: scalar registers
  const int g = lane >> 4, c = lane & 15;
  int m0, r0;
  if (!tile_of((N + T::TM - 1) / T::TM, (a.R + T::TR - 1) / T::TR, m0, r0)) return;
  m0 *= T::TM;
  r0 *= T::TR;
  const int wm = 16 * RT * (wave / WR), wr = 16 * CT * (wave % WR);

  // direct-to-LDS loads: 1 KB blocks of whole tile rows (four of S), first the J tile's, then the S
  // tile's; wave w issues blocks LPW w .. LPW w + LPW - 1. Lane l fills position l % (units per row) of
  // tile row (rows per block) b' + l / (units per row) (b' the block within its tile) with the global
  // unit the swizzle puts there.
  const size_t jrow = P == PREC_BF16 ? (size_t)Kp * JRB / T::BLK : (size_t)Kp * ES;  // bytes of a J row
  size_t goff[LPW];
#pragma unroll
  for (int u = 0; u < LPW; ++u) {
    const int b = LPW * wave + u;
    const bool is_j = b < T::JB;
    const int q = is_j ? 1024 / JRB * b + lane / UPR : 4 * (b - T::JB) + (lane >> 4);
    const int unit = is_j ? (lane % UPR) ^ T::swz(q) : (lane & 15) ^ (q & 15);
    const size_t k = P == PREC_FP32 ? (size_t)(unit >> 2) * Kp + 16 * (unit & 3) : 16 * unit;  // bytes (Kp / 4 words)
    goff[u] = (is_j ? (size_t)(m0 + q) * jrow : (size_t)(r0 + q) * Kp * ES) + k;
  }
  const unsigned char* Jb = reinterpret_cast<const unsigned char*>(a.J);
  const unsigned char* Sb = reinterpret_cast<const unsigned char*>(S_cur);
  unsigned char* ring = smem_sf;
  auto issue = [&](int kb, int stage) {
#pragma unroll
    for (int u = 0; u < LPW; ++u) {
      const int b = LPW * wave + u;
      const unsigned char* src = (b < T::JB ? Jb + (size_t)kb * T::JADV : Sb + (size_t)kb * T::SADV) + goff[u];
      __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint32_t*>(src), ring + stage * T::STAGE + b * 1024,
                                       16, 0, 0);
    }
  };
  // fragment offsets within a stage
  int aoff[RT][4], boff[CT][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int unit = P == PREC_FP32 ? 4 * g + i : 4 * i + g;
    constexpr int JPU = 1 << JFMT;  // S units that a 16-byte unit of J covers
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int q = wm + 16 * rt + Tr::a_row(c);
      aoff[rt][i] = q * JRB + (((unit / JPU) ^ T::swz(q)) * 16) + (unit % JPU) * (16 / JPU);
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int q = wr + 16 * ct + c;
      boff[ct][i] = T::JT + q * 256 + ((unit ^ (q & 15)) * 16);
    }
  }

  // this wave's master states (issued ahead of the first blocks, so the first wait covers them)
  acc_t* state = reinterpret_cast<acc_t*>(a.state);
  acc_t st[RT][CT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int row0 = m0 + wm + 16 * rt + 4 * g, r = r0 + wr + 16 * ct + c;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        st[rt][ct][v] = (r < a.R && row0 + v < N) ? state[(size_t)r * N + row0 + v] : (acc_t)0;
    }

  acc4_t acc[RT][CT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[rt][ct][v] = (acc_t)0;

  // blocks beyond N would add zeros (in FP32 every block holds some k below N)
  const int nkb = P == PREC_FP32 ? Kp / T::BLK : (N + T::BLK - 1) / T::BLK;
  // The fragments of a window are read into one register set while the MFMAs of the window before
  // it run on the other, across the block boundaries too: the barrier that makes block kb + 1
  // visible stands before the last window of block kb.
  junit_t af[2][RT];
  unit_t bfr[2][CT];
  auto load = [&](int set, int stage, int i) {
    const unsigned char* base = ring + stage * T::STAGE;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) af[set][rt] = *reinterpret_cast<const junit_t*>(base + aoff[rt][i]);
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) bfr[set][ct] = *reinterpret_cast<const unit_t*>(base + boff[ct][i]);
  };
#pragma unroll
  for (int p = 0; p < LA; ++p)
    if (p < nkb) issue(p, p);
  if (nkb >= LA) step_wait_vm<LPW * (LA - 1)>();
  else step_wait_vm<0>();
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  load(0, 0, 0);
  int cur = 0;  // stage of block kb
  for (int kb = 0; kb < nkb; ++kb) {
    const int nxt = cur + 1 == NS ? 0 : cur + 1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i < 3) {
        load((i + 1) & 1, cur, i + 1);
      } else if (kb + 1 < nkb) {
        // this wave's part of block kb + 1 has landed (up to LA - 2 blocks after it may still be in flight)
        if (kb + LA <= nkb) step_wait_vm<LPW * (LA - 2)>();
        else step_wait_vm<0>();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();  // every wave's part landed; every wave is done with block kb - 1
        __builtin_amdgcn_sched_barrier(0);
        if (kb + LA < nkb) issue(kb + LA, cur == 0 ? NS - 1 : cur - 1);
        load(0, nxt, 0);
      }
      __builtin_amdgcn_sched_barrier(0);  // the reads go out ahead of the MFMAs
      unit_t aw[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const junit_t w = af[i & 1][rt];
        if constexpr (JFMT == 2) aw[rt] = tiled_widen_fp4(w[0]);
        else if constexpr (JFMT == 1) aw[rt] = tiled_widen_fp8(make_uint2(w[0], w[1]));
        else aw[rt] = __builtin_bit_cast(unit_t, w);
      }
#pragma unroll
      for (int s = 0; s < SPU; ++s)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            if constexpr (SPU == 1) acc[rt][ct] = Tr::mfma(aw[rt], bfr[i & 1][ct], acc[rt][ct]);
            else acc[rt][ct] = Tr::mfma(aw[rt][s], bfr[i & 1][ct][s], acc[rt][ct]);
          }
      __builtin_amdgcn_sched_barrier(0);
    }
    cur = nxt;
  }

  // ---- fused epilogue (the one every kernel of the precision shares) ----------------------------
  const acc_t* inv_g = reinterpret_cast<const acc_t*>(a.inv_norm);
  const acc_t* h_g = reinterpret_cast<const acc_t*>(a.hterm);
  acc_t* traj = reinterpret_cast<acc_t*>(a.traj);
  const acc_t coef_t = reinterpret_cast<const acc_t*>(a.coef)[t - 1];
  const int k_rec = t - a.t_begin;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int row0 = m0 + wm + 16 * rt + 4 * g;
    acc_t inv[4], hv[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      inv[v] = inv_g[row0 + v];
      hv[v] = h_g[row0 + v];
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int r = r0 + wr + 16 * ct + c;
      const bool live_r = r < a.R;
      acc_t fld[4];
      acc_t* s = st[rt][ct];
#pragma unroll
      for (int v = 0; v < 4; ++v) fld[v] = acc[rt][ct][v];
      Epilogue<P>::apply(fld, inv, hv, s, a, coef_t, (uint32_t)(row0 >> 2), (uint32_t)r, (uint32_t)t);
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (row0 + v >= N || !live_r) s[v] = (acc_t)0;
      typedef op_t op4_t __attribute__((ext_vector_type(4)));
      *reinterpret_cast<op4_t*>(S_next + (size_t)r * Kp + row0) =
          op4_t{(op_t)s[0], (op_t)s[1], (op_t)s[2], (op_t)s[3]};
      if (live_r) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (row0 + v < N) {
            state[(size_t)r * N + row0 + v] = s[v];
            if (traj && k_rec < a.record) traj[((size_t)k_rec * a.R + r) * N + row0 + v] = s[v];
          }
      }
    }
  }
}

template <int P, int JFMT, int RT, int CT, int WM, int WR, int WPC>
__global__ __launch_bounds__(64 * WM * WR, WM * WR * WPC / 4) void anneal_step_tiled_f(
    AnnealArgs a, const void* __restrict__ S_cur, void* __restrict__ S_next, int t) {
  step_tiled_f_body<P, JFMT, RT, CT, WM, WR, WPC>(a, S_cur, S_next, t);
}

template <int JFMT>
static hipError_t launch_step_tiled(const AnnealArgs& a, const void* S_cur, void* S_next, int t, hipStream_t st) {
  const size_t lds = (size_t)StFmt<JFMT>::NS * StFmt<JFMT>::STAGE;
  hipError_t e = hipFuncSetAttribute((const void*)anneal_step_tiled<JFMT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  const dim3 grid = tile_grid((a.N + ST_M - 1) / ST_M, (a.R + ST_R - 1) / ST_R);
  hipLaunchKernelGGL(anneal_step_tiled<JFMT>, grid, dim3(512), lds, st, a, (const __bf16*)S_cur, (__bf16*)S_next, t);
  return hipGetLastError();
}

template <int P, int JFMT, int RT, int CT, int WM, int WR, int WPC>
static hipError_t launch_step_f(const AnnealArgs& a, const void* S_cur, void* S_next, int t, hipStream_t st) {
  using T = SfTile<P, JFMT, RT, CT, WM, WR, WPC>;
  const size_t lds = (size_t)T::NS * T::STAGE;
  hipError_t e = hipFuncSetAttribute((const void*)anneal_step_tiled_f<P, JFMT, RT, CT, WM, WR, WPC>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const dim3 grid = tile_grid((a.N + T::TM - 1) / T::TM, (a.R + T::TR - 1) / T::TR);
  hipLaunchKernelGGL((anneal_step_tiled_f<P, JFMT, RT, CT, WM, WR, WPC>), grid, dim3(64 * T::W), lds, st, a, S_cur,
                     S_next, t);
  return hipGetLastError();
}

// Tile of the FP64 / FP32 iteration: 128 x 64 or 64 x 64 with eight waves, one workgroup per CU, or
// 32 x 32 with four waves and two workgroups per CU. The measured time of one round of tiles over
// the CUs is 155 / 87 us (FP64, N = 2000; FP32 84 / 46), and 9 + 25.5 us (FP32 4.5 + 14) per 32 x 32
// tile that a CU gets, i.e. in both precisions 6.2 : 3.3 : 1/3 + 1 per tile; the cheapest by this
// count is taken. (N = 2000: 128 x 64 from R = 1024, where it takes 178 us in FP64 against 192 with
// 64 x 64 and 213 with 32 x 32; 64 x 64 at R = 512; 32 x 32 at R = 256, 55 us against 89 and 158.)
template <int P>
static hipError_t launch_step_f_pick(const AnnealArgs& a, const void* S_cur, void* S_next, int t, hipStream_t st) {
  const int cus = device_cus();
  auto rounds = [&](int tm, int tr) {
    const long tiles = (long)((a.N + tm - 1) / tm) * ((a.R + tr - 1) / tr);
    return (double)((tiles + cus - 1) / cus);
  };
  const double big = 6.2 * rounds(128, 64), mid = 3.3 * rounds(64, 64), small = 1.0 / 3 + rounds(32, 32);
  if (big <= mid && big <= small) return launch_step_f<P, 0, 2, 2, 4, 2, 1>(a, S_cur, S_next, t, st);
  if (mid <= small) return launch_step_f<P, 0, 1, 2, 4, 2, 1>(a, S_cur, S_next, t, st);
  return launch_step_f<P, 0, 1, 1, 2, 2, 2>(a, S_cur, S_next, t, st);
}

template <int JFMT>
static hipError_t launch_step_b(const AnnealArgs& a, const void* S_cur, void* S_next, int t, hipStream_t st) {
  constexpr int P = PREC_BF16;
  const StepTile tile = step_pick(JFMT, a.N, a.R, device_cus()).tile;
  if (tile == STEP_64X32) return launch_step_f<P, JFMT, 1, 2, 4, 1, 2>(a, S_cur, S_next, t, st);
  if constexpr (JFMT == 0) {
    if (tile == STEP_64X32_ALONE) return launch_step_f<P, JFMT, 1, 2, 4, 1, 1>(a, S_cur, S_next, t, st);
    if (tile == STEP_128) return launch_step_f<P, JFMT, 2, 2, 4, 2, 1>(a, S_cur, S_next, t, st);
  } else {
    if (tile == STEP_128) return launch_step_f<P, JFMT, 1, 2, 8, 1, 2>(a, S_cur, S_next, t, st);
    if (tile == STEP_256X64) return launch_step_f<P, JFMT, 2, 4, 8, 1, 1>(a, S_cur, S_next, t, st);
  }
  return launch_step_tiled<JFMT>(a, S_cur, S_next, t, st);
}

hipError_t launch_anneal_step(int prec, int jfmt, const AnnealArgs& a, const void* S_cur, void* S_next, int t,
                              hipStream_t st) {
  if (a.Mp % 256 != 0 || a.Kp != a.Mp) return hipErrorInvalidValue;
  switch (prec) {
    case PREC_FP64: return launch_step_f_pick<PREC_FP64>(a, S_cur, S_next, t, st);
    case PREC_FP32: return launch_step_f_pick<PREC_FP32>(a, S_cur, S_next, t, st);
    case PREC_BF16:
    case PREC_FP8J_BF16S:
      if (jfmt == 2) return launch_step_b<2>(a, S_cur, S_next, t, st);
      if (jfmt == 1) return launch_step_b<1>(a, S_cur, S_next, t, st);
      return launch_step_b<0>(a, S_cur, S_next, t, st);
  }
  return hipErrorInvalidValue;
}

size_t sparse_lds_bytes(int prec, int N, int RB) {
  return (size_t)2 * 4 * ((N + 3) / 4) * RB * (prec == PREC_FP64 ? 8 : 4);
}

// Register-ELL variants: RB replicas per thread (4, 2, 1), DM = D rounded up to 3, 4, 6, 8, 10, 12 or
// 16 (a slot beyond D costs a gather and an FMA per spin all the same), QP quads per thread (1 up to
// 512 quads, 2 up to 1024), with QP * (D rounded up to 4, 8 or 16) * (value words + 1) <= 32. FP64
// keeps RB <= 2, and RB = 2 only for DM <= 4, QP = 1: its epilogue, unrolled over the replicas, would
// spill otherwise (with 4 slots it spills six registers: N = 2000, R = 1024 17.4 us before, 16.8 with them).
template <int P, int RB>
static const void* rq_fn_d(int DM, int QP) {
  if (QP == 1) {
    switch (DM) {
      case 3: return (const void*)anneal_sparse_rq<P, RB, 3, 1>;
      case 4: return (const void*)anneal_sparse_rq<P, RB, 4, 1>;
      case 6: return (const void*)anneal_sparse_rq<P, RB, 6, 1>;
      case 8: return (const void*)anneal_sparse_rq<P, RB, 8, 1>;
    }
    if constexpr (P != PREC_FP64) {
      switch (DM) {
        case 10: return (const void*)anneal_sparse_rq<P, RB, 10, 1>;
        case 12: return (const void*)anneal_sparse_rq<P, RB, 12, 1>;
        case 16: return (const void*)anneal_sparse_rq<P, RB, 16, 1>;
      }
    }
  } else if (QP == 2) {
    switch (DM) {
      case 3: return (const void*)anneal_sparse_rq<P, RB, 3, 2>;
      case 4: return (const void*)anneal_sparse_rq<P, RB, 4, 2>;
    }
    if constexpr (P != PREC_FP64) {
      switch (DM) {
        case 6: return (const void*)anneal_sparse_rq<P, RB, 6, 2>;
        case 8: return (const void*)anneal_sparse_rq<P, RB, 8, 2>;
      }
    }
  }
  return nullptr;
}

static const void* rq_fn(int prec, int RB, int DM, int QP) {
  if (prec == PREC_FP64) {
    if (RB == 2) {
      if (QP != 1 || DM > 4) return nullptr;
      return DM == 3 ? (const void*)anneal_sparse_rq<PREC_FP64, 2, 3, 1>
                     : (const void*)anneal_sparse_rq<PREC_FP64, 2, 4, 1>;
    }
    return RB == 1 ? rq_fn_d<PREC_FP64, 1>(DM, QP) : nullptr;
  }
  if (RB == 4) return rq_fn_d<PREC_FP32, 4>(DM, QP);
  if (RB == 2) return rq_fn_d<PREC_FP32, 2>(DM, QP);
  return RB == 1 ? rq_fn_d<PREC_FP32, 1>(DM, QP) : nullptr;
}

struct SparseRq {
  const void* fn;
  int RB, threads;
  size_t lds;
};

// Picks the variant for (prec, N, D, R): the largest RB whose state fits in LDS and whose grid
// still covers every CU (RB = 1 when none does); then RB = 4 gives way to RB = 2 when it leaves
// the CUs under 16 resident waves and two RB = 2 workgroups fit on a CU (more waves hide the LDS
// and transcendental latencies better than a third and fourth replica per thread). Returns 0
// where the generic kernel must run.
static int sparse_rq_pick(int prec, int N, int D, int R, SparseRq* o) {
  const int Nq = (N + 3) / 4;
  const int QP = Nq <= 512 ? 1 : (Nq <= 1024 ? 2 : 0);
  const int cls = D <= 4 ? 4 : (D <= 8 ? 8 : (D <= 16 ? 16 : 0));  // registers of the slots: the kernel's limit
  if (!QP || !cls || QP * cls * (prec == PREC_FP64 ? 3 : 2) > 32) return 0;
  int DM = 16;
  for (int m : {12, 10, 8, 6, 4, 3})
    if (D <= m) DM = m;
  int dev = 0, cus = 256, max_lds = 65536;
  if (hipGetDevice(&dev) == hipSuccess) {
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
  }
  const size_t word = prec == PREC_FP64 ? 8 : 4;
  const int threads = ((Nq + QP - 1) / QP + 63) / 64 * 64;
  auto lds_of = [&](int rb) { return (size_t)2 * 4 * Nq * rb * word; };
  auto fits = [&](int rb) { return lds_of(rb) <= (size_t)max_lds && rq_fn(prec, rb, DM, QP) != nullptr; };
  auto per_cu = [&](int rb) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, rq_fn(prec, rb, DM, QP), threads, lds_of(rb)) != hipSuccess)
      return 0;
    return nb;
  };
  int RB = 0;
  for (int rb : {4, 2, 1}) {
    if (!fits(rb)) continue;
    RB = rb;
    if ((R + rb - 1) / rb >= cus) break;
  }
  if (!RB) return 0;
  if (RB == 4 && fits(2)) {
    const int g4 = (R + 3) / 4, g2 = (R + 1) / 2, waves = threads / 64;
    const long res4 = (long)std::min(g4, cus * std::max(per_cu(4), 1)) * waves;
    if (res4 < 16L * cus && g2 >= 2 * cus && per_cu(2) >= 2) RB = 2;
  }
  o->fn = rq_fn(prec, RB, DM, QP);
  // one replica, 8 slots: unrolled it has 129 registers, so one workgroup of more than four waves on a CU. Where
  // the grid asks for more, the rolled loop (degree 7, us per iteration, N = 1500, R = 400 2.18, rolled 1.83).
  if (prec != PREC_FP64 && RB == 1 && DM == 8 && QP == 1 && R > cus)
    o->fn = (const void*)anneal_sparse_rq<PREC_FP32, 1, 8, 1, false>;
  o->RB = RB;
  o->threads = threads;
  o->lds = lds_of(RB);
  return o->fn != nullptr;
}

int sparse_rq_applies(int prec, int N, int D) {
  SparseRq c;
  return sparse_rq_pick(prec, N, D, 1, &c);
}

hipError_t launch_anneal_sparse(int prec, const AnnealArgs& a, const int* ell_col, const void* ell_val, int D,
                                int RB, int allow_rq, int* used_rq, hipStream_t st) {
  SparseRq c;
  const bool rq = allow_rq && sparse_rq_pick(prec, a.N, D, a.R, &c);
  if (used_rq) *used_rq = rq ? 1 : 0;
  if (rq) {
    hipError_t e = hipFuncSetAttribute(c.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)c.lds);
    if (e != hipSuccess) return e;
    AnnealArgs args = a;
    const void* col = ell_col;
    const void* val = ell_val;
    int d = D;
    void* kargs[] = {&args, &col, &val, &d};
    return hipLaunchKernel(c.fn, dim3((a.R + c.RB - 1) / c.RB), dim3(c.threads), kargs, c.lds, st);
  }
  const int grid = (a.R + RB - 1) / RB;
  const size_t lds = sparse_lds_bytes(prec, a.N, RB);
  const void* fn = prec == PREC_FP64 ? (const void*)anneal_sparse<PREC_FP64> : (const void*)anneal_sparse<PREC_FP32>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  // 16 waves per workgroup (4 per SIMD; 8 waves in FP64, whose epilogue needs more registers): the
  // gathers and the epilogue of one wave hide behind the others
  if (prec == PREC_FP64)
    hipLaunchKernelGGL((anneal_sparse<PREC_FP64>), dim3(grid), dim3(512), lds, st, a, ell_col, ell_val, D, RB);
  else
    hipLaunchKernelGGL((anneal_sparse<PREC_FP32>), dim3(grid), dim3(1024), lds, st, a, ell_col, ell_val, D, RB);
  return hipGetLastError();
}

hipError_t launch_pack_state(int prec, const void* state, void* S, int N, int R, int Kp, int ld, int Rp, int zero,
                             hipStream_t st) {
  const size_t total = (size_t)Rp * Kp;
  const int blocks = (int)std::min<size_t>((total + 255) / 256, 4096);
  switch (prec) {
    case PREC_FP64:
      hipLaunchKernelGGL((pack_state_kernel<double, double>), dim3(blocks), dim3(256), 0, st,
                         (const double*)state, (double*)S, N, R, Kp, ld, Rp, zero);
      break;
    case PREC_FP32:
      hipLaunchKernelGGL((pack_state_kernel<float, float>), dim3(blocks), dim3(256), 0, st,
                         (const float*)state, (float*)S, N, R, Kp, ld, Rp, zero);
      break;
    case PREC_FP8J_FP8S:
      hipLaunchKernelGGL(pack_state_fp8_kernel, dim3(blocks), dim3(256), 0, st, (const float*)state, (uint8_t*)S, N,
                         R, Kp, ld, Rp, zero);
      break;
    default:
      hipLaunchKernelGGL((pack_state_kernel<__bf16, float>), dim3(blocks), dim3(256), 0, st,
                         (const float*)state, (__bf16*)S, N, R, Kp, ld, Rp, zero);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_readout(int prec, const void* state, int8_t* spins, size_t count, hipStream_t st) {
  const int blocks = (int)std::min<size_t>((count + 255) / 256, 8192);
  if (prec == PREC_FP64)
    hipLaunchKernelGGL((readout_kernel<double>), dim3(blocks), dim3(256), 0, st, (const double*)state,
                       spins, count);
  else
    hipLaunchKernelGGL((readout_kernel<float>), dim3(blocks), dim3(256), 0, st, (const float*)state,
                       spins, count);
  return hipGetLastError();
}

hipError_t launch_noise_words(uint32_t k0, uint32_t k1, uint32_t t, uint32_t r0, int nrep, int nq,
                              uint32_t* out, hipStream_t st) {
  const int total = nrep * nq;
  hipLaunchKernelGGL(noise_words_kernel, dim3((total + 255) / 256), dim3(256), 0, st, k0, k1, t, r0, nrep,
                     nq, out);
  return hipGetLastError();
}

hipError_t launch_noise_values(uint32_t k0, uint32_t k1, uint32_t t, uint32_t r0, int nrep, int nq,
                               int fp64, double* out, hipStream_t st) {
  const int total = nrep * nq;
  hipLaunchKernelGGL(noise_values_kernel, dim3((total + 255) / 256), dim3(256), 0, st, k0, k1, t, r0,
                     nrep, nq, fp64, out);
  return hipGetLastError();
}

}  // namespace nmfa
