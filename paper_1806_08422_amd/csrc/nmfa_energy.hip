// Ising energies of Eq. 1 (pairs i < j) for R spin vectors: E = (1/2) sum_i s_i y_i + sum_i h_i s_i
// with y = J s, a matrix product over the replicas. Integral couplings |J_ij| <= 127 use the int8
// matrix cores (exact, in any order), other couplings the FP64 ones, their sums added in one fixed
// order. The field term is added in ascending i by one thread per replica (integers where h is
// integral), so that its FP64 sum is the plain loop's bit for bit; its blocks ride in the launch of
// the pair kernels, whose time covers that serial chain.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "nmfa_device.h"
#include "nmfa_internal.h"

namespace nmfa {

typedef int i32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------------
// Field term of 64 replicas (r0 ..) by a block of 256 threads: chunks of 256 spins per replica are
// staged through LDS by all threads (coalesced), and thread q < 64 adds replica r0 + q's terms in
// ascending i. Bound by the chain of dependent additions (a thread per replica reading its own row:
// n = 777, R = 256, energies in all 144 us; now 27). T: long long (integral h) or double.
// ------------------------------------------------------------------------------------------
constexpr int FLD_K = 256;             // spins per chunk
constexpr int FLD_STRIDE = FLD_K + 4;  // LDS bytes per replica: 64 replicas' words fall on distinct banks

// 4 spins from p on (any alignment), of which the first `left` exist (zeros beyond)
__device__ __forceinline__ int load4(const int8_t* p, int left) {
  int w = 0;
  if (left >= 4) {
    __builtin_memcpy(&w, p, 4);
  } else {
    for (int j = 0; j < left; ++j) w |= (int)(uint8_t)p[j] << (8 * j);
  }
  return w;
}

template <typename T>
struct FieldSh {
  int8_t s[64 * FLD_STRIDE];
  T h[FLD_K];
};

__device__ __forceinline__ double field_term(double h, int s, double acc) { return __builtin_fma(h, (double)s, acc); }
__device__ __forceinline__ long long field_term(long long h, int s, long long acc) { return acc + h * s; }

template <typename T>
__device__ __forceinline__ T field_sum(FieldSh<T>& sh, const double* __restrict__ h, const int8_t* __restrict__ spins,
                                       int N, int R, int r0) {
  T acc = (T)0;
  // thread t stages words t % 64 (4 spins) of replicas t / 64 + 4 j, and h_t, of a chunk; the next
  // chunk's loads are in flight while a chunk is added up
  const int q0 = threadIdx.x >> 6, kw = 4 * (threadIdx.x & 63);
  int pre[16];
  double hp = 0.0;
  auto fetch = [&](int k0) {
    const int8_t* p = spins + (size_t)r0 * N + k0 + kw;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int q = q0 + 4 * j;
      pre[j] = r0 + q < R ? load4(p + (size_t)q * N, N - k0 - kw) : 0;
    }
    hp = k0 + (int)threadIdx.x < N ? h[k0 + threadIdx.x] : 0.0;
  };
  fetch(0);
  for (int k0 = 0; k0 < N; k0 += FLD_K) {
    const int len = min(FLD_K, N - k0);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) *reinterpret_cast<int*>(sh.s + (q0 + 4 * j) * FLD_STRIDE + kw) = pre[j];
    sh.h[threadIdx.x] = (T)hp;
    __syncthreads();
    if (k0 + FLD_K < N) fetch(k0 + FLD_K);
    if (threadIdx.x < 64) {
      const int8_t* s = sh.s + threadIdx.x * FLD_STRIDE;
      int k = 0;
      for (; k + 8 <= len; k += 8) {
        const int w0 = *reinterpret_cast<const int*>(s + k), w1 = *reinterpret_cast<const int*>(s + k + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = field_term(sh.h[k + j], (int)(int8_t)(w0 >> (8 * j)), acc);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = field_term(sh.h[k + 4 + j], (int)(int8_t)(w1 >> (8 * j)), acc);
      }
      for (; k < len; ++k) acc = field_term(sh.h[k], (int)s[k], acc);
    }
  }
  return acc;
}

// ------------------------------------------------------------------------------------------
// Integral couplings |J_ij| <= 127. Operands of the pair kernel are zero-padded copies, J8p [Np][Np]
// and the signs Sp [Rp][Np] (Np and Rp multiples of 64).
// ------------------------------------------------------------------------------------------
__global__ void pad_spins_kernel(const int8_t* __restrict__ s, int N, int R, int8_t* __restrict__ Sp, int Np, int Rp,
                                 unsigned long long* __restrict__ E2) {
  const size_t total = (size_t)Rp * Np;
  const size_t first = (size_t)blockIdx.x * blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
  for (size_t idx = first; idx < (size_t)R; idx += step) E2[idx] = 0ull;
  for (size_t idx = first; idx < total; idx += step) {
    const int r = (int)(idx / Np), i = (int)(idx - (size_t)r * Np);
    Sp[idx] = (r < R && i < N) ? s[(size_t)r * N + i] : (int8_t)0;
  }
}

// Pair sums of a 128-row x 128-replica tile per block (grid: row tiles x (replica tiles + field
// blocks, over y and z)): wave w owns 64 x 64 of it, 4 x 4 accumulators. J and the signs stream through
// a 4-stage LDS ring of 128-k blocks by direct-to-LDS loads; the 16-byte unit u of tile row q sits at
// u ^ ((q >> 1) & 7) of its 128-byte row, so that a fragment read hits distinct banks. The wave forms
// s_i y_i for its rows and adds the per-replica sums to E2 with 64-bit integer atomics (exact, order-
// free). Np need not be a multiple of 128: rows and replicas past the end repeat the last one and
// are left out of the sums, and a last block of 64 k stops after its first step. Bound by the LDS reads
// (one 16-byte read per two MFMAs) and, where the tiles do not cover the chip, by one tile's k loop.
// All launches of one evaluation, against operands read from L2 and the field term in a launch of its
// own: n = 8192, R = 1024 600 -> 161 us; n = 2000, R = 1024 with real fields 247 -> 49 us.
// The blocks with by >= pair_by (where h is given) write the field term of 64 replicas each to fld.
constexpr int EP_T = 128, EP_KB = 128, EP_NS = 4, EP_STAGE = 2 * EP_T * EP_KB, EP_LPW = EP_STAGE / 1024 / 4;

__global__ __launch_bounds__(256) void energy_pairs_i8(const int8_t* __restrict__ J8p, const int8_t* __restrict__ Sp,
                                                       int Np, int R, unsigned long long* __restrict__ E2, int pair_by,
                                                       const double* __restrict__ h, int h_integral,
                                                       const int8_t* __restrict__ spins, int N,
                                                       long long* __restrict__ fld) {
  extern __shared__ __align__(16) unsigned char smem_ep[];  // the ring, or a field block's staging
  FieldSh<long long>& sh = *reinterpret_cast<FieldSh<long long>*>(smem_ep);
  const int by = (int)(blockIdx.y + gridDim.y * blockIdx.z);
  if (by >= pair_by) {
    const int r0 = 64 * ((int)blockIdx.x + (int)gridDim.x * (by - pair_by));
    if (!h || r0 >= R) return;
    const int r = r0 + (int)threadIdx.x;
    if (h_integral) {
      const long long f = field_sum(sh, h, spins, N, R, r0);
      if (threadIdx.x < 64 && r < R) fld[r] = f;
    } else {
      const double f = field_sum(reinterpret_cast<FieldSh<double>&>(sh), h, spins, N, R, r0);
      if (threadIdx.x < 64 && r < R) reinterpret_cast<double*>(fld)[r] = f;
    }
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, g4 = lane >> 4;
  const int m0 = blockIdx.x * EP_T, rep0 = by * EP_T, Rp = (R + 63) / 64 * 64;
  const int wm = 64 * (wave >> 1), wr = 64 * (wave & 1);
  // 1 KB loads of eight tile rows: 0 .. 15 the J tile, 16 .. 31 the signs; wave w issues 8 w .. 8 w + 7
  const int8_t* src[EP_LPW];
  int unit[EP_LPW];
#pragma unroll
  for (int u = 0; u < EP_LPW; ++u) {
    const int b = EP_LPW * wave + u, q = 8 * (b & 15) + (lane >> 3);
    unit[u] = (lane & 7) ^ ((q >> 1) & 7);
    src[u] = b < 16 ? J8p + (size_t)min(m0 + q, Np - 1) * Np : Sp + (size_t)min(rep0 + q, Rp - 1) * Np;
  }
  const int nkb = (Np + EP_KB - 1) / EP_KB;
  auto issue = [&](int kb) {
#pragma unroll
    for (int u = 0; u < EP_LPW; ++u) {
      const int k = kb * EP_KB + 16 * unit[u];
      __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint32_t*>(src[u] + (k < Np ? k : k - 64)),
                                       smem_ep + (kb % EP_NS) * EP_STAGE + (EP_LPW * wave + u) * 1024, 16, 0, 0);
    }
  };
  i32x4 acc[4][4];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) acc[rt][ct] = i32x4{0, 0, 0, 0};
#pragma unroll
  for (int p = 0; p < EP_NS - 1; ++p)
    if (p < nkb) issue(p);
  for (int kb = 0; kb < nkb; ++kb) {
    // this wave's part of block kb has landed (up to two blocks after it may still be in flight)
    const int rem = nkb - 1 - kb;
    if (rem >= 2) __builtin_amdgcn_s_waitcnt(0xF70 | ((2 * EP_LPW) & 15) | (((2 * EP_LPW) >> 4) << 14));
    else if (rem == 1) __builtin_amdgcn_s_waitcnt(0xF70 | EP_LPW);
    else __builtin_amdgcn_s_waitcnt(0xF70);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();  // every wave's part landed; every wave is done with block kb - 1
    __builtin_amdgcn_sched_barrier(0);
    if (kb + EP_NS - 1 < nkb) issue(kb + EP_NS - 1);
    const unsigned char* At = smem_ep + (kb % EP_NS) * EP_STAGE + wm * EP_KB;
    const unsigned char* Bt = smem_ep + (kb % EP_NS) * EP_STAGE + (EP_T + wr) * EP_KB;
    const int steps = kb * EP_KB + 64 < Np ? 2 : 1;
    for (int st = 0; st < steps; ++st) {
      const int off = c * EP_KB + (((4 * st + g4) ^ ((c >> 1) & 7)) * 16);
      i32x4 af[4], bf[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        af[i] = *reinterpret_cast<const i32x4*>(At + 16 * EP_KB * i + off);
        bf[i] = *reinterpret_cast<const i32x4*>(Bt + 16 * EP_KB * i + off);
      }
#pragma unroll
      for (int rt = 0; rt < 4; ++rt)
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
          acc[rt][ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[rt], bf[ct], acc[rt][ct], 0, 0, 0);
    }
    // the reads of this block are complete before the next barrier frees its buffer
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_sched_barrier(0);
  }
  // lane (c, g4) holds y of rows m0 + wm + 16 rt + 4 g4 + v for replica rep0 + wr + 16 ct + c
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
    const int r = rep0 + wr + 16 * ct + c;
    long long part = 0;  // other values than +-1 are taken as the integers they are: a product may need 36 bits
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
      const int row = m0 + wm + 16 * rt + 4 * g4;
      const int sv = (r < R && row < Np) ? *reinterpret_cast<const int*>(Sp + (size_t)r * Np + row) : 0;  // 4 signs
#pragma unroll
      for (int v = 0; v < 4; ++v) part += (long long)(int8_t)(sv >> (8 * v)) * acc[rt][ct][v];
    }
    part += __shfl_xor(part, 16, 64);
    part += __shfl_xor(part, 32, 64);
    if (g4 == 0 && r < R) atomicAdd(&E2[r], (unsigned long long)part);
  }
}

// E_int = (sum_i s_i y_i) / 2 + the integral field term; E adds an FP64 field term. fld and E (or
// E_int) may be the same memory.
__device__ __forceinline__ void energy_finish(long long pair2, bool has_h, int h_integral, long long fld, int r,
                                              long long* E_int, double* E) {
  const long long e2 = pair2 + (has_h && h_integral ? 2 * fld : 0);
  if (E_int) E_int[r] = e2 / 2;
  E[r] = has_h && !h_integral ? (double)(e2 / 2) + __longlong_as_double(fld) : (double)(e2 / 2);
}

__global__ void energy_finish_kernel(const unsigned long long* __restrict__ E2, int has_h, int h_integral,
                                     const long long* fld, int R, long long* E_int, double* E) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= R) return;
  energy_finish((long long)E2[r], has_h != 0, h_integral, has_h ? fld[r] : 0ll, r, E_int, E);
}

// n <= 256: one launch does all of it (the launches above take about 4.5 us each, whatever their work:
// n = 173, R = 64 with fields 31 -> 10 us; n = 100, R = 16384 16 -> 8 us). A block owns 16 replicas and
// all rows: wave w the 16-row tiles w, w + 4, ...; the signs are staged, zero-padded, in LDS, and J8p
// comes from L2.
constexpr int ESM_NP = 256;
__global__ __launch_bounds__(256) void energy_small_i8(const int8_t* __restrict__ J8p, int Np,
                                                       const double* __restrict__ h, int h_integral,
                                                       const int8_t* __restrict__ spins, int N, int R,
                                                       long long* __restrict__ E_int, double* __restrict__ E) {
  __shared__ __align__(16) int8_t sp[16 * (ESM_NP + 16)];
  __shared__ double hs[ESM_NP];
  __shared__ long long red[4][16];
  const int st = Np + 16;  // row stride: the 16 rows of a fragment read fall on distinct banks
  const int r0 = blockIdx.x * 16;
  for (int idx = threadIdx.x; idx < 16 * Np; idx += 256) {
    const int q = idx / Np, k = idx - q * Np;
    sp[q * st + k] = (r0 + q < R && k < N) ? spins[(size_t)(r0 + q) * N + k] : (int8_t)0;
  }
  if (h)
    for (int k = threadIdx.x; k < N; k += 256) hs[k] = h[k];
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane & 15, g4 = lane >> 4;
  long long part = 0;
  for (int row0 = 16 * wave; row0 < Np; row0 += 64) {
    i32x4 acc = i32x4{0, 0, 0, 0};
    const int8_t* a_ptr = J8p + (size_t)(row0 + c) * Np + 16 * g4;
    for (int k0 = 0; k0 < Np; k0 += 64)
      acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(*reinterpret_cast<const i32x4*>(a_ptr + k0),
                                                  *reinterpret_cast<const i32x4*>(sp + c * st + 16 * g4 + k0), acc, 0,
                                                  0, 0);
    const int sv = *reinterpret_cast<const int*>(sp + c * st + row0 + 4 * g4);
#pragma unroll
    for (int v = 0; v < 4; ++v) part += (long long)(int8_t)(sv >> (8 * v)) * acc[v];
  }
  part += __shfl_xor(part, 16, 64);
  part += __shfl_xor(part, 32, 64);
  if (g4 == 0) red[wave][c] = part;
  __syncthreads();
  const int r = r0 + (int)threadIdx.x;
  if (threadIdx.x >= 16 || r >= R) return;
  long long fld = 0;
  if (h && h_integral) {
    for (int i = 0; i < N; ++i) fld = field_term((long long)hs[i], (int)sp[threadIdx.x * st + i], fld);
  } else if (h) {
    double f = 0.0;
    for (int i = 0; i < N; ++i) f = field_term(hs[i], (int)sp[threadIdx.x * st + i], f);
    fld = __double_as_longlong(f);
  }
  long long pair2 = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) pair2 += red[w][threadIdx.x];
  energy_finish(pair2, h != nullptr, h_integral, fld, r, E_int, E);
}

// ------------------------------------------------------------------------------------------
// FP64 couplings: y on v_mfma_f64_16x16x4f64. A block owns 64 rows x 16 CT replicas, 16 rows per wave;
// J comes from memory (lane group g carries k = 4 m + g in step m: four consecutive doubles per
// row and step), the signs through LDS, 256 k at a time, as bytes ordered so that a lane reads its 16
// steps' signs of a 64-k block with one ds_read_b128. The block's partial sum of s_i y_i goes to
// part[row block][R], and the finishing kernel adds the row blocks in ascending order. With part =
// null one block runs over all row blocks and adds them in the same order: the same bits without
// scratch. What bounds it: the matrix cores where the blocks cover the chip (n = 8192, R = 256: 0.79
// ms, 43 TFLOP/s), else the k loop of one block. Against one block per replica reading all of J: n =
// 1000, R = 512 984 -> 74 us; n = 4000, R = 1024 15.9 -> 0.75 ms; n = 8192, R = 256 89.5 -> 0.79 ms.
// ------------------------------------------------------------------------------------------
constexpr int EF_K = 256;             // k per staged chunk
constexpr int EF_STRIDE = EF_K + 16;  // LDS bytes per replica

template <int CT>
__global__ __launch_bounds__(256) void energy_f64(const double* __restrict__ J, const int8_t* __restrict__ spins, int N,
                                                  int R, int pair_by, double* __restrict__ part,
                                                  const double* __restrict__ h, int exact, double* __restrict__ fld,
                                                  long long* __restrict__ E_int, double* __restrict__ E) {
  using Tr = Traits<PREC_FP64>;
  __shared__ __align__(16) int8_t sp[16 * CT * EF_STRIDE];
  __shared__ double red[4][16 * CT];
  __shared__ FieldSh<double> fsh;
  const int by = (int)(blockIdx.y + gridDim.y * blockIdx.z);
  if (by >= pair_by) {  // field term of 64 replicas (or past the grid's end)
    const int r0 = 64 * ((int)blockIdx.x + (int)gridDim.x * (by - pair_by));
    if (!h || !fld) return;
    if (r0 >= R) return;
    const double f = field_sum(fsh, h, spins, N, R, r0);
    if (threadIdx.x < 64 && r0 + (int)threadIdx.x < R) fld[r0 + threadIdx.x] = f;
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, c = lane & 15;
  const int rep0 = by * 16 * CT;
  const int nb = (N + 63) / 64;
  double total = 0.0;  // of replica rep0 + threadIdx.x
  for (int b = blockIdx.x; b < nb; b += gridDim.x) {
    const int arow = min(64 * b + 16 * wave + Tr::a_row(c), N - 1);  // rows beyond N are left out of the sums
    const double* Jr = J + (size_t)arow * N + g;
    f64x4 acc[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[ct][v] = 0.0;
    for (int k0 = 0; k0 < N; k0 += EF_K) {
      __syncthreads();
      // thread t: spins 4 (t % 64) .. +3 of replicas t / 64 + 4 j
      const int kw = 4 * (threadIdx.x & 63);
      int pre[4 * CT];
#pragma unroll
      for (int j = 0; j < 4 * CT; ++j) {
        const int r = rep0 + (int)(threadIdx.x >> 6) + 4 * j;
        pre[j] = r < R ? load4(spins + (size_t)r * N + k0 + kw, N - k0 - kw) : 0;
      }
#pragma unroll
      for (int j = 0; j < 4 * CT; ++j) {
        int8_t* d = sp + ((threadIdx.x >> 6) + 4 * j) * EF_STRIDE + (kw & 192) + ((kw & 63) >> 2);
#pragma unroll
        for (int v = 0; v < 4; ++v) d[16 * v] = (int8_t)(pre[j] >> (8 * v));
      }
      __syncthreads();
      for (int sub = 0; sub < EF_K && k0 + sub < N; sub += 64) {
        double af[16];
        const double* p = Jr + k0 + sub;
        if (k0 + sub + 64 <= N) {
#pragma unroll
          for (int m = 0; m < 16; ++m) af[m] = p[4 * m];
        } else {
#pragma unroll
          for (int m = 0; m < 16; ++m) af[m] = k0 + sub + 4 * m + g < N ? p[4 * m] : 0.0;
        }
        int4 sv[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
          sv[ct] = *reinterpret_cast<const int4*>(sp + (16 * ct + c) * EF_STRIDE + sub + 16 * g);
#pragma unroll
        for (int m = 0; m < 16; ++m)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            const int w = m < 4 ? sv[ct].x : (m < 8 ? sv[ct].y : (m < 12 ? sv[ct].z : sv[ct].w));
            acc[ct] = Tr::mfma(af[m], (double)(int)(int8_t)(w >> (8 * (m & 3))), acc[ct]);
          }
      }
    }
    // lane (c, g) holds y of rows 64 b + 16 wave + 4 g + v for replica rep0 + 16 ct + c
    __syncthreads();
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int r = rep0 + 16 * ct + c;
      double p = 0.0;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 64 * b + 16 * wave + 4 * g + v;
        // rows beyond N are left out: they repeat row N - 1, whose y may be infinite (0 x inf)
        if (r < R && i < N) p = __builtin_fma((double)spins[(size_t)r * N + i], acc[ct][v], p);
      }
      p += __shfl_xor(p, 16, 64);
      p += __shfl_xor(p, 32, 64);
      if (g == 0) red[wave][16 * ct + c] = p;
    }
    __syncthreads();
    if (threadIdx.x < 16 * CT) {
      const double p = (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
      const int r = rep0 + (int)threadIdx.x;
      if (part && r < R) part[(size_t)b * R + r] = p;
      total += p;
    }
  }
  if (part) return;
  // one block over all rows: finish here
  double field = 0.0;
  if (h) field = field_sum(fsh, h, spins, N, R, rep0);
  const int r = rep0 + (int)threadIdx.x;
  if (threadIdx.x >= 16 * CT || r >= R) return;
  if (E_int) E_int[r] = exact ? (long long)total / 2 + (long long)field : 0;
  E[r] = 0.5 * total + field;
}

// fld and E may be the same memory
__global__ void energy_f64_finish(const double* __restrict__ part, int nb, const double* fld, int exact, int R,
                                  long long* __restrict__ E_int, double* E) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= R) return;
  double total = 0.0;
  for (int b = 0; b < nb; ++b) total += part[(size_t)b * R + r];
  const double field = fld ? fld[r] : 0.0;
  if (E_int) E_int[r] = exact ? (long long)total / 2 + (long long)field : 0;
  E[r] = 0.5 * total + field;
}

size_t energy_f64_part(int N) { return (size_t)(N + 63) / 64; }

// values of by that the field blocks of R replicas take beside a grid of gx columns
static int field_rows(const double* h, int R, int gx) { return h ? ((R + 63) / 64 + gx - 1) / gx : 0; }
// grid of gx x by blocks, by over y and z (a grid's y extent is limited to 65535)
static dim3 grid_of(int gx, int by) {
  const int z = (by + 32767) / 32768;
  return dim3(gx, (by + z - 1) / z, z);
}

hipError_t launch_energy_f64(const double* J64, const double* h, int exact, const int8_t* spins, int N, int R,
                             double* part, long long* E_int, double* E, hipStream_t st) {
  const int nb = (N + 63) / 64;
  if (!part || nb == 1) {  // one launch
    hipLaunchKernelGGL(energy_f64<1>, grid_of(1, (R + 15) / 16), dim3(256), 0, st, J64, spins, N, R, (R + 15) / 16,
                       (double*)nullptr, h, exact, (double*)nullptr, E_int, E);
    return hipGetLastError();
  }
  // 64 replicas per block where such blocks cover the chip, else 16 (the sums are the same)
  if ((long)nb * ((R + 63) / 64) >= 256) {
    const int by = (R + 63) / 64;
    hipLaunchKernelGGL(energy_f64<4>, grid_of(nb, by + field_rows(h, R, nb)), dim3(256), 0, st, J64, spins, N, R, by,
                       part, h, exact, E, E_int, E);
  } else {
    const int by = (R + 15) / 16;
    hipLaunchKernelGGL(energy_f64<1>, grid_of(nb, by + field_rows(h, R, nb)), dim3(256), 0, st, J64, spins, N, R, by,
                       part, h, exact, E, E_int, E);
  }
  hipLaunchKernelGGL(energy_f64_finish, dim3((R + 127) / 128), dim3(128), 0, st, (const double*)part, nb,
                     h ? (const double*)E : nullptr, exact, R, E_int, E);
  return hipGetLastError();
}

hipError_t launch_energy_i8(const int8_t* J8p, int Np, const double* h, int h_integral, const int8_t* spins,
                            int N, int R, int8_t* Sp, unsigned long long* E2, long long* E_int, double* E,
                            hipStream_t st) {
  if (Np <= ESM_NP) {
    hipLaunchKernelGGL(energy_small_i8, dim3((R + 15) / 16), dim3(256), 0, st, J8p, Np, h, h_integral, spins, N, R,
                       E_int, E);
    return hipGetLastError();
  }
  const int Rp = (R + 63) / 64 * 64;
  const size_t total = (size_t)Rp * Np;
  const int pb = (int)std::min<size_t>((total + 255) / 256, 4096);
  hipLaunchKernelGGL(pad_spins_kernel, dim3(pb), dim3(256), 0, st, spins, N, R, Sp, Np, Rp, E2);
  long long* fld = reinterpret_cast<long long*>(E);  // the field terms wait in E
  const size_t lds = (size_t)EP_NS * EP_STAGE;
  hipError_t e =
      hipFuncSetAttribute((const void*)energy_pairs_i8, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const int gx = (Np + EP_T - 1) / EP_T, by = (R + EP_T - 1) / EP_T;
  hipLaunchKernelGGL(energy_pairs_i8, grid_of(gx, by + field_rows(h, R, gx)), dim3(256), lds, st, J8p,
                     (const int8_t*)Sp, Np, R, E2, by, h, h_integral, spins, N, fld);
  hipLaunchKernelGGL(energy_finish_kernel, dim3((R + 127) / 128), dim3(128), 0, st, (const unsigned long long*)E2,
                     h ? 1 : 0, h_integral, (const long long*)fld, R, E_int, E);
  return hipGetLastError();
}

}  // namespace nmfa
