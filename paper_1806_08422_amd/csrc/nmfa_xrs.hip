// Small tiles of the register-J group kernel for gfx950 (Algorithm 1, paper Sec. II).
//
// anneal_xrj gives a workgroup 256 rows x 32 replicas, which fills the chip at N = 2000 from R = 1024
// on; with fewer replicas most CUs are idle while each iteration still takes its 7.3 us. Here a
// workgroup covers 64 x 16, 128 x 16 or 128 x 32 (64 RT rows, 16 CT replicas), so that a replica's
// iteration is spread over 2 to 8 times as many CUs; the launcher takes the tile by the estimated
// time (ctx_group_plan). The scheme is that of anneal_xrj: persistent, J in registers for the whole
// anneal, BF16 spins streamed from the group's L2 by direct-to-LDS loads in chunks of 128 k, FP32
// state in registers, one group barrier per iteration with the next noise drawn inside it. What
// differs:
//   * v_mfma_f32_16x16x32_bf16 on four k octets per step instead of two steps of 32x32x16: both add
//     their octets one after the other in ascending lane-group order, so the results are the same
//     bits (measured on gfx950 over 51,200 random outputs; no other octet order is). The k order is
//     anneal_xrj's with FP4 J and ascending otherwise, and so is the epilogue's arithmetic: every
//     tile, and the LDS-J and per-iteration kernels for FP8 / BF16 J, give the same bits.
//   * All chunks of an iteration fit in LDS (64 KB or 128 KB at Kp = 2048), so none waits for a
//     buffer; PRO chunks are issued up front and one more per chunk multiplied (an issue of all of
//     them at once held the waves back by 1085 cycles of 8145 at N = 2000).
//   * J is kept as BF16 in registers as far as they go, because the widening of FP4 (8 v_cvt per step
//     and wave) takes longer than the step's two MFMAs.
// With FP8 spins (XRS_FP8S) the decomposition is the same and the arithmetic, k order and operand layouts
// are those of anneal_xrj8: FP4 J and FP8 spins go to the mixed-format instruction as they are stored.
// What bounds it (cycles of one iteration, N = 2000, 128 x 16 tiles, one workgroup per CU): 4440 of
// 8420 the k loop, where widening and MFMAs share the issue slots of the single wave; 560 the
// epilogue; 760 two noise draws; the rest the exchange (stores, arrival, poll, first chunks), which
// is nearly all of the time at N = 300. Measured per iteration against anneal_xrj (FP4) and the
// LDS-J and tiled kernels (BF16 J): N = 2000, R = 100 8.0 -> 2.4 us, R = 256 7.3 -> 3.5, R = 512
// 7.3 -> 5.0; N = 1000, R = 1024 4.8 -> 3.2; N = 300, R = 64 3.7 -> 1.4; BF16 J, N = 1000, R = 512
// 12.0 -> 2.3, N = 1500, R = 256 34.8 -> 4.4, N = 2000, R = 1024 42 -> 23; FP8 spins against
// anneal_xrj8, N = 2000, R = 100 5.0 -> 2.0, R = 256 5.0 -> 2.2, R = 512 5.0 -> 3.3, N = 1000, R = 256
// 3.5 -> 1.5, R = 1024 3.6 -> 2.4, N = 300, R = 64 3.1 -> 1.1.
#include <hip/hip_runtime.h>

#include "nmfa_device.h"
#include "nmfa_group.h"
#include "nmfa_internal.h"

namespace nmfa {

typedef int i32x8 __attribute__((ext_vector_type(8)));

// JFMT: format of J in memory (0 BF16, 1 FP8 E4M3, 2 FP4 E2M1), spins in BF16; XRS_FP8S: FP4 J and FP8
// E4M3 spins, both taken by the matrix instruction as they are stored (a chunk of 256 bytes per replica
// is 256 k then, else 128). The first NB chunks of J are held in registers as BF16, widened once at the
// start; with FP4 J the others stay in FP4 and are widened at every use. NB is what the registers of
// one wave per SIMD have room for beside about 110 (one column tile) or 150 (two) others; a tile whose
// FP8 or BF16 J does not fit is not built.
template <int JFMT, int RT, int CT, int NCH>
struct XrsCfg {
  static constexpr int ROWS = 64 * RT;         // rows of J per workgroup (16 RT per wave)
  static constexpr int RG = 16 * CT;           // replicas per group
  static constexpr int CHB = RG * 256;         // bytes of one chunk of spins
  static constexpr bool S8 = JFMT == XRS_FP8S;
  static constexpr int ES = S8 ? 1 : 2;        // bytes per spin
  static constexpr int NST = S8 ? 2 : 4;       // matrix steps per chunk (of 128 or 32 k)
  static constexpr int MW = JFMT == 0 ? 4 : (JFMT == 1 ? 2 : 1);  // 32-bit words per 8 couplings in memory
  static constexpr int JBUDGET = CT == 1 ? 336 : 304;             // registers for J
  static constexpr int NBMAX = (JBUDGET / (4 * RT) - NCH) / 3;
  static constexpr int NB = S8 ? 0 : (JFMT != 2 || NBMAX > NCH ? NCH : NBMAX);
  static constexpr int JREGS = S8 ? 8 * RT * NCH : 4 * RT * (4 * NB + MW * (NCH - NB));
};

// 8 couplings of format JFMT as BF16 (exact in every format)
template <int JFMT>
__device__ __forceinline__ bf16x8 xrs_widen(const uint32_t (&m)[JFMT == 0 ? 4 : (JFMT == 1 ? 2 : 1)]) {
  if constexpr (JFMT >= 2) return fp4x8_to_bf16x8(m[0]);
  else if constexpr (JFMT == 1) return fp8x8_to_bf16x8(m[0], m[1]);
  else return __builtin_bit_cast(bf16x8, uint4{m[0], m[1], m[2], m[3]});
}

template <int JFMT, int RT, int CT, int NCH>
__device__ __forceinline__ void xrs_body(const AnnealArgs& a, const XcdArgs& x) {
  using C = XrsCfg<JFMT, RT, CT, NCH>;
  constexpr bool S8 = C::S8;
  constexpr int NC = NCH, NST = C::NST, NSTEP = NC * NST, ES = C::ES;
  constexpr int D = NST;                              // spin fragments read D steps (one chunk) ahead
  constexpr int GB = (CT == 1 ? 2 : 4) / (S8 ? 2 : 1);  // chunks per workgroup barrier
  constexpr int PRO = NC < 7 ? NC : 7;                // chunks issued before the k loop
  constexpr int CHB = C::CHB, ROWS = C::ROWS, RG = C::RG, MW = C::MW, NB = C::NB;
  constexpr int DPW = CHB / 1024 / 4;                 // 1 KB direct-to-LDS loads per wave and chunk
  constexpr bool XRJ = JFMT >= 2;  // arithmetic and k order of anneal_xrj, else those of anneal_xcd
  static_assert(NC * DPW <= 63 && D % NST == 0, "wait counts fit the vmcnt field");
  extern __shared__ __align__(16) unsigned char smem[];  // one buffer per chunk
  __shared__ unsigned abort_word;                        // the group barrier's decision
  const int N = a.N, ks = x.ks;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: scalar registers
  const int g = lane >> 4, c = lane & 15;

  const XcdSlot slot = xcd_register(x, tid);
  const unsigned my_group = slot.my_group;
  if (my_group >= (unsigned)x.groups) return;
  const int group = (int)my_group + x.group_base;
  const int rb = slot.rb;
  const bool xcd_mode = slot.xcd_mode;
  bool aborted = slot.aborted;
  const int ch0 = XRJ ? (rb * ROWS / 256) * (S8 ? 1 : 2) : 0;  // first chunk of the pass over k

  // J of this wave: jr[i][st][rt] = the 8 couplings of row rb ROWS + 16 (RT wave + rt) + c at
  // k = 128 ch + 32 st + 8 g .. +7 with ch = (ch0 + i) mod NC
  // (FP8 spins: j8[i][st][rt] = the 32 of that row at k = 256 ch + 128 st + 32 g ..)
  bf16x8 jb[NB > 0 ? NB : 1][NST][RT];                // chunks 0 .. NB - 1, widened
  uint32_t jn[NC > NB ? NC - NB : 1][NST][RT][MW];    // the others
  uint4 j8[S8 ? NC : 1][NST][RT];
  if constexpr (S8) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const unsigned char* p = reinterpret_cast<const unsigned char*>(a.J) +
                               (size_t)(rb * ROWS + 16 * (RT * wave + rt) + c) * (128 * NC) + 16 * g;
#pragma unroll
      for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int st = 0; st < NST; ++st)
          j8[i][st][rt] = *reinterpret_cast<const uint4*>(p + 128 * ((ch0 + i) % NC) + 64 * st);
    }
  } else {
    const size_t jrow = (size_t)64 * NC * MW;  // bytes of one row (Kp couplings)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const unsigned char* p = reinterpret_cast<const unsigned char*>(a.J) +
                               (size_t)(rb * ROWS + 16 * (RT * wave + rt) + c) * jrow + 4 * MW * g;
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int ch = (ch0 + i) % NC;
#pragma unroll
        for (int st = 0; st < NST; ++st) {
          uint32_t m[MW];
#pragma unroll
          for (int q = 0; q < MW; ++q)
            m[q] = *reinterpret_cast<const uint32_t*>(p + 64 * MW * ch + 16 * MW * st + 4 * q);
          if (i < NB) {
            jb[i < NB ? i : 0][st][rt] = xrs_widen<JFMT>(m);
          } else {
#pragma unroll
            for (int q = 0; q < MW; ++q) jn[i < NB ? 0 : i - NB][st][rt][q] = m[q];
          }
        }
      }
    }
  }
  float* state = reinterpret_cast<float*>(a.state);
  float* traj = reinterpret_cast<float*>(a.traj);
  const float* coef = reinterpret_cast<const float*>(a.coef);
  // outputs of this lane: rows row0 + 16 rt + v, replicas rgroup0 + 16 ct + c
  const int row0 = rb * ROWS + 16 * RT * wave + 4 * g;
  const int rgroup0 = group * RG;
  f32x4 inv[RT], hinv[RT];  // 1 / norm_i and h_i / norm_i of this lane's rows
  float s[RT][CT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    inv[rt] = reinterpret_cast<const f32x4*>(a.inv_norm)[(row0 + 16 * rt) >> 2];
    hinv[rt] = reinterpret_cast<const f32x4*>(a.hterm)[(row0 + 16 * rt) >> 2];
    // rows beyond N: a field that no 1 / T, however large, turns into a NaN (0 x NaN would spread it)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (row0 + 16 * rt + v >= N) hinv[rt][v] = 1.0f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int r = rgroup0 + 16 * ct + c;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = row0 + 16 * rt + v;
        s[rt][ct][v] = (a.load_state && r < a.R && row < N) ? state[(size_t)r * N + row] : 0.0f;
      }
    }
  }
  const float sg = (float)a.sigma;
  const float neg2ln2_s2 = -2.0f * 0.6931471805599453f * sg * sg;
  const float alpha = (float)a.alpha, oma = (float)(1.0 - a.alpha);
  const float alpha2 = (float)(2.0 * a.alpha), nalpha = (float)(-a.alpha);

  // Spin chunks: replica rows of 16 units of 16 bytes; unit u of replica q sits at u ^ (q & 15), so
  // the 16 lanes that one ds_read_b128 serves at a time hit all 64 banks once
  // (BF16: unit 4 st + g in step st; FP8, whose operand takes k = 16 g .. and 64 + 16 g .. of a step: units
  // 8 st + g and 8 st + 4 + g)
  int boff[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) boff[j] = c * 256 + (((4 * j + g) ^ c) * 16);
  unsigned dma_off[DPW];
#pragma unroll
  for (int u = 0; u < DPW; ++u) {
    const int q = 4 * (DPW * wave + u) + lane / 16;
    dma_off[u] = (unsigned)(q * ks * ES + ((lane % 16) ^ (q & 15)) * 16);
  }
  // where this lane's new spins go in the group's rows of S
  const unsigned out_off = (unsigned)(c * ks + row0) * ES;

  // The noise of one iteration, drawn while the group barrier of the one before completes: w is
  // (h_i + sigma z) / (T_t norm_i) in exp2 units with anneal_xrj's arithmetic, else sigma z
  float w[RT][CT][4];
  f32x4 invc[RT];
  float coef_next = coef[a.t_begin - 1];
  auto draw = [&](int tt, int d, float coef_tt) {
    const int rt = d / CT, ct = d % CT;
    float z[4];
    sigma_gauss4_f32(philox4x32_10((uint32_t)((row0 + 16 * rt) >> 2), (uint32_t)(rgroup0 + 16 * ct + c), (uint32_t)tt,
                                   0u, a.key0, a.key1),
                     neg2ln2_s2, z);
    if constexpr (XRJ) {
      const float coef_z = a.negate_noise ? -coef_tt : coef_tt;
      const f32x4 hc = hinv[rt] * coef_tt;
      invc[rt] = inv[rt] * coef_tt;
#pragma unroll
      for (int v = 0; v < 4; ++v) w[rt][ct][v] = fmaf(z[v], coef_z, hc[v]);
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) w[rt][ct][v] = a.negate_noise ? -z[v] : z[v];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) asm volatile("" : "+v"(w[rt][ct][v]));  // drawn here, not at its use
  };
#pragma unroll
  for (int d = 0; d < RT * CT; ++d) draw(a.t_begin, d, coef_next);

  unsigned char* S0 = reinterpret_cast<unsigned char*>(x.S[0]) + (size_t)group * RG * ks * ES;
  unsigned char* S1 = reinterpret_cast<unsigned char*>(x.S[1]) + (size_t)group * RG * ks * ES;
  unsigned* bar = &x.ctl[CTL_BAR + 16 * (int)my_group];
  int epoch = 0;
  __syncthreads();

  for (int t = a.t_begin; t <= a.t_end && !aborted; ++t) {
    const float coef_t = coef_next;
    unsigned char* Sg = (t & 1) ? S1 : S0;
    unsigned char* Sn = (t & 1) ? S0 : S1;
    const __amdgpu_buffer_rsrc_t srs = __builtin_amdgcn_make_buffer_rsrc(Sg, 0, RG * ks * ES, 0x00020000);
    int ch_t = ch0, wb = DPW * 1024 * wave;  // opaque, so that no address is held across the loop
    asm volatile("" : "+s"(ch_t));
    asm volatile("" : "+s"(wb));
    auto issue = [&](int i) {
      int ch = ch_t + i;
      if (ch >= NC) ch -= NC;
#pragma unroll
      for (int u = 0; u < DPW; ++u)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(srs, smem + wb + i * CHB + u * 1024, 16, dma_off[u], ch * 256, 0,
                                                 AUX_SC1);
    };
#pragma unroll
    for (int i = 0; i < PRO; ++i) issue(i);
    // FP8 spins are read as BF16 vectors too: an integer read would wait for every direct-to-LDS load in
    // flight, which the compiler takes to be integer stores (N = 2000, R = 100, BF16: 2.4 -> 3.4 us)
    bf16x8 fb[D + 1][CT][S8 ? 2 : 1];
    auto load = [&](int sidx) {
      constexpr int NU = S8 ? 2 : 1;  // 16-byte units of a step
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int u = 0; u < NU; ++u)
          fb[sidx % (D + 1)][ct][u] = *reinterpret_cast<const bf16x8*>(smem + (sidx / NST) * CHB + ct * 4096 +
                                                                       boff[sidx % NST * NU + u]);
    };
    f32x4 acc[RT][CT];
    wait_vm<(PRO > GB ? PRO - GB : 0) * DPW>();
    bare_barrier();
#pragma unroll
    for (int sidx = 0; sidx < D; ++sidx) load(sidx);
    // step sidx: the spins of step sidx + D are read while the MFMAs of step sidx run; the workgroup
    // meets before the first read of each batch of GB chunks, when every wave's loads of that batch
    // have landed. One further chunk is issued per chunk multiplied, so that the loads run beside
    // the matrix work instead of ahead of it.
    static_for(
        [&](auto sc) {
          constexpr int sidx = decltype(sc)::value;
          constexpr int i = sidx / NST, st = sidx % NST;
          constexpr int nxt = sidx + D;
          if constexpr (nxt < NSTEP && nxt % (NST * GB) == 0) {
            constexpr int ci = nxt / NST;                                 // first chunk of the batch
            constexpr int issued = PRO + i < NC ? PRO + i : NC;           // chunks issued so far
            constexpr int need = ci + GB < NC ? ci + GB : NC;
            static_assert(issued >= need, "the batch has been issued");
            wait_vm<(issued - need) * DPW>();
            __builtin_amdgcn_sched_barrier(0);
            bare_barrier();
            __builtin_amdgcn_sched_barrier(0);
          }
          if constexpr (st == 0 && PRO + i < NC) issue(PRO + i);
          if constexpr (nxt < NSTEP) load(nxt);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            if constexpr (S8) {
              const uint4 j = j8[i][st][rt];
              const i32x8 af = i32x8{(int)j.x, (int)j.y, (int)j.z, (int)j.w, 0, 0, 0, 0};
#pragma unroll
              for (int ct = 0; ct < CT; ++ct) {
                const uint4 lo = __builtin_bit_cast(uint4, fb[sidx % (D + 1)][ct][0]);
                const uint4 hi = __builtin_bit_cast(uint4, fb[sidx % (D + 1)][ct][S8 ? 1 : 0]);
                const i32x8 bf = i32x8{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w,
                                       (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
                acc[rt][ct] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                    af, bf, sidx == 0 ? f32x4{} : acc[rt][ct], 4, 0, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f);
              }
            } else {
              bf16x8 af;
              if constexpr (i < NB) af = jb[i][st][rt];
              else af = xrs_widen<JFMT>(jn[i - NB][st][rt]);
#pragma unroll
              for (int ct = 0; ct < CT; ++ct)
                acc[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    af, fb[sidx % (D + 1)][ct][0], sidx == 0 ? f32x4{} : acc[rt][ct], 0, 0, 0);
            }
          }
          __builtin_amdgcn_sched_barrier(0);  // keeps the reads D steps ahead of their use
        },
        std::make_integer_sequence<int, NSTEP>{});

    // ---- fused epilogue --------------------------------------------------------------------
    if (t < a.t_end) coef_next = coef[t];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float sv;
          if constexpr (XRJ) {
            // -tanh(Phi / T) = 2 / (1 + exp2(arg)) - 1 with arg = 2 log2(e) Phi / T; damped update
            const float e = __builtin_amdgcn_exp2f(fmaf(acc[rt][ct][v], invc[rt][v], w[rt][ct][v]));
            sv = fmaf(alpha2, __builtin_amdgcn_rcpf(1.0f + e), fmaf(oma, s[rt][ct][v], nalpha));
          } else {
            const float phi = fmaf(acc[rt][ct][v], inv[rt][v], hinv[rt][v]) + w[rt][ct][v];
            sv = fmaf(alpha, neg_tanh_from_exp2_arg(phi * coef_t), oma * s[rt][ct][v]);
          }
          s[rt][ct][v] = sv;
        }
        unsigned char* dst = Sn + (out_off + (unsigned)(16 * rt + ct * 16 * ks) * ES);
        if constexpr (S8) {
          const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(s[rt][ct][0], s[rt][ct][1], 0, false);
          *reinterpret_cast<int*>(dst) = __builtin_amdgcn_cvt_pk_fp8_f32(s[rt][ct][2], s[rt][ct][3], lo, true);
        } else {
          const __bf16 outv[4] = {(__bf16)s[rt][ct][0], (__bf16)s[rt][ct][1], (__bf16)s[rt][ct][2],
                                  (__bf16)s[rt][ct][3]};
          *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<const uint2*>(outv);
        }
      }
    const int k_rec = t - a.t_begin;
    if (traj && k_rec < a.record) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int r = rgroup0 + 16 * ct + c;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int row = row0 + 16 * rt + v;
            if (r < a.R && row < N) traj[((size_t)k_rec * a.R + r) * N + row] = s[rt][ct][v];
          }
      }
    }
    if (t < a.t_end) {
      // half of the next iteration's noise while the spin stores complete, the other half while the
      // other workgroups arrive
      constexpr int ND = RT * CT, H = (ND + 1) / 2;
#pragma unroll
      for (int d = 0; d < H; ++d) draw(t + 1, d, coef_next);
      xcd_group_arrive(bar, xcd_mode, tid);
#pragma unroll
      for (int d = H; d < ND; ++d) draw(t + 1, d, coef_next);
      aborted = xrj_group_wait(x, bar, (unsigned)++epoch, xcd_mode, tid, 0u, &abort_word);
    }
  }

  // ---- final state and readout ---------------------------------------------------------------
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const int r = rgroup0 + 16 * ct + c;
    if (r >= a.R) continue;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = row0 + 16 * rt + v;
        if (row < N) {
          state[(size_t)r * N + row] = s[rt][ct][v];
          if (a.spins) a.spins[(size_t)r * N + row] = (s[rt][ct][v] >= 0.0f) ? (int8_t)1 : (int8_t)-1;
        }
      }
  }
}

template <int JFMT, int RT, int CT, int NCH>
__global__ __launch_bounds__(256, 1) void anneal_xrs(AnnealArgs a, XcdArgs x) {
  xrs_body<JFMT, RT, CT, NCH>(a, x);
}

int xrs_rows(int tile) { return tile == 0 ? 64 : 128; }
int xrs_group_replicas(int tile) { return tile == 2 ? 32 : 16; }

template <int JFMT, int RT, int CT, int NCH>
static const void* xrs_fn_n() {
  if constexpr (XrsCfg<JFMT, RT, CT, NCH>::JREGS <= XrsCfg<JFMT, RT, CT, NCH>::JBUDGET)
    return (const void*)anneal_xrs<JFMT, RT, CT, NCH>;
  else
    return nullptr;
}

template <int JFMT, int RT, int CT>
static const void* xrs_fn_k(int Kp) {
  constexpr int CPK = JFMT == XRS_FP8S ? 1 : 2;  // chunks per 256 k
  switch (Kp) {
    case 512: return xrs_fn_n<JFMT, RT, CT, 2 * CPK>();
    case 768: return xrs_fn_n<JFMT, RT, CT, 3 * CPK>();
    case 1024: return xrs_fn_n<JFMT, RT, CT, 4 * CPK>();
    case 1280: return xrs_fn_n<JFMT, RT, CT, 5 * CPK>();
    case 1536: return xrs_fn_n<JFMT, RT, CT, 6 * CPK>();
    case 1792: return xrs_fn_n<JFMT, RT, CT, 7 * CPK>();
    case 2048: return xrs_fn_n<JFMT, RT, CT, 8 * CPK>();
    default: return nullptr;
  }
}

template <int JFMT>
static const void* xrs_fn_t(int tile, int Kp) {
  if (tile == 0) return xrs_fn_k<JFMT, 1, 1>(Kp);
  if (tile == 1) return xrs_fn_k<JFMT, 2, 1>(Kp);
  return tile == 2 ? xrs_fn_k<JFMT, 2, 2>(Kp) : nullptr;
}

static const void* xrs_fn(int jfmt, int tile, int Kp) {
  switch (jfmt) {
    case 0: return xrs_fn_t<0>(tile, Kp);
    case 1: return xrs_fn_t<1>(tile, Kp);
    case 2: return xrs_fn_t<2>(tile, Kp);
    case XRS_FP8S: return xrs_fn_t<XRS_FP8S>(tile, Kp);
    default: return nullptr;
  }
}

bool xrs_applies(int jfmt, int tile, int Kp) { return xrs_fn(jfmt, tile, Kp) != nullptr; }

hipError_t launch_anneal_xrs(int jfmt, int tile, const AnnealArgs& a, const XcdArgs& x, int grid, hipStream_t st) {
  const void* fn = xrs_fn(jfmt, tile, a.Kp);
  if (!fn) return hipErrorInvalidValue;
  return launch_group_resident(fn, grid, 256, (size_t)a.Kp * (jfmt == XRS_FP8S ? 1 : 2) * xrs_group_replicas(tile), a,
                               x, st);
}

}  // namespace nmfa
