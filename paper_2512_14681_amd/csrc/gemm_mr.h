// Many-row GEMM of the decoder's projections, Y[R][N] = X[R][K] * W[N][K]^T,
// for the wide Jacobi steps (multi-block drafts with recycled candidates,
// Sec. 3.2 and App. A Alg. 1; the packed training forward; prompt chunks).
// Planned and launched by gemm_mr.hip, instantiated per row-tile count in
// gemm_mr_rt*.hip.
//
// What bounds it: up to about 128 rows the weight stream (6.7 TB/s measured
// for a streaming read), beyond it the matrix cores (every activation is two
// bf16 planes, so twice the algorithmic operations; 1.75 PFLOP/s measured
// for bare 16x16x32 instructions) and what moves through LDS.  So
//   * a workgroup of 8 waves (one per compute unit) takes all rows of up to
//     256 (more rows: equal chunks) and a group of columns, so the weights
//     come from HBM once and are requested by one compute unit;
//   * both operands go from global memory to LDS without passing registers,
//     in 1 KB pieces that already have the matrix instructions' operand order
//     (no bank conflicts, no address work on the way out), into rings of 3 to
//     12 stages; the activations, which every workgroup reads, come from L2
//     (27 TB/s measured for 256 compute units reading one buffer);
//   * the waves tile the workgroup's block WM x WN, so a fragment read from
//     LDS feeds NT or MT matrix instructions;
//   * a step's LDS reads and loads are spread between its matrix instructions;
//   * split K (narrow matrices): each workgroup writes its raw partial tile
//     and a second kernel sums the partials in split order (deterministic)
//     and runs the epilogue.
// Measured (7B shapes, us with the reduction; before: a kernel whose waves
// each streamed their own weights through registers and re-read all
// activations from LDS): gate/up at 64 / 192 / 320 / 512 rows 62 / 116 / 211
// / 285 -> 52 / 86 / 156 / 211; down 47 / 68 / 114 / 139 -> 38 / 62 / 91 /
// 131; QKV 24 / 35 / 48 / 62 -> 20 / 30 / 38 / 51; the LM head at 64 rows
// 284 -> 240.
#pragma once

#include <type_traits>

#include "jf_device.h"
#include "jf_epilogue.h"
#include "jf_internal.h"

namespace jf {

constexpr int kMrWaves = 8;
constexpr int kMrThreads = 64 * kMrWaves;

// Accumulator sets of a wave: the activation's lo plane has its own where
// the registers allow (2 sets: half the fp32 additions in the chain that
// carries the rounding error), and the even and odd steps theirs (4).
constexpr int mr_acc(int MT, int NT) {
  const int frags = 8 * (2 * MT + NT);        // two stages' fragments
  return 16 * MT * NT + frags <= 200 ? 4 : (8 * MT * NT + frags <= 200 ? 2 : 1);
}

// Block shape and LDS rings of one instantiation: WM x WN waves, each MT row
// tiles x NT column tiles.  A stage is one 32-wide fragment step of K: per
// row tile a 1 KB piece of each activation plane, per column tile a 1 KB
// piece of the packed weights.  The waves below LW bring the weight pieces
// and the others the activation pieces, each into a ring of its own depth
// (DW, DX stages): the counter of outstanding loads retires a wave's loads
// in issue order, so a wave that brought both would hold its activations
// (L2 hits) behind its weights (HBM).  Measured with 24 KB of shared and
// 10 KB of private bytes a stage on every compute unit: 57 us for 268 MB of
// weights when each wave brings both, 52 us with the roles split (75 us
// without the streaming hint on the weights).
template <int MT, int NT, int WM, int WN, int KB> struct MrCfg {
  static_assert(WM * WN == kMrWaves, "8 waves");
  static constexpr int RT = MT * WM, CT = NT * WN;
  static constexpr int XP = 2 * RT, WP = CT;   // 1 KB pieces a stage
  static constexpr int worst(int lw) {
    const int a = (WP + lw - 1) / lw, b = (XP + kMrWaves - lw - 1) / (kMrWaves - lw);
    return a > b ? a : b;
  }
  static constexpr int best_lw() {
    int best = 1;
    for (int l = 2; l < kMrWaves; ++l)
      if (worst(l) < worst(best)) best = l;
    return best;
  }
  static constexpr int LW = best_lw();
  static constexpr int CW = (WP + LW - 1) / LW, CX = (XP + kMrWaves - LW - 1) / (kMrWaves - LW);
  // Ring depths within KB kilobytes: activations 8 deep where they are small
  // (a stage is short then, and 4 of them no longer cover a load's latency),
  // else 4, or 3 where the weights would be left with fewer than 3; the
  // weights what remains, at most 12.
  static constexpr int DX = 8 * XP + 8 * WP <= KB ? 8 : (6 * XP + 6 * WP <= KB ? 6 : (4 * XP + 3 * WP <= KB ? 4 : 3));
  static constexpr int DW0 = (KB - DX * XP) / WP;
  static constexpr int DW = DW0 > 12 ? 12 : DW0;
  static_assert(DW >= 3 && DX * XP + DW * WP <= KB, "LDS ring");
  static_assert(16 * RT <= kMrThreads, "a row per thread");
  static_assert((DW - 1) * CW <= 63 && (DX - 1) * CX <= 63, "outstanding-load counter");
  static constexpr int kRing = (DX * XP + DW * WP) * 1024;
  // the epilogue's fp32 tile (aliased over the rings): ER row tiles a round
  static constexpr int TLD = CT * 16 + 4;
  static constexpr int ER0 = kRing / (16 * TLD * 4);
  static constexpr int ER = ER0 > RT ? RT : ER0;
  static_assert(ER >= 1, "epilogue tile");
  static constexpr int kLds = kRing + RT * 16 * 4;  // + the rows' 1 / rms
  static constexpr int ACC = mr_acc(MT, NT);
};

template <int N> __device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// Waits until at most `a` (<= A) stages of C loads each are outstanding.
template <int C, int A> __device__ __forceinline__ void wait_stages(int a) {
  if constexpr (A == 0) {
    wait_vm<0>();
  } else {
    if (a >= A) wait_vm<A * C>();
    else wait_stages<C, A - 1>(a);
  }
}
// One 1 KB piece from global memory to LDS without passing registers: lane
// l's 16 bytes at src + lane16 go to LDS byte dst + 16 l (M0 holds dst; one
// wait state between its write and the load).  Written as the instruction:
// the compiler would take every LDS read for a reader of every such load in
// flight and wait for all of them.  The ring's waits below order them.
// kStream: the weights of a launch whose blocks share none are read once,
// with the streaming hint.
template <bool kStream> __device__ __forceinline__ void dma_1k(const char* src, int lane16, uint32_t dst) {
  if constexpr (kStream)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(dst), "v"(lane16), "s"(src)
                 : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(lane16), "s"(src)
                 : "memory", "m0");
}

template <int MT, int NT> struct MrFrags {
  uint4 x[MT][2];  // hi, lo
  uint4 w[NT];
};

// What a wave brings: its pieces e = first + step i of a stage (C of them,
// or C - 1), from the bases src[i], into a ring of D stages of NP pieces.
template <int C> struct MrLoader {
  const char* src[C];
  uint32_t ring;       // LDS byte address of piece `first` of slot 0
  bool full;           // C pieces a stage, else C - 1
};

// The K loop of a wave over nst stages.  Step s multiplies the fragments of
// stage s (read one step ahead) while those of stage s + 1 come from LDS.
// One barrier a step: at it every wave has stage s in registers, so its slot
// is refilled (stage s + D), and every wave's loads of stage s + 1 have
// landed.  kWeights: the wave brings weight pieces (K-block stride kstride
// bytes, fragment step f at 1024 (f % 4) in it), else activation pieces
// (contiguous stages).
template <typename Cfg, int MT, int NT, bool kWeights, bool kStream>
__device__ __forceinline__ void mr_kloop(f32x4_t (&acc)[Cfg::ACC][MT][NT], const MrLoader<kWeights ? Cfg::CW : Cfg::CX>& ld,
                                         int s0, int nst, size_t kstride, const char* rx, const char* rw, int lane16) {
  constexpr int C = kWeights ? Cfg::CW : Cfg::CX, D = kWeights ? Cfg::DW : Cfg::DX;
  constexpr int NP = kWeights ? Cfg::WP : Cfg::XP, STEP = kWeights ? Cfg::LW : kMrWaves - Cfg::LW;
  constexpr int kReads = NT + 2 * MT;         // fragments: the weights', then the row tiles' hi and lo
  auto offset = [&](int s) {
    const int f = s0 + s;
    return kWeights ? (size_t)(f >> 2) * kstride + (size_t)(f & 3) * 1024 : (size_t)f * 1024;
  };
  auto issue1 = [&](int i, size_t off, uint32_t d) {
    if (i < C - 1 || ld.full) dma_1k<kStream>(ld.src[i] + off, lane16, d + STEP * i * 1024);
  };
  auto read1 = [&](int j, MrFrags<MT, NT>& f, const char* px, const char* pw) {
    if (j < NT) f.w[j] = *reinterpret_cast<const uint4*>(pw + j * 1024);
    else f.x[(j - NT) >> 1][(j - NT) & 1] = *reinterpret_cast<const uint4*>(px + (j - NT) * 1024);
  };
  // plane k % 2 of row tile k / 2, for a step of parity par
  auto mma1 = [&](auto par, int k, const MrFrags<MT, NT>& f) {
    constexpr int p = decltype(par)::value;
    const int a = Cfg::ACC == 4 ? 2 * p + (k & 1) : (Cfg::ACC == 2 ? k & 1 : 0);
#pragma unroll
    for (int t = 0; t < NT; ++t)
      acc[a][k >> 1][t] =
          __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f.x[k >> 1][k & 1]),
                                                  __builtin_bit_cast(bf16x8_t, f.w[t]), acc[a][k >> 1][t], 0, 0, 0);
  };
  auto mma = [&](auto par, const MrFrags<MT, NT>& f) {
#pragma unroll
    for (int k = 0; k < 2 * MT; ++k) mma1(par, k, f);
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
  // at most a (<= D - 2) stages outstanding
  auto wait = [&](int a) {
    if (ld.full) wait_stages<C, D - 2>(a);
    else wait_stages<C - 1, D - 2>(a);
  };
  auto barrier = [&] {
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto next = [](int q, int d) { return q + 1 == d ? 0 : q + 1; };
  // One step's work in 2 MT slices: a slice is its share of the next stage's
  // LDS reads and of the refill's loads, then the matrix instructions of one
  // plane of one row tile.  Issued in one go at the start of the step, the
  // refill's loads (16 clocks of address work each, 8 waves at once) hold
  // every wave's matrix instructions back; left alone, the compiler sinks
  // the reads to the end of the step, where the next step waits for them.
  auto slices = [&](auto par, const MrFrags<MT, NT>& cur, MrFrags<MT, NT>& nxt, bool refill, size_t off, uint32_t d,
                    const char* px, const char* pw) {
    constexpr int kSl = 2 * MT;
#pragma unroll
    for (int k = 0; k < kSl; ++k) {
#pragma unroll
      for (int j = 0; j < kReads; ++j)
        if (j * kSl / kReads == k) read1(j, nxt, px, pw);
      if (refill) {
#pragma unroll
        for (int i = 0; i < C; ++i)
          if (i * kSl / C == k) issue1(i, off, d);
      }
      mma1(par, k, cur);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int d = 0; d < D && d < nst; ++d) {
#pragma unroll
    for (int i = 0; i < C; ++i) issue1(i, offset(d), ld.ring + d * (NP * 1024));
  }
  MrFrags<MT, NT> f0, f1;
  wait(nst - 1);
  barrier();
#pragma unroll
  for (int j = 0; j < kReads; ++j) read1(j, f0, rx, rw);
  int si = 0, qx = 1, qw = 1;                 // ring slots: the next stage to issue and to read
  auto full_step = [&](auto par, int s, const MrFrags<MT, NT>& cur, MrFrags<MT, NT>& nxt) {  // s + D < nst
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (ld.full) wait_vm<(D - 2) * C>();
    else wait_vm<(D - 2) * (C - 1)>();
    barrier();
    slices(par, cur, nxt, true, offset(s + D), ld.ring + si * (NP * 1024), rx + qx * (Cfg::XP * 1024),
           rw + qw * (Cfg::WP * 1024));
    si = next(si, D);
    qx = next(qx, Cfg::DX);
    qw = next(qw, Cfg::DW);
  };
  auto tail_step = [&](auto par, int s, const MrFrags<MT, NT>& cur, MrFrags<MT, NT>& nxt) {  // s + 1 < nst
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wait(nst - 2 - s);
    barrier();
    if (s + D < nst) {
      const size_t off = offset(s + D);
#pragma unroll
      for (int i = 0; i < C; ++i) issue1(i, off, ld.ring + si * (NP * 1024));
    }
    slices(par, cur, nxt, false, 0, 0, rx + qx * (Cfg::XP * 1024), rw + qw * (Cfg::WP * 1024));
    si = next(si, D);
    qx = next(qx, Cfg::DX);
    qw = next(qw, Cfg::DW);
  };
  int s = 0;
  for (; s + 1 + D < nst; s += 2) {
    full_step(even, s, f0, f1);
    full_step(odd, s + 1, f1, f0);
  }
  for (; s + 2 < nst; s += 2) {
    tail_step(even, s, f0, f1);
    tail_step(odd, s + 1, f1, f0);
  }
  if (s + 1 < nst) {
    tail_step(even, s, f0, f1);
    mma(odd, f1);
  } else {
    mma(even, f0);
  }
}

// The K loop for operands off a 16-byte boundary, which the loads above do not
// take: every wave brings C pieces a fragment step through registers, two
// stages of two steps ahead, into two LDS slots (stage s + 1 is written while
// stage s is read; the barrier between them waits for LDS only, so the loads
// stay in flight).  Piece i of a wave comes from src[i] and goes to dst[i] of
// slot 0; the weight pieces (isw[i]) advance by K-blocks of kstride bytes, the
// others are contiguous, and a step's pieces of the two kinds are WP and XP apart
// in a slot.  A piece with on[i] false (a wave's last) re-reads another and is
// not written.
template <int C> struct MrAnyPieces {
  const char* src[C];
  char* dst[C];
  bool isw[C], on[C];
};
template <typename Cfg, int MT, int NT, int C>
__device__ __forceinline__ void mr_kloop_any(f32x4_t (&acc)[Cfg::ACC][MT][NT], const MrAnyPieces<C>& pc, int s0, int nst,
                                             size_t kstride, const char* rx, const char* rw, int lane16) {
  static_assert(Cfg::DX >= 4 && Cfg::DW >= 4, "two slots of two steps");
  u32x4_t stg[2][2][C];
  auto load = [&](u32x4_t (&r)[2][C], int s) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int f = s0 + 2 * s + j;
      const size_t wo = (size_t)(f >> 2) * kstride + (size_t)(f & 3) * 1024, xo = (size_t)f * 1024;
#pragma unroll
      for (int i = 0; i < C; ++i)
        r[j][i] = *reinterpret_cast<const u32x4_t*>(pc.src[i] + (pc.isw[i] ? wo : xo) + lane16);
    }
  };
  auto store = [&](const u32x4_t (&r)[2][C], int slot) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < C; ++i)
        if (pc.on[i])
          *reinterpret_cast<u32x4_t*>(pc.dst[i] + (2 * slot + j) * (pc.isw[i] ? Cfg::WP : Cfg::XP) * 1024 + lane16) =
              r[j][i];
  };
  auto barrier = [] {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto compute = [&](int slot) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const char *px = rx + (2 * slot + j) * (Cfg::XP * 1024), *pw = rw + (2 * slot + j) * (Cfg::WP * 1024);
      uint4 w[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) w[t] = *reinterpret_cast<const uint4*>(pw + t * 1024);
#pragma unroll
      for (int k = 0; k < 2 * MT; ++k) {
        const uint4 x = *reinterpret_cast<const uint4*>(px + k * 1024);
        const int a = Cfg::ACC == 4 ? 2 * j + (k & 1) : (Cfg::ACC == 2 ? k & 1 : 0);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[a][k >> 1][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8_t, x), __builtin_bit_cast(bf16x8_t, w[t]), acc[a][k >> 1][t], 0, 0, 0);
      }
    }
  };
  const int ns = nst / 2;                     // stages (nst is even)
  load(stg[0], 0);
  if (ns > 1) load(stg[1], 1);
  store(stg[0], 0);
  barrier();
  int s = 0;
#pragma unroll 1
  for (; s + 4 <= ns; s += 2) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      compute(d);
      load(stg[d], s + d + 2);
      store(stg[d ^ 1], d ^ 1);
      barrier();
    }
  }
  // fewer than 4 stages left
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    if (s + d < ns) {
      compute(d & 1);
      if (s + d + 2 < ns) load(stg[d & 1], s + d + 2);
      if (s + d + 1 < ns) store(stg[(d & 1) ^ 1], (d & 1) ^ 1);
      barrier();
    }
  }
}

// kAny: operands of any alignment (mr_kloop_any).
template <int MT, int NT, int WM, int WN, int KB, bool kAny>
__global__ void __launch_bounds__(kMrThreads, 2)
k_gemm_mr(const bf16_t* __restrict__ X, size_t xplane, const bf16_t* __restrict__ Wp, MrPlan m, Epi ep) {
  using Cfg = MrCfg<MT, NT, WM, WN, KB>;
  constexpr int XP = Cfg::XP, WP = Cfg::WP, LW = Cfg::LW, CX = Cfg::CX, CW = Cfg::CW;
  extern __shared__ __align__(16) char lds[];
  char* lx = lds;                             // [DX][XP][1 KB]
  char* lw = lds + Cfg::DX * XP * 1024;       // [DW][WP][1 KB]
  float* s_rs = reinterpret_cast<float*>(lds + Cfg::kRing);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Block order: unit u = (column group, K split), the split fastest, and the
  // row chunks of a unit on one XCD (ids congruent mod 8) next to each other
  // in dispatch order, so that they share the weights in its L2.  With 2, 4
  // or 8 splits every XCD works on one K range, whose activations then stay
  // in its L2.
  const int b = blockIdx.x;
  const int z = (b >> 3) % m.chunks, u = ((b >> 3) / m.chunks) * 8 + (b & 7);
  if (u >= m.n_cg * m.S) return;              // ids past the last unit (block-uniform)
  const int sk = u % m.S, g = u / m.S;
  const int KC = m.KC, P = m.P;
  const int r0 = z * 16 * Cfg::RT;            // first row of the chunk
  const int rtiles = (min(16 * Cfg::RT, m.R - r0) + 15) / 16;
  const int U = m.T / m.gr;                   // column units
  const int t0 = (int)(((long)U * g) / m.n_cg) * m.gr, t1 = (int)(((long)U * (g + 1)) / m.n_cg) * m.gr;
  const int nt = t1 - t0;                     // column tiles of the group (<= CT)
  // fragment steps (kAny: a whole number of its two-step stages)
  const int s0 = kAny ? (2 * KC * sk) / m.S * 2 : (4 * KC * sk) / m.S;
  const int s1 = kAny ? (2 * KC * (sk + 1)) / m.S * 2 : (4 * KC * (sk + 1)) / m.S;
  const int nst = s1 - s0;

  // Folded RMSNorm: the row sums of squares (a row per thread) are loaded
  // ahead of the rings' loads, which retire after them, and used at the end.
  uint64_t ssw[3] = {0, 0, 0};
  if (ep.ss_in && m.S == 1)
    ss_load(ep.ss_in, ep.ss_stride, min(r0 + min((int)threadIdx.x, 16 * Cfg::RT - 1), m.R - 1), ssw);

  const int lane16 = lane * 16;
  const int wm = wave / WN, wn = wave % WN;
  const char* rx = lx + wm * MT * 2048 + lane16;
  const char* rw = lw + wn * NT * 1024 + lane16;
  f32x4_t acc[Cfg::ACC][MT][NT];
#pragma unroll
  for (int a = 0; a < Cfg::ACC; ++a)
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[a][i][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto lds_addr = [](char* p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)p; };
  // This wave's pieces (absent row and column tiles re-read the last one, an
  // L2 hit whose products are not stored): bases at fragment step 0.
  auto w_base = [&](int e) {                  // weight piece e: column tile e of the group
    const int t = t0 + min(e, nt - 1);
    return reinterpret_cast<const char*>(Wp + ((size_t)(t / P) * KC * P + t % P) * kBlockElems);
  };
  auto x_base = [&](int e) {                  // activation piece e: plane e % 2 of row tile e / 2
    const int rt = min(e >> 1, rtiles - 1);
    return reinterpret_cast<const char*>(X + (size_t)(e & 1) * xplane + (((size_t)(r0 / 16 + rt) * KC) << 11));
  };
  const size_t ks = (size_t)P * kBlockElems * sizeof(bf16_t);
  if constexpr (kAny) {
    constexpr int C = (XP + WP + kMrWaves - 1) / kMrWaves;
    MrAnyPieces<C> pc;
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const int e = wave + kMrWaves * i, ex = min(max(e - WP, 0), XP - 1);
      pc.isw[i] = e < WP;
      pc.on[i] = e < WP + XP;
      pc.src[i] = pc.isw[i] ? w_base(e) : x_base(ex);
      pc.dst[i] = pc.isw[i] ? lw + e * 1024 : lx + ex * 1024;
    }
    mr_kloop_any<Cfg, MT, NT, C>(acc, pc, s0, nst, ks, rx, rw, lane16);
  } else if (wave < LW) {
    MrLoader<CW> ld;
#pragma unroll
    for (int i = 0; i < CW; ++i) ld.src[i] = w_base(min(wave + LW * i, WP - 1));
    ld.ring = lds_addr(lw + wave * 1024);
    ld.full = wave + LW * (CW - 1) < WP;
    if (m.chunks == 1) mr_kloop<Cfg, MT, NT, true, true>(acc, ld, s0, nst, ks, rx, rw, lane16);
    else mr_kloop<Cfg, MT, NT, true, false>(acc, ld, s0, nst, ks, rx, rw, lane16);
  } else {
    MrLoader<CX> ld;
#pragma unroll
    for (int i = 0; i < CX; ++i) ld.src[i] = x_base(min(wave - LW + (kMrWaves - LW) * i, XP - 1));
    ld.ring = lds_addr(lx + (wave - LW) * 1024);
    ld.full = wave - LW + (kMrWaves - LW) * (CX - 1) < XP;
    mr_kloop<Cfg, MT, NT, false, false>(acc, ld, s0, nst, 0, rx, rw, lane16);
  }

  // the sets' sum: (hi + hi) + (lo + lo)
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if constexpr (Cfg::ACC == 4) {
        acc[0][i][t] += acc[2][i][t];
        acc[1][i][t] += acc[3][i][t];
      }
      if constexpr (Cfg::ACC >= 2) acc[0][i][t] += acc[1][i][t];
    }

  // Epilogue through an LDS tile over the rings, ER row tiles at a time;
  // with split K the tile goes out raw, row-major per split, for the
  // reduction kernel.
  constexpr int ER = Cfg::ER, TLD = Cfg::TLD;
  float* tile = reinterpret_cast<float*>(lds);
  const int cols = nt * 16, N = m.T * 16;
  const int mrow = wm * MT, ncol = wn * NT;
  if (ep.ss_in && m.S == 1 && threadIdx.x < 16 * Cfg::RT) s_rs[threadIdx.x] = ss_rstd(ssw, ep.norm_inv_d, ep.norm_eps);
  // the other RMSNorm accumulator (filled by the next producer) is cleared
  // by the first workgroup
  if (ep.ss_clear && b == 0)
    for (int i = threadIdx.x; i < 3 * ep.ss_stride; i += kMrThreads)
      __hip_atomic_store(ep.ss_clear + i, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int er = 0; er < rtiles; er += ER) {
    const int hr0 = r0 + er * 16;
    const int hR = min(16 * min(ER, rtiles - er), m.R - hr0);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int rt = mrow + i - er;           // wave-uniform
      if (rt >= 0 && rt < ER) {
        float4 k = {1.f, 1.f, 1.f, 1.f};
        if (ep.ss_in && m.S == 1) k = *reinterpret_cast<const float4*>(s_rs + (mrow + i) * 16 + 4 * (lane >> 4));
#pragma unroll
        for (int t = 0; t < NT; ++t)
          if (ncol + t < nt) {
            float* p = tile + (rt * 16 + 4 * (lane >> 4)) * TLD + (ncol + t) * 16 + (lane & 15);
            p[0 * TLD] = acc[0][i][t][0] * k.x;
            p[1 * TLD] = acc[0][i][t][1] * k.y;
            p[2 * TLD] = acc[0][i][t][2] * k.z;
            p[3 * TLD] = acc[0][i][t][3] * k.w;
          }
      }
    }
    __syncthreads();
    if (m.S > 1) {
      float* kp = ep.kpart + ((size_t)sk * m.R + hr0) * N + t0 * 16;
      const int q = cols / 4;
      for (int e = threadIdx.x; e < hR * q; e += kMrThreads) {
        const int r = e / q, c = 4 * (e - r * q);
        *reinterpret_cast<float4*>(kp + (size_t)r * N + c) = *reinterpret_cast<const float4*>(tile + r * TLD + c);
      }
    } else {
      epilogue_wide(tile, TLD, cols, t0 * 16, ep, g, threadIdx.x, kMrThreads, hr0, hR);
    }
  }
}

template <int MT, int NT, int WM, int WN, int KB, bool kAny = false>
static hipError_t launch_mr_cfg(const void* X, size_t xplane, const void* Wp, const MrPlan& m, const Epi& ep,
                                hipStream_t st) {
  using Cfg = MrCfg<MT, NT, WM, WN, KB>;
  if (m.RT != Cfg::RT || m.CT != Cfg::CT || m.any != (int)kAny) return hipErrorInvalidValue;
  const unsigned units = (unsigned)m.n_cg * m.S;
  hipLaunchKernelGGL((k_gemm_mr<MT, NT, WM, WN, KB, kAny>), dim3((units + 7) / 8 * 8 * m.chunks), dim3(kMrThreads),
                     Cfg::kLds, st, reinterpret_cast<const bf16_t*>(X), xplane, reinterpret_cast<const bf16_t*>(Wp), m,
                     ep);
  return hipGetLastError();
}

}  // namespace jf
