// Many-row GEMM of the decoder's projections, Y[R][N] = X[R][K] * W[N][K]^T:
// plans, dispatch and the split-K reduction (the main kernel is gemm_mr.h).
#include <algorithm>
#include <cmath>

#include "jf_device.h"
#include "jf_epilogue.h"
#include "gemm_mr.h"
#include "jf_internal.h"

namespace jf {

// Split-K reduction: block (x, y) sums the S partials of rows 16 y .. and
// columns 64 x .. in split order (deterministic), applies the folded RMSNorm
// and runs the epilogue (its per-block argmax slot is x).  Each thread owns
// 4 adjacent columns of one row (the 16 lanes of a row are in one wave) and
// keeps 8 partial loads in flight.  It is little more than its memory round
// trips, so the residual and QKV epilogues run in registers on operands
// loaded along with the partials (residual and gain; position, RoPE row and
// cache page), with row sums and RoPE partners exchanged between lanes: no
// LDS tile, no second round trip (192 rows: residual 8.1 -> 7.3 us, QKV 8.2
// -> 5.6 us a launch; the 64-row step 335.9 -> 325.1 us).
constexpr int kRedRows = 16, kRedCols = 64, kRedThreads = 256;

__global__ void __launch_bounds__(kRedThreads) k_mr_reduce(MrPlan m, Epi ep) {
  constexpr int tld = kRedCols + 4;
  __shared__ __align__(16) float tile[kRedRows * tld];
  const int N = m.T * 16;
  const int c0 = blockIdx.x * kRedCols, r0 = blockIdx.y * kRedRows;
  const int cols = min(kRedCols, N - c0), rows = min(kRedRows, m.R - r0);
  const size_t split = (size_t)m.R * N;
  const int r = threadIdx.x / (kRedCols / 4), c = 4 * (threadIdx.x % (kRedCols / 4));
  const bool mine = r < rows && c < cols;                   // cols is a multiple of 16
  const int row = r0 + min(r, rows - 1), col = c0 + min(c, cols - 4);
  const bool resid = ep.kind == EPI_RESID && ep.gain_next, qkv = ep.kind == EPI_QKV;
  // the epilogue's operands, in flight with the partials
  uint64_t ssw[3] = {0, 0, 0};
  if (ep.ss_in) ss_load(ep.ss_in, ep.ss_stride, row, ssw);
  float4 h = {0.f, 0.f, 0.f, 0.f}, gn = h;                  // residual, gain; or cos, sin
  int page = 0, slot = 0;
  // QKV: packed rows are q, k and v heads; RoPE pairs 8 columns apart
  const int half = ep.hd >> 1;
  const int head = qkv ? col / ep.hd : 0, w = qkv ? col - head * ep.hd : 0;
  const int cc = w & 15, ri = 8 * (w >> 4) + (cc & 7);
  const bool rope = qkv && head < ep.H + ep.G;
  if (resid) {
    h = *reinterpret_cast<const float4*>(ep.f32 + (size_t)row * ep.ldf + col);
    gn = *reinterpret_cast<const float4*>(ep.gain_next + col);
  } else if (qkv) {
    slot = ep.state[0] + row;
    if (head >= ep.H && slot < ep.max_ctx) page = ep.page_table[slot / kPage];
    if (rope) {
      const size_t o = (size_t)ep.pos[row] * half + ri;
      h = *reinterpret_cast<const float4*>(ep.rope_cos + o);
      gn = *reinterpret_cast<const float4*>(ep.rope_sin + o);
    }
  }
  float4 v = {0.f, 0.f, 0.f, 0.f};
  {
    const float4* p = reinterpret_cast<const float4*>(ep.kpart + (size_t)row * N + col);
    const size_t sp = split / 4;
    int s = 0;
    for (; s + 8 <= m.S; s += 8) {
      float4 x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = p[(size_t)(s + j) * sp];
#pragma unroll
      for (int j = 0; j < 8; ++j) { v.x += x[j].x; v.y += x[j].y; v.z += x[j].z; v.w += x[j].w; }
    }
    float4 x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (s + j < m.S) x[j] = p[(size_t)(s + j) * sp];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (s + j < m.S) { v.x += x[j].x; v.y += x[j].y; v.z += x[j].z; v.w += x[j].w; }
  }
  if (ep.ss_in) {
    const float k = ss_rstd(ssw, ep.norm_inv_d, ep.norm_eps);
    v.x *= k; v.y *= k; v.z *= k; v.w *= k;
  }
  if (resid) {
    h.x += v.x; h.y += v.y; h.z += v.z; h.w += v.w;
    float sq = mine ? h.x * h.x + h.y * h.y + h.z * h.z + h.w * h.w : 0.f;
#pragma unroll
    for (int o = 1; o < kRedCols / 4; o <<= 1) sq += __shfl_xor(sq, o);
    if (!mine) return;
    *reinterpret_cast<float4*>(ep.f32 + (size_t)row * ep.ldf + col) = h;
    const float x[4] = {h.x * gn.x, h.y * gn.y, h.z * gn.z, h.w * gn.w};
    act_store4<bf16_t>(reinterpret_cast<bf16_t*>(ep.xg) + act_offset(row, col, ep.ldf), ep.xg_plane, x);
    if (c == 0) ss_add(ep.ss_out, ep.ss_stride, row, sq);
    return;
  }
  if (qkv) {
    // the partner columns c ^ 8: two lanes away
    const float4 y = {__shfl_xor(v.x, 2), __shfl_xor(v.y, 2), __shfl_xor(v.z, 2), __shfl_xor(v.w, 2)};
    if (!mine) return;
    float o[4] = {v.x, v.y, v.z, v.w};
    int dim = w;
    if (rope) {
      const float sg = cc < 8 ? -1.f : 1.f;
      o[0] = v.x * h.x + sg * (y.x * gn.x);
      o[1] = v.y * h.y + sg * (y.y * gn.y);
      o[2] = v.z * h.z + sg * (y.z * gn.z);
      o[3] = v.w * h.w + sg * (y.w * gn.w);
      dim = cc < 8 ? ri : half + ri;
    }
    if (head < ep.H) {
      act_store4<bf16_t>(reinterpret_cast<bf16_t*>(ep.q) + ((size_t)row * ep.H + head) * ep.hd + dim, ep.q_plane, o);
      return;
    }
    if (slot >= ep.max_ctx) {
      if (ep.flags) atomicOr(ep.flags, 2);
      return;
    }
    bf16_t* pg = reinterpret_cast<bf16_t*>(ep.kv) + (size_t)page * 2 * ep.G * kPage * ep.hd;
    const int st = slot % kPage;
    if (head < ep.H + ep.G) {
      *reinterpret_cast<uint2*>(pg + ((size_t)(head - ep.H) * kPage + st) * ep.hd + dim) =
          make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
    } else {
      bf16_t* pv = pg + (size_t)ep.G * kPage * ep.hd + ((size_t)(head - ep.H - ep.G) * ep.hd + dim) * kPage + st;
#pragma unroll
      for (int k = 0; k < 4; ++k) pv[(size_t)k * kPage] = f32_to_bf16(o[k]);
    }
    return;
  }
  *reinterpret_cast<float4*>(tile + r * tld + c) = mine ? v : float4{0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  epilogue_wide(tile, tld, cols, c0, ep, blockIdx.x, threadIdx.x, kRedThreads, r0, rows);
}

// ---- plans ------------------------------------------------------------------------
// The instantiated block shapes: RT row tiles as WM x MT, column tiles as
// WN x NT for NT = 1 .. max_nt.
struct MrShape { int RT, MT, WN, max_nt; };
static const MrShape kMrShapes[] = {{2, 1, 4, 3}, {4, 1, 2, 6}, {6, 3, 4, 3}, {8, 2, 2, 6}, {10, 5, 4, 4},
                                    {12, 3, 2, 6}, {16, 4, 2, 5}};

// Estimated clocks of a launch.  A stage (a 32-wide step of K) costs its
// matrix work (16 clocks an instruction at 0.8 of the peak rate) and its
// requested bytes (17 a clock and compute unit of weights from HBM while all
// of them stream, 42 a clock of what L2 serves: the activations, and the
// weights of all but one of a unit's row chunks), which overlap but for 0.37
// of the smaller, and no less than 340 clocks of barrier and load latency.
// The constants are fitted to 3850 launches (the 7B- and mid-shaped
// projections, 24 to 512 rows, every shape, split and chunk count).  Without
// split K the QKV epilogue (2-byte stores behind RoPE and page loads, element
// by element) costs 1100 clocks for each element a thread owns, which the
// reduction's QKV epilogue does not (4608 x 2560 at 448 rows: one split 44.9
// us, two 35.9).  Each further row chunk counts 3%: launched back to back, with
// the activations still in every L2, more chunks look cheaper than they are
// inside a step (three layers, without -> with it: d = 3584 at 224 / 288 rows
// 868 -> 839 / 1103 -> 1070 us, d = 4096 at 448 rows 1392 -> 1346; it costs
// short launches, d = 256 and a prompt of 1024 tokens 356 -> 368).  Over 41600
// launches of 46 matrices (256 to 4096 wide decoders, 17 to 512 rows) the picked
// plans are 2.6% slower than the fastest on average, 1.6% without the chunks'
// 3%, 3.8% without the QKV term.
static double mr_cost(const MrPlan& m, const MrShape& sh, int NT, int cus, int epi_kind) {
  // units go round-robin over the XCDs, the row chunks of a unit to one XCD
  const double units = std::ceil((double)m.n_cg * m.S / 8) * 8;
  const double rounds = std::ceil(units * m.chunks / cus);
  const double blocks = std::min<double>(cus, (double)m.n_cg * m.S * m.chunks);
  const long U = m.T / m.gr;
  const double tiles = (double)((U + m.n_cg - 1) / m.n_cg * m.gr);
  const double w_rate = std::min(30.0, 17.0 * cus / blocks);
  const double mma = 64.0 * sh.MT * NT / 0.8;
  const double mem = tiles * 1024 / w_rate / m.chunks + tiles * 1024 / 42 * (m.chunks - 1) / m.chunks +
                     2.0 * sh.RT * 1024 / 42;
  double stage = std::max(std::max(mma, mem) + 0.37 * std::min(mma, mem), 340.0);
  // operands through registers: matrix work, LDS traffic and the hand-over in turn
  if (m.any) stage = std::max(stage, mma + (64.0 * (2 * sh.MT + NT) + 8.0 * (2 * sh.RT + m.CT)) / 2 + 280);
  double clocks = rounds * (std::ceil(4.0 * m.KC / m.S) * stage + 14500) + 6500;
  // a thread's 16 x 16 RT x tiles / 512 elements of the QKV epilogue
  if (m.S == 1 && epi_kind == EPI_QKV) clocks += rounds * 0.5 * sh.RT * tiles * 1100;
  // the partials written and read again (5 TB/s), and the reduction's launch
  if (m.S > 1) clocks += 2.0 * m.S * m.R * m.T * 64 / (2170.0 * cus / 256) + 5200;
  return clocks * (1 + 0.03 * (m.chunks - 1));
}

// Which shapes run here rather than on the weight-streaming kernel (us,
// there -> here, measured at 7B and mid shapes).  From 65 rows all: its
// 32-row chunks stream the weights three times or more (96 rows: QKV 32.8
// -> 22.2, O 25.4 -> 21.1).  33 to 64 rows (two chunks): matrices of 16M
// elements or more (64 rows: gate/up 97 -> 52, QKV 23.7 -> 19.8; smaller
// ones lose: O 16.3 -> 18.2), of 26M where its two chunks make one full round
// of 7 or 8 waves a unit that share K (at 48 rows: 4096 x 4096 / 5504 / 6912 /
// 7552 16.4 / 20.0 / 23.3 / 25.4 -> 20.3 / 21.9 / 23.8 / 24.4; but 4352 x 4096, a
// round and a bit, 28.8 -> 19.5, and wide matrices, 32000 x 512 and 16384 x 1024
// in a step, 20.5 -> 13.6 and 18.1 -> 15.0), and long K of any size (a down projection of 8192 x 512 / 1024 /
// 1536 at 64 rows 19.0 / 20.6 / 21.6 -> 12.4 / 14.6 / 17.5).  17 to 32 rows
// (its two-row-tile blocks): long K, and matrices that give every compute unit
// 8 column tiles (32 rows: gate/up 60.6 -> 47.7, down 36.4 -> 32.9, LM head 218
// -> 211, but QKV 16.2 -> 18.1); up to 24 rows, where its blocks still load
// each weight once, long K (N x 8192 at 17 rows: 1024 / 2048 / 3072 16.6 / 17.2 /
// 18.3 -> 12.9 / 15.9 / 18.3; a layer with a down projection of 3328 x 13312 /
// 3584 x 14336 / 18944 / 4096 x 16384 107.7 / 119.2 / 130.1 / 131.2 -> 104.4 / 115.4 /
// 129.2 / 130.3, of 3840 / 4096 x 8192 even), and of the others only what one
// round of workgroups holds (24 rows: gate/up 56.0 -> 47.5, LM head 198 ->
// 210).  10 to 16 rows: of those, the ones whose 64-column groups do
// not make full rounds there (gate/up at 10 / 16 rows in a step 47.5 -> 46.4 /
// 48.0 -> 46.1, at 8 rows 45.8 -> 46.2; 40960 x 512 / 2048, two and a half rounds,
// at 10 rows 14.0 / 31.9 -> 12.4 / 30.4, but 49152 x 1024 and 32768 x 3072, three
// and two, 19.7 / 34.9 -> 20.9 / 36.4), and a step's LM head (49152 x 256 / 32768
// x 3584 10.8 / 41.8 -> 10.1 / 40.4) and matrices of 200M elements (32768 x 8192
// without the scratch 87.7 -> 80.7).  Fewer rows: none.
// Without scratch for split K (split false: the LM-head component) a workgroup
// walks all of K here, where there the waves of a block share it, so long K
// counts for nothing (LM heads of 1024 / 4096 / 16384 x 8192 at 17 rows 34.5 /
// 36.2 / 46.4 -> 48.6 / 50.8 / 51.1); a head of fewer than 3 column tiles a unit
// stays up to 64 rows where it makes a full round there (8192 x 2048 / 5120 at
// 33 rows 15.0 / 29.0 -> 16.4 / 31.7; 12288 x 3584 33.3 -> 28.5), and one of
// less than a tile a unit stays while the chunks do not fill the chip (2048 x
// 3584 at 192 / 256 rows 29.1 / 37.5 -> 33.6 / 24.2) or K is long (1024 / 2048 x
// 8192 at 448 rows 30.0 / 58.5 -> 61.1 / 61.8).
static bool mr_takes(int R, int N, int K, int epi_kind, int cus, bool split) {
  const int T = N / 16;
  const bool long_k = K >= 8192 && split;
  const bool one_round = T >= 8 * cus && T <= 12 * cus;
  if (R < 10) return false;
  if (R <= 16)
    return one_round &&
           (T % (4 * cus) != 0 || (split && epi_kind == EPI_ARGMAX) || (long)N * K >= 200000000);
  if (R <= 24) return one_round || long_k;
  if (R <= 32) return long_k || T >= 8 * cus;
  if (R <= 64) {
    if (long_k) return true;
    GemmShape g{R, N, K, 1, 1, 1};
    gemm_plan(g, epi_kind);
    const long waves = (long)gemm_blocks(g) * g.S * g.C * g.WK;
    const bool full = T <= 2 * cus && waves >= 7 * cus && waves <= 8 * cus;
    if (full && !split && T < 3 * cus) return false;
    return (long)N * K >= (full ? 26000000 : 16000000);
  }
  return split || T >= cus || (K < 8192 && (long)R * T > 96 * cus);
}

// Operands off a 16-byte boundary go through registers on their way to LDS
// (mr_kloop_any), in 64-, 96- and 128-row chunks, from 33 rows on: up to 32 the
// weight-streaming kernel's blocks load each weight once (the 7B LM head at 32
// rows 201 us there, 239 here).  Three 7B layers at 48 / 96 / 192 / 320 / 512
// rows with the weights and the workspace 8 bytes off: 543 / 656 / 993 / 1512 /
// 1976 us, on the weight-streaming kernel 645 / 888 / 1265 / 1925 / 2958, aligned
// 443 / 576 / 729 / 1128 / 1528.
bool gemm_mr_plan(MrPlan& m, int R, int N, int K, int epi_kind, int n_cus, int max_splits, bool aligned) {
  if (!aligned && R < 33) return false;
  if (N % 16 || K % 128 || !mr_takes(R, N, K, epi_kind, std::max(1, n_cus), max_splits > 1)) return false;
  const int gr = epi_kind == EPI_SWIGLU ? 2 : 1;
  if ((N / 16) % gr) return false;
  const int cus = std::max(1, n_cus);
  const bool narrow = max_splits > 1 && N / 16 < 8 * std::max(1, cus / ((R + 127) / 128));
  double best = -1;
  for (const MrShape& sh : kMrShapes) {
    if (!aligned && sh.RT != 4 && sh.RT != 6 && sh.RT != 8) continue;
    MrPlan t{};
    t.any = !aligned;
    t.R = R;
    t.RT = sh.RT;
    t.KC = K / 128;
    t.P = pack_group(N);
    t.T = N / 16;
    t.gr = gr;
    t.chunks = (R + 16 * sh.RT - 1) / (16 * sh.RT);
    const int U = t.T / gr;
    for (int S = 1; S <= std::min(max_splits, 16); S *= 2) {
      // a split of at least 6 stages
      if (S > 1 && (4 * t.KC < 6 * S || (size_t)S * R * N > kGemmPartFloats)) break;
      t.S = S;
      for (int NT = 1; NT <= sh.max_nt; ++NT) {
        t.CT = sh.WN * NT;
        const int per = t.CT / gr;            // units a workgroup holds
        if (per < 1) continue;
        // fp32 additions in the longest chain (two planes a step): for a
        // matrix too narrow to fill the chip without split K no more than
        // with 4 splits and one accumulator set, so that the plan's choice
        // does not cost accuracy
        if (narrow && S * mr_acc(sh.MT, NT) < 4) continue;
        // the fewest groups, or as many as fill a round
        const int need = (U + per - 1) / per;
        const long round = std::max(1, cus / (S * t.chunks));
        t.n_cg = (int)std::min<long>(U, need <= round ? round : need);
        const double c = mr_cost(t, sh, NT, cus, epi_kind);
        if (best < 0 || c < best) {
          best = c;
          m = t;
        }
      }
    }
  }
  return best >= 0;
}

int gemm_mr_part_blocks(const MrPlan& m) { return m.S > 1 ? (m.T * 16 + kRedCols - 1) / kRedCols : m.n_cg; }

hipError_t launch_gemm_mr(const void* X, size_t xplane, const void* Wp, const MrPlan& m, const Epi& ep,
                          hipStream_t st) {
  if (m.R < 1 || m.R > kMaxRows || m.T < 1 || m.KC < 1 || m.gr < 1 || m.T % m.gr || m.n_cg < 1 ||
      m.n_cg > m.T / m.gr || m.S < 1 || m.S > (m.any ? 2 : 4) * m.KC || m.RT < 1 ||
      m.chunks != (m.R + 16 * m.RT - 1) / (16 * m.RT) || ep.row0 != 0)
    return hipErrorInvalidValue;
  // every group must fit the workgroup's column tiles
  const int U = m.T / m.gr;
  if ((U + m.n_cg - 1) / m.n_cg * m.gr > m.CT) return hipErrorInvalidValue;
  if (m.S > 1 && (!ep.kpart || (size_t)m.S * m.R * m.T * 16 > kGemmPartFloats)) return hipErrorInvalidValue;
  if (!m.any && (((uintptr_t)X | (uintptr_t)Wp | (xplane * sizeof(bf16_t))) & 15)) return hipErrorInvalidValue;
  hipError_t e = hipErrorInvalidValue;
  if (m.any) e = launch_mr_any(X, xplane, Wp, m, ep, st);
  else switch (m.RT) {
    case 2: e = launch_mr_rt2(X, xplane, Wp, m, ep, st); break;
    case 4: e = launch_mr_rt4(X, xplane, Wp, m, ep, st); break;
    case 6: e = launch_mr_rt6(X, xplane, Wp, m, ep, st); break;
    case 8: e = launch_mr_rt8(X, xplane, Wp, m, ep, st); break;
    case 10: e = launch_mr_rt10(X, xplane, Wp, m, ep, st); break;
    case 12: e = launch_mr_rt12(X, xplane, Wp, m, ep, st); break;
    case 16: e = launch_mr_rt16(X, xplane, Wp, m, ep, st); break;
    default: break;
  }
  if (e != hipSuccess || m.S == 1) return e;
  hipLaunchKernelGGL(k_mr_reduce, dim3((m.T * 16 + kRedCols - 1) / kRedCols, (m.R + kRedRows - 1) / kRedRows),
                     dim3(kRedThreads), 0, st, m, ep);
  return hipGetLastError();
}

}  // namespace jf
