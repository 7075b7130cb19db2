// Jacobi trajectories (Sec. 2.1) and the noise-schedule point selection
// (Sec. 3.1, Eq. 7; App. C) -- the data-collection side of Jacobi Forcing.
//
// k_traj_record writes iterate y^(j+1) of an n-token block from y^(j) and the
// argmaxes of the step that fed y^(j)'s unaccepted tail: one HBM pass over n
// tokens.
//
// Point selection reads every point of every block once: HBM-bound, with
// little data per block (a 16-token block's 17 points are 1088 bytes), so
// the design goal is bytes in flight.  k_traj_select_multi gives each wave B
// blocks: one load of their B lengths, then every point of all B blocks and
// their fixed points y* loaded at once through range-checked buffer loads
// (when n <= 64 a load covers floor(64 / n) points: 4 points of a 16-token
// block per coalesced 256-byte load); lane j then owns point j (so
// max_points <= 64 there).  k_traj_select_wide does the same for n = 16 and
// 32 without counts, four tokens a lane (traj_select_form).
// k_traj_select (one block per wave, any n and length) is the general path.
// The unconverged count of a point is a popcount of the wave's mismatch
// ballot; the choice is exact integer arithmetic, |u w - t_num n| minimal
// (the fraction u / n closest to t_num / w), ties to the earliest point.
#include "jf_internal.h"

namespace jf {
namespace {

constexpr int kSelWaves = 4;   // waves (blocks of tokens) per workgroup
constexpr int kSelBatch = 8;   // loads issued back to back per wave
constexpr int kStreamHint = 2;   // cache policy of a buffer load: nontemporal (each point is read once)
constexpr int kBufferFlags = 0x00020000;  // buffer descriptor word 3 (gfx9 family): 32-bit raw data

__global__ void __launch_bounds__(256) k_traj_record(const int32_t* prev, const int32_t* __restrict__ g,
                                                     int n, int rows, int32_t* out) {
  // positions < n - rows were accepted before the step; position n - rows is
  // the step's first row (the pending token): all of them stay.  Row r's
  // argmax is the update of position n - rows + 1 + r.
  const int keep = n - rows + 1;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256)
    out[i] = i < keep ? prev[i] : g[i - keep];
}

__global__ void __launch_bounds__(256) k_traj_select(const int32_t* __restrict__ traj,
                                                     const int32_t* __restrict__ len, int n_blocks, int n,
                                                     int max_points, int w, const int32_t* __restrict__ t_num,
                                                     int32_t* __restrict__ sel, int32_t* __restrict__ unconv) {
  const int lane = threadIdx.x & 63;
  const int b = blockIdx.x * kSelWaves + (threadIdx.x >> 6);
  if (b >= n_blocks) return;
  const int L = len[b];
  const size_t base = (size_t)b * max_points * n;
  int32_t* U = unconv ? unconv + (size_t)b * max_points : nullptr;
  if (L < 1 || L > max_points) {
    if (lane == 0) sel[b] = -1;
    if (U)
      for (int j = lane; j < max_points; j += 64) U[j] = -1;
    return;
  }
  const long long tn = (long long)(t_num ? t_num[b] : b % w) * n;
  const int32_t* T = traj + base;
  const int32_t* ys = T + (size_t)(L - 1) * n;
  long long best_d = -1;
  int best = 0;
  if (n <= 64) {
    const int per = 64 / n;                 // points per load
    const int used = per * n;
    const int sub = lane / n;
    const int pos = lane - sub * n;
    const bool active = lane < used;
    const int ystar = active ? ys[pos] : 0;
    const unsigned long long nmask = n == 64 ? ~0ull : ((1ull << n) - 1);
    for (int j0 = 0; j0 < L; j0 += per * kSelBatch) {
      int v[kSelBatch];
#pragma unroll
      for (int q = 0; q < kSelBatch; ++q) {
        const int j = j0 + q * per + sub;
        v[q] = (active && j < L) ? T[(size_t)j * n + pos] : ystar;
      }
#pragma unroll
      for (int q = 0; q < kSelBatch; ++q) {
        const int jq = j0 + q * per;
        if (jq >= L) break;
        const unsigned long long m = __ballot(v[q] != ystar);
        for (int s = 0; s < per; ++s) {
          const int j = jq + s;
          if (j >= L) break;
          const int u = __popcll((m >> (s * n)) & nmask);
          long long d = (long long)u * w - tn;
          d = d < 0 ? -d : d;
          if (best_d < 0 || d < best_d) { best_d = d; best = j; }
          if (U && lane == s) U[j] = u;
        }
      }
    }
  } else {
    for (int j = 0; j < L; ++j) {
      int u = 0;
      for (int c = 0; c < n; c += 64) {
        const int p = c + lane;
        const bool in = p < n;
        const bool diff = in && T[(size_t)j * n + p] != ys[p];
        u += __popcll(__ballot(diff));
      }
      long long d = (long long)u * w - tn;
      d = d < 0 ? -d : d;
      if (best_d < 0 || d < best_d) { best_d = d; best = j; }
      if (U && lane == 0) U[j] = u;
    }
  }
  if (U)
    for (int j = L + lane; j < max_points; j += 64) U[j] = -1;
  if (lane == 0) sel[b] = best;
}

// Minimum of a non-negative int over the 64 lanes: DPP within each row of
// 16 lanes (xor 1, xor 2, half-row mirror, row mirror), then the four row
// results through scalar registers.  All lanes must be active.
__device__ __forceinline__ int wave_min_nonneg(int x) {
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, false));  // row_half_mirror
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, false));  // row_mirror
  const int a = __builtin_amdgcn_readlane(x, 0), b = __builtin_amdgcn_readlane(x, 16);
  const int c = __builtin_amdgcn_readlane(x, 32), d = __builtin_amdgcn_readlane(x, 48);
  return min(min(a, b), min(c, d));
}

// B blocks per wave, all of their points held in K registers per block and
// the fixed point in one more (K * floor(64 / n) >= max_points, n <= 64,
// max_points <= 64, w < 2^24, n w < 2^25).
// Lane j takes point j's unconverged count u_j; a wave minimum over the key
// (d_j << 6) | j, d_j = |u_j w - t n|, picks the point, the earliest on
// ties.  The numerator t is clamped to [0, w] first: beyond that range d is
// monotone in u either way, so the choice is unchanged, and d <= n w keeps
// the key within 31 bits.
template <int B, int K>
__global__ void __launch_bounds__(256) k_traj_select_multi(const int32_t* __restrict__ traj,
                                                           const int32_t* __restrict__ len, int n_blocks,
                                                           int n, int max_points, int w,
                                                           const int32_t* __restrict__ t_num,
                                                           int32_t* __restrict__ sel,
                                                           int32_t* __restrict__ unconv) {
  const int lane = threadIdx.x & 63;
  // wave-uniform: a scalar register, so the buffer descriptors below are too
  const int b0 = __builtin_amdgcn_readfirstlane((blockIdx.x * kSelWaves + (threadIdx.x >> 6)) * B);
  if (b0 >= n_blocks) return;
  const int per = 64 / n;
  const int pos = lane % n;
  const bool active = lane < per * n;
  const unsigned long long nmask = n == 64 ? ~0ull : ((1ull << n) - 1);
  const bool mine = lane < B && b0 + lane < n_blocks;   // lane i carries block b0 + i's scalars
  const int Lr = mine ? len[b0 + lane] : 0;
  const int tr = mine ? (t_num ? min(max(t_num[b0 + lane], 0), w) : (b0 + lane) % w) : 0;
  // Loads through a buffer descriptor per block whose range is the block's
  // valid points (L n tokens): lanes past it read 0 from the hardware's range
  // check instead of branching.  Lane l of load q reads token l of the
  // per * n tokens that start at point q * per.
  // The fixed point y* (point L - 1) is one more load of the same batch.
  int v[B][K], ys[B];
#pragma unroll
  for (int i = 0; i < B; ++i) {
    const int L = __builtin_amdgcn_readlane(Lr, i);
    const int valid = (L >= 1 && L <= max_points) ? L * n * 4 : 0;
    __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int32_t*>(traj + (size_t)(b0 + i) * max_points * n), 0, valid, kBufferFlags);
#pragma unroll
    // whole offsets in the vector operand, the range-checked one
    for (int q = 0; q < K; ++q) v[i][q] = __builtin_amdgcn_raw_buffer_load_b32(rs, (q * per * n + lane) * 4, 0, 0);
    ys[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, ((L - 1) * n + pos) * 4, 0, 0);
  }
  // this lane's own point (j = lane): load lq, slice lsl
  const int lq = lane / per;
  const int lsh = (lane - lq * per) * n;
  int res = 0;
#pragma unroll
  for (int i = 0; i < B; ++i) {
    const int b = b0 + i;
    if (b >= n_blocks) break;
    const int L = __builtin_amdgcn_readlane(Lr, i);
    int32_t* U = unconv ? unconv + (size_t)b * max_points : nullptr;
    if (L < 1 || L > max_points) {
      if (lane == i) res = -1;
      if (U && lane < max_points) U[lane] = -1;
      continue;
    }
    const int tn = __builtin_amdgcn_readlane(tr, i) * n;
    unsigned long long mine_m = 0;
#pragma unroll
    for (int q = 0; q < K; ++q) {
      if (q * per < L) {                                   // uniform: loads past L hold nothing
        const unsigned long long m = __builtin_amdgcn_ballot_w64(active && v[i][q] != ys[i]);
        mine_m = q == lq ? m : mine_m;
      }
    }
    const int u = __popcll((mine_m >> lsh) & nmask);
    const int d = abs((int)__umul24(u, w) - tn);   // u <= 64, w < 2^24: one 24-bit multiply
    const int key = lane < L ? (d << 6) | lane : 0x7FFFFFFF;
    const int best = wave_min_nonneg(key) & 63;
    if (U && lane < max_points) U[lane] = lane < L ? u : -1;
    if (lane == i) res = best;
  }
  if (mine) sel[b0 + lane] = res;
}

// The same choice, without the counts, for n = 16 or 32 (Q = n / 4 lanes a
// point) and at least two points: a lane loads four tokens at once, so a
// block of 16 is one 16-byte load for its points before the fixed point and
// one for the fixed point itself (whose own count is 0), where the kernel
// above issues six 4-byte loads and a ballot, a compare and a select for
// each.  The counts are summed over a point's Q lanes and the keys minimised
// over the wave in DPP steps: about 30 vector instructions a block instead of
// 70, which bounded it.  The loads carry the streaming hint (each point is
// read once; 33.6 -> 32.4 us).  K loads hold max_points - 1 points: 64 K >=
// (max_points - 1) Q.  Where it is used: traj_select_form.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_min(int x) {
  return min(x, __builtin_amdgcn_update_dpp(x, x, CTRL, ROWS, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ int dpp_add(int x) {
  return x + __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, false);
}

template <int B, int K, int Q>
__global__ void __launch_bounds__(256) k_traj_select_wide(const int32_t* __restrict__ traj,
                                                          const int32_t* __restrict__ len, int n_blocks,
                                                          int max_points, int w, const int32_t* __restrict__ t_num,
                                                          int32_t* __restrict__ sel) {
  static_assert(Q == 4 || Q == 8, "lanes a point");
  typedef int v4i __attribute__((ext_vector_type(4)));
  constexpr int n = 4 * Q, PP = 64 / Q;                 // tokens of a point, points of a load
  const int lane = threadIdx.x & 63;
  // wave-uniform: a scalar register, so the buffer descriptors below are too
  const int b0 = __builtin_amdgcn_readfirstlane((blockIdx.x * kSelWaves + (threadIdx.x >> 6)) * B);
  if (b0 >= n_blocks) return;
  const int pos = lane % Q, pt = lane / Q;
  const bool mine = lane < B && b0 + lane < n_blocks;   // lane i carries block b0 + i's scalars
  const int Lr = mine ? len[b0 + lane] : 0;
  const int tr = mine ? (t_num ? min(max(t_num[b0 + lane], 0), w) : (b0 + lane) % w) : 0;
  // Loads through buffer descriptors whose ranges are the block's points
  // before the fixed point, and the fixed point: lanes past them read 0 from
  // the hardware's range check.
  v4i v[B][K], ys[B];
#pragma unroll
  for (int i = 0; i < B; ++i) {
    const int L = __builtin_amdgcn_readlane(Lr, i);
    const int before = (L >= 1 && L <= max_points) ? L - 1 : 0;
    int32_t* base = const_cast<int32_t*>(traj + (size_t)min(b0 + i, n_blocks - 1) * max_points * n);
    __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(base, 0, before * n * 4, kBufferFlags);
    __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(base + before * n, 0, n * 4, kBufferFlags);
#pragma unroll
    for (int q = 0; q < K; ++q)
      v[i][q] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, (q * 64 + lane) * 16, 0, kStreamHint));
    ys[i] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(ry, pos * 16, 0, kStreamHint));
  }
  int res = 0;
#pragma unroll
  for (int i = 0; i < B; ++i) {
    const int b = b0 + i;
    if (b >= n_blocks) break;
    const int L = __builtin_amdgcn_readlane(Lr, i);
    if (L < 1 || L > max_points) {
      if (lane == i) res = -1;
      continue;
    }
    const int tn = __builtin_amdgcn_readlane(tr, i) * n;
    int key = 0x7FFFFFFF;
#pragma unroll
    for (int q = 0; q < K; ++q) {
      if (q * PP < L - 1) {                             // uniform: loads past the points hold nothing
        const v4i x = v[i][q], y = ys[i];
        int u = (int)(x.x != y.x) + (int)(x.y != y.y) + (int)(x.z != y.z) + (int)(x.w != y.w);
        u = dpp_add<0xB1>(u);                           // quad_perm [1,0,3,2]
        u = dpp_add<0x4E>(u);                           // quad_perm [2,3,0,1]
        if constexpr (Q == 8) u = dpp_add<0x141>(u);    // row_half_mirror
        const int j = q * PP + pt;
        const int d = abs((int)__umul24(u, w) - tn);    // u <= 32, w < 2^24
        key = min(key, j < L - 1 ? (d << 6) | j : 0x7FFFFFFF);
      }
    }
    if constexpr (Q == 4) key = dpp_min<0x141, 0xF>(key);
    key = dpp_min<0x140, 0xF>(key);                     // row_mirror: the row's minimum in each lane
    key = dpp_min<0x142, 0xA>(key);                     // row_bcast15 into rows 1 and 3
    key = dpp_min<0x143, 0xC>(key);                     // row_bcast31 into rows 2 and 3
    // the fixed point: no token differs, d = tn
    const int best = min(__builtin_amdgcn_readlane(key, 63), (tn << 6) | (L - 1)) & 63;
    if (lane == i) res = best;
  }
  if (mine) sel[b0 + lane] = res;
}

}  // namespace

hipError_t launch_traj_record(const int32_t* prev, const int32_t* g, int n, int rows, int32_t* out,
                              hipStream_t st) {
  const int blocks = (n + 255) / 256;
  hipLaunchKernelGGL(k_traj_record, dim3(blocks), dim3(256), 0, st, prev, g, n, rows, out);
  return hipGetLastError();
}

template <int B, int K>
static void launch_multi(const int32_t* traj, const int32_t* len, int n_blocks, int n, int max_points, int w,
                         const int32_t* t_num, int32_t* sel, int32_t* unconv, hipStream_t st) {
  const int blocks = (n_blocks + kSelWaves * B - 1) / (kSelWaves * B);
  hipLaunchKernelGGL((k_traj_select_multi<B, K>), dim3(blocks), dim3(64 * kSelWaves), 0, st, traj, len,
                     n_blocks, n, max_points, w, t_num, sel, unconv);
}

template <int B, int K, int Q>
static void launch_wide(const int32_t* traj, const int32_t* len, int n_blocks, int max_points, int w,
                        const int32_t* t_num, int32_t* sel, hipStream_t st) {
  const int blocks = (n_blocks + kSelWaves * B - 1) / (kSelWaves * B);
  hipLaunchKernelGGL((k_traj_select_wide<B, K, Q>), dim3(blocks), dim3(64 * kSelWaves), 0, st, traj, len, n_blocks,
                     max_points, w, t_num, sel);
}

// Which kernel a selection runs on.  Four tokens a lane for n = 16 and 32,
// without counts, as far as its loads hold the points (n + 1 of them, the
// most a block that converges has, fit), with the fewest loads that do: one
// issued for points that are not there costs as much as the others (n = 32 of
// 5 points with four loads: 32.2 -> 59.4 us).  2^18 blocks of random lengths,
// us, k_traj_select_multi -> here: n = 16 of 2 / 9 / 17 points 30.9 / 31.8 /
// 34.0 -> 26.8 / 30.2 / 32.6; n = 32 of 2 / 9 points 31.0 / 34.5 -> 27.6 /
// 33.2, of 18 / 25 / 33 69.1 / 76.4 / 93.7 -> 60.0 / 66.6 / 83.0 (two blocks a
// wave there: four leave 2^15 blocks short of waves, 11.7 -> 12.8 of 26
// points).  Not for n = 32 of 10 to 16 points (10: 35.3 -> 44.1, 13: 42.0 ->
// 46.4), for n = 8 (16 of 64 lanes would load: 32.8 -> 34.0) and with counts (a
// store of 16 or 8 lanes a load instead of one a block: n = 16 41.1 -> 42.4,
// n = 32 111 -> 121).
int traj_select_form(int n, int max_points, int w, bool counts) {
  const bool fast = n <= 64 && max_points <= 64 && w < (1 << 24) && (long long)n * w < (1 << 25);
  if (!fast) return SEL_GENERAL;
  if (!counts && max_points >= 2) {
    if (n == 16 && max_points <= 17) return SEL_WIDE_16;
    if (n == 32 && max_points <= 9) return SEL_WIDE_32_1;
    if (n == 32 && max_points >= 17 && max_points <= 25) return SEL_WIDE_32_3;
    if (n == 32 && max_points >= 26 && max_points <= 33) return SEL_WIDE_32_4;
  }
  const int loads = (max_points + 64 / n - 1) / (64 / n);
  return loads <= 5 ? SEL_MULTI_5 : (loads <= 8 ? SEL_MULTI_8 : (loads <= 17 ? SEL_MULTI_17 : SEL_GENERAL));
}

hipError_t launch_traj_select(const int32_t* traj, const int32_t* len, int n_blocks, int n, int max_points,
                              int w, const int32_t* t_num, int32_t* sel, int32_t* unconv, hipStream_t st) {
  switch (traj_select_form(n, max_points, w, unconv != nullptr)) {
    case SEL_WIDE_16: launch_wide<8, 1, 4>(traj, len, n_blocks, max_points, w, t_num, sel, st); break;
    case SEL_WIDE_32_1: launch_wide<4, 1, 8>(traj, len, n_blocks, max_points, w, t_num, sel, st); break;
    case SEL_WIDE_32_3: launch_wide<2, 3, 8>(traj, len, n_blocks, max_points, w, t_num, sel, st); break;
    case SEL_WIDE_32_4: launch_wide<2, 4, 8>(traj, len, n_blocks, max_points, w, t_num, sel, st); break;
    case SEL_MULTI_5: launch_multi<8, 5>(traj, len, n_blocks, n, max_points, w, t_num, sel, unconv, st); break;
    case SEL_MULTI_8: launch_multi<4, 8>(traj, len, n_blocks, n, max_points, w, t_num, sel, unconv, st); break;
    case SEL_MULTI_17: launch_multi<2, 17>(traj, len, n_blocks, n, max_points, w, t_num, sel, unconv, st); break;
    default:
      hipLaunchKernelGGL(k_traj_select, dim3((n_blocks + kSelWaves - 1) / kSelWaves), dim3(64 * kSelWaves), 0, st,
                         traj, len, n_blocks, n, max_points, w, t_num, sel, unconv);
  }
  return hipGetLastError();
}

}  // namespace jf
