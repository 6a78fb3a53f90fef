// Per-head block selection: optimal sparse indices of Sec. 4.1 (top-k of the
// block masses), text sink and row-wise uniform counts of Sec. 4.3, and the
// per-head coverage count (smallest uniform k reaching a Recall target).
//
// Determinism: the order of candidate blocks is a strict total order (text
// blocks, then the fp32 mass descending, then the index ascending), and
// cumulative masses are exact 64-bit integers, so every output is independent
// of thread scheduling.
//
// No row is sorted to find its kept blocks: a wave holds the row's masses in
// registers as ordered 32-bit keys, finds the key of the last kept block by
// counting the keys that reach a value (find_cut), and writes the kept indices
// in ascending order from ballots.  Only the coverage count needs sorted
// rows, and of those only the cumulative masses, so it sorts bare 32-bit
// keys (blocks of equal mass may change places without changing a sum).
// At 1,724 blocks per row and 24 heads (41,376 rows, 285 MB of masses),
// against a bitonic sort of 64-bit keys per row with its order and running
// sums stored: top-k selection 1,732 -> 154 us, 2.0 TB/s of the masses.  What
// is left is bound by the vector instructions (counts and exact sums): the
// vector units issue in 86% of the kernel's cycles.
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace adaspa {

constexpr int SEL_NT = 256;
constexpr int SEL_WAVES = SEL_NT / 64;

// Order-preserving 32-bit image of an fp32 value; -0 maps like +0 and NaN
// maps below every other value.  +inf maps to 0xFF800000, the largest image.
__device__ __forceinline__ uint32_t float_order_bits(float f) {
  uint32_t b = __float_as_uint(f);
  if (f != f) return 0u;
  if (b == 0x80000000u) b = 0u;
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// round_half_even(m * 2^32), at most cap, of the value with order bits u; 0
// for NaN, zeros and negatives.  m = mant * 2^(e - 150) in whole numbers, so
// the product is a shift of the 24-bit mantissa (a subnormal m rounds to 0).
__device__ __forceinline__ int64_t q32(uint32_t u, int64_t cap) {
  const uint32_t b = (u & 0x80000000u) ? u ^ 0x80000000u : 0u;
  const int e = (int)(b >> 23);
  const uint32_t mant = e > 0 ? ((b & 0x7FFFFFu) | 0x800000u) : 0u;
  const int sh = e - 118;
  if (sh >= 0) {
    const uint64_t r = (uint64_t)mant << (sh < 39 ? sh : 39);   // 2^62 and more: past every cap
    return (int64_t)r > cap ? cap : (int64_t)r;
  }
  const int rs = -sh < 31 ? -sh : 31;
  const uint32_t q = mant >> rs, rem = mant & ((1u << rs) - 1u), half = 1u << (rs - 1);
  const int64_t r = q + ((rem > half || (rem == half && (q & 1u))) ? 1 : 0);
  return r > cap ? cap : r;
}

__device__ __forceinline__ bool in_text(int c, int lo, int hi) { return c >= lo && c <= hi; }

// Sums over the wave, returned to every lane: DPP moves within each row of 16
// lanes (no LDS round trips), then the four row sums on the scalar unit.
template <int CTRL>
__device__ __forceinline__ int dpp_int(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ int64_t dpp_plus_i64(int64_t v) {
  const uint32_t lo = (uint32_t)dpp_int<CTRL>((int)v), hi = (uint32_t)dpp_int<CTRL>((int)(v >> 32));
  return v + (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int64_t lane_i64(int64_t v, int lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), lane);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int wave_sum_i32(int v) {
  v += dpp_int<0xB1>(v);     // quad_perm [1,0,3,2]
  v += dpp_int<0x4E>(v);     // quad_perm [2,3,0,1]
  v += dpp_int<0x124>(v);    // row_ror:4
  v += dpp_int<0x128>(v);    // row_ror:8
  return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
         __builtin_amdgcn_readlane(v, 48);
}
__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
  v = dpp_plus_i64<0xB1>(v);
  v = dpp_plus_i64<0x4E>(v);
  v = dpp_plus_i64<0x124>(v);
  v = dpp_plus_i64<0x128>(v);
  return lane_i64(v, 0) + lane_i64(v, 16) + lane_i64(v, 32) + lane_i64(v, 48);
}

// A row's masses in registers: key r of lane l belongs to block 64 r + l and
// holds its order bits plus one, 0 past the row's end and the given key for a
// text block (0: never a candidate).
template <int R>
__device__ __forceinline__ void load_keys(const SelectParams& P, const float* w, int lane, uint32_t (&u)[R],
                                          uint32_t text_key = 0u) {
  float f[R];
#pragma unroll
  for (int r = 0; r < R; ++r) f[r] = r * 64 + lane < P.nb ? w[r * 64 + lane] : 0.f;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = r * 64 + lane;
    u[r] = i >= P.nb ? 0u : (in_text(i, P.text_lo, P.text_hi) ? text_key : float_order_bits(f[r]) + 1u);
  }
}

// The candidates kept by a count of n: those with key > thr, and of those
// with key == thr the `ties` of lowest index.
struct Cut {
  uint32_t thr;
  int ties;
};

// Number of keys of the row that reach c, the same in every lane.  The lanes
// count their own keys (a compare and an add with carry per key) and the sum
// goes over the wave once: with a ballot and a scalar population count per
// key instead, the scalar unit that the CU's waves share was the bound.
template <int R>
__device__ __forceinline__ int count_reaching(const uint32_t (&u)[R], uint32_t c) {
  int n = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) n += u[r] >= c ? 1 : 0;
  return wave_sum_i32(n);
}

// The cut that keeps n of the row's `all` candidates.  lo is a value that
// more than n keys reach, hi one that fewer do; once exactly n keys reach the
// value between them that is tried, every one of those is kept.  The keys of a
// row are spread about like a bell curve (they go by the logarithm of the
// masses), so the value is placed where the logits of the two counts, taken
// as linear in between, meet that of n, and every fourth time in the middle:
// 7.8 counts on average over rows of 1,724 blocks (18 at most), 6.7 of 862 and
// 4.0 of 32, where a search bit by bit took fifteen.
template <int R>
__device__ __forceinline__ Cut find_cut(const uint32_t (&u)[R], int n, int all) {
  if (n <= 0) return Cut{0xFFFFFFFFu, 0};
  if (n >= all) return Cut{0u, 0};
  uint32_t least = 0xFFFFFFFFu, most = 0u;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    least = min(least, u[r] - 1u);          // an empty key turns into the largest value
    most = max(most, u[r]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    least = min(least, (uint32_t)__shfl_xor((int)least, o, 64));
    most = max(most, (uint32_t)__shfl_xor((int)most, o, 64));
  }
  uint32_t lo = __builtin_amdgcn_readfirstlane(least) + 1u, hi = __builtin_amdgcn_readfirstlane(most) + 1u;
  auto logit = [&](int k) {                 // base 2, of k keys out of all
    return __builtin_amdgcn_logf((float)k + 0.5f) - __builtin_amdgcn_logf((float)(all - k) + 0.5f);
  };
  const float want = logit(n);
  int n_hi = 0;                             // keys that reach hi
  float g_lo = logit(all), g_hi = logit(0);
  for (int it = 0; hi - lo > 1u; ++it) {
    const uint32_t span = hi - lo;
    uint32_t d = span / 2u;
    if (it % 4 != 3)
      d = min(max((uint32_t)((float)span * (g_lo - want) * __builtin_amdgcn_rcpf(g_lo - g_hi)), 1u), span - 1u);
    const uint32_t c = __builtin_amdgcn_readfirstlane(lo + d);
    const int cnt = count_reaching<R>(u, c);
    if (cnt == n) return Cut{c - 1u, 0};
    if (cnt > n) {
      lo = c;
      g_lo = logit(cnt);
    } else {
      hi = c;
      n_hi = cnt;
      g_hi = logit(cnt);
    }
  }
  return Cut{lo, n - n_hi};                 // the keys equal to lo share the last places
}

// This lane's shares of the exact mass kept by each of N cuts, and of the
// row's total (text blocks in neither).  Tied blocks have equal masses, so
// which of them are kept does not matter here: lane 0 adds them.  While no
// sum of the row can reach 2^53 the sums are whole numbers in double
// precision, exact, at a third of the instructions of the 64-bit integers.
template <int R, int N>
__device__ __forceinline__ void mass_shares(const uint32_t (&u)[R], const Cut (&cut)[N], int64_t cap, int nb,
                                            int lane, int64_t (&kept)[N], int64_t& total) {
  uint32_t most = 0u;
#pragma unroll
  for (int r = 0; r < R; ++r) most = max(most, u[r]);
  // A key holds its mass's bits from 0x80000001 on; lower ones count nothing.
  const float lane_max = __uint_as_float(__builtin_elementwise_sub_sat(most, 0x80000001u));
  const double two32 = 4294967296.0, two53 = 9007199254740992.0;
  const double dcap = (double)cap < two53 ? (double)cap : two53;
  if (!__any((double)lane_max * two32 * (double)nb >= two53) || (double)cap * (double)nb < two53) {
    double t = 0.0, s[N];
#pragma unroll
    for (int j = 0; j < N; ++j) s[j] = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float m = __uint_as_float(__builtin_elementwise_sub_sat(u[r], 0x80000001u));
      double x = __builtin_rint((double)m * two32);          // half to even
      x = x < dcap ? x : dcap;
      t += x;
#pragma unroll
      for (int j = 0; j < N; ++j) s[j] += u[r] > cut[j].thr ? x : 0.0;
    }
    total = (int64_t)t;
#pragma unroll
    for (int j = 0; j < N; ++j) kept[j] = (int64_t)s[j];
  } else {
    total = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) kept[j] = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t q = u[r] > 0u ? q32(u[r] - 1u, cap) : 0;
      total += q;
#pragma unroll
      for (int j = 0; j < N; ++j) kept[j] += u[r] > cut[j].thr ? q : 0;
    }
  }
#pragma unroll
  for (int j = 0; j < N; ++j)
    if (lane == 0 && cut[j].ties > 0) kept[j] += (int64_t)cut[j].ties * q32(cut[j].thr - 1u, cap);
}

// The text blocks' exact mass of a row, this lane's share.
__device__ __forceinline__ int64_t text_share(const SelectParams& P, const float* w, int lane) {
  int64_t s = 0;
  for (int i = P.text_lo + lane; i <= P.text_hi; i += 64) s += q32(float_order_bits(w[i]), P.cap);
  return s;
}

__device__ __forceinline__ int n_text(const SelectParams& P) {
  return P.text_lo <= P.text_hi ? P.text_hi - P.text_lo + 1 : 0;
}

// Entries of head h when its video rows keep k blocks each.
__device__ __forceinline__ int head_entries(const SelectParams& P, int k) {
  const int nt = n_text(P);
  return nt * P.nb + (P.nb - nt) * k;
}

// Writes a row's kept indices, ascending, from out on, and its row_ptr entry
// (the last row also the end).
template <int R>
__device__ __forceinline__ void emit_row(const SelectParams& P, int row, int k, int head_start, Cut cut,
                                         const uint32_t (&u)[R], int lane) {
  const int nb = P.nb, p = row % nb, nt = n_text(P);
  int text_before = 0;
  if (nt > 0) {
    const int hi = min(p, P.text_hi + 1);
    text_before = hi > P.text_lo ? hi - P.text_lo : 0;
  }
  const bool full = in_text(p, P.text_lo, P.text_hi);
  const int start = head_start + text_before * nb + (p - text_before) * k;
  if (lane == 0) {
    P.row_ptr[row] = start;
    if (row == P.batch_heads * nb - 1) P.row_ptr[row + 1] = start + (full ? nb : k);
  }
  int32_t* out = P.col_idx + start;
  if (full) {
    for (int i = lane; i < nb; i += 64) out[i] = i;
    return;
  }
  const uint64_t below = (1ull << lane) - 1ull;
  int pos = 0, ties = cut.ties;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (r * 64 >= nb) break;
    const int i = r * 64 + lane;
    const bool text = in_text(i, P.text_lo, P.text_hi);
    bool keep = text || u[r] > cut.thr;
    if (ties > 0) {
      const bool eq = !text && u[r] == cut.thr;
      const uint64_t m = __ballot(eq);
      keep = keep || (eq && __builtin_popcountll(m & below) < ties);
      ties -= min(ties, (int)__builtin_popcountll(m));
    }
    const uint64_t m = __ballot(keep);
    if (keep) out[pos + __builtin_popcountll(m & below)] = i;
    pos += __builtin_popcountll(m);
  }
}

// TOPK: the counts are known, so one pass over the masses finds each row's
// kept blocks, writes them, and leaves the row's kept and total mass for the
// head's Recall.  One wave per row.
template <int R>
__global__ __launch_bounds__(SEL_NT) void select_topk_kernel(SelectParams P) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * SEL_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = P.nb;
  if (row >= P.batch_heads * nb) return;
  const int bh = row / nb, p = row % nb, hh = bh % P.heads;
  const float* w = P.w + (size_t)row * nb;
  uint32_t u[R];
  load_keys<R>(P, w, lane, u);
  const int k = P.head_param[hh];
  int before = 0, batch = 0;       // entries of this batch element's earlier heads, and of all its heads
  for (int h = lane; h < P.heads; h += 64) {
    const int e = head_entries(P, P.head_param[h]);
    batch += e;
    before += h < hh ? e : 0;
  }
  const int start = (int)wave_sum_i64((int64_t)(bh / P.heads) * batch + before);
  const Cut cut = in_text(p, P.text_lo, P.text_hi) ? Cut{0u, 0} : find_cut<R>(u, k - n_text(P), nb - n_text(P));
  emit_row<R>(P, row, k, start, cut, u, lane);
  const int64_t ts = text_share(P, w, lane);
  const Cut cuts[1] = {cut};
  int64_t kept[1], total;
  mass_shares<R, 1>(u, cuts, P.cap, nb, lane, kept, total);
  kept[0] = wave_sum_i64(kept[0] + ts);
  total = wave_sum_i64(total + ts);
  if (lane == 0) {
    P.ws_sums[(size_t)row * 2] = kept[0];
    P.ws_sums[(size_t)row * 2 + 1] = total;
  }
}

// HIERARCHICAL: the mass kept at the three possible counts and the total mass
// of a workgroup's four rows (which head gets which count is decided from
// their sums).
template <int R>
__global__ __launch_bounds__(SEL_NT) void select_levels_kernel(SelectParams P) {
  __shared__ int64_t sums[SEL_WAVES][4];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = P.nb, bh = blockIdx.y, p = blockIdx.x * SEL_WAVES + wave;
  int64_t kept[3] = {0, 0, 0}, total = 0;
  if (p < nb) {
    const float* w = P.w + ((size_t)bh * nb + p) * nb;
    uint32_t u[R];
    load_keys<R>(P, w, lane, u);
    const int64_t ts = text_share(P, w, lane);
    const bool full = in_text(p, P.text_lo, P.text_hi);
    const int ks[3] = {P.k_base, P.k_hi, P.k_lo};
    Cut cuts[3];
#pragma unroll
    for (int j = 0; j < 3; ++j)
      cuts[j] = full ? Cut{0u, 0} : find_cut<R>(u, ks[j] - n_text(P), nb - n_text(P));
    mass_shares<R, 3>(u, cuts, P.cap, nb, lane, kept, total);
#pragma unroll
    for (int j = 0; j < 3; ++j) kept[j] = wave_sum_i64(kept[j] + ts);
    total = wave_sum_i64(total + ts);
  }
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < 3; ++j) sums[wave][j] = kept[j];
    sums[wave][3] = total;
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    int64_t v = 0;
#pragma unroll
    for (int i = 0; i < SEL_WAVES; ++i) v += sums[i][threadIdx.x];
    P.ws_sums[((size_t)bh * gridDim.x + blockIdx.x) * 4 + threadIdx.x] = v;
  }
}

// COVERAGE and HIERARCHICAL, once the counts are known: the kept blocks.
template <int R>
__global__ __launch_bounds__(SEL_NT) void select_emit_kernel(SelectParams P) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * SEL_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = P.nb;
  if (row >= P.batch_heads * nb) return;
  const int bh = row / nb, p = row % nb;
  uint32_t u[R];
  load_keys<R>(P, P.w + (size_t)row * nb, lane, u);
  const int k = P.ws_headk[bh];
  int start;
  if (P.base_ready) {
    start = P.ws_base[bh];
  } else {
    int before = 0;
    for (int h = lane; h < bh; h += 64) before += head_entries(P, P.ws_headk[h]);
    start = (int)wave_sum_i64(before);
  }
  const Cut cut = in_text(p, P.text_lo, P.text_hi) ? Cut{0u, 0} : find_cut<R>(u, k - n_text(P), nb - n_text(P));
  emit_row<R>(P, row, k, start, cut, u, lane);
}

// Lane l ^ X's value.
template <int X>
__device__ __forceinline__ uint32_t from_xor(uint32_t v) {
  auto dpp = [](uint32_t x, auto ctrl) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, 0xF, 0xF, false);
  };
  if constexpr (X == 1) return dpp(v, std::integral_constant<int, 0xB1>{});          // quad_perm [1,0,3,2]
  else if constexpr (X == 2) return dpp(v, std::integral_constant<int, 0x4E>{});     // quad_perm [2,3,0,1]
  else if constexpr (X == 3) return dpp(v, std::integral_constant<int, 0x1B>{});     // quad_perm [3,2,1,0]
  else if constexpr (X == 7) return dpp(v, std::integral_constant<int, 0x141>{});    // row_half_mirror
  else if constexpr (X == 4) return from_xor<3>(from_xor<7>(v));
  else if constexpr (X == 8) return dpp(v, std::integral_constant<int, 0x128>{});    // row_ror:8
  else if constexpr (X == 15) return dpp(v, std::integral_constant<int, 0x140>{});   // row_mirror
  else if constexpr (X == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return (threadIdx.x & 16) ? r[0] : r[1];
  } else if constexpr (X == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (threadIdx.x & 32) ? r[0] : r[1];
  } else if constexpr (X == 31) return from_xor<16>(from_xor<15>(v));
  else return from_xor<32>(from_xor<31>(v));                                         // 63
}

// Sorts the wave's 64 R keys in descending order, key r of lane l being
// number l R + r: the bitonic network whose merges begin by comparing with
// the mirrored position, so every comparison keeps the larger key first and
// the strides below R stay inside a lane (two instructions per pair).
template <int R, int J>
__device__ __forceinline__ void lane_strides(uint32_t (&u)[R]) {
  if constexpr (J > 0) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if ((r & J) == 0) {
        const uint32_t a = u[r], b = u[r + J];
        u[r] = max(a, b);
        u[r + J] = min(a, b);
      }
    lane_strides<R, J / 2>(u);
  }
}
template <int R, int X>
__device__ __forceinline__ void wave_strides(uint32_t (&u)[R], int lane) {
  if constexpr (X > 0) {
    const bool high = (lane & X) != 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t v = from_xor<X>(u[r]);
      u[r] = ((v > u[r]) != high) ? v : u[r];
    }
    wave_strides<R, X / 2>(u, lane);
  }
}
template <int R, int K>
__device__ __forceinline__ void merges_in_lane(uint32_t (&u)[R]) {    // runs of K <= R keys
  if constexpr (K <= R) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if ((r & (K / 2)) == 0) {
        const int s = r ^ (K - 1);
        const uint32_t a = u[r], b = u[s];
        u[r] = max(a, b);
        u[s] = min(a, b);
      }
    lane_strides<R, K / 4>(u);
    merges_in_lane<R, K * 2>(u);
  }
}
template <int R, int X>
__device__ __forceinline__ void merges_in_wave(uint32_t (&u)[R], int lane) {   // runs of X lanes
  if constexpr (X <= 64) {
    const bool high = (lane & (X / 2)) != 0;
    uint32_t m[R];
#pragma unroll
    for (int r = 0; r < R; ++r) m[r] = from_xor<X - 1>(u[R - 1 - r]);
#pragma unroll
    for (int r = 0; r < R; ++r) u[r] = ((m[r] > u[r]) != high) ? m[r] : u[r];
    wave_strides<R, X / 4>(u, lane);
    lane_strides<R, R / 2>(u);
    merges_in_wave<R, X * 2>(u, lane);
  }
}

// COVERAGE: kept(k) summed over a workgroup's rows for every k.  Each wave
// sorts its rows' keys in registers, one row after another, and adds their
// running exact sums in registers; the waves' sums meet in LDS (integers, so
// in any order) and go out as one partial curve per workgroup.  A text query
// row keeps everything: its total counts at every k.  Text blocks come first
// (the key above every mass) and their mass is in every running sum, which
// is then right from k = #text on, the smallest count in use.
template <int R>
__global__ __launch_bounds__(SEL_NT) void select_curve_kernel(SelectParams P) {
  __shared__ unsigned long long part[64 * R];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = P.nb, bh = blockIdx.y;
  for (int i = threadIdx.x; i < nb; i += SEL_NT) part[i] = 0ull;
  __syncthreads();
  int64_t acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0;
  auto q_of = [&](uint32_t k) -> int64_t {
    return k == 0u || k == 0xFFFFFFFFu ? 0 : q32(k - 1u, P.cap);
  };
  const int p0 = blockIdx.x * P.rows_per_wg;
  const int p1 = min(nb, p0 + P.rows_per_wg);
  for (int p = p0 + wave; p < p1; p += SEL_WAVES) {
    const float* w = P.w + ((size_t)bh * nb + p) * nb;
    uint32_t u[R];
    load_keys<R>(P, w, lane, u, 0xFFFFFFFFu);
    const bool full = in_text(p, P.text_lo, P.text_hi);
    int64_t before = text_share(P, w, lane);
    if (full) {
#pragma unroll
      for (int r = 0; r < R; ++r) before += q_of(u[r]);
    }
    before = wave_sum_i64(before);
    if (full) {
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] += before;
      continue;
    }
    merges_in_lane<R, 2>(u);
    merges_in_wave<R, 2>(u, lane);
    int64_t s = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      s += q_of(u[r]);
      asm volatile("" : "+v"(u[r]));      // taken again below: 2 R registers less than keeping it
    }
    int64_t incl = s;                     // inclusive scan over the lanes
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t v = __shfl_up((long long)incl, o, 64);
      if (lane >= o) incl += v;
    }
    int64_t run = before + incl - s;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      run += q_of(u[r]);
      acc[r] += run;
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (lane * R + r < nb) atomicAdd(&part[lane * R + r], (unsigned long long)acc[r]);
  __syncthreads();
  int64_t* out = P.ws_sums + ((size_t)bh * gridDim.x + blockIdx.x) * nb;
  for (int i = threadIdx.x; i < nb; i += SEL_NT) out[i] = (int64_t)part[i];
}

// The same for rows of more than 2,048 blocks, whose keys do not fit a wave's
// registers beside the sums: a workgroup sorts one row after another in LDS
// (n keys, the power of two that holds nb), thread t keeping the sums of
// positions [t PER, (t + 1) PER).
template <int PER>
__global__ __launch_bounds__(SEL_NT) void select_curve_long_kernel(SelectParams P) {
  constexpr int n = PER * SEL_NT;
  __shared__ uint32_t keys[n];
  __shared__ int64_t scan[SEL_NT];
  const int tid = threadIdx.x, nb = P.nb, bh = blockIdx.y;
  int64_t acc[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r) acc[r] = 0;
  auto block_inclusive = [&](int64_t v) {
    scan[tid] = v;
    __syncthreads();
    for (int off = 1; off < SEL_NT; off <<= 1) {
      const int64_t add = tid >= off ? scan[tid - off] : 0;
      __syncthreads();
      scan[tid] += add;
      __syncthreads();
    }
    return scan[tid];
  };
  const int p1 = min(nb, (int)(blockIdx.x + 1) * P.rows_per_wg);
  for (int p = blockIdx.x * P.rows_per_wg; p < p1; ++p) {
    const float* w = P.w + ((size_t)bh * nb + p) * nb;
    const bool full = in_text(p, P.text_lo, P.text_hi);
    int64_t first = 0;                    // counted at every k
    for (int i = tid; i < n; i += SEL_NT) {
      uint32_t u = 0u;
      if (i < nb) {
        const uint32_t b = float_order_bits(w[i]);
        const bool text = in_text(i, P.text_lo, P.text_hi);
        if (text || full) first += q32(b, P.cap);
        u = text ? 0xFFFFFFFFu : b + 1u;
      }
      keys[i] = u;
    }
    __syncthreads();
    block_inclusive(first);
    const int64_t before = scan[SEL_NT - 1];
    __syncthreads();
    if (full) {
#pragma unroll
      for (int r = 0; r < PER; ++r) acc[r] += before;
      continue;
    }
    // Bitonic sort, descending.  Each stage visits its n / 2 compare-exchange
    // pairs (i, i + j) directly: i has bit j clear.
    for (int k = 2; k <= n; k <<= 1) {
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int pr = tid; pr < (n >> 1); pr += SEL_NT) {
          const int i = ((pr & ~(j - 1)) << 1) | (pr & (j - 1));
          const uint32_t x = keys[i], y = keys[i + j];
          if ((i & k) == 0 ? (x < y) : (x > y)) {
            keys[i] = y;
            keys[i + j] = x;
          }
        }
        __syncthreads();
      }
    }
    int64_t s = 0;
    for (int r = 0; r < PER; ++r) {
      const uint32_t u = keys[tid * PER + r];
      s += (u == 0u || u == 0xFFFFFFFFu) ? 0 : q32(u - 1u, P.cap);
    }
    int64_t run = before + block_inclusive(s) - s;
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const uint32_t u = keys[tid * PER + r];
      run += (u == 0u || u == 0xFFFFFFFFu) ? 0 : q32(u - 1u, P.cap);
      acc[r] += run;
    }
    __syncthreads();
  }
  int64_t* out = P.ws_sums + ((size_t)bh * gridDim.x + blockIdx.x) * nb;
#pragma unroll
  for (int r = 0; r < PER; ++r)
    if (tid * PER + r < nb) out[tid * PER + r] = acc[r];
}

__device__ __forceinline__ float recall_of(int64_t kept, int64_t total) {
  return total == 0 ? 1.f : (float)((double)kept / (double)total);
}

// TOPK: each head's Recall from its rows' sums (one workgroup per head).
__global__ __launch_bounds__(SEL_NT) void select_recall_kernel(SelectParams P) {
  __shared__ int64_t sk[SEL_WAVES], st[SEL_WAVES];
  const int bh = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t* s = P.ws_sums + (size_t)bh * P.nb * 2;
  int64_t kept = 0, total = 0;
  for (int i = threadIdx.x; i < P.nb; i += SEL_NT) {
    kept += s[2 * i];
    total += s[2 * i + 1];
  }
  kept = wave_sum_i64(kept);
  total = wave_sum_i64(total);
  if (lane == 0) {
    sk[wave] = kept;
    st[wave] = total;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < SEL_WAVES; ++i) {
      kept += sk[i];
      total += st[i];
    }
    if (P.head_k_out) P.head_k_out[bh] = P.head_param[bh % P.heads];
    if (P.head_recall_out) P.head_recall_out[bh] = recall_of(kept, total);
  }
}

// COVERAGE: the partial curves of each head added up over 64 positions per
// workgroup, into the first of them (its positions are read by the workgroup
// that writes them, before it does).
constexpr int kSumPositions = 64;
__global__ __launch_bounds__(SEL_NT) void select_curve_sum_kernel(SelectParams P) {
  __shared__ int64_t part[SEL_WAVES][kSumPositions];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = blockIdx.x * kSumPositions + lane, nb = P.nb;
  int64_t* s = P.ws_sums + (size_t)blockIdx.y * P.n_parts * nb;
  int64_t v = 0;
  if (i < nb) {
#pragma unroll 8
    for (int c = wave; c < P.n_parts; c += SEL_WAVES) v += s[(size_t)c * nb + i];
  }
  part[wave][lane] = v;
  __syncthreads();
  if (wave == 0 && i < nb) {
#pragma unroll
    for (int j = 1; j < SEL_WAVES; ++j) v += part[j][lane];
    s[i] = v;
  }
}

// COVERAGE: the head's curve from the partial curves, and the smallest count
// whose kept share reaches the target (one workgroup per head).
constexpr int SEL_HEAD_NT = 1024;
__global__ __launch_bounds__(SEL_HEAD_NT) void select_coverage_kernel(SelectParams P) {
  __shared__ unsigned long long cv[kMaxBlocks];
  const int bh = blockIdx.x, nb = P.nb;
  const int64_t* s = P.ws_sums + (size_t)bh * P.n_parts * nb;
  const int n_parts = P.summed ? 1 : P.n_parts;
  // Where a head has fewer positions than threads, the partial curves are
  // dealt out over the spare ones.
  const int cols = (nb + 63) / 64 * 64, groups = cols < SEL_HEAD_NT ? SEL_HEAD_NT / cols : 1;
  for (int i = threadIdx.x; i < nb; i += SEL_HEAD_NT) cv[i] = 0ull;
  __syncthreads();
  const int g = groups > 1 ? (int)threadIdx.x / cols : 0;
  if (g < groups)
    for (int i = (int)threadIdx.x - g * cols; i < nb; i += SEL_HEAD_NT) {
      int64_t v = 0;
#pragma unroll 8
      for (int c = g; c < n_parts; c += groups) v += s[(size_t)c * nb + i];
      atomicAdd(&cv[i], (unsigned long long)v);
    }
  __syncthreads();
  if (threadIdx.x != 0) return;
  const int64_t total = (int64_t)cv[nb - 1];
  const unsigned __int128 need = (unsigned __int128)(uint64_t)total * (uint64_t)P.head_param[bh % P.heads];
  int lo = P.kmin, hi = nb;       // smallest k in [lo, hi] with kept(k)*10000 >= need
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    const unsigned __int128 have = (unsigned __int128)cv[mid - 1] * 10000u;
    if (have >= need) hi = mid; else lo = mid + 1;
  }
  P.ws_headk[bh] = lo;
  if (P.head_k_out) P.head_k_out[bh] = lo;
  if (P.head_recall_out) P.head_recall_out[bh] = recall_of((int64_t)cv[lo - 1], total);
}

// HIERARCHICAL (one workgroup per batch element): the heads' sums, then each
// head's count from the rank of its Recall at the base count among the heads
// (a head with no mass has Recall 1; ranks compare kept/total exactly).
__global__ __launch_bounds__(SEL_HEAD_NT) void select_hierarchy_kernel(SelectParams P) {
  __shared__ unsigned long long sum[kMaxHeads][4];      // kept at k_base, k_hi, k_lo, total
  __shared__ int rank_of[kMaxHeads], n_above;
  const int b = blockIdx.x, H = P.heads, lane = threadIdx.x & 63;
  for (int i = threadIdx.x; i < 4 * H; i += SEL_HEAD_NT) sum[i >> 2][i & 3] = 0ull;
  for (int i = threadIdx.x; i < H; i += SEL_HEAD_NT) rank_of[i] = 0;
  if (threadIdx.x == 0) n_above = 0;
  __syncthreads();
  // A wave adds up 64 of a head's groups of rows at a time.
  const int per = (P.n_parts + 63) / 64;
  for (int t = threadIdx.x >> 6; t < H * per; t += SEL_HEAD_NT / 64) {
    const int h = t / per, g = (t % per) * 64 + lane;
    int64_t v[4] = {0, 0, 0, 0};
    if (g < P.n_parts) {
      const int64_t* s = P.ws_sums + ((size_t)(b * H + h) * P.n_parts + g) * 4;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = s[j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = wave_sum_i64(v[j]);
    if (lane == 0)
#pragma unroll
      for (int j = 0; j < 4; ++j) atomicAdd(&sum[h][j], (unsigned long long)v[j]);
  }
  __syncthreads();
  // The rank of every head: each pair of heads compared by its own thread.
  for (int t = threadIdx.x; t < H * H; t += SEL_HEAD_NT) {
    const int hh = t / H, h2 = t % H;
    uint64_t ka = sum[hh][0], ta = sum[hh][3], k2 = sum[h2][0], t2 = sum[h2][3];
    if (ta == 0) { ka = 1; ta = 1; }
    if (t2 == 0) { k2 = 1; t2 = 1; }
    const unsigned __int128 lhs = (unsigned __int128)k2 * ta, rhs = (unsigned __int128)ka * t2;
    if (lhs > rhs || (lhs == rhs && h2 < hh)) atomicAdd(&rank_of[hh], 1);
    if (hh == 0 && (unsigned __int128)k2 * 10000u > (unsigned __int128)t2 * (uint64_t)P.recall_thr_bp)
      atomicAdd(&n_above, 1);
  }
  __syncthreads();
  for (int hh = threadIdx.x; hh < H; hh += SEL_HEAD_NT) {
    const int64_t total = (int64_t)sum[hh][3];
    const int rank = rank_of[hh];
    const int n = n_above < H / 2 ? n_above : H / 2;
    const int level = rank < n ? 1 : (rank >= H - n ? 2 : 0);
    const int k = level == 1 ? P.k_hi : (level == 2 ? P.k_lo : P.k_base);
    const int bh = b * H + hh;
    P.ws_headk[bh] = k;
    if (P.head_k_out) P.head_k_out[bh] = k;
    if (P.head_recall_out) P.head_recall_out[bh] = recall_of((int64_t)sum[hh][level], total);
  }
}

// The first col_idx entry of every head, for more heads than each row's wave
// adds up by itself.
constexpr int kInlineHeads = 2048;
__global__ __launch_bounds__(64) void select_base_kernel(SelectParams P) {
  const int lane = threadIdx.x;
  int carry = 0;
  for (int b0 = 0; b0 < P.batch_heads; b0 += 64) {
    const int bh = b0 + lane;
    const int v = bh < P.batch_heads ? head_entries(P, P.ws_headk[bh]) : 0;
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int x = __shfl_up(incl, o, 64);
      if (lane >= o) incl += x;
    }
    if (bh < P.batch_heads) P.ws_base[bh] = carry + incl - v;
    carry += __shfl(incl, 63, 64);
  }
}

// One instantiation per number of keys a lane holds: a row takes the smallest
// that covers it, and its compares on the keys past its end are wasted.  The
// steps lie where the usual sequences need them (140, 862 and 1,724 blocks, 2,582
// and 5,164 of the longest clips: 3, 14, 27, 41 and 81 keys); in between up to
// half of the keys are empty (2,689 blocks, 43 keys, take 82), and from 82 on the
// registers leave two waves per SIMD, then one.
template <typename F>
static void with_keys_per_lane(int nb, F&& f) {
  const int need = (nb + 63) / 64;
  if (need <= 1) f(std::integral_constant<int, 1>{});
  else if (need <= 2) f(std::integral_constant<int, 2>{});
  else if (need <= 4) f(std::integral_constant<int, 4>{});
  else if (need <= 8) f(std::integral_constant<int, 8>{});
  else if (need <= 14) f(std::integral_constant<int, 14>{});
  else if (need <= 20) f(std::integral_constant<int, 20>{});
  else if (need <= 27) f(std::integral_constant<int, 27>{});
  else if (need <= 42) f(std::integral_constant<int, 42>{});
  else if (need <= 82) f(std::integral_constant<int, 82>{});
  else f(std::integral_constant<int, 128>{});
}

// Entries of a head's partial curves from which they are added up by a launch of
// their own, over the whole chip, instead of by the one workgroup that looks for
// the head's count (a whole selection, us, without and with that launch: 24,727
// entries, 313 blocks x 2 heads, 25.4 and 26.1; 31,500, 500 x 24, 68.1 and 67.3;
// 62,500, 500 x 3, 33.5 and 30.0; 743,000, 1,724 x 3, 235 and 154; 1.05 million,
// 2,049 x 1, 566 and 445).
constexpr int64_t kSumEntries = 30000;

hipError_t launch_select(SelectParams P, hipStream_t st) {
  const int rows = P.batch_heads * P.nb;
  const dim3 per_row((rows + SEL_WAVES - 1) / SEL_WAVES), nt(SEL_NT);
  P.base_ready = 0;
  if (P.mode == 0) {
    with_keys_per_lane(P.nb, [&](auto R) {
      hipLaunchKernelGGL((select_topk_kernel<decltype(R)::value>), per_row, nt, 0, st, P);
    });
    hipLaunchKernelGGL(select_recall_kernel, dim3(P.batch_heads), nt, 0, st, P);
    return hipGetLastError();
  }
  if (P.mode == 1) {
    P.rows_per_wg = select_rows_per_wg(rows, P.nb);
    P.n_parts = (P.nb + P.rows_per_wg - 1) / P.rows_per_wg;
    const dim3 grid(P.n_parts, P.batch_heads);
    const int need = (P.nb + 63) / 64;
    if (need <= 1) hipLaunchKernelGGL((select_curve_kernel<1>), grid, nt, 0, st, P);
    else if (need <= 2) hipLaunchKernelGGL((select_curve_kernel<2>), grid, nt, 0, st, P);
    else if (need <= 4) hipLaunchKernelGGL((select_curve_kernel<4>), grid, nt, 0, st, P);
    else if (need <= 8) hipLaunchKernelGGL((select_curve_kernel<8>), grid, nt, 0, st, P);
    else if (need <= 16) hipLaunchKernelGGL((select_curve_kernel<16>), grid, nt, 0, st, P);
    else if (need <= 32) hipLaunchKernelGGL((select_curve_kernel<32>), grid, nt, 0, st, P);
    else if (need <= 64) hipLaunchKernelGGL((select_curve_long_kernel<16>), grid, nt, 0, st, P);
    else hipLaunchKernelGGL((select_curve_long_kernel<32>), grid, nt, 0, st, P);
    P.summed = (int64_t)P.n_parts * P.nb >= kSumEntries;
    if (P.summed)
      hipLaunchKernelGGL(select_curve_sum_kernel, dim3((P.nb + kSumPositions - 1) / kSumPositions, P.batch_heads), nt,
                         0, st, P);
    hipLaunchKernelGGL(select_coverage_kernel, dim3(P.batch_heads), dim3(SEL_HEAD_NT), 0, st, P);
  } else {
    P.n_parts = (P.nb + SEL_WAVES - 1) / SEL_WAVES;
    with_keys_per_lane(P.nb, [&](auto R) {
      hipLaunchKernelGGL((select_levels_kernel<decltype(R)::value>), dim3(P.n_parts, P.batch_heads), nt, 0, st, P);
    });
    hipLaunchKernelGGL(select_hierarchy_kernel, dim3(P.batch_heads / P.heads), dim3(SEL_HEAD_NT), 0, st, P);
  }
  if (P.batch_heads > kInlineHeads) {
    hipLaunchKernelGGL(select_base_kernel, dim3(1), dim3(64), 0, st, P);
    P.base_ready = 1;
  }
  with_keys_per_lane(P.nb, [&](auto R) {
    hipLaunchKernelGGL((select_emit_kernel<decltype(R)::value>), per_row, nt, 0, st, P);
  });
  return hipGetLastError();
}

}  // namespace adaspa
