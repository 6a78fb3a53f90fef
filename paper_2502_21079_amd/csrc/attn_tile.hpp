// Tile-level building blocks shared by the attention and block-mass kernels
// (gfx950): bounds-checked global->LDS tile loads, the transposed-score MFMA
// tile, online-softmax pieces and the P V update.
//
// Orientation.  Scores are formed transposed, S^T[key][query] = K Q^T, with K
// as the MFMA A operand (read from LDS) and a 32-query Q fragment as the B
// operand (kept in registers).  In the 32x32 accumulator each lane then holds
// 16 keys of ONE query, so the softmax row statistics are lane-local plus one
// exchange between the two half-waves.  The probabilities P^T are already laid
// out as the B operand of the second product O^T[d][query] += V^T P^T, once
// the 16 keys of each MFMA step are ordered to match the accumulator rows; the
// V^T operand is read from a row-major V tile with the LDS transpose read.
//
// Online softmax.  Probabilities are taken against a per-row reference that
// moves only when a row's running sum grows too large, so neither a per-tile
// maximum nor a rescale of the output accumulator is needed for almost every
// tile; the final normalisation uses the same reference, so the result is
// unchanged.  The running sums are formed on the matrix pipe (RowSums).
#pragma once

#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace adaspa {

constexpr int KT = 64;          // keys per tile

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}

// Buffer resource words (base, stride 0, size in bytes, the format word of
// make_rsrc) in scalar registers, for the loads issued by dma16.
__device__ __forceinline__ u32x4 rsrc_words(const void* base, uint32_t bytes) {
  const uint64_t b = (uint64_t)base;
  u32x4 r;
  r.x = __builtin_amdgcn_readfirstlane((uint32_t)b);
  r.y = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  r.z = __builtin_amdgcn_readfirstlane(bytes);
  r.w = 0x00020000u;
  return r;
}

// One 16-byte-per-lane direct load into LDS: lane l's 16 bytes at voff +
// soff of the buffer go to LDS byte lds + OFS + 16 l.  It is issued as inline
// asm so that the compiler does not track it: otherwise it makes every later
// LDS read wait for the load (vmcnt) unless it can prove the two touch
// different addresses, which it cannot for the ring slots.  The ordering is
// explicit instead: a loaded tile is read only after a vmcnt(0) wait and a
// barrier, and a slot is refilled only after the barrier that follows its
// last read.  M0 carries the LDS address; the compiler sets M0 itself before
// each of its own uses, so clobbering it here is harmless.  The add that
// forms M0 also sets SCC, which is declared clobbered too (a compare whose
// result the compiler kept in SCC across the load would otherwise be lost).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int OFS>
__device__ __forceinline__ void dma16(u32x4 rsrc, uint32_t lds, uint32_t voff, uint32_t soff) {
  asm volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff), "n"(OFS) : "m0", "scc");
}
#pragma clang diagnostic pop

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(size_t)(const __attribute__((address_space(3))) void*)p;
}

// One [KEYS, D] bf16 tile in LDS, its rows back to back and the 16-byte chunks
// of a row in an order of the row's own: chunk c of row r sits at place
// c ^ swz(r).  So 16 consecutive rows of a K tile read at one column fall in
// distinct banks, and so do the four rows of 64 bytes that 32 lanes of a
// transposed read of a V tile take; and a lane's operand addresses differ in
// compile-time offsets and one exclusive or per column (k_lane, v_lane).  The
// loads write LDS in lane order, so the order is made by what each lane loads.
// (Rows padded by one and two chunks instead took 19 load instructions per
// pair of tiles where these take 16 at d 64, and 35 for 32 at d 128.)
enum { K_TILE = 1, V_TILE = 2 };
template <int D, int NW, int KIND, int KEYS = KT>
struct TileDMA {
  static constexpr int CPR = D / 8;                 // chunks per row
  static constexpr int RPI = 64 / CPR;              // rows per 64-lane instruction
  static constexpr int NINST = KEYS / RPI;
  static constexpr int SLOTS = KEYS * CPR;          // chunks per tile
  static constexpr int ELEMS = KEYS * D;            // bf16 elements per tile

  __device__ __forceinline__ static int swz(int row) {
    if (KIND == K_TILE) return D == 64 ? (row >> 1) & 7 : row & 15;
    return D == 64 ? ((row >> 1) & 1) << 2 : (row & 3) << 2;
  }
  // Chunk of its row that slot p of the tile holds.
  __device__ __forceinline__ static int chunk_of(int p) { return (p % CPR) ^ swz(p / CPR); }

  // Issue the loads of rows [kbase, kbase + KEYS).  Rows past the buffer's end
  // are skipped by its bounds check: the slot keeps what it held.
  __device__ __forceinline__ static void issue(__amdgpu_buffer_rsrc_t r, u16* dst, int kbase,
                                               int wave, int lane) {
#pragma unroll
    for (int i0 = 0; i0 < NINST; i0 += NW) {
      const int i = i0 + wave;
      if (i < NINST) {
        const int p = i * 64 + lane;
        const uint32_t off = (uint32_t)((kbase + p / CPR) * D + chunk_of(p) * 8) * 2u;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(dst + i * 64 * 8), 16, off, 0, 0, 0);
      }
    }
  }

  // Issue the loads of a dual tile: rows [0, 32) from keys [ka, ka + 32),
  // rows [32, 64) from keys [kb, kb + 32) (both inside the sequence).
  __device__ __forceinline__ static void issue_dual(__amdgpu_buffer_rsrc_t r, u16* dst, int ka, int kb,
                                                    int wave, int lane) {
#pragma unroll
    for (int i0 = 0; i0 < NINST; i0 += NW) {
      const int i = i0 + wave;
      if (i < NINST) {
        const int p = i * 64 + lane, row = p / CPR;
        const int key = row < 32 ? ka + row : kb + (row - 32);
        const uint32_t off = (uint32_t)(key * D + chunk_of(p) * 8) * 2u;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(dst + i * 64 * 8), 16, off, 0, 0, 0);
      }
    }
  }

  // Byte offset, inside a tile that lies whole in the sequence, of the chunk
  // that slot i * 64 + lane holds.
  __device__ __forceinline__ static uint32_t rel_offset(int i, int lane) {
    const int p = i * 64 + lane;
    return (uint32_t)(p / CPR * D + chunk_of(p) * 8) * 2u;
  }
};
using std::integral_constant;

// A lane's K operand address in a tile, in elements: row c32, chunk hw; its
// chunk 2 ks + hw of row 32 g + c32 is at (k_lane ^ 16 ks) + 32 g D.
template <int D>
__device__ __forceinline__ int k_lane(int c32, int hw) {
  return c32 * D + (hw ^ TileDMA<D, 1, K_TILE>::swz(c32)) * 8;
}
// A lane's transposed V read: row 4 hw + gi / 4, elements 16 (grp & 1) +
// 4 (gi & 3); output block d of row r further down is at (v_lane ^ 32 d) + r D
// (r a multiple of 8).
template <int D>
__device__ __forceinline__ int v_lane(int gi, int grp, int hw) {
  const int row = 4 * hw + (gi >> 2);
  const int chunk = (2 * (grp & 1) + ((gi & 3) >> 1)) ^ TileDMA<D, 1, V_TILE>::swz(row);
  return row * D + chunk * 8 + 4 * (gi & 1);
}

// Loads of one full K tile per step (the block-mass pass), uniform over the
// waves: wave w issues the tile's DMA instructions j * NW + w, j = 0 .. PW-1.
// Their in-tile offsets differ by whole periods of the row order, so one
// register holds them all and the rest goes into the scalar offset.
template <int D, int NW>
struct KLoader {
  using K = TileDMA<D, NW, K_TILE>;
  static constexpr int PW = K::NINST / NW;
  static constexpr int STEP = K::RPI * NW * D * 2;     // source bytes between a wave's loads
  static_assert(K::NINST % NW == 0 && K::RPI * NW % 16 == 0, "every wave loads alike, whole periods apart");
  uint32_t rel;              // per lane: in-tile source offset of load 0
  uint32_t wbase;            // LDS byte offset of this wave's piece of load 0

  __device__ __forceinline__ void init(int wave, int lane) {
    wbase = (uint32_t)wave * 1024u;
    rel = K::rel_offset(wave, lane);
  }
  // Load n (a constant once the caller's loop is unrolled) of the tile whose
  // first byte is kbyte into the tile at LDS byte address tile.
  template <int J = 0>
  __device__ __forceinline__ void issue_n(int n, uint32_t tile, u32x4 rK, uint32_t kbyte) const {
    if constexpr (J < PW) {
      if (n == J) dma16<J * NW * 1024>(rK, tile + wbase, rel, kbyte + J * STEP);
      else issue_n<J + 1>(n, tile, rK, kbyte);
    }
  }
};

// Loads of one full K tile and one full V tile per step into one ring slot
// laid out [K tile | V tile].  Wave w issues instructions j * NW + w of the K
// tile (j < PWK), then those of the V tile, each filling a 1 KB piece of the
// slot.  The source of a load is the tile's first byte and a constant (scalar
// offset) plus a per-lane in-tile offset in a register, and its destination
// the slot plus a per-wave constant.
template <int D, int NW, int KEYS = KT>
struct KVLoader {
  using K = TileDMA<D, NW, K_TILE, KEYS>;
  using V = TileDMA<D, NW, V_TILE, KEYS>;
  static constexpr int PWK = K::NINST / NW;                 // loads per wave, tile and step
  static constexpr int PW = 2 * PWK;
  static constexpr int ELEMS = K::ELEMS + V::ELEMS;         // bf16 elements per ring slot
  static constexpr int VOFF = K::ELEMS;                     // V tile within the slot
  static constexpr int ROWS = K::RPI * NW;                  // rows between a wave's loads
  static constexpr int NP = ROWS % 16 == 0 ? 1 : 16 / ROWS; // loads until the K rows' order repeats
  static_assert(K::NINST % NW == 0 && ROWS % 4 == 0 && 16 % (NP * ROWS < 16 ? NP * ROWS : 16) == 0,
                "every wave loads alike, whole periods of the row orders apart");
  static constexpr uint32_t row_bytes(int rows) { return (uint32_t)rows * D * 2u; }

  uint32_t relK[NP], relV;   // per lane: in-tile source offsets, without their row of load j
  uint32_t wbase;            // LDS byte offset of this wave's piece of entry j = 0

  __device__ __forceinline__ void init(int wave, int lane) {
    wbase = (uint32_t)wave * 1024u;
#pragma unroll
    for (int j = 0; j < NP; ++j) relK[j] = K::rel_offset(j * NW + wave, lane) - row_bytes(j * ROWS);
    relV = V::rel_offset(wave, lane);
  }
  // Load J of this wave into the slot at LDS byte address slot; kbyte / vbyte
  // are the first bytes of the K and the V tile.
  template <int J>
  __device__ __forceinline__ void issue(uint32_t slot, u32x4 rK, u32x4 rV, uint32_t kbyte, uint32_t vbyte) const {
    constexpr int F = J * NW * 1024;
    if constexpr (J < PWK) dma16<F>(rK, slot + wbase, relK[J % NP], kbyte + row_bytes(J * ROWS));
    else dma16<F>(rV, slot + wbase, relV, vbyte + row_bytes((J - PWK) * ROWS));
  }
  // Load n (a constant once the caller's loop is unrolled).
  template <int J = 0>
  __device__ __forceinline__ void issue_n(int n, uint32_t slot, u32x4 rK, u32x4 rV, uint32_t kbyte,
                                          uint32_t vbyte) const {
    if constexpr (J < PW) {
      if (n == J) issue<J>(slot, rK, rV, kbyte, vbyte);
      else issue_n<J + 1>(n, slot, rK, rV, kbyte, vbyte);
    }
  }

  // Dual slots: rows [0, 32) of the K and V tiles come from one 32-key half
  // tile, rows [32, 64) from another; ka / va are the first bytes of the first
  // half's K / V keys, kb / vb those of the second's.  All rows of a load
  // belong to one half.
  template <int J>
  __device__ __forceinline__ void issue_dual(uint32_t slot, u32x4 rK, u32x4 rV, uint32_t ka, uint32_t kb,
                                             uint32_t va, uint32_t vb) const {
    constexpr int F = J * NW * 1024, ROW = (J < PWK ? J : J - PWK) * ROWS;
    static_assert(32 % ROWS == 0, "a load lies in one half");
    if constexpr (J < PWK) dma16<F>(rK, slot + wbase, relK[J % NP], (ROW < 32 ? ka : kb) + row_bytes(ROW % 32));
    else dma16<F>(rV, slot + wbase, relV, (ROW < 32 ? va : vb) + row_bytes(ROW % 32));
  }
  template <int J = 0>
  __device__ __forceinline__ void issue_dual_n(int n, uint32_t slot, u32x4 rK, u32x4 rV, uint32_t ka,
                                               uint32_t kb, uint32_t va, uint32_t vb) const {
    if constexpr (J < PW) {
      if (n == J) issue_dual<J>(slot, rK, rV, ka, kb, va, vb);
      else issue_dual_n<J + 1>(n, slot, rK, rV, ka, kb, va, vb);
    }
  }
};

// The K or V part of the ring slots: part[b] is the tile in slot b.
template <int ELEMS, int OFF>
struct SlotPart {
  u16 (*slots)[ELEMS];
  __device__ __forceinline__ u16* operator[](int b) const { return slots[b] + OFF; }
};

// Maximum without the sNaN canonicalisation that fmaxf needs in IEEE mode
// (a NaN score propagates, which is fine: the row is then NaN either way).
__device__ __forceinline__ float vmax(float a, float b) { return __builtin_elementwise_maximum(a, b); }

// Keeps the computation of v at this point of the instruction stream: the
// empty volatile asm is ordered with the scheduling fences around it, so the
// compiler can neither sink the work that produces v past them (out of the
// MFMA slot it was placed in) nor hoist it.
__device__ __forceinline__ void pin(float& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void pin(bf16x2& v) { asm volatile("" : "+v"(v)); }

__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

template <int D>
__device__ __forceinline__ void load_q(const u16* qh, int qrow, int L, int hw, bf16x8 (&qf)[D / 16]) {
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) {
    if (qrow < L)
      qf[ks] = *reinterpret_cast<const bf16x8*>(qh + (size_t)qrow * D + ks * 16 + hw * 8);
    else
      qf[ks] = bf16x8{};
  }
}

// S^T tile for G groups of 32 keys (G = 2: a 64-key tile; G = 1: its first
// 32 keys): lane (hw, c32) gets keys 32g + 8(e/4) + 4hw + e%4 of query c32 in
// s[g][e].  ka is the lane's k_lane.
template <int D, int G = 2>
__device__ __forceinline__ void qk_tile(const u16* sK, int ka, const bf16x8 (&qf)[D / 16], f32x16 (&s)[2]) {
#pragma unroll
  for (int g = 0; g < G; ++g) {
    s[g] = f32x16{};
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      bf16x8 kf = *reinterpret_cast<const bf16x8*>(sK + (ka ^ (16 * ks)) + 32 * g * D);
      s[g] = mfma32(kf, qf[ks], s[g]);
    }
  }
}

template <int G = 2>
__device__ __forceinline__ void mask_tile(f32x16 (&s)[2], int kvalid, int hw) {
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int key = 32 * g + 8 * (e >> 2) + 4 * hw + (e & 3);
      if (key >= kvalid) s[g][e] = -INFINITY;
    }
}

template <int NCH>
__device__ __forceinline__ void zero_lds(u16* p, int tid, int nt) {
  for (int i = tid; i < NCH; i += nt) *reinterpret_cast<u32x4*>(p + i * 8) = u32x4{0, 0, 0, 0};
}

// Online softmax against a lazy reference.  Probabilities of a row are taken
// as exp2(s * sl2 - mc) with mc = m * sl2 for a reference m (raw score units)
// that is NOT the running maximum, so no per-tile maximum is computed on the
// common path; the final normalisation uses the same reference, so the
// result is the softmax whatever the reference.  The first tile sets it to
// that tile's maximum, however negative (against mc = 0 a
// row whose scaled scores all lie below the fp32 exponent range would sum to
// zero).  In the pipeline it then moves only when the row's running sum
// passes kRowSumLimit (move_reference below); on the masked, exact path it
// moves when the tile's probabilities, summed over one lane's keys, exceed
// kTileSumLimit (RowRef::lim, checked before the tile enters P V), so there no
// probability exceeds 2^16 whatever the scores.  When the reference moves,
// sums taken against the old one are rescaled.
constexpr float kTileSumLimit = 65536.f;

struct RowRef {
  float m = -INFINITY;   // reference, raw score units; -inf until a finite score is seen
  float mc = 0.f;        // m * sl2 (0 while m is -inf)
  float lim = -1.f;      // tile sum above which the reference must move (below any sum while m is -inf)

  // m <- max(m, row maximum of s) for the rows of this wave (the two
  // half-waves holding a row agree); returns the rescale factor of sums
  // taken against the old reference.
  template <int G = 2>
  __device__ __forceinline__ float raise(const f32x16 (&s)[2], float sl2) {
    float mt = -INFINITY;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < 16; e += 2) mt = vmax(mt, vmax(s[g][e], s[g][e + 1]));
    float lo, hi;
    half_pair(mt, lo, hi);
    mt = vmax(lo, hi);
    const float mnew = fmaxf(m, mt);
    const float a = (mnew == -INFINITY) ? 1.f : fast_exp2((m - mnew) * sl2);
    m = mnew;
    mc = (m == -INFINITY) ? 0.f : m * sl2;
    lim = (m == -INFINITY) ? -1.f : kTileSumLimit;
    return a;
  }
  // Moves a set reference up by d (log2 units): sums taken against the old
  // one scale by 2^-d.
  __device__ __forceinline__ void shift(float d, float sl2) {
    mc += d;
    m = mc / sl2;
  }
};

// Running row sums of the rounded probabilities, formed on the matrix pipe.
// The 16x16x32 bf16 MFMA takes a P^T operand of the P V product as its B
// operand (lane l holds 8 keys of query row l % 32, so output column n
// gathers lanes n, n+16, n+32 and n+48, i.e. rows n and n+16) and a 0/1
// selector as A: output rows 0-7 keep k-groups 0 and 2 (lanes n, n+32:
// row n), output rows 8-15 keep k-groups 1 and 3 (row n+16).  Lane l then
// holds the sum of query row (l % 16) + 16 (l / 32), the same in all four
// accumulator entries.  (A v_dot2c per pair on the VALU holds the matrix
// pipe ~20 cycles each; four of these MFMAs take 64 cycles per step.)
// Sums above kRowSumLimit move the reference by log2 of the sum; a sum above
// kRowSumBad (or not finite) means a single tile jumped so far above the
// reference that a product may have overflowed, and the caller redoes the
// row on the exact path.
constexpr float kRowSumLimit = 1099511627776.f;                   // 2^40
constexpr float kRowSumBad = 1267650600228229401496703205376.f;   // 2^100

struct RowSums {
  f32x4 acc;
  bf16x8 sel;
  __device__ __forceinline__ void init(int lane) {
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
    const __bf16 v = (((lane & 15) < 8) == (((lane >> 4) & 1) == 0)) ? (__bf16)1.0f : (__bf16)0.0f;
    sel = bf16x8{v, v, v, v, v, v, v, v};
  }
  __device__ __forceinline__ void add(const bf16x8& p) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sel, p, acc, 0, 0, 0);
  }
  // The sum of query row c32 (the row of the P V layout), from its lane.
  __device__ __forceinline__ static float for_row(float v, int c32) {
    return __shfl(v, c32 < 16 ? c32 : c32 + 16, 64);
  }
};

// P = bf16(exp2(s * sl2 - mc)) for one S^T tile; returns this lane's sum of
// exactly the rounded values that enter P V, so numerator and denominator
// use the same weights.
template <int G = 2>
__device__ __forceinline__ float exp_tile(const f32x16 (&s)[2], float sl2, float mc, bf16x8 (&pb)[2][2]) {
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  float ts = 0.f;
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
      const bf16x2 pr = {(__bf16)fast_exp2(fmaf(s[g][e], sl2, -mc)),
                         (__bf16)fast_exp2(fmaf(s[g][e + 1], sl2, -mc))};
      pb[g][e >> 3][e & 7] = pr[0];
      pb[g][e >> 3][(e & 7) + 1] = pr[1];
      ts = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, ts, false);
    }
  return ts;
}

// As exp_tile, and fsum also receives this lane's sum of the unrounded fp32
// exponentials (for block masses, which must not carry the rounding of P).
template <int G = 2>
__device__ __forceinline__ float exp_tile_fsum(const f32x16 (&s)[2], float sl2, float mc, bf16x8 (&pb)[2][2],
                                               float& fsum) {
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  float ts = 0.f, fs = 0.f;
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
      const float x0 = fast_exp2(fmaf(s[g][e], sl2, -mc)), x1 = fast_exp2(fmaf(s[g][e + 1], sl2, -mc));
      const bf16x2 pr = {(__bf16)x0, (__bf16)x1};
      pb[g][e >> 3][e & 7] = pr[0];
      pb[g][e >> 3][(e & 7) + 1] = pr[1];
      ts = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, ts, false);
      fs += x0 + x1;
    }
  fsum = fs;
  return ts;
}

// Start of a pipelined step of the block-64 pairs while some row of the wave
// has no reference yet: such rows take the maximum of the tile whose
// probabilities the step forms (their sums so far are 0).  A tile that only
// the other query block keeps (hidden) never sets it.  Returns whether some row
// is still without one; the caller keeps that in a scalar, since looking at the
// rows again in every step cost a text row's walk 2% (110,336 tokens x 2 heads,
// keep 7%, d 128: 1809 us, with the scalar 1773).
template <int G = 2>
__device__ __forceinline__ bool first_reference(RowRef& ref, const f32x16 (&s_cur)[2], float sl2, bool hidden) {
  if (hidden) return true;
  RowRef r = ref;
  r.template raise<G>(s_cur, sl2);
  if (ref.m == -INFINITY) ref = r;
  return __any(ref.m == -INFINITY);
}

// End of a pipelined step (rare branch, taken by the whole wave): rows whose
// running sum (tiles up to the previous one) passed kRowSumLimit move their
// reference up by a whole number of log2 units, about log2 of the sum, so the
// sum becomes about 1.  What was taken against the old reference scales by
// an exact power of two: the sums and the current tile's probabilities (and
// with BS their fp32 sum, *tsum) here, the output accumulator at the start of
// the next step (pend).  So the tile's scores are not needed any more once
// its probabilities are taken, and the registers of its two 32-key groups go
// to the next tile's scores group by group; taking the probabilities again
// against the new reference kept all of them to the end of every step (dense
// attention at d 64: 182 registers, now 163).  bad is set when a sum has left
// the safe range.  A row's first reference is set before the pipeline from its
// first tile; a row that has none then (no finite score) is redone on the
// exact path (block-64 pairs, whose first tile may be the other block's, look
// for it at the start of every step instead).
template <int G = 2, bool BS = false>
__device__ __forceinline__ void move_reference(RowRef& ref, RowSums& rsum, bool& bad, bf16x8 (&p_cur)[2][2],
                                               bool& pend, float& pend_alpha, float sl2, int c32,
                                               float* tsum = nullptr) {
  const float sr = rsum.acc[0];
  if (!__any(sr > kRowSumLimit)) return;
  bad = bad || !(sr <= kRowSumBad);
  const float dr = sr > kRowSumLimit ? __builtin_floorf(__builtin_amdgcn_logf(sr)) : 0.f;   // log2 of the sum
  const float ar = fast_exp2(-dr);
#pragma unroll
  for (int j = 0; j < 4; ++j) rsum.acc[j] *= ar;
  const float d = RowSums::for_row(dr, c32);        // the same value for this lane's row
  const float al = fast_exp2(-d);
  if (d > 0.f) ref.shift(d, sl2);
  pend_alpha = al;
  pend = true;
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int e = 0; e < 8; ++e) p_cur[g][s2][e] = (__bf16)((float)p_cur[g][s2][e] * al);
  if constexpr (BS) *tsum *= al;
}

// After the last pipelined tile: its probabilities join the sums, a sum out
// of the safe range sets bad, and the row's sum is returned in the form the
// masked path continues from (the whole sum on the hw = 0 lane of the row, 0
// on the other).
template <int G = 2>
__device__ __forceinline__ float finish_sums(RowSums& rsum, bool& bad, const bf16x8 (&p_last)[2][2],
                                             int hw, int c32) {
#pragma unroll
  for (int j = 0; j < 2 * G; ++j) rsum.add(p_last[j >> 1][j & 1]);
  const float sr = rsum.acc[0];
  bad = bad || !(sr <= kRowSumBad);
  const float v = RowSums::for_row(sr, c32);
  return hw == 0 ? v : 0.f;
}

// Whether every entry of the output accumulator is finite.  The row-sum test
// bounds the probabilities, not their products with V: with large |V| a
// product can overflow fp32 while the sums stay in range, so a non-finite
// accumulator after the pipeline also sends the wave to the exact path (whose
// tile-sum test keeps every probability below 2^16).  The maximum propagates
// NaN, and the comparison fails for NaN and infinity.
template <int ND>
__device__ __forceinline__ bool acc_finite(const f32x16 (&o)[ND]) {
  float m = 0.f;
#pragma unroll
  for (int d = 0; d < ND; ++d)
#pragma unroll
    for (int e = 0; e < 16; ++e) m = vmax(m, __builtin_fabsf(o[d][e]));
  return m <= 3.4028234663852886e38f;
}

// Softmax of one tile outside the pipeline (masked tiles): P against the
// current reference, moved first if this tile needs it.  Returns the factor
// by which the output accumulator must be rescaled before this tile's P V
// (1 when the reference did not move); lsum includes the tile afterwards.
template <int G = 2>
__device__ __forceinline__ float softmax_tile(const f32x16 (&s)[2], RowRef& ref, float& lsum, float sl2,
                                              bf16x8 (&pb)[2][2]) {
  float ts = exp_tile<G>(s, sl2, ref.mc, pb);
  float a = 1.f;
  if (__any(ts > ref.lim)) {
    a = ref.template raise<G>(s, sl2);
    lsum *= a;
    ts = exp_tile<G>(s, sl2, ref.mc, pb);
  }
  lsum += ts;
  return a;
}

// As softmax_tile; fsum receives this lane's fp32 sum of the tile's
// exponentials against the reference they were finally taken against.
template <int G = 2>
__device__ __forceinline__ float softmax_tile_fsum(const f32x16 (&s)[2], RowRef& ref, float& lsum, float sl2,
                                                   bf16x8 (&pb)[2][2], float& fsum) {
  float ts = exp_tile_fsum<G>(s, sl2, ref.mc, pb, fsum);
  float a = 1.f;
  if (__any(ts > ref.lim)) {
    a = ref.template raise<G>(s, sl2);
    lsum *= a;
    ts = exp_tile_fsum<G>(s, sl2, ref.mc, pb, fsum);
  }
  lsum += ts;
  return a;
}

// O^T += V^T P^T for one tile.  MFMA step (g, s2) covers keys
// 32g + 16s2 + 8u + 4hw + j; lane (hw, e) supplies key index 8*(e/4) + 4*hw +
// e%4 of the step.  In each 16-lane group, lane j names row r0 + j/4 and 4
// elements at column d*32 + 16*(grp&1) + 4*(j%4); va is the lane's v_lane.
template <int ND, int G = 2>
__device__ __forceinline__ void pv_tile(const u16* sV, int va, const bf16x8 (&pb)[2][2], f32x16 (&o)[ND]) {
#pragma unroll
  for (int d = 0; d < ND; ++d)
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        const u16* p0 = sV + (va ^ (32 * d)) + (32 * g + 16 * s2) * (ND * 32);
        const s16x4 lo = lds_read_tr16(p0);
        const s16x4 hi = lds_read_tr16(p0 + 8 * (ND * 32));
        bf16x8 vf;
        __builtin_memcpy(&vf, &lo, 8);
        __builtin_memcpy(reinterpret_cast<char*>(&vf) + 8, &hi, 8);
        o[d] = mfma32(vf, pb[g][s2], o[d]);
      }
}

// Writes one wave's 32 x D output tile (o scaled by inv, rounded to bf16) as
// whole rows: the tile goes through stage, this wave's region of the K/V ring
// (32 rows of D elements, their 16-byte chunks in an order of the row's own as
// in the tiles; free once every wave has passed a barrier after its last use
// of the ring), and each store instruction then writes 64 / (D / 8) complete
// rows of 2 D bytes instead of 8-byte pieces of 32 rows.  Row row0 + r of out
// gets tile row r; rows at or past L are skipped.
template <int D>
__device__ __forceinline__ void store_rows(const f32x16 (&o)[D / 32], float inv, u16* stage, u16* out,
                                           int row0, int L, int lane) {
  constexpr int ND = D / 32, CPR = D / 8, RPI = 64 / CPR;
  const int hw = lane >> 5, c32 = lane & 31;
#pragma unroll
  for (int d = 0; d < ND; ++d)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bf16x4 w;
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = (__bf16)(o[d][4 * i + j] * inv);
      *reinterpret_cast<bf16x4*>(stage + c32 * D + ((4 * d + i) ^ (c32 & (CPR - 1))) * 8 + 4 * hw) = w;
    }
#pragma unroll 4
  for (int j = 0; j < 32 / RPI; ++j) {
    const int r = lane / CPR + RPI * j;
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(stage + r * D + ((lane ^ r) & (CPR - 1)) * 8);
    if (row0 + r < L) *reinterpret_cast<bf16x8*>(out + (size_t)(row0 + r) * D + (lane % CPR) * 8) = v;
  }
}
template <int D, int NW>
constexpr int kStageElems = NW * 32 * D;    // ring elements store_rows uses

// One pipelined step, scheduled by hand: NM = 2*NK + 4*ND MFMA slots that
// alternate a QK MFMA (scores of the next tile) and a PV MFMA (output update
// of the previous tile).  The QK MFMAs form one 32-key score group after the
// other (the current tile's groups are exponentiated in the same order, so a
// group's registers are free for the next tile's by then) and the PV MFMAs
// rotate over the ND output blocks, so two MFMAs into the same accumulator
// are 2 (QK) or 2*ND (PV) slots apart; each accumulator sums in the same order.
// Each slot first issues the LDS operand reads of the slot LA places ahead,
// then its MFMA, then hook(slot) (the caller's tile loads, at most one per
// slot), then its share of the softmax of the current tile against the
// reference mc (below); a scheduling fence closes the slot, so the matrix
// pipe and the VALU work side by side within the wave.  Four slots also add
// the previous tile's rounded probabilities (the operands of its P V) to the
// running row sums: the middle slot of each quarter of the step, or with
// RS_FIRST its first slot, so the last of them is done well before the sum
// test at the end of the step (dense attention: -1%; block-sparse
// attention, whose loads and index picks crowd the first slots, keeps the
// middle).  The sums are the same either way.
// With BS, *tsum receives this lane's sum of the current tile's unrounded
// exponentials, added pair by pair as the pairs are rounded.
template <int D, int G = 2, bool BS = false, bool RS_FIRST = false, typename Hook>
__device__ __forceinline__ void pipelined_step(Hook&& hook, const u16* sK, int ka, const u16* sV, int va,
                                               const bf16x8 (&qf)[D / 16], const f32x16 (&s_cur)[2],
                                               const bf16x8 (&p_prev)[2][2], f32x16 (&s_next)[2],
                                               bf16x8 (&p_cur)[2][2], f32x16 (&o)[D / 32], float sl2,
                                               float mc, RowSums& rsum, float* tsum = nullptr) {
  constexpr int NK = D / 16, ND = D / 32;
  constexpr int NQK = G * NK, NPV = 2 * G * ND;      // G score groups of 32 keys
  static_assert(NQK == NPV, "QK and PV slots alternate");
  constexpr int NM = NQK + NPV;
  constexpr int NS = 16 * G;                           // scores per lane
  static_assert(NS % NM == 0 && NM % 2 == 0, "whole exponential pairs per slot pair");
  constexpr int LA = 2;                       // operand lookahead, in slots

  bf16x8 op[NM];
  auto fetch = [&](int i) {
    const int j = i >> 1;
    if ((i & 1) == 0) {       // QK j: g = j / NK, ks = j % NK
      const int g = j / NK, ks = j % NK;
      op[i] = *reinterpret_cast<const bf16x8*>(sK + (ka ^ (16 * ks)) + 32 * g * D);
    } else {                  // PV j: d = j % ND, (g, s2) = j / ND
      const int d = j % ND, g = (j / ND) >> 1, s2 = (j / ND) & 1;
      const u16* p0 = sV + (va ^ (32 * d)) + (32 * g + 16 * s2) * D;
      const s16x4 lo = lds_read_tr16(p0);
      const s16x4 hi = lds_read_tr16(p0 + 8 * D);
      __builtin_memcpy(&op[i], &lo, 8);
      __builtin_memcpy(reinterpret_cast<char*>(&op[i]) + 8, &hi, 8);
    }
  };
  auto mfma = [&](int i) {
    const int j = i >> 1;
    if ((i & 1) == 0) {
      const int g = j / NK, ks = j % NK;
      if (ks == 0) s_next[g] = mfma32(op[i], qf[ks], f32x16{});
      else s_next[g] = mfma32(op[i], qf[ks], s_next[g]);
    } else {
      const int d = j % ND, g = (j / ND) >> 1, s2 = (j / ND) & 1;
      o[d] = mfma32(op[i], p_prev[g][s2], o[d]);
    }
  };

  // Slot i owns scores e in [i*PER, (i+1)*PER) of the tile's 32, in (group,
  // element) order.  Their softmax is pipelined over three slots: slot i
  // forms the exponent arguments, slot i+1 takes the exponentials, slot i+2
  // rounds each completed pair to bf16, so no instruction waits on the result
  // of the one just before it.  The last two slots' shares are finished after
  // the MFMAs.
  constexpr int PER = NS / NM;
  constexpr int RSP = NM / (2 * G);           // row-sum MFMAs in slots RS0 + j*RSP
  constexpr int RS0 = RS_FIRST ? 0 : RSP / 2;
  float arg[NS], ex[NS];
  float fs = 0.f;
  auto stage_arg = [&](int i) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = i * PER + u;
      arg[e] = fmaf(s_cur[e >> 4][e & 15], sl2, -mc);
      pin(arg[e]);
    }
  };
  auto stage_exp = [&](int i) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = i * PER + u;
      ex[e] = fast_exp2(arg[e]);
      pin(ex[e]);
    }
  };
  auto stage_sum = [&](int i) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = i * PER + u, g = e >> 4, r = e & 15;
      if (e & 1) {
        bf16x2 pr = {(__bf16)ex[e - 1], (__bf16)ex[e]};
        pin(pr);
        p_cur[g][r >> 3][(r & 7) - 1] = pr[0];
        p_cur[g][r >> 3][r & 7] = pr[1];
        if constexpr (BS) {
          fs += ex[e - 1] + ex[e];
          pin(fs);              // in this slot: deferred, the adds keep every exponential live
        }
      }
    }
  };

#pragma unroll
  for (int i = 0; i < LA; ++i) fetch(i);
#pragma unroll
  for (int i = 0; i < NM; ++i) {
    if (i + LA < NM) fetch(i + LA);
    mfma(i);
    if (i % RSP == RS0) rsum.add(p_prev[(i / RSP) >> 1][(i / RSP) & 1]);
    hook(i);
    stage_arg(i);
    if (i >= 1) stage_exp(i - 1);
    if (i >= 2) stage_sum(i - 2);
    __builtin_amdgcn_sched_barrier(0);
  }
  stage_exp(NM - 1);
  stage_sum(NM - 2);
  stage_sum(NM - 1);
  if constexpr (BS) *tsum = fs;
}

// One pipelined step of the block-mass pass: the NM = 2*NK QK MFMAs of the
// next tile (alternating the two 32-key groups) with, slot by slot, an equal
// share of the exp2(s * sl2 - lse2) terms of the current tile added to acc in
// (group, element) order; hook(slot) issues the caller's tile loads.
template <int D, typename Hook>
__device__ __forceinline__ void mass_step(Hook&& hook, const u16* sK, int ka, const bf16x8 (&qf)[D / 16],
                                          const f32x16 (&s_cur)[2], f32x16 (&s_next)[2], float& acc,
                                          float sl2, float nlse2) {
  constexpr int NK = D / 16, NM = 2 * NK, LA = 2;
  bf16x8 op[NM];
  // At d 128 half of the columns' addresses are formed in every step: kept over
  // the loop, all eight would take the pass past 128 registers.
  int half_row = 64;
  if constexpr (D == 128) asm volatile("" : "+s"(half_row));
  auto fetch = [&](int j) {
    const int g = j & 1, ks = j >> 1;
    int at = ka ^ (16 * (ks & 3));
    if (ks >= 4) at ^= half_row;
    op[j] = *reinterpret_cast<const bf16x8*>(sK + at + 32 * g * D);
  };
  auto mfma = [&](int j) {
    const int g = j & 1, ks = j >> 1;
    if (ks == 0) s_next[g] = mfma32(op[j], qf[ks], f32x16{});
    else s_next[g] = mfma32(op[j], qf[ks], s_next[g]);
  };
  // Slot j owns scores [j*PER, (j+1)*PER); as in pipelined_step, slot j forms
  // their exponent arguments, slot j+1 the exponentials and slot j+2 adds
  // them to acc (in score order), the last two shares after the MFMAs.
  constexpr int PER = 32 / NM;
  float arg[32], ex[32];
  auto stage_arg = [&](int j) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = j * PER + u;
      arg[e] = fmaf(s_cur[e >> 4][e & 15], sl2, nlse2);
      pin(arg[e]);
    }
  };
  auto stage_exp = [&](int j) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = j * PER + u;
      ex[e] = fast_exp2(arg[e]);
      pin(ex[e]);
    }
  };
  auto stage_sum = [&](int j) {
#pragma unroll
    for (int u = 0; u < PER; ++u) acc += ex[j * PER + u];
    pin(acc);
  };
#pragma unroll
  for (int i = 0; i < LA; ++i) fetch(i);
#pragma unroll
  for (int i = 0; i < NM; ++i) {
    if (i + LA < NM) fetch(i + LA);
    mfma(i);
    hook(i);
    stage_arg(i);
    if (i >= 1) stage_exp(i - 1);
    if (i >= 2) stage_sum(i - 2);
    __builtin_amdgcn_sched_barrier(0);
  }
  stage_exp(NM - 1);
  stage_sum(NM - 2);
  stage_sum(NM - 1);
}

}  // namespace adaspa
