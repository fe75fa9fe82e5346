// Chunk scan kernel: the sequential part of the recurrence.
//
// One workgroup per (sequence, value head): d_v/16 waves (two per SIMD for
// d_v = 128), each owning 16 columns of M = S^T (d_k x d_v) in registers for the
// whole sequence.  Per 64-token chunk, with M0 the state at chunk start:
//   R      = diag(beta) V - diag(beta e^G) (K M0)
//   Delta  = T R                                                  (T from k_intra)
//   O      = diag(scale e^G) (Q M0) + P Delta                     (outputs only)
//   M1     = e^{G_last} M0 + K^T diag(e^{G_last - G}) Delta
// All four products run on MFMA.  The contraction order inside every 32-wide k
// step is permuted (kperm) so each accumulator is directly the next product's
// B operand.  fp32 operands (M0, R, Delta, T, P) are split into bf16 hi + lo.
// For bf16 inputs T R takes two passes, hi(T) (hi + lo)(R); every other
// product keeps both parts of its fp32 operands.  With hi(T) alone the state's
// error stays below about 5e-4 relative (gate scales 0 to 0.5, beta up to 1,
// tails of 3277 tokens and a 32768-token prefix), measured on the CPU with a
// model of exactly these roundings; dropping any other pass (hi(M0) alone in
// K M0, or the lo part of R, Delta or P) takes it past 1e-3 somewhere.
//
// A chunk's operands come global -> LDS by DMA (global_load_lds, 16 bytes per
// lane) into one of two LDS buffers while the waves compute on the other: the
// key, query and value rows from the inputs (bf16; for fp32 inputs keys and
// queries from a record of hi and lo fragments), T, P and the scalars from the
// records k_intra wrote.  A wave fetches each operand with 16-byte or
// transposing LDS reads whose addresses are a lane constant plus an immediate
// (the chunk loop takes the two buffers in turn, see each_chunk).  Inside a
// chunk the waves issue each group of LDS reads one region ahead of its use.
//
// What bounds it: a chunk is a chain of dependent products, and a wave issues
// its ~290 vector and 76 MFMA instructions of 16 columns in order, one every
// ~5.5 clocks (3.2k clocks a chunk, of which the matrix pipe is busy 1.2k).
#pragma once

#include "gdn_device.h"
#include "gdn_intra.h"
#include "gdn_plan.h"

#include <type_traits>

namespace gdn {

constexpr int kLdsBytes = 160 * 1024;

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __attribute__((address_space(3))) unsigned char lds_byte;   // LDS bytes

// 16 bytes per lane from `src` (per lane) to LDS `dst + 16 * lane` (dst uniform).
__device__ __forceinline__ void dma16(const void* src, lds_byte* dst) {
  __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)dst, 16, 0, 0);
}

__device__ __forceinline__ void wait_dma() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// The same, but for the N youngest.
template <int N>
__device__ __forceinline__ void wait_dma_but() {
  static_assert(N < 64, "vmcnt holds six bits");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// The same from `base + off`: a uniform base and a 32-bit lane offset, so the
// load takes the scalar-base form and its address costs no 64-bit lane
// arithmetic.  Offsets stay below 2^32: a chunk spans 64 rows of at most
// 65535 heads x 128 x 4 bytes.
__device__ __forceinline__ void dma16_at(const void* base, uint32_t off, lds_byte* dst) {
  dma16(static_cast<const unsigned char*>(base) + off, dst);
}


// Byte offset of byte `byte_in_row` of row `row` in a value row tile whose rows
// hold ROW_BYTES / 16 pieces of 16 bytes, piece p of row R stored at p ^
// v_swz(R): the transposing reads (32 lanes, eight rows of two pieces, at a
// time) then touch every bank once.
template <int ROW_BYTES>
__device__ __forceinline__ constexpr int v_swz(int row) {
  if (ROW_BYTES == 256) return row_swz<256>(row);
  if (ROW_BYTES == 64) return 2 * ((row >> 2) & 1);
  return row % (ROW_BYTES / 16);
}
template <int ROW_BYTES>
__device__ __forceinline__ int swz(int row, int byte_in_row) {
  return row * ROW_BYTES + 16 * ((byte_in_row / 16) ^ v_swz<ROW_BYTES>(row)) + byte_in_row % 16;
}

// DMA of rows [0, 64) of a token-major tensor (row 0 at `row0`, 1 KiB block
// `blk` of the tile) into a swizzled LDS row tile; rows past `rows` repeat the
// last valid row.
template <int ROW_BYTES, typename T>
__device__ __forceinline__ void dma_rows(const T* row0, int64_t row_stride, int rows, lds_byte* dst,
                                         int blk, int lane) {
  constexpr int pieces = ROW_BYTES / 16;
  constexpr int rows_per_block = 1024 / ROW_BYTES;
  const int r = blk * rows_per_block + lane / pieces;
  const int p = (lane % pieces) ^ v_swz<ROW_BYTES>(r);
  const uint32_t stride_b = static_cast<uint32_t>(row_stride) * static_cast<uint32_t>(sizeof(T));
  dma16_at(row0, static_cast<uint32_t>(min(r, rows - 1)) * stride_b + 16u * p, dst + blk * 1024);
}

// Element j (0..3) of four bf16 values packed in two dwords, as float.
__device__ __forceinline__ float bf16_elt(const u32x2& x, int j) {
  const uint32_t w = j < 2 ? x.x : x.y;
  return __uint_as_float((j & 1) ? (w & 0xFFFF0000u) : (w << 16));
}

// Buffer resource over `bytes` bytes from `base` (gfx9 raw buffer: stride 0,
// byte offsets).  The hardware drops a store whose VGPR offset is at or past
// `bytes`; the SGPR offset is not range-checked, so callers pass 0 there.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t out_rsrc(void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000);
}
// Four consecutive output elements of one row, as bf16 (8 bytes) or fp32 (16).
__device__ __forceinline__ void store_out4(__amdgpu_buffer_rsrc_t r, int voff, const f32x4& x, uint16_t*) {
  const uint32_t a = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x[0], x[1]}, bf16x2));
  const uint32_t b = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x[2], x[3]}, bf16x2));
  __builtin_amdgcn_raw_buffer_store_b64(u32x2{a, b}, r, voff, 0, 0);
}
__device__ __forceinline__ void store_out4(__amdgpu_buffer_rsrc_t r, int voff, const f32x4& x, float*) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), r, voff, 0, 0);
}

// LDS layout of one chunk buffer of a workgroup that covers VC state columns;
// P (outputs only) is staged in LDS when P_LDS, else read from global memory.
template <typename TIn, int DK, int VC, bool FWD, bool P_LDS>
struct ScanLds {
  static constexpr int kDK = DK;
  static constexpr bool kSplit = sizeof(TIn) == 4;
  static constexpr bool kPInLds = FWD && P_LDS;
  static constexpr int kKFrags = k_record_frags(DK, FWD);         // per bf16 part
  static constexpr int kKBytes = static_cast<int>(k_tile_bytes(DK, FWD, kSplit));
  static constexpr int kTBytes = static_cast<int>(t_record_bytes(kSplit));
  static constexpr int kSBytes = static_cast<int>(kSRecordBytes);
  static constexpr int kVRowBytes = VC * static_cast<int>(sizeof(TIn));
  static constexpr int kVBytes = kChunk * kVRowBytes;
  static constexpr int kOffK = 0;                 // K (and Q) fragments
  static constexpr int kOffT = kOffK + kKBytes;
  static constexpr int kPBytes = kPInLds ? static_cast<int>(kPRecordBytes) : 0;
  static constexpr int kOffP = kOffT + kTBytes;
  static constexpr int kOffS = kOffP + kPBytes;
  static constexpr int kOffV = kOffS + 2048;      // S padded to two DMA blocks
  static constexpr int kBytes = kOffV + kVBytes;
  static constexpr int kBuffers = 2 * kBytes <= kLdsBytes ? 2 : 1;
  // DMA jobs per chunk (one 1 KiB global_load_lds each): K (and Q) fragments,
  // T, P, V rows, then the scalars as one full and one quarter block
  static constexpr int kKJobs = kKBytes / 1024, kTJobs = kTBytes / 1024, kPJobs = kPBytes / 1024;
  static constexpr int kVJobs = kVBytes / 1024;
  static constexpr int kJobs = kKJobs + kTJobs + kPJobs + kVJobs + 2;
};

// Where one chunk's operands come from.
struct ChunkSrc {
  const unsigned char* krec;   // K record of (slot, key head), fp32 inputs
  const void* k0;              // key row 0 of the chunk (bf16 inputs: the fragments come from the rows)
  const void* q0;              // query row 0 of the chunk (bf16 inputs, outputs only)
  int64_t krow;                // elements between consecutive key (query) rows
  const unsigned char* trec;   // T record of (slot, value head)
  const unsigned char* prec;   // P record of (slot, value head), outputs only
  const unsigned char* srow;   // scalars of (slot, value head)
  const void* v0;              // V row 0 of the chunk, first column of the workgroup
  int clen;                    // valid rows
};

// DMA job j of a chunk of fp32 inputs (0 <= j < L::kJobs) into LDS buffer `base`.
template <typename L, typename TIn>
__device__ __forceinline__ void dma_job(const ChunkSrc& c, int64_t vrow, lds_byte* base, int j, int lane) {
  static_assert(L::kPJobs == 0, "fp32 inputs: the output waves read P from memory");
  if (j < L::kKJobs) {
    dma16_at(c.krec + 1024 * j, 16u * lane, base + L::kOffK + 1024 * j);
  } else if (j < L::kKJobs + L::kTJobs) {
    const int t = j - L::kKJobs;
    dma16_at(c.trec + 1024 * t, 16u * lane, base + L::kOffT + 1024 * t);
  } else if (j < L::kKJobs + L::kTJobs + L::kVJobs) {
    // V rows; pad rows repeat the last row (their beta is 0, so they add nothing)
    dma_rows<L::kVRowBytes>(static_cast<const TIn*>(c.v0), vrow, c.clen, base + L::kOffV,
                            j - L::kKJobs - L::kTJobs, lane);
  } else if (j == L::kJobs - 2) {
    dma16_at(c.srow, 16u * lane, base + L::kOffS);                 // scalars, bytes 0..1023
  } else if (lane < 16) {
    dma16_at(c.srow + 1024, 16u * lane, base + L::kOffS + 1024);   // bytes 1024..1279
  }
}

// A chunk's key rows in LDS (bf16 inputs; rows 64.. are the queries), as MFMA
// operands.
template <int DK>
struct KeyTile {
  static constexpr int kRB = 2 * DK;
  const unsigned char* rows;
  int lane;
  // A operand of K M0 (and B operand of (Q M0)^T): lane (g, r) gets columns 32
  // kk + 8 g .. +7 of row 16 ti + r.
  __device__ __forceinline__ bf16x8 frag(int ti, int kk) const {
    const int lg = lane / 16, lr = lane % 16;
    return *reinterpret_cast<const bf16x8*>(rows + (16 * ti + lr) * kRB + 16 * ((4 * kk + lg) ^ row_swz<kRB>(lr)));
  }
  // A operand of K^T Delta by transposing reads: lane (g, c) needs K[32 kk +
  // kperm(g, j)][column c of state row tile td] (see strow).  In a transposing
  // read each lane of a 16-lane group addresses four consecutive columns of one
  // row and receives one column of four rows; lane (g, c) addresses row 32 kk +
  // 4 g + c / 4 (then 16 rows further, for j >= 4), columns strow(td, c % 4, 0..3).
  __device__ __forceinline__ bf16x8 frag_t(int td, int kk) const {
    const int lg = lane / 16, lr = lane % 16;
    const int rr = 4 * lg + lr / 4;
    const unsigned char* p = rows + (32 * kk + rr) * kRB + 16 * ((4 * (td / 2) + lr % 4) ^ row_swz<kRB>(rr)) +
                             8 * (td % 2);
    return __builtin_bit_cast(bf16x8, join_halves(lds_read_tr16(p), lds_read_tr16(p + 16 * kRB)));
  }
};

// One 64-token chunk for one wave: 16 state columns, M (and its split mb) in
// registers.  `base` is the chunk's LDS buffer, `vc0` the wave's first column
// within the buffer's V tile.  The chunk runs as a chain of regions: each region issues the
// LDS reads of a later region, runs MFMAs on operands that are ready, and does
// VALU work (scaling, hi/lo splits) for the next region that is independent of
// its own MFMAs.  hook(k) runs at the start of region k (the whole-head kernel
// issues its DMA share there).  With outputs, the chunk's O is left in `pout`:
// pout[ti][i] = O[16 ti + lane % 16][4 (lane / 16) + i] of the wave's columns.
// With EXPORT (and FWD false), the wave leaves the outputs to another wave: it
// writes Delta (four 16-byte tiles per lane) to LDS `xd` before hook(5) and
// the split of M1 (the next chunk's B operand of K M0, layout [k step][hi |
// lo][lane]) to `xm` at the end.
template <typename L, int DK, bool FWD, bool EXPORT, typename Hook>
__device__ __forceinline__ void chunk_step(const unsigned char* base, int vc0, int lane,
                                           f32x4 (&M)[DK / 16], Frag (&mb)[DK / 32], f32x4 (&pout)[4],
                                           Hook&& hook, unsigned char* xd = nullptr,
                                           unsigned char* xm = nullptr) {
  static_assert(!(FWD && EXPORT), "a wave that exports Delta leaves the outputs to another");
  constexpr bool SPLIT = L::kSplit;
  static_assert(!(FWD && SPLIT), "fp32 inputs leave the outputs to output waves");
  constexpr int NT = DK / 16, NK = DK / 32;
  constexpr int NKF = L::kKFrags;
  constexpr int VRB = L::kVRowBytes;
  const int lg = lane / 16, lr = lane % 16;
  const u32x4* kf = reinterpret_cast<const u32x4*>(base + L::kOffK);
  const u32x4* tf = reinterpret_cast<const u32x4*>(base + L::kOffT);
  const float* sc = reinterpret_cast<const float*>(base + L::kOffS);
  const unsigned char* vtile = base + L::kOffV;
  // fp32 inputs: fragments of the K record, lanes in kslot order; bf16 inputs:
  // the rows themselves, the queries' behind the keys'
  const int klane = kslot(lane);
  const KeyTile<DK> kt{base + L::kOffK, lane};
  auto ldf = [&](Frag& x, int ti, int kk, bool isq) __attribute__((always_inline)) {
    if constexpr (SPLIT) {
      const int f = ti * NK + kk;
      x.hi = __builtin_bit_cast(bf16x8, kf[f * kWave + klane]);
      x.lo = __builtin_bit_cast(bf16x8, kf[(NKF + f) * kWave + klane]);
    } else {
      x.hi = kt.frag(ti + (isq ? 4 : 0), kk);
    }
  };
  // fp32-derived records: P always hi and lo, T hi (and lo for fp32 inputs)
  auto ld_split = [&](Frag& x, const u32x4* rec, int f) __attribute__((always_inline)) {
    x.hi = __builtin_bit_cast(bf16x8, rec[f * kWave + lane]);
    x.lo = __builtin_bit_cast(bf16x8, rec[(kTFrags + f) * kWave + lane]);
  };
  auto ld_t = [&](Frag& x, const u32x4* rec, int f) __attribute__((always_inline)) {
    x.hi = __builtin_bit_cast(bf16x8, rec[f * kWave + lane]);
    if constexpr (SPLIT) x.lo = __builtin_bit_cast(bf16x8, rec[(kTFrags + f) * kWave + lane]);
  };
  // K M0: K exact (bf16 inputs) or split (fp32 inputs), M0 split
  auto mma_km = [&](const Frag& a, const Frag& m, f32x4 c) __attribute__((always_inline)) {
    return mma_a<SPLIT>(a, m, c);
  };
  // T R: fp32 inputs 3 passes; bf16 inputs hi(T) times both parts of R
  auto mma_tr = [&](const Frag& t, const Frag& r, f32x4 c) __attribute__((always_inline)) {
    if constexpr (SPLIT) return mma_x3(t, r, c);
    else return mma_x2(t.hi, r, c);
  };
  // K (and Q) operands of row tiles 2 tp, 2 tp + 1 for every k step
  auto ld_ka = [&](Frag (&a)[2][NK], Frag (&aq)[2][NK], int tp) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        ldf(a[u][kk], 2 * tp + u, kk, false);
        if constexpr (FWD) ldf(aq[u][kk], 2 * tp + u, kk, true);
      }
  };
  // K^T operands of every row tile td of M for token k step kk, by
  // transposing reads of the keys (see KeyTile): lane (g, c) addresses row 32 kk
  // + 4 g + c / 4, columns strow(td, c % 4, 0..3); in K record fragment (row tile
  // 2 kk (+1), k step td / 2) that is lane 16 (c % 4) + 4 g + c / 4 (at its kslot
  // position), bytes 8 (td % 2)..+7.
  const int kt_off = 16 * kslot(16 * (lr % 4) + 4 * lg + lr / 4);
  auto ld_kt = [&](Frag (&a)[NT], int kk) __attribute__((always_inline)) {
#pragma unroll
    for (int td = 0; td < NT; ++td) {
      if constexpr (!SPLIT) {
        a[td].hi = kt.frag_t(td, kk);
      } else {
        const unsigned char* f0 = reinterpret_cast<const unsigned char*>(kf + ((2 * kk) * NK + td / 2) * kWave);
        const unsigned char* f1 = reinterpret_cast<const unsigned char*>(kf + ((2 * kk + 1) * NK + td / 2) * kWave);
        const int o = kt_off + 8 * (td % 2);
        a[td].hi = __builtin_bit_cast(bf16x8, join_halves(lds_read_tr16(f0 + o), lds_read_tr16(f1 + o)));
        constexpr int lo = NKF * kWave * 16;
        a[td].lo = __builtin_bit_cast(bf16x8, join_halves(lds_read_tr16(f0 + lo + o), lds_read_tr16(f1 + lo + o)));
      }
    }
  };

  // The chunk runs as a chain of regions.  Each region issues the LDS reads of
  // a later region, runs MFMAs on operands that are ready, and does VALU work
  // (scaling, hi/lo splits) for the next region, independent of its own MFMAs
  // so the two overlap.
  Frag ka0[2][NK], qa0[2][NK], ka1[2][NK], qa1[2][NK];
  Frag tfr[kTFrags];
  Frag kta[NT], ktb[NT];
  f32x4 km[4], qm[4], bv[4], R[4], D[4];
  u32x2 vraw[4];
  float vf[4][4];

  hook(0);
  // ---- region 0: first operands
  ld_ka(ka0, qa0, 0);
  if constexpr (!SPLIT) {
    // transposing read: lane (g, c) gets V[16 ti + 4 g + r][c], r = 0..3
#pragma unroll
    for (int ti = 0; ti < 4; ++ti)
      vraw[ti] = lds_read_tr16(vtile + swz<VRB>(16 * ti + 4 * lg + lr / 4, 2 * (vc0 + 4 * (lr % 4))));
  } else {
#pragma unroll
    for (int ti = 0; ti < 4; ++ti)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        vf[ti][r] = *reinterpret_cast<const float*>(vtile + swz<VRB>(16 * ti + 4 * lg + r, 4 * (vc0 + lr)));
  }
  __builtin_amdgcn_sched_barrier(0);

  hook(1);
  // ---- region 1: K M0 for row tiles 0, 1 | beta V; the row tiles 2, 3
  //      operands arrive
  ld_ka(ka1, qa1, 1);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    km[u] = zero4();
    qm[u] = zero4();
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      km[u] = mma_km(ka0[u][kk], mb[kk], km[u]);
      if constexpr (FWD) qm[u] = mma_b<false>(mb[kk], qa0[u][kk], qm[u]);
    }
  }
#pragma unroll
  for (int ti = 0; ti < 4; ++ti) {
    const f32x4 bta = *reinterpret_cast<const f32x4*>(sc + 0 * kChunk + 16 * ti + 4 * lg);
#pragma unroll
    for (int r = 0; r < 4; ++r) bv[ti][r] = bta[r] * (SPLIT ? vf[ti][r] : bf16_elt(vraw[ti], r));
  }
  __builtin_amdgcn_sched_barrier(0);

  hook(2);
  // ---- region 2: K M0 for row tiles 2, 3 | R rows 0..31 and their split;
  //      T arrives
#pragma unroll
  for (int f = 0; f < kTFrags; ++f) ld_t(tfr[f], tf, f);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    km[2 + u] = zero4();
    qm[2 + u] = zero4();
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      km[2 + u] = mma_km(ka1[u][kk], mb[kk], km[2 + u]);
      if constexpr (FWD) qm[2 + u] = mma_b<false>(mb[kk], qa1[u][kk], qm[2 + u]);
    }
  }
  auto make_r = [&](int ti) __attribute__((always_inline)) {
    const f32x4 bge = *reinterpret_cast<const f32x4*>(sc + 1 * kChunk + 16 * ti + 4 * lg);
#pragma unroll
    for (int r = 0; r < 4; ++r) R[ti][r] = bv[ti][r] - bge[r] * km[ti][r];
  };
  make_r(0);
  make_r(1);
  const Frag rb0 = chain_frag(R[0], R[1]);
  __builtin_amdgcn_sched_barrier(0);

  hook(3);
  // ---- region 3: Delta = T R, k step 0 for all row tiles | R rows 32..63
  //      and their split; K^T (k step 0) and P (outputs) arrive
  ld_kt(kta, 0);
  Frag pfr[FWD ? kTFrags : 1];
  if constexpr (FWD) {
    // P (fp32-derived: hi and lo parts)
    static_assert(L::kPInLds, "a wave that forms its own outputs reads P from LDS");
    const u32x4* pl = reinterpret_cast<const u32x4*>(base + L::kOffP);
#pragma unroll
    for (int f = 0; f < kTFrags; ++f) ld_split(pfr[f], pl, f);
  }
#pragma unroll
  for (int ti = 0; ti < 4; ++ti) D[ti] = mma_tr(tfr[tri_frag(ti, 0)], rb0, zero4());
  make_r(2);
  make_r(3);
  const Frag rb1 = chain_frag(R[2], R[3]);
  __builtin_amdgcn_sched_barrier(0);

  hook(4);
  // ---- region 4: Delta, k step 1 for row tiles 2, 3 | split of the
  //      weighted Delta rows 0..31 (and of Delta for the outputs); K^T
  //      arrives
  ld_kt(ktb, 1);
  if constexpr (EXPORT) {
#pragma unroll
    for (int ti = 0; ti < 2; ++ti) reinterpret_cast<f32x4*>(xd)[ti * kWave + lane] = D[ti];   // final
  }
#pragma unroll
  for (int ti = 2; ti < 4; ++ti) D[ti] = mma_tr(tfr[tri_frag(ti, 1)], rb1, D[ti]);
  f32x4 Dw[4];
  auto make_dw = [&](int ti) __attribute__((always_inline)) {
    const f32x4 w = *reinterpret_cast<const f32x4*>(sc + 2 * kChunk + 16 * ti + 4 * lg);
#pragma unroll
    for (int r = 0; r < 4; ++r) Dw[ti][r] = w[r] * D[ti][r];
  };
  make_dw(0);
  make_dw(1);
  const Frag db0 = chain_frag(Dw[0], Dw[1]);
  Frag dd0;
  if constexpr (FWD) dd0 = chain_frag(D[0], D[1]);
  __builtin_amdgcn_sched_barrier(0);

  if constexpr (EXPORT) {
#pragma unroll
    for (int ti = 2; ti < 4; ++ti) reinterpret_cast<f32x4*>(xd)[ti * kWave + lane] = D[ti];
  }
  hook(5);
  // ---- region 5: M1 partial, k step 0 (tokens 0..31) | split of the
  //      weighted Delta rows 32..63
  const float eg = sc[4 * kChunk];
#pragma unroll
  for (int td = 0; td < NT; ++td) {
#pragma unroll
    for (int r = 0; r < 4; ++r) M[td][r] *= eg;
    M[td] = mma_a<SPLIT>(kta[td], db0, M[td]);
  }
  make_dw(2);
  make_dw(3);
  const Frag db1 = chain_frag(Dw[2], Dw[3]);
  Frag dd1;
  if constexpr (FWD) dd1 = chain_frag(D[2], D[3]);
  __builtin_amdgcn_sched_barrier(0);

  // ---- outputs, transposed: O^T = diag-scaled (Q M0)^T + Delta^T P^T, whose
  //      MFMA layout gives a lane four consecutive columns of one token row
  //      (row 16 ti + lane % 16, columns 4 (lane / 16) + 0..3 of the wave's 16).
  //      The split Delta (dd) is the A operand and the P fragments the B
  //      operand; qm already holds (Q M0)^T (A = split M0, B = Q fragments).
  //      Stored at the start of the next chunk.
  if constexpr (FWD) {
#pragma unroll
    for (int ti = 0; ti < 4; ++ti) {
      const float qe = sc[3 * kChunk + 16 * ti + lr];
#pragma unroll
      for (int r = 0; r < 4; ++r) pout[ti][r] = qe * qm[ti][r];
      pout[ti] = mma_x3(dd0, pfr[tri_frag(ti, 0)], pout[ti]);
      if (ti >= 2) pout[ti] = mma_x3(dd1, pfr[tri_frag(ti, 1)], pout[ti]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  hook(6);
  // ---- region 6: M1, k step 1 (tokens 32..63) | split of M1 for the next chunk
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    M[2 * kk] = mma_a<SPLIT>(ktb[2 * kk], db1, M[2 * kk]);
    M[2 * kk + 1] = mma_a<SPLIT>(ktb[2 * kk + 1], db1, M[2 * kk + 1]);
    mb[kk] = chain_frag(M[2 * kk], M[2 * kk + 1]);
  }
  if constexpr (EXPORT) {
    u32x4* x = reinterpret_cast<u32x4*>(xm);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      x[(2 * kk) * kWave + lane] = __builtin_bit_cast(u32x4, mb[kk].hi);
      x[(2 * kk + 1) * kWave + lane] = __builtin_bit_cast(u32x4, mb[kk].lo);
    }
  }
}

// One 64-token chunk of tail replay (no outputs, bf16 inputs) for a wave that
// carries NC tiles of 16 state columns: the products of chunk_step in the same
// order with the same roundings (so the state is bit for bit that of NC waves
// of one tile each), but every operand that does not depend on the state (K,
// T, K^T) is read from LDS once for all NC tiles, and K M0 runs k step by k
// step (the four row tiles' K fragments of one step, shared by the tiles), so
// only two steps' operands are held at a time.  The tiles' chains are
// independent, so each phase has NC times the MFMAs to cover the LDS reads
// issued for the next.  hook(p) runs at the start of phase p, p = 0 ..
// tiles_phases(DK) - 1 (a workgroup without a DMA wave issues the next
// chunk's DMA there).  Of the two waves of a SIMD the one in a phase of many
// MFMAs (K M0, K^T Dw) goes first, so the other's vector work fills in behind
// it (12 sequences of 52 chunks 247 -> 238 us, 36 of them 532 -> 517).
constexpr int tiles_phases(int dk) { return dk / 32 + 6; }
template <typename L, int DK, int NC, typename Hook>
__device__ __forceinline__ void chunk_step_tiles(const unsigned char* base, int vc0, int lane,
                                                 f32x4 (&M)[NC][DK / 16], Frag (&mb)[NC][DK / 32],
                                                 Hook&& hook) {
  static_assert(!L::kSplit, "bf16 inputs: K, K^T and hi(T) are single bf16 operands");
  constexpr int NT = DK / 16, NK = DK / 32;
  constexpr int VRB = L::kVRowBytes;
  const int lg = lane / 16, lr = lane % 16;
  const u32x4* tf = reinterpret_cast<const u32x4*>(base + L::kOffT);
  const float* sc = reinterpret_cast<const float*>(base + L::kOffS);
  const unsigned char* vtile = base + L::kOffV;
  const KeyTile<DK> kt{base + L::kOffK, lane};

  // ---- V (transposing reads: lane (g, c) gets V[16 ti + 4 g + r][c]) and the
  //      first k step's K
  hook(0);
  __builtin_amdgcn_s_setprio(0);
  u32x2 vraw[NC][4];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int ti = 0; ti < 4; ++ti)
      vraw[c][ti] = lds_read_tr16(vtile + swz<VRB>(16 * ti + 4 * lg + lr / 4, 2 * (vc0 + 16 * c + 4 * (lr % 4))));
  bf16x8 ka[2][4];
#pragma unroll
  for (int ti = 0; ti < 4; ++ti) ka[0][ti] = kt.frag(ti, 0);
  __builtin_amdgcn_sched_barrier(0);

  // ---- K M0, one k step at a time; the next step's K (after the last, T) arrives
  __builtin_amdgcn_s_setprio(1);
  f32x4 km[NC][4];
  bf16x8 tfr[kTFrags];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    hook(1 + kk);
    if (kk + 1 < NK) {
#pragma unroll
      for (int ti = 0; ti < 4; ++ti) ka[(kk + 1) & 1][ti] = kt.frag(ti, kk + 1);
    } else {
#pragma unroll
      for (int f = 0; f < kTFrags; ++f) tfr[f] = __builtin_bit_cast(bf16x8, tf[f * kWave + lane]);
    }
#pragma unroll
    for (int ti = 0; ti < 4; ++ti)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        km[c][ti] = mma_x2(ka[kk & 1][ti], mb[c][kk], kk == 0 ? zero4() : km[c][ti]);
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- R = diag(beta) V - diag(beta e^G) (K M0), split by 32-row halves
  hook(NK + 1);
  __builtin_amdgcn_s_setprio(0);
  bf16x8 kt0[NT], kt1[NT];
  Frag rb[NC][2];
  auto make_rb = [&](int h) __attribute__((always_inline)) {
    f32x4 R[NC][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int ti = 2 * h + u;
      const f32x4 bta = *reinterpret_cast<const f32x4*>(sc + 0 * kChunk + 16 * ti + 4 * lg);
      const f32x4 bge = *reinterpret_cast<const f32x4*>(sc + 1 * kChunk + 16 * ti + 4 * lg);
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) R[c][u][r] = bta[r] * bf16_elt(vraw[c][ti], r) - bge[r] * km[c][ti][r];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) rb[c][h] = chain_frag(R[c][0], R[c][1]);
  };
  make_rb(0);
  __builtin_amdgcn_sched_barrier(0);

  // ---- Delta = hi(T) R, k step 0 | R rows 32..63; K^T for tokens 0..31 arrives
  hook(NK + 2);
#pragma unroll
  for (int td = 0; td < NT; ++td) kt0[td] = kt.frag_t(td, 0);
  f32x4 D[NC][4];
#pragma unroll
  for (int ti = 0; ti < 4; ++ti)
#pragma unroll
    for (int c = 0; c < NC; ++c) D[c][ti] = mma_x2(tfr[tri_frag(ti, 0)], rb[c][0], zero4());
  make_rb(1);
  __builtin_amdgcn_sched_barrier(0);

  // ---- Delta, k step 1 for row tiles 2, 3 | the weighted Delta rows 0..31,
  //      split; K^T for tokens 32..63 arrives
  hook(NK + 3);
#pragma unroll
  for (int td = 0; td < NT; ++td) kt1[td] = kt.frag_t(td, 1);
#pragma unroll
  for (int ti = 2; ti < 4; ++ti)
#pragma unroll
    for (int c = 0; c < NC; ++c) D[c][ti] = mma_x2(tfr[tri_frag(ti, 1)], rb[c][1], D[c][ti]);
  Frag db[NC][2];
  auto make_db = [&](int h) __attribute__((always_inline)) {
    f32x4 Dw[NC][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const f32x4 w = *reinterpret_cast<const f32x4*>(sc + 2 * kChunk + 16 * (2 * h + u) + 4 * lg);
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) Dw[c][u][r] = w[r] * D[c][2 * h + u][r];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) db[c][h] = chain_frag(Dw[c][0], Dw[c][1]);
  };
  make_db(0);
  const float eg = sc[4 * kChunk];
  __builtin_amdgcn_sched_barrier(0);

  // ---- M1 = e^{G_last} M0 + K^T Dw, tokens 0..31 | weighted Delta rows 32..63
  hook(NK + 4);
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int td = 0; td < NT; ++td)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int r = 0; r < 4; ++r) M[c][td][r] *= eg;
      M[c][td] = mma_x2(kt0[td], db[c][0], M[c][td]);
    }
  make_db(1);
  __builtin_amdgcn_sched_barrier(0);

  // ---- tokens 32..63 | split of M1 for the next chunk
  hook(NK + 5);
#pragma unroll
  for (int kk = 0; kk < NK; ++kk)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      M[c][2 * kk] = mma_x2(kt1[2 * kk], db[c][1], M[c][2 * kk]);
      M[c][2 * kk + 1] = mma_x2(kt1[2 * kk + 1], db[c][1], M[c][2 * kk + 1]);
      mb[c][kk] = chain_frag(M[c][2 * kk], M[c][2 * kk + 1]);
    }
}

// f(j, b) for chunks j = 0 .. n - 1, b (a compile-time constant) the LDS buffer
// of chunk j.  The loop takes as many chunks a turn as there are buffers, so
// every LDS address of a chunk is a lane address that never changes plus a
// constant.
template <int BUFFERS, typename F>
__device__ __forceinline__ void each_chunk(int n, F&& f) {
  for (int j = 0; j < n; j += BUFFERS) {
    f(j, std::integral_constant<int, 0>{});
    if constexpr (BUFFERS > 1) {
      if (j + 1 < n) f(j + 1, std::integral_constant<int, 1>{});
    }
    if constexpr (BUFFERS > 2) {
      if (j + 2 < n) f(j + 2, std::integral_constant<int, 2>{});
    }
  }
}

// The loop of the DMA wave beside output waves, over chunks 0 .. n - 1 into a
// ring of RING buffers.
// With three buffers and a long chain it runs two chunks ahead, so a chunk's
// operands have two chunks' time to arrive: over 32768 tokens, whose records
// and inputs come from HBM, the forward scan takes 750 us so and 900 one chunk
// ahead.  A short chain stays one ahead: its first chunk then waits for its own
// operands alone (16 chunks 27.5 against 28.5 us).  The barriers are those of
// the recurrence and output waves' loops.
constexpr int kFarChunks = 32;
template <int RING, typename D>
__device__ __forceinline__ void dma_ring(D& dma, lds_byte* lds, int buf_bytes, int n) {
  static_assert(RING == 2 || RING == 3, "one or two chunks ahead");
  const int ahead = RING == 3 && n >= kFarChunks ? 2 : 1;
  int b = 0;
  // the next chunk's DMA, while the compute waves work on the other buffers
  auto issue = [&]() __attribute__((always_inline)) {
    dma.chunk(lds + b * buf_bytes);
    b = b + 1 == RING ? 0 : b + 1;
  };
  // the next chunk's has landed, the youngest, a further one's, may be under way
  auto wait_next = [&](bool further) __attribute__((always_inline)) {
    if (further) wait_dma_but<D::kPerWave>();
    else wait_dma();
  };
  if (n > 0) issue();
  if (ahead == 2) issue();
  wait_next(ahead == 2);
  lds_barrier();
  for (int j = 0; j < n; ++j) {
    const bool more = j + ahead < n;
    if (more) issue();
    lds_barrier();   // mid-chunk
    wait_next(more && ahead == 2);
    lds_barrier();   // the next chunk's operands are in LDS; this chunk's buffer is free
  }
}

// Shared set-up of a scan workgroup for sequence n, value head h, state
// columns [col0, col0 + VC).
struct ScanUnit {
  int n, h, kh, tok0, len, slot0, nch;
};
// `slot` is the workgroup's logical sequence slot; `order` (NULL or n = 0:
// identity) maps it to the sequence, longest first.  When a scan grid exceeds
// the chip, workgroups start in logical order as earlier ones finish, so a
// long sequence that comes late in a varlen batch would finish late.
__device__ __forceinline__ ScanUnit scan_unit(const int32_t* __restrict__ cu, int slot, int h, int hv, int hk,
                                              const SeqOrder* order = nullptr) {
  const int n = (order && order->n > 0) ? order->seq[slot] : slot;
  ScanUnit u;
  u.n = n;
  u.h = h;
  u.kh = h / (hv / hk);
  u.tok0 = cu[n];
  u.len = cu[n + 1] - u.tok0;
  u.slot0 = u.tok0 / kChunk + n;
  u.nch = (u.len + kChunk - 1) / kChunk;
  return u;
}

template <typename L, typename TIn>
__device__ __forceinline__ ChunkSrc chunk_src(const ScanUnit& u, int ci, int hk, int hv, int dv, int col0,
                                              const TIn* v, const TIn* kin, const TIn* qin, const u32x4* Kw,
                                              const u32x4* Tw, const float* Sw, const u32x4* Pw) {
  const int64_t srec = static_cast<int64_t>(u.slot0 + ci);
  const int64_t vrow = static_cast<int64_t>(hv) * dv;
  ChunkSrc c;
  c.krec = reinterpret_cast<const unsigned char*>(Kw) + (srec * hk + u.kh) * L::kKBytes;
  c.krow = static_cast<int64_t>(hk) * L::kDK;
  const int64_t krow0 = static_cast<int64_t>(u.tok0 + ci * kChunk) * c.krow + static_cast<int64_t>(u.kh) * L::kDK;
  c.k0 = kin + krow0;
  c.q0 = qin ? qin + krow0 : nullptr;
  c.trec = reinterpret_cast<const unsigned char*>(Tw) + (srec * hv + u.h) * L::kTBytes;
  c.prec = reinterpret_cast<const unsigned char*>(Pw) + (srec * hv + u.h) * static_cast<int64_t>(kPRecordBytes);
  c.srow = reinterpret_cast<const unsigned char*>(Sw) + (srec * hv + u.h) * L::kSBytes;
  c.v0 = v + static_cast<int64_t>(u.tok0 + ci * kChunk) * vrow + static_cast<int64_t>(u.h) * dv + col0;
  c.clen = min(kChunk, u.len - ci * kChunk);
  return c;
}

// The DMA of a bf16 scan's chunks, one after the other, as issued by wave w of
// NW: its share is the same jobs every chunk (key, query and value row blocks
// w, w + NW, .., then T blocks and scalars), so a chunk costs it a few scalar
// additions and four vector instructions per row block.  With the addresses
// formed anew for every job, the issuing waves of the wide scan spent ~250
// scalar instructions and two dozen branches a chunk on them.
template <typename L, int NW, bool FWD>
struct ScanDma {
  static_assert(!L::kSplit, "key rows come from the inputs");
  static_assert(L::kOffP == L::kOffT + 1024 * L::kTJobs && L::kOffS == L::kOffP + 1024 * L::kPJobs, "T, P, scalars");
  static constexpr int kRB = 2 * L::kDK, kKPieces = kRB / 16, kKRows = 1024 / kRB;   // key rows
  static constexpr int kKBlocks = kChunk * kRB / 1024;
  // eight waves: four fetch the keys, four the queries
  static constexpr int kKW = NW == 8 ? 4 : NW;
  static_assert(kKBlocks % kKW == 0 && (NW <= 4 || (NW == 8 && FWD)), "equal shares of the key rows");
  static constexpr int kKPer = kKBlocks / kKW;
  static constexpr int kKQ = kKPer * (FWD && NW <= 4 ? 2 : 1);
  static constexpr int kPieces = L::kVRowBytes / 16, kRowsPerBlock = 1024 / L::kVRowBytes;
  static constexpr int kVPer = (L::kVJobs + NW - 1) / NW;
  static constexpr int kTP = L::kTJobs + L::kPJobs;
  static constexpr int kTSPer = (kTP + 2 + NW - 1) / NW;   // T blocks, P blocks if any, then the scalars' two
  static constexpr int kPerWave = kKQ + kVPer + kTSPer;

  int w, lane;
  int left;                               // rows from the chunk's first to the sequence's end
  uint32_t krow_b, vrow_b, t_b, p_b, s_b; // bytes between rows, and between chunks' records
  const unsigned char *k, *q, *v, *t, *p, *s;   // the chunk's first rows and records
  uint32_t krow, kpiece, vrow, vpiece;    // this lane's row and piece of the wave's first row blocks

  __device__ __forceinline__ void start(const ScanUnit& u, int ci, int wave, int lane_, int hk, int hv, int dv,
                                        int col0, const uint16_t* vin, const uint16_t* kin, const uint16_t* qin,
                                        const u32x4* Kw, const u32x4* Tw, const float* Sw, const u32x4* Pw) {
    const ChunkSrc c = chunk_src<L>(u, ci, hk, hv, dv, col0, vin, kin, qin, Kw, Tw, Sw, Pw);
    w = wave;
    lane = lane_;
    left = u.len - ci * kChunk;
    krow_b = static_cast<uint32_t>(hk) * kRB;
    vrow_b = static_cast<uint32_t>(hv) * static_cast<uint32_t>(dv) * 2u;
    t_b = static_cast<uint32_t>(hv) * L::kTBytes;
    p_b = static_cast<uint32_t>(hv) * static_cast<uint32_t>(kPRecordBytes);
    s_b = static_cast<uint32_t>(hv) * L::kSBytes;
    k = static_cast<const unsigned char*>(NW == 8 && w >= 4 ? c.q0 : c.k0);
    q = static_cast<const unsigned char*>(c.q0);
    v = static_cast<const unsigned char*>(c.v0);
    t = c.trec;
    p = c.prec;
    s = c.srow;
    krow = (w % kKW) * kKRows + lane / kKPieces;
    kpiece = 16u * ((lane % kKPieces) ^ row_swz<kRB>(krow));
    vrow = w * kRowsPerBlock + lane / kPieces;
    vpiece = 16u * ((lane % kPieces) ^ v_swz<L::kVRowBytes>(vrow));
  }
  // Lane offset of row `row` (rows past the chunk's end repeat the last valid
  // row: their beta is 0, so they add nothing).  Strides are below 2^24: at
  // most 65535 heads of 128 bf16.
  __device__ __forceinline__ uint32_t row_off(uint32_t row, uint32_t stride_b, uint32_t piece) const {
    return __umul24(min(row, static_cast<uint32_t>(min(kChunk, left) - 1)), stride_b) + piece;
  }
  // Job J of the wave's share into LDS buffer `base`; `values` false: no value rows.
  template <int J>
  __device__ __forceinline__ void job(lds_byte* base, bool values = true) const {
    if constexpr (J < kKQ) {
      constexpr int i = J % kKPer, row = i * kKW * kKRows;
      constexpr bool isq = J >= kKPer;    // queries after the keys
      const int blk = w % kKW + kKW * i + (isq || (NW == 8 && w >= 4) ? kKBlocks : 0);
      dma16_at(isq ? q : k, row_off(krow + row, krow_b, kpiece ^ (16u * row_swz<kRB>(row))),
               base + L::kOffK + 1024 * blk);
    } else if constexpr (J < kKQ + kVPer) {
      constexpr int i = J - kKQ, row = i * NW * kRowsPerBlock;
      const int blk = w + NW * i;
      if (values && (L::kVJobs % NW == 0 || blk < L::kVJobs))
        dma16_at(v, row_off(vrow + row, vrow_b, vpiece ^ (16u * v_swz<L::kVRowBytes>(row))),
                 base + L::kOffV + 1024 * blk);
    } else {
      // block of T, then of P, then of the scalars (1 KiB and 256 bytes)
      const int x = w * kTSPer + (J - kKQ - kVPer);
      const unsigned char* src = x < L::kTJobs ? t + 1024 * x : x < kTP ? p + 1024 * (x - L::kTJobs) : s + 1024 * (x - kTP);
      if (x <= kTP || (x == kTP + 1 && lane < 16)) dma16_at(src, 16u * lane, base + L::kOffT + 1024 * x);
    }
  }
  template <int J0, int J1>
  __device__ __forceinline__ void jobs(lds_byte* base, bool values = true) const {
    if constexpr (J0 < J1) {
      job<J0>(base, values);
      jobs<J0 + 1, J1>(base, values);
    }
  }
  __device__ __forceinline__ void next() {
    k += static_cast<uint64_t>(krow_b) * kChunk;
    q += static_cast<uint64_t>(krow_b) * kChunk;
    v += static_cast<uint64_t>(vrow_b) * kChunk;
    t += t_b;
    p += p_b;
    s += s_b;
    left -= kChunk;
  }
  // A whole chunk's share, and on to the next chunk.
  __device__ __forceinline__ void chunk(lds_byte* base, bool values = true) {
    jobs<0, kPerWave>(base, values);
    next();
  }
  // The p-th of N parts of it (p a constant in each instance).
  template <int N, int P = 0>
  __device__ __forceinline__ void phase(int p, lds_byte* base) {
    if constexpr (P < N) {
      if (p == P) {
        jobs<P * kPerWave / N, (P + 1) * kPerWave / N>(base);
        if (P == N - 1) next();
      } else {
        phase<N, P + 1>(p, base);
      }
    }
  }
};

// The same for fp32 inputs, whose K record is contiguous: wave w takes jobs w,
// w + NW, ..
template <typename L, typename TIn, int NW>
struct RecordDma {
  static constexpr int kPerWave = (L::kJobs + NW - 1) / NW;
  ChunkSrc c;
  int w, lane, left;
  int64_t vrow, k_b, t_b, s_b;   // elements between value rows; bytes between chunks' records
  __device__ __forceinline__ void start(const ScanUnit& u, int ci, int wave, int lane_, int hk, int hv, int dv,
                                        int col0, const TIn* vin, const TIn* kin, const TIn* qin, const u32x4* Kw,
                                        const u32x4* Tw, const float* Sw, const u32x4* Pw) {
    c = chunk_src<L>(u, ci, hk, hv, dv, col0, vin, kin, qin, Kw, Tw, Sw, Pw);
    w = wave;
    lane = lane_;
    left = u.len - ci * kChunk;
    vrow = static_cast<int64_t>(hv) * dv;
    k_b = static_cast<int64_t>(hk) * L::kKBytes;
    t_b = static_cast<int64_t>(hv) * L::kTBytes;
    s_b = static_cast<int64_t>(hv) * L::kSBytes;
  }
  __device__ __forceinline__ void jobs(lds_byte* base, int j0, int j1, bool values = true) const {
    constexpr int kV0 = L::kKJobs + L::kTJobs;   // first value row job
#pragma unroll
    for (int jj = j0; jj < j1; ++jj) {
      const int j = w + NW * jj;
      if (!values && j >= kV0 && j < kV0 + L::kVJobs) continue;
      if (j < L::kJobs) dma_job<L, TIn>(c, vrow, base, j, lane);
    }
  }
  __device__ __forceinline__ void next() {
    c.krec += k_b;
    c.trec += t_b;
    c.srow += s_b;
    c.v0 = static_cast<const TIn*>(c.v0) + vrow * kChunk;
    left -= kChunk;
    c.clen = min(kChunk, left);
  }
  __device__ __forceinline__ void chunk(lds_byte* base, bool values = true) {
    jobs(base, 0, kPerWave, values);
    next();
  }
  template <int N>
  __device__ __forceinline__ void phase(int p, lds_byte* base) {
    if (p < N) jobs(base, p * kPerWave / N, (p + 1) * kPerWave / N);
    if (p == N - 1) next();
  }
};
template <typename L, typename TIn, int NW, bool FWD>
struct ChunkDmaOf { using type = ScanDma<L, NW, FWD>; };
template <typename L, int NW, bool FWD>
struct ChunkDmaOf<L, float, NW, FWD> { using type = RecordDma<L, float, NW>; };
template <typename L, typename TIn, int NW, bool FWD>
using ChunkDma = typename ChunkDmaOf<L, TIn, NW, FWD>::type;

// Per-wave state load/store and the deferred output store.
template <int DK>
__device__ __forceinline__ void load_state(const float* __restrict__ state_in, int64_t sbase, int dv, int lg,
                                           f32x4 (&M)[DK / 16], Frag (&mb)[DK / 32]) {
#pragma unroll
  for (int td = 0; td < DK / 16; ++td)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      M[td][r] = state_in ? state_in[sbase + static_cast<int64_t>(strow(td, lg, r)) * dv] : 0.f;
#pragma unroll
  for (int kk = 0; kk < DK / 32; ++kk) mb[kk] = chain_frag(M[2 * kk], M[2 * kk + 1]);
}
// Stores a chunk's outputs (`pout` as chunk_step leaves it) for the wave whose
// first column is `colw`; rows past the chunk's end fall outside the buffer
// range and are dropped by the hardware.
template <typename TIn>
__device__ __forceinline__ void store_chunk_out(TIn* o, const ScanUnit& u, int ci, int hv, int dv, int colw,
                                                int lane, const f32x4 (&pout)[4]) {
  constexpr int E = static_cast<int>(sizeof(TIn));
  const int64_t vrow = static_cast<int64_t>(hv) * dv;
  const int row_bytes = static_cast<int>(vrow) * E;
  const int clen = min(kChunk, u.len - ci * kChunk);
  const __amdgpu_buffer_rsrc_t r =
      out_rsrc(o + static_cast<int64_t>(u.tok0 + ci * kChunk) * vrow + static_cast<int64_t>(u.h) * dv,
               clen * row_bytes);
  const int voff = (lane % 16) * row_bytes + (colw + 4 * (lane / 16)) * E;
#pragma unroll
  for (int ti = 0; ti < 4; ++ti) store_out4(r, voff + 16 * ti * row_bytes, pout[ti], o);
}

// ---------------------------------------------------------------- latency kernel
// grid = N x Hv x d_v/32, one workgroup per CU.  Used when this grid fits on
// the chip at once, where per-chunk latency is all that matters.  Tail replay:
// two compute waves (16 columns each) and one wave that only issues DMA.  With
// outputs: the two waves that carry the recurrence hand Delta and the split
// state to two output waves (one per 16 columns), so the outputs' products
// stay off the sequential chain, and a fifth wave issues the DMA.
constexpr int kColsPerGroup = 32;
// With outputs: roles of the workgroup's waves (waves go to the four SIMDs in
// turn).
constexpr int kOutTiles = 4, kOutCols = 16 * kOutTiles;   // of a throughput workgroup with outputs
enum ColsRole { kRoleChain, kRoleOut, kRoleDma };
constexpr int cols_dma_waves(bool split, int tiles) { return split || tiles == kOutTiles ? 0 : 1; }
constexpr int cols_threads(bool fwd, bool split, int tiles = 2) {
  return (fwd ? 2 * tiles + cols_dma_waves(split, tiles) : 3) * kWave;
}
// DMA wave first, then the recurrence waves, then the output waves.
__device__ __forceinline__ int cols_role(bool split, int tiles, int wave) {
  const int x = wave - cols_dma_waves(split, tiles);
  return x < 0 ? kRoleDma : x < tiles ? kRoleChain : kRoleOut;
}
__device__ __forceinline__ int cols_tile(bool split, int tiles, int wave) {
  const int x = wave - cols_dma_waves(split, tiles);
  return x < 0 ? 0 : x % tiles;
}

template <typename TIn, int DK, int COLS = kColsPerGroup>
using ColsLds = ScanLds<TIn, DK, COLS, false, false>;

// Tail replay of bf16 inputs whose grid does not fit on the chip at once (a
// throughput batch) may run the wide column scan (see TailScan): COLS = 128 columns (a whole
// head; 64 for d_v = 64) per workgroup, two 16-column tiles per compute wave
// (chunk_step_tiles: the K, T and K^T operands are read from LDS once for both
// tiles), no DMA wave (each compute wave issues a share of the next chunk's
// DMA), and two workgroups per CU, so every SIMD holds two waves whose chains
// interleave.  Measured on MI355X (16 sequences x 32 heads x 52 chunks):
// 1.25x the columns per CU per unit time of the 64-column workgroup of four
// one-tile waves and a DMA wave it replaces.
constexpr int kWideTiles = 2;   // 16-column tiles per compute wave
constexpr int kDmaPhases = 4;   // parts of a chunk over which its compute waves issue the next one's DMA
constexpr int cols_wide_threads(int cols) { return cols / (16 * kWideTiles) * kWave; }

// Tail replay in two halves: the recurrence over a chunk is affine in the
// state, M1 = A_c M0 + B_c with A_c = e^{G_last} I - K^T diag(e^{G_last - G}) T
// diag(beta e^G) K (d_k x d_k), so the state after chunks [0, n) from zero is
// A M' + M'' where M' is the state after the first c1 chunks, M'' the state
// after the remaining chunks started from zero, and A the product of their
// A_c: the same recurrence run with V = 0 from M0 = I.  The parts run side by
// side in one launch (k_scan_cols_split):
//   first half  (kFirstHalf):  chunks [0, c1), zero start, state -> state_out
//   second half (kSecondHalf): chunks [c1, n), zero start, state -> m2, and
//                              identity start with V = 0, d_k columns -> a2
// and k_state_combine forms A M' + M'' in state_out.  Each part is the
// unsplit scan's arithmetic on its chunks.  The first half runs 32 columns
// per workgroup, the second 64 (four waves read the chunk's operands from LDS,
// and the part starts later), so the first half takes the first
// round(0.54 n) chunks: on MI355X at n = 52 and 26 the halves then end
// closest together (28 of 52: the split scan 47.0 -> 46.3 us against 29).
enum ScanPart { kWhole = 0, kFirstHalf = 1, kSecondHalf = 2 };
struct SplitOut {
  float* m2;   // [N, Hv, d_k, d_v] second half from zero
  float* a2;   // [N, Hv, d_k, d_k] second half's transition, transposed (A^T)
};
__device__ __forceinline__ int split_point(int nch) { return (27 * nch + 25) / 50; }

// One column-split workgroup (block `block` of `nblocks`), LDS in `lds`, COLS
// columns per workgroup, NC tiles of 16 columns per compute wave.  Waves 0 ..
// COLS / (16 NC) - 1 compute.  With DMA_WAVE the next issues the DMA and any
// further waves only take part in the barriers; without, the compute waves
// issue the next chunk's DMA themselves, a share at each phase of the chunk
// (multi-tile steps only).
template <typename TIn, int DK, int COLS = kColsPerGroup, int PART = kWhole, int NC = 1, bool DMA_WAVE = true>
__device__ __forceinline__ void scan_cols_body(lds_byte* lds_l, int block, int nblocks,
                                               const int32_t* __restrict__ cu, int32_t hk, int32_t hv,
                                               int32_t dv, const TIn* __restrict__ v,
                                               const TIn* __restrict__ kin, const u32x4* __restrict__ Kw,
                                               const u32x4* __restrict__ Tw, const float* __restrict__ Sw,
                                               float* __restrict__ state_out, SplitOut split = {},
                                               const SeqOrder* order = nullptr) {
  using L = ColsLds<TIn, DK, COLS>;
  static_assert(L::kBuffers == 2, "the next chunk's DMA runs beside a chunk");
  constexpr bool SPLIT = PART != kWhole;
  constexpr int NT = DK / 16;
  constexpr int CW = COLS / (16 * NC);   // compute waves
  static_assert(CW * 16 * NC == COLS, "whole column tiles per wave");
  static_assert(DMA_WAVE || NC > 1, "the compute waves issue the DMA in multi-tile steps");
  const int tid = threadIdx.x;
  // wave index made provably uniform: DMA destinations (M0) stay scalar
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const bool data_wave = DMA_WAVE && wave >= CW;
  const bool dma_wave = DMA_WAVE && wave == CW;
  const int lane = tid % kWave, lg = lane / 16, lr = lane % 16;
  const int ngroups = PART == kSecondHalf ? dv / COLS + DK / COLS : dv / COLS;
  // logical unit: the column groups of a value head, then the value heads of a
  // key head, are adjacent and one cluster (same XCD, shared records in its L2)
  const int unit = xcd_cluster_remap(block, nblocks, ngroups * (hv / hk));
  const ScanUnit u = scan_unit(cu, unit / (ngroups * hv), (unit / ngroups) % hv, hv, hk, order);
  // this workgroup's chunks [cb, ce), columns, start and destination
  int g = unit % ngroups, cb = 0, ce = u.nch, ld = dv;
  bool ident = false;
  float* dst = state_out;
  if constexpr (PART == kFirstHalf) {
    ce = split_point(u.nch);
  } else if constexpr (PART == kSecondHalf) {
    cb = split_point(u.nch);
    if (g < dv / COLS) {
      dst = split.m2;
    } else {
      g -= dv / COLS;
      ident = true;
      ld = DK;
      dst = split.a2;
    }
  }
  const int col0 = COLS * g;
  const int colw = col0 + 16 * NC * wave;   // the wave's first column; tile c: colw + 16 c + lr
  // the chunks' DMA, in order: all of it on the DMA wave, or an equal share on
  // each compute wave (the transition's value rows are the zeros written below)
  constexpr int NI = DMA_WAVE ? 1 : CW;
  ChunkDma<L, TIn, NI, false> dma;
  if (DMA_WAVE ? dma_wave : true)
    dma.start(u, cb, DMA_WAVE ? 0 : wave, lane, hk, hv, dv, ident ? 0 : col0, v, kin, nullptr, Kw, Tw, Sw,
              nullptr);

  const int64_t sbase = (static_cast<int64_t>(u.n) * hv + u.h) * DK * ld + colw + lr;   // tile c: + 16 c
  if (SPLIT && ident) {
    // the transition's V tiles (both buffers) are zero
    for (int b = 0; b < L::kBuffers; ++b)
      for (int x = 16 * tid; x < L::kVBytes; x += 16 * static_cast<int>(blockDim.x))
        *reinterpret_cast<__attribute__((address_space(3))) u32x4*>(lds_l + b * L::kBytes + L::kOffV + x) =
            u32x4{0u, 0u, 0u, 0u};
  }
  const int nch = ce - cb;
  // The data waves and the compute waves run loops of their own with the same
  // barriers (one before the first chunk and one per chunk), so the state lives
  // in the compute waves' loop alone.
  if (data_wave) {
    if (dma_wave && nch > 0) {
      dma.chunk(lds_l, !ident);
      wait_dma();
    }
    __syncthreads();
    for (int j = 0; j < nch; ++j) {
      const int b = j & 1;
      if (dma_wave && j + 1 < nch) {
        dma.chunk(lds_l + (b ^ 1) * L::kBytes, !ident);   // lands while the compute waves work on buffer b
        wait_dma();
      }
      __syncthreads();     // next chunk's operands are in LDS; this buffer is free
    }
    return;
  }

  f32x4 M[NC][NT];
  Frag mb[NC][DK / 32];
  if (SPLIT && ident) {
    // M0 = identity columns
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int td = 0; td < NT; ++td)
#pragma unroll
        for (int r = 0; r < 4; ++r) M[c][td][r] = (strow(td, lg, r) == colw + 16 * c + lr) ? 1.f : 0.f;
#pragma unroll
      for (int kk = 0; kk < DK / 32; ++kk) mb[c][kk] = chain_frag(M[c][2 * kk], M[c][2 * kk + 1]);
    }
  } else {
#pragma unroll
    for (int c = 0; c < NC; ++c)
      load_state<DK>(nullptr, 0, ld, lg, M[c], mb[c]);
  }
  if (!DMA_WAVE && nch > 0) {
    dma.chunk(lds_l, !ident);
    wait_dma();
  }
  __syncthreads();
  auto chunk = [&](int j, auto bc) __attribute__((always_inline)) {
    const int b = bc;
    const unsigned char* buf = (const unsigned char*)(lds_l + b * L::kBytes);
    if constexpr (NC > 1) {
      // without a DMA wave: the next chunk's share, spread over the phases
      const bool prefetch = !DMA_WAVE && j + 1 < nch;
      chunk_step_tiles<L, DK, NC>(buf, 16 * NC * wave, lane, M, mb, [&](int p) __attribute__((always_inline)) {
        if constexpr (!DMA_WAVE) {
          if (prefetch) dma.template phase<kDmaPhases>(p, lds_l + (b ^ 1) * L::kBytes);
        }
      });
      if (!DMA_WAVE) wait_dma();   // this wave's share of the next chunk has landed
    } else {
      f32x4 none[4];
      chunk_step<L, DK, false, false>(buf, 16 * wave, lane, M[0], mb[0], none, [](int) {});
    }
    __syncthreads();     // next chunk's operands are in LDS (every wave's share)
  };
  // The buffers in turn with constant LDS addresses, but for bf16 chains of d_k =
  // 64 in 64 columns: their short chunk gains less from them than the doubled
  // loop costs (one of 52 chunks among 6 sequences of 32 heads: 68.9 us so, 65.6
  // with the buffer as a variable; at d_k = 128 89.2 and 89.5, and the two halves'
  // split scan is ahead with constants, 42.0 against 42.5).
  if constexpr (DK == 64 && COLS == kSplitCols2 && NC == 1 && !SPLIT && !L::kSplit) {
    for (int j = 0; j < nch; ++j) chunk(j, j & 1);
  } else {
    each_chunk<L::kBuffers>(nch, chunk);
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if (SPLIT && ident) {
      // the transition goes out transposed, A^T [d_k x d_k]: a lane's four
      // rows of its column are one 16-byte piece of that row of A^T
      float* at = dst + ((static_cast<int64_t>(u.n) * hv + u.h) * DK + colw + 16 * c + lr) * DK;
#pragma unroll
      for (int td = 0; td < NT; ++td) *reinterpret_cast<f32x4*>(at + strow(td, lg, 0)) = M[c][td];
    } else if (dst) {
#pragma unroll
      for (int td = 0; td < NT; ++td)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          dst[sbase + 16 * c + static_cast<int64_t>(strow(td, lg, r)) * ld] = M[c][td][r];
    }
  }
}

// LDS of the workgroup with outputs: chunk buffers (P read from global
// memory) and, per 16-column tile, the exchange from the recurrence wave to
// the output wave: Delta (4 KiB) and the split state (d_k / 32 x 2 KiB).
template <typename TIn, int DK, int TILES = 2>
struct ColsOutLayout {
  using L = ScanLds<TIn, DK, 16 * TILES, true, false>;
  static constexpr int kDBytes = 4 * kWave * 16;
  static constexpr int kMBytes = DK / 32 * 2 * kWave * 16;
  static constexpr int kTileBytes = kDBytes + kMBytes;
  static constexpr int fits(int n) { return n * L::kBytes + TILES * kTileBytes <= kLdsBytes; }
  static constexpr int kBuffers = cols_dma_waves(L::kSplit, TILES) > 0 && fits(3) ? 3 : fits(2) ? 2 : 1;
  static constexpr int kOffX = kBuffers * L::kBytes;
  static constexpr int kBytes = kOffX + TILES * kTileBytes;
  static_assert(kBytes <= kLdsBytes, "column scan with outputs does not fit in LDS");
};

// One column-split workgroup with outputs (block `block` of `nblocks`), LDS in
// `lds_l`: TILES waves carry the recurrence of 16 columns each (chunk_step
// without outputs, exporting Delta before its region 5 and the split of M1 at
// its end) and TILES waves write the outputs of the same columns:
//   before the mid-chunk barrier: (Q M0)^T from the split M0 of the chunk;
//   after it: O^T = diag-scaled (Q M0)^T + Delta^T P^T, stored at the start
//   of the next chunk.
// The products are those of chunk_step with outputs, in the same order, so the
// results are the same bit for bit.
template <typename TIn, int DK, int TILES = 2>
__device__ __forceinline__ void scan_cols_out_body(lds_byte* lds_l, int block, int nblocks,
                                                   const int32_t* __restrict__ cu, int32_t hk, int32_t hv,
                                                   int32_t dv, const TIn* __restrict__ v,
                                                   const TIn* __restrict__ kin, const TIn* __restrict__ qin,
                                                   const u32x4* __restrict__ Kw, const u32x4* __restrict__ Tw,
                                                   const float* __restrict__ Sw, const u32x4* __restrict__ Pw,
                                                   const float* __restrict__ state_in, TIn* __restrict__ o,
                                                   float* __restrict__ state_out,
                                                   const SeqOrder* order = nullptr) {
  using CL = ColsOutLayout<TIn, DK, TILES>;
  using L = typename CL::L;
  constexpr bool SPLIT = L::kSplit;
  constexpr int NT = DK / 16, NK = DK / 32;
  constexpr int NKA = ka_frags(DK);
  constexpr int NKF = L::kKFrags;
  constexpr int DW = cols_dma_waves(SPLIT, TILES);
  constexpr bool TWO = CL::kBuffers > 1;
  // Output waves beside a DMA wave store a chunk's outputs at once (32768 bf16
  // tokens: 855 us so, 900 in the next chunk, with two buffers).  Those that
  // issue the DMA wait for it, and for their stores, at the chunk's end: they
  // store in the next chunk.  Only fp32 chunks of d_k = 128, held one at a time,
  // are ahead at once (one of 52 chunks 101.9 us against 103.3, 24 sequences of
  // 6 479 against 484; at d_k = 64 62.9 against 61.6 and 198 against 188, at d_k =
  // 64, d_v = 128 64.4 against 61.8 and 308 against 287).
  constexpr bool kDefer = DW == 0 && !(SPLIT && DK == 128);
  static_assert(TILES == 2 || !SPLIT, "fp32 inputs: two tiles per workgroup");
  static_assert(TWO || DW == 0, "a DMA wave fills the other buffer");
  const int tid = threadIdx.x;
  // wave index made provably uniform: DMA destinations (M0) stay scalar
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int role = cols_role(SPLIT, TILES, wave);
  const int tile = cols_tile(SPLIT, TILES, wave);
  const bool issues = role == (DW > 0 ? kRoleDma : kRoleOut);
  const int lane = tid % kWave, lg = lane / 16, lr = lane % 16;
  constexpr int COLS = 16 * TILES;
  const int ngroups = dv / COLS;
  // logical unit: the column groups of a value head, then the value heads of a
  // key head, are adjacent and one cluster (same XCD, shared records in its L2)
  const int unit = xcd_cluster_remap(block, nblocks, ngroups * (hv / hk));
  const int col0 = COLS * (unit % ngroups);
  const ScanUnit u = scan_unit(cu, unit / (ngroups * hv), (unit / ngroups) % hv, hv, hk, order);
  const int colw = col0 + 16 * tile;
  unsigned char* xd = (unsigned char*)(lds_l + CL::kOffX + tile * CL::kTileBytes);
  unsigned char* xm = xd + CL::kDBytes;

  ChunkDma<L, TIn, (DW > 0 ? DW : TILES), true> dma;
  if (issues) dma.start(u, 0, tile, lane, hk, hv, dv, col0, v, kin, qin, Kw, Tw, Sw, Pw);

  // each role runs a loop of its own with the same barriers
  if (DW == 0 && issues && u.nch > 0) dma.chunk(lds_l);
  auto chunk_end = [&](int ci) __attribute__((always_inline)) {
    if (!TWO) {
      lds_barrier();   // every wave is done with the only buffer
      if (issues && ci + 1 < u.nch) dma.chunk(lds_l);
    }
    if (issues) wait_dma();
    lds_barrier();     // next chunk's operands are in LDS; this buffer is free
  };
  if (role == kRoleChain) {
    f32x4 M[NT];
    Frag mb[NK];
    f32x4 none[4];
    const int64_t sbase = (static_cast<int64_t>(u.n) * hv + u.h) * DK * dv + colw + lr;
    load_state<DK>(state_in, sbase, dv, lg, M, mb);
    u32x4* x = reinterpret_cast<u32x4*>(xm);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      x[(2 * kk) * kWave + lane] = __builtin_bit_cast(u32x4, mb[kk].hi);
      x[(2 * kk + 1) * kWave + lane] = __builtin_bit_cast(u32x4, mb[kk].lo);
    }
    lds_barrier();
    each_chunk<CL::kBuffers>(u.nch, [&](int ci, auto bc) __attribute__((always_inline)) {
      const unsigned char* base = (const unsigned char*)(lds_l + decltype(bc)::value * L::kBytes);
      chunk_step<L, DK, false, true>(base, 16 * tile, lane, M, mb, none,
                                     [](int k) __attribute__((always_inline)) {
                                       if (k == 5) lds_barrier();   // Delta is out
                                     },
                                     xd, xm);
      chunk_end(ci);
    });
    if (state_out) {
#pragma unroll
      for (int td = 0; td < NT; ++td)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          state_out[sbase + static_cast<int64_t>(strow(td, lg, r)) * dv] = M[td][r];
    }
  } else if (role == kRoleOut) {
    f32x4 pout[4];
    if (issues) wait_dma();
    lds_barrier();
    each_chunk<CL::kBuffers>(u.nch, [&](int ci, auto bc) __attribute__((always_inline)) {
      constexpr int b = decltype(bc)::value;
      const unsigned char* base = (const unsigned char*)(lds_l + b * L::kBytes);
      // P (split, six nonzero fragments) from global memory
      const u32x4* pg = Pw + (static_cast<int64_t>(u.slot0 + ci) * hv + u.h) * (2 * kTFrags * kWave);
      Frag pfr[kTFrags];
      auto load_p = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < kTFrags; ++f) {
          pfr[f].hi = __builtin_bit_cast(bf16x8, pg[f * kWave + lane]);
          pfr[f].lo = __builtin_bit_cast(bf16x8, pg[(kTFrags + f) * kWave + lane]);
        }
      };
      load_p();
      __builtin_amdgcn_sched_barrier(0);
      if (DW == 0 && TWO && ci + 1 < u.nch) dma.chunk(lds_l + (b ^ 1) * L::kBytes);
      if (kDefer && ci > 0) store_chunk_out(o, u, ci - 1, hv, dv, colw, lane, pout);
      // (Q M0)^T: A = split M0 from the recurrence wave, B = Q fragments
      const u32x4* kf = reinterpret_cast<const u32x4*>(base + L::kOffK);
      const KeyTile<DK> qt{base + L::kOffK, lane};
      const u32x4* x = reinterpret_cast<const u32x4*>(xm);
      Frag m0[NK];
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        m0[kk].hi = __builtin_bit_cast(bf16x8, x[(2 * kk) * kWave + lane]);
        m0[kk].lo = __builtin_bit_cast(bf16x8, x[(2 * kk + 1) * kWave + lane]);
      }
      // one token tile's Q fragments at a time (fp32 inputs carry hi and lo)
      f32x4 qm[4];
#pragma unroll
      for (int ti = 0; ti < 4; ++ti) {
        Frag qa[NK];
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
          if constexpr (SPLIT) {
            const int f = NKA + ti * NK + kk;
            qa[kk].hi = __builtin_bit_cast(bf16x8, kf[f * kWave + kslot(lane)]);
            qa[kk].lo = __builtin_bit_cast(bf16x8, kf[(NKF + f) * kWave + kslot(lane)]);
          } else {
            qa[kk].hi = qt.frag(4 + ti, kk);
          }
        }
        qm[ti] = zero4();
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) qm[ti] = mma_b<SPLIT>(m0[kk], qa[kk], qm[ti]);
      }
      lds_barrier();   // Delta is in
      const f32x4* xdv = reinterpret_cast<const f32x4*>(xd);
      f32x4 D[4];
#pragma unroll
      for (int ti = 0; ti < 4; ++ti) D[ti] = xdv[ti * kWave + lane];
      const Frag dd0 = chain_frag(D[0], D[1]);
      const Frag dd1 = chain_frag(D[2], D[3]);
      const float* sc = reinterpret_cast<const float*>(base + L::kOffS);
#pragma unroll
      for (int ti = 0; ti < 4; ++ti) {
        const float qe = sc[3 * kChunk + 16 * ti + lr];
#pragma unroll
        for (int r = 0; r < 4; ++r) pout[ti][r] = qe * qm[ti][r];
        pout[ti] = mma_x3(dd0, pfr[tri_frag(ti, 0)], pout[ti]);
        if (ti >= 2) pout[ti] = mma_x3(dd1, pfr[tri_frag(ti, 1)], pout[ti]);
      }
      if (!kDefer) store_chunk_out(o, u, ci, hv, dv, colw, lane, pout);
      chunk_end(ci);
    });
    if (kDefer && u.nch > 0) store_chunk_out(o, u, u.nch - 1, hv, dv, colw, lane, pout);
  } else if constexpr (DW > 0) {
    dma_ring<CL::kBuffers>(dma, lds_l, L::kBytes, u.nch);
  }
}

template <typename TIn, int DK, bool FWD, int TILES = 2>
__global__ __launch_bounds__(cols_threads(FWD, sizeof(TIn) == 4, TILES)) __attribute__((amdgpu_waves_per_eu(1, 1)))
void k_scan_cols(const int32_t* __restrict__ cu, int32_t hk, int32_t hv, int32_t dv,
                 const TIn* __restrict__ v, const TIn* __restrict__ kin, const TIn* __restrict__ qin,
                 const u32x4* __restrict__ Kw, const u32x4* __restrict__ Tw,
                 const float* __restrict__ Sw, const u32x4* __restrict__ Pw,
                 const float* __restrict__ state_in, TIn* __restrict__ o, float* __restrict__ state_out) {
  if constexpr (FWD) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[ColsOutLayout<TIn, DK, TILES>::kBytes];
    scan_cols_out_body<TIn, DK, TILES>((lds_byte*)lds, blockIdx.x, gridDim.x, cu, hk, hv, dv, v, kin, qin, Kw, Tw,
                                       Sw, Pw, state_in, o, state_out);
  } else {
    using L = ColsLds<TIn, DK>;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[L::kBuffers * L::kBytes];
    scan_cols_body<TIn, DK>((lds_byte*)lds, blockIdx.x, gridDim.x, cu, hk, hv, dv, v, kin, Kw, Tw, Sw, state_out);
  }
}

// The scan with output waves, 16 TILES columns per workgroup, over the P
// sequences `order` names (all of them, in index order, when its n is 0; grid
// P x Hv x d_v / (16 TILES), any number of rounds): TILES = 2 for fp32 batches
// that do not fit on the chip, TILES = 4 for bf16 batches and for the sequences
// peeled off a whole-head grid's partly empty last round (see launch_scan).
template <typename TIn, int DK, int TILES>
__global__ __launch_bounds__(cols_threads(true, sizeof(TIn) == 4, TILES))
__attribute__((amdgpu_waves_per_eu(TILES == kOutTiles ? 2 : 1, TILES == kOutTiles ? 2 : 1)))
void k_scan_cols_out_ord(const int32_t* __restrict__ cu, const SeqOrder order, int32_t hk, int32_t hv, int32_t dv,
                          const TIn* __restrict__ v, const TIn* __restrict__ kin, const TIn* __restrict__ qin,
                          const u32x4* __restrict__ Kw, const u32x4* __restrict__ Tw,
                          const float* __restrict__ Sw, const u32x4* __restrict__ Pw,
                          const float* __restrict__ state_in, TIn* __restrict__ o, float* __restrict__ state_out) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[ColsOutLayout<TIn, DK, TILES>::kBytes];
  scan_cols_out_body<TIn, DK, TILES>((lds_byte*)lds, blockIdx.x, gridDim.x, cu, hk, hv, dv, v, kin, qin, Kw, Tw, Sw,
                                     Pw, state_in, o, state_out, &order);
}

// The wide column scan, tail replay only (grid N x Hv x d_v / COLS).
template <typename TIn, int DK, int COLS>
__global__ __launch_bounds__(cols_wide_threads(COLS)) __attribute__((amdgpu_waves_per_eu(COLS / 64, 2)))
void k_scan_cols_wide(const int32_t* __restrict__ cu, const SeqOrder order, int32_t hk, int32_t hv, int32_t dv,
                      const TIn* __restrict__ v, const TIn* __restrict__ kin,
                      const u32x4* __restrict__ Kw, const u32x4* __restrict__ Tw,
                      const float* __restrict__ Sw, float* __restrict__ state_out) {
  using L = ColsLds<TIn, DK, COLS>;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[L::kBuffers * L::kBytes];
  scan_cols_body<TIn, DK, COLS, kWhole, kWideTiles, false>((lds_byte*)lds, blockIdx.x, gridDim.x, cu, hk, hv, dv, v,
                                                           kin, Kw, Tw, Sw, state_out, SplitOut{}, &order);
}

// Tail replay, 64 columns per workgroup: one 16-column tile per compute wave
// beside a DMA wave (the chains of the split scan's second half, which finish a
// chunk sooner than the wide scan's two-tile waves), grid P x Hv x d_v / 64 over
// the P sequences `order` names (all of them when its n is 0).  Used for batches
// whose grid fits on the chip, for those that run in rounds of it (see
// TailScan), and for the sequences of a wide grid's partly empty last round.
template <typename TIn, int DK>
__global__ __launch_bounds__((kSplitCols2 / 16 + 1) * kWave)
void k_scan_cols_64(const int32_t* __restrict__ cu, const SeqOrder order, int32_t hk, int32_t hv, int32_t dv,
                      const TIn* __restrict__ v, const TIn* __restrict__ kin,
                      const u32x4* __restrict__ Kw, const u32x4* __restrict__ Tw,
                      const float* __restrict__ Sw, float* __restrict__ state_out) {
  using L = ColsLds<TIn, DK, kSplitCols2>;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[L::kBuffers * L::kBytes];
  scan_cols_body<TIn, DK, kSplitCols2>((lds_byte*)lds, blockIdx.x, gridDim.x, cu, hk, hv, dv, v, kin, Kw, Tw, Sw,
                                       state_out, SplitOut{}, &order);
}

// Tail replay in two halves, one launch: blocks [0, n_first) run the first
// half kSplitCols1 = 32 columns wide (grid N x Hv x d_v / 32; waves 3 and 4
// only take part in the barriers), the rest the second half and its
// transition kSplitCols2 = 64 columns wide (N x Hv x (d_v + d_k) / 64), one
// 16-column tile per compute wave.  state_out holds the first half's state
// until the combine runs.
constexpr int cols_split_threads() { return (kSplitCols2 / 16 + 1) * kWave; }
template <typename TIn, int DK>
__global__ __launch_bounds__(cols_split_threads())
void k_scan_cols_split(int32_t n_first, const int32_t* __restrict__ cu, int32_t hk, int32_t hv, int32_t dv,
                       const TIn* __restrict__ v, const TIn* __restrict__ kin,
                       const u32x4* __restrict__ Kw, const u32x4* __restrict__ Tw,
                       const float* __restrict__ Sw, float* __restrict__ state_out, float* __restrict__ m2,
                       float* __restrict__ a2) {
  using L1 = ColsLds<TIn, DK, kSplitCols1>;
  using L2 = ColsLds<TIn, DK, kSplitCols2>;
  constexpr int kB1 = L1::kBuffers * L1::kBytes, kB2 = L2::kBuffers * L2::kBytes;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kB1 > kB2 ? kB1 : kB2];
  const int b = blockIdx.x;
  if (b < n_first)
    scan_cols_body<TIn, DK, kSplitCols1, kFirstHalf>((lds_byte*)lds, b, n_first, cu, hk, hv, dv, v, kin, Kw, Tw, Sw,
                                                     state_out);
  else
    scan_cols_body<TIn, DK, kSplitCols2, kSecondHalf>((lds_byte*)lds, b - n_first,
                                                      static_cast<int>(gridDim.x) - n_first, cu, hk, hv, dv, v, kin,
                                                      Kw, Tw, Sw, nullptr, SplitOut{m2, a2});
}

// state = A state + B per (sequence, value head): A^T [d_k x d_k], state and
// B [d_k x d_v], fp32 row-major.  grid N x Hv x d_v / 16; a workgroup owns 16
// whole columns of one state (it reads them all before it writes any) and
// stages those columns in LDS, every load in flight at once.  The product
// runs on fp32 MFMA (16x16x4, fp32 products and sums): wave w takes the
// 16-row tiles w, w + 4, ..; per 4-step slice of k, lane l supplies
// A[16 t + l % 16][k + l / 16] (= A^T[k + l / 16][..], read from memory into
// registers up front) and column l % 16 of row k + l / 16 of the staged
// state, and holds D[4 (l / 16) + i][l % 16] of the tile.  With 8 KiB of LDS
// the combine leaves room for four preparation workgroups per CU beside it
// in k_combine_intra.
constexpr int kCombineThreads = 256;
constexpr int kCombineCols = 16;
template <int DK>
struct CombineLds {
  alignas(16) float ms[DK * kCombineCols];
};

// `block` of `nblocks`: the column groups of one (sequence, head) are one
// cluster on one XCD, so the head's transition is fetched from memory once
// and its other workgroups find it in that XCD's L2.
template <int DK>
__device__ __forceinline__ void combine_body(CombineLds<DK>& sm, int block, int nblocks, int32_t dv,
                                             const float* __restrict__ At, const float* __restrict__ B,
                                             float* __restrict__ state) {
  constexpr int PER = DK * kCombineCols / kCombineThreads;   // staged column values per thread
  constexpr int TILES = DK / 16 / (kCombineThreads / kWave);  // row tiles per wave
  float* ms = sm.ms;
  const int groups = dv / kCombineCols;
  const int unit = xcd_cluster_remap(block, nblocks, groups);
  const int64_t head = unit / groups;
  const int c0 = kCombineCols * (unit % groups);
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int li = lane % 16, lk = lane / 16;
  float* st = state + head * DK * dv + c0;
  const float* bm = B + head * DK * dv + c0;
  const float* at = At + head * DK * DK;
  // the wave's A operands straight from memory (A^T rows are 16 consecutive
  // floats per tile: 64-byte pieces), every load in flight at once
  float av[DK / 4][TILES];
#pragma unroll
  for (int k = 0; k < DK; k += 4)
#pragma unroll
    for (int t = 0; t < TILES; ++t) av[k / 4][t] = at[(k + lk) * DK + 16 * (wave + 4 * t) + li];
  float mv[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int x = tid + kCombineThreads * i;
    mv[i] = st[static_cast<int64_t>(x / kCombineCols) * dv + x % kCombineCols];
  }
  f32x4 acc[TILES];
#pragma unroll
  for (int t = 0; t < TILES; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      acc[t][i] = bm[static_cast<int64_t>(16 * (wave + 4 * t) + 4 * lk + i) * dv + li];
#pragma unroll
  for (int i = 0; i < PER; ++i) ms[tid + kCombineThreads * i] = mv[i];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < DK; k += 4) {
    const float b = ms[(k + lk) * kCombineCols + li];
#pragma unroll
    for (int t = 0; t < TILES; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[k / 4][t], b, acc[t], 0, 0, 0);
  }
#pragma unroll
  for (int t = 0; t < TILES; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) st[static_cast<int64_t>(16 * (wave + 4 * t) + 4 * lk + i) * dv + li] = acc[t][i];
}
template <int DK>
__global__ __launch_bounds__(kCombineThreads)
void k_state_combine(int32_t dv, const float* __restrict__ At, const float* __restrict__ B,
                     float* __restrict__ state) {
  __shared__ CombineLds<DK> sm;
  combine_body<DK>(sm, blockIdx.x, gridDim.x, dv, At, B, state);
}

// The combine of a split tail replay beside the suffix's chunk preparation,
// one launch: blocks [0, n_comb) run k_state_combine, the rest k_intra for the
// suffix chunks (with outputs).  The combine is short and light, so the
// preparation workgroups fill the chip around it.  No workgroup waits for
// another.
template <typename TIn, int DK>
__global__ __launch_bounds__(kCombineThreads)
void k_combine_intra(int32_t n_comb, int32_t dv, const float* __restrict__ At, const float* __restrict__ B,
                     float* __restrict__ state, int32_t slots_s, const int32_t* __restrict__ cu_s, int32_t num_seqs,
                     int32_t hk, int32_t hv, const TIn* __restrict__ q_s, const TIn* __restrict__ k_s,
                     const float* __restrict__ g_s, const float* __restrict__ beta_s, float scale,
                     u32x4* __restrict__ Kw_s, u32x4* __restrict__ Tw_s, float* __restrict__ Sw_s,
                     u32x4* __restrict__ Pw_s) {
  static_assert(kCombineThreads == 4 * kWave, "the preparation body runs on four waves");
  using LC = CombineLds<DK>;
  using LI = IntraLds<TIn, DK, true>;
  constexpr size_t kBytes = sizeof(LC) > sizeof(LI) ? sizeof(LC) : sizeof(LI);
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kBytes];
  const int b = blockIdx.x;
  if (b < n_comb) {
    combine_body<DK>(*reinterpret_cast<LC*>(smem), b, n_comb, dv, At, B, state);
  } else {
    const int i = b - n_comb;
    int slot, h;
    intra_unit(i, slots_s * hv, hv, hv / hk, slot, h);
    intra_body<TIn, DK, true>(*reinterpret_cast<LI*>(smem), slot, h, cu_s, num_seqs, hk, hv,
                              q_s, k_s, g_s, beta_s, scale, Kw_s, Tw_s, Sw_s, Pw_s);
  }
}

// ---------------------------------------------------------------- replay scan + suffix intra
// One launch, two kinds of workgroup (256 threads): blocks [0, n_scan) run the
// column-split tail replay (FWD = false, zero start, final state to
// `state_mid`; the fourth wave only takes part in the barriers), the rest run
// k_intra for the suffix chunks (with outputs), so the suffix's records are
// built on the CUs the replay leaves idle.  No workgroup waits for another.
template <typename TIn, int DK>
__global__ __launch_bounds__(4 * kWave) __attribute__((amdgpu_waves_per_eu(1, 1)))
void k_scan_cols_intra(int32_t n_scan, const int32_t* __restrict__ cu_t, int32_t hk, int32_t hv, int32_t dv,
                       const TIn* __restrict__ v_t, const TIn* __restrict__ k_t, const u32x4* __restrict__ Kw_t,
                       const u32x4* __restrict__ Tw_t, const float* __restrict__ Sw_t,
                       float* __restrict__ state_mid,
                       int32_t slots_s, const int32_t* __restrict__ cu_s, int32_t num_seqs,
                       const TIn* __restrict__ q_s, const TIn* __restrict__ k_s,
                       const float* __restrict__ g_s, const float* __restrict__ beta_s, float scale,
                       u32x4* __restrict__ Kw_s, u32x4* __restrict__ Tw_s, float* __restrict__ Sw_s,
                       u32x4* __restrict__ Pw_s) {
  using LS = ColsLds<TIn, DK>;
  using LI = IntraLds<TIn, DK, true>;
  constexpr size_t kScanBytes = static_cast<size_t>(LS::kBuffers) * LS::kBytes;
  constexpr size_t kBytes = kScanBytes > sizeof(LI) ? kScanBytes : sizeof(LI);
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kBytes];
  if (static_cast<int>(blockIdx.x) < n_scan) {
    scan_cols_body<TIn, DK>((lds_byte*)smem, blockIdx.x, n_scan, cu_t, hk, hv, dv, v_t, k_t, Kw_t, Tw_t, Sw_t,
                            state_mid);
  } else {
    const int i = blockIdx.x - n_scan;
    int slot, h;
    intra_unit(i, slots_s * hv, hv, hv / hk, slot, h);
    intra_body<TIn, DK, true>(*reinterpret_cast<LI*>(smem), slot, h, cu_s, num_seqs, hk, hv,
                              q_s, k_s, g_s, beta_s, scale, Kw_s, Tw_s, Sw_s, Pw_s);
  }
}

// ---------------------------------------------------------------- throughput kernel
// d_v = 128, grid = N x Hv: eight waves (two per SIMD), each 16 columns, sharing
// one copy of the chunk's records per head; every wave issues an equal share of
// the next chunk's DMA, spread over the chunk's regions (fp32 inputs at d_k = 128
// hold one chunk in LDS and issue it between two).  Used for bf16 batches with
// outputs and fp32 tail replay batches beyond the chip (see launch_scan and
// TailScan).
constexpr int kHeadCols = 128;
constexpr int kHeadThreads = kHeadCols / 16 * kWave;

template <typename TIn, int DK, bool FWD>
__global__ __launch_bounds__(kHeadThreads)
void k_scan_head(const int32_t* __restrict__ cu, const SeqOrder order, int32_t hk, int32_t hv,
                 const TIn* __restrict__ v, const TIn* __restrict__ kin, const TIn* __restrict__ qin,
                 const u32x4* __restrict__ Kw, const u32x4* __restrict__ Tw,
                 const float* __restrict__ Sw, const u32x4* __restrict__ Pw,
                 const float* __restrict__ state_in, TIn* __restrict__ o, float* __restrict__ state_out) {
  constexpr int DV = kHeadCols;
  using L = ScanLds<TIn, DK, DV, FWD, true>;
  constexpr int NT = DK / 16;
  constexpr int W = DV / 16;
  __shared__ __attribute__((aligned(1024))) unsigned char lds_g[L::kBuffers * L::kBytes];
  lds_byte* lds = (lds_byte*)lds_g;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave, lg = lane / 16, lr = lane % 16;
  // logical unit: the value heads of a key head are adjacent and one cluster (same XCD)
  const int unit = xcd_cluster_remap(blockIdx.x, gridDim.x, hv / hk);
  const ScanUnit u = scan_unit(cu, unit / hv, unit % hv, hv, hk, &order);
  const int col = 16 * wave + lr;
  ChunkDma<L, TIn, W, FWD> dma;
  dma.start(u, 0, wave, lane, hk, hv, DV, 0, v, kin, qin, Kw, Tw, Sw, Pw);

  f32x4 M[NT];
  Frag mb[DK / 32];
  f32x4 pout[4];
  const int64_t sbase = (static_cast<int64_t>(u.n) * hv + u.h) * DK * DV + col;
  load_state<DK>(state_in, sbase, DV, lg, M, mb);

  if (u.nch > 0) {
    dma.chunk(lds);
    wait_dma();
  }
  __syncthreads();
  for (int ci = 0; ci < u.nch; ++ci) {
    const int b = L::kBuffers == 2 ? (ci & 1) : 0;
    if constexpr (FWD) {
      if (ci > 0) store_chunk_out(o, u, ci - 1, hv, DV, col - lr, lane, pout);
    }
    const bool prefetch = L::kBuffers == 2 && ci + 1 < u.nch;
    // the next chunk's DMA share, a few jobs at the start of each region
    auto hook = [&](int k) __attribute__((always_inline)) {
      if (prefetch) dma.template phase<kDmaPhases>(k, lds + (b ^ 1) * L::kBytes);
    };
    chunk_step<L, DK, FWD, false>((const unsigned char*)(lds + b * L::kBytes), 16 * wave, lane, M, mb, pout, hook);
    if (L::kBuffers == 1) {
      __syncthreads();   // every wave is done with the only buffer
      if (ci + 1 < u.nch) dma.chunk(lds);
    }
    wait_dma();          // this wave's share of the next chunk has landed
    __syncthreads();     // ... and everyone else's; this chunk's buffer is free
  }
  if constexpr (FWD) {
    if (u.nch > 0) store_chunk_out(o, u, u.nch - 1, hv, DV, col - lr, lane, pout);
  }
  if (state_out) {
#pragma unroll
    for (int td = 0; td < NT; ++td)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        state_out[sbase + static_cast<int64_t>(strow(td, lg, r)) * DV] = M[td][r];
  }
}

}  // namespace gdn
