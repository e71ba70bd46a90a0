// gfx950 macro-tile kernels whose operand tiles travel from global memory
// straight into LDS (buffer_load ... lds: no staging registers, no register
// transposes) through S LDS stages, so that S - 1 k-blocks of loads are in
// flight while one is multiplied out (the Multi-Buffer module of Table 2;
// the schedule of Eq. 13 with a deeper pipeline).
//
//   A tile  BM x 64 k, row-major as in memory, 16-byte chunks XOR-swizzled
//           per row; MFMA fragments read with ds_read_b128.
//   B tile  64 k x BN, row-major as in memory (chunks swizzled per k-row);
//           MFMA fragments read with the LDS transpose read
//           ds_read_b64_tr_b16, which hands each lane four consecutive k of
//           one column: the k-contiguous operand the MFMA needs, without the
//           v_perm transposes of the register-staged kernel.
//   C       4 waves in a 2 x 2 grid, each a (BM/2) x (BN/2) quadrant of
//           32 x 32 x 16 MFMAs (tiles of at most 64 rows: 4 waves side by
//           side along N); fp32 accumulation in the accumulation registers;
//           bf16 output converted through a per-wave LDS slab and written as
//           whole 16-byte row segments.
//
// The swizzle of a stage is applied on the global side: a wave-wide LDS load
// writes 1024 contiguous bytes (lane l to bytes 16l .. 16l+15), so each lane
// fetches the global chunk that belongs at its slot.
//
// (A column-major operand read in place, k_dlc, trades places: a B of N rows
// of k is tiled and read like A here, an A of K rows of M like B.)
//
// k_dl needs row-major operands with 16-byte aligned rows (A and B base
// addresses 16-byte aligned, lda and ldb multiples of 8 below 2^22) and K, N
// multiples of 8. A plan for other shapes either copies the operand
// zero-padded first (k_pad16 below, the Padding module) or runs k_dlu, the
// register-load form of the same tiling (16-byte loads at any 2-byte
// alignment, two LDS stages); an operand found misaligned at run time takes
// k_dlu, or the register-staged tile kernel of the same tiling where the
// configuration has no k_dlu. Chunks outside the matrices (rows past M,
// columns past N, k past K) are read as zeros through out-of-range buffer
// offsets, so edge tiles take the same path.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernel_args.h"
#include "registry.h"

#ifndef AC_INPUT_F16
#define AC_INPUT_F16 0
#endif
#ifndef AC_DL_PART
#define AC_DL_PART 0
#endif

namespace ac {
#if AC_INPUT_F16
namespace f16 {
#endif

#include "device_common.h"
#include "grouped_map.h"

namespace {

// the transpose read moves 16-bit patterns; its bf16 form serves fp16 too
typedef __bf16 tr16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) tr16x4 lds_tr16x4;

enum DlOut : int { DL_F32 = 0, DL_BF16 = 1, DL_PARTIAL = 2 };

// One operand's tile of a stage: EXT rows of A (or columns of B) by BK of k.
// KC: k runs along the stored rows (a row-major A, a column-major B): EXT rows
// of BK, MFMA fragments read with ds_read_b128. Otherwise the extent does (a
// row-major B, a column-major A): BK rows of EXT, fragments read with the
// transpose read. Either way 16-byte chunks swizzled within their row, and a
// lane gets the same 8 consecutive k of the same row or column.
template <int EXT_, int BK, bool KC_>
struct DlOp {
  static constexpr int EXT = EXT_;
  static constexpr bool KC = KC_;
  static constexpr int ROW = (KC ? BK : EXT) * 2;  // bytes of a stored row
  static constexpr int BYTES = EXT * BK * 2;
  static constexpr int LPR = ROW / 16;     // 16-byte chunks of a row
  static constexpr int RPI = 64 / LPR;     // rows per wave-wide load
  static constexpr int NI = BYTES / 4096;  // wave-wide loads per wave and stage
  static constexpr int READS = KC ? 1 : 2; // LDS reads of a fragment
  static_assert(KC || EXT >= 128, "the k-row swizzle spans 16 chunks");
};

// LAY: bit 0, A column-major in memory; bit 1, B column-major.
template <int BM, int BN, int BK_, int S_, int LAY = 0>
struct Dl {
  static constexpr int BN_ = BN, BK = BK_, S = S_, NT = 256;
  // waves: 2 x 2 quadrants, or (tiles of at most 64 rows: the decode-style
  // shapes) 1 x 4 along N
  static constexpr int WM = BM >= 128 ? 2 : 1, WN = 4 / WM;
  static constexpr int WTM = BM / WM, WTN = BN / WN;  // a wave's part of the tile
  static constexpr int TM = WTM / 32, TN = WTN / 32;
  typedef DlOp<BM, BK, (LAY & 1) == 0> OA;
  typedef DlOp<BN, BK, (LAY & 2) != 0> OB;
  static constexpr int A_BYTES = OA::BYTES, B_BYTES = OB::BYTES;
  static constexpr int A_LPR = OA::LPR, A_RPI = OA::RPI, B_LPR = OB::LPR, B_RPI = OB::RPI;
  static constexpr int NIA = OA::NI, NIB = OB::NI;
  static constexpr int LOADS = NIA + NIB;
  static constexpr int CT_LD = WTN + 4;       // padded row of the bf16 output slab
  // workgroups per CU the configuration is built for: two when two fit the
  // LDS and the register file (two waves per SIMD, at most 256 registers
  // each): one workgroup's epilogue stores then overlap the other's loads
  // and MFMAs
  static constexpr int WPE = (S * (BM + BN) * BK * 2 <= 80 * 1024 && BM * BN <= 256 * 128) ? 2 : 1;
  static_assert(BM % 32 == 0 && BM >= 32 && BN >= 128 && BN <= 512 && (BK == 32 || BK == 64) && WTN % 32 == 0,
                "tile");
  // the bf16 epilogue's per-wave slab of 32 output rows goes into one stage
  // buffer per wave: A0, A1, B0, B1 if both kinds are large enough, else
  // the first four of the kind that is, else two slabs in each of B0, B1
  static constexpr int SLAB = 32 * CT_LD * 2;
  static constexpr int SLAB_KIND = (SLAB <= A_BYTES && SLAB <= B_BYTES) ? 0
                                   : (SLAB <= B_BYTES && S >= 4)        ? 1
                                   : (2 * SLAB <= B_BYTES)              ? 3
                                                                        : 2;
  static_assert(SLAB_KIND != 2 || (SLAB <= A_BYTES && S >= 4), "output slab fits a stage buffer");
};

// B stage: chunk c of k-row r sits at slot c ^ f(r & 3), f = 0, 6, 12, 10.
// One transpose read covers 4 consecutive k-rows and 2 (16 lanes) or 4 (32
// lanes) consecutive chunks; f keeps those on distinct banks for both 32
// and 64 banks.
__device__ __forceinline__ int swz_b(int r) { return (0xAC60 >> (4 * (r & 3))) & 15; }

// Workgroup barrier of the pipeline: this wave waits until at most N of its
// loads into LDS are in flight and its own LDS reads and writes are done,
// then all waves meet. After it every wave's older loads have landed and no
// wave still reads what it read before. (__syncthreads would add a workgroup
// fence, which waits for ALL loads into LDS, the prefetched stages included.)
// The empty asm with a memory clobber keeps the compiler from moving LDS
// accesses across it.
template <int N>
__device__ __forceinline__ void stage_barrier() {
  static_assert(N >= 0 && N <= 63, "vmcnt range");
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(N));
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Addressing of a workgroup's loads of one operand: the byte offset of every
// 16-byte chunk this lane loads (OOB_OFF for rows and columns outside the
// matrix), and the k of that chunk within the block for the K tail.
template <class O, int BK>
struct DlOpTile {
  const char* base;       // the tile's first row (column) at k = 0
  int64_t kstep;          // bytes from one k to the next
  int32_t off[O::NI];
  int32_t k[O::KC ? O::NI : 1];  // KC: k of each chunk; else the k-row of the first one

  // p: the operand, ld its row pitch, e0 the tile's first row or column, left
  // how many of them the matrix has from there on
  __device__ __forceinline__ void init(const uint16_t* p, int64_t ld, int64_t e0, int64_t left, int w) {
    const int lane = threadIdx.x & 63;
    base = reinterpret_cast<const char*>(p + e0 * (O::KC ? ld : 1));
    kstep = 2 * (O::KC ? 1 : ld);
    if constexpr (!O::KC) k[0] = lane / O::LPR;
#pragma unroll
    for (int q = 0; q < O::NI; ++q) {
      const int row = (w * O::NI + q) * O::RPI + lane / O::LPR;  // stored row of the tile
      const int c = (lane % O::LPR) ^ (O::KC ? swz_a<BK>(row) : swz_b(row));  // the chunk this slot holds
      off[q] = (O::KC ? row : c * 8) < left ? (int32_t)(row * ld * 2) + c * 16 : OOB_OFF;
      if constexpr (O::KC) k[q] = c * 8;
    }
  }
  // load q (a compile-time index) of wave w into a stage: cur = the block's
  // first k, rem = k left from there
  __device__ __forceinline__ void issue(const char* cur, int rem, char* stage, int w, int q) const {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(cur), (short)0,
                                                                       (int)0x7FFFFFF0, (int)RSRC_WORD3);
    const bool in = O::KC ? k[O::KC ? q : 0] < rem : k[0] < rem - (w * O::NI + q) * O::RPI;
    const int32_t o = in ? off[q] : OOB_OFF;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(stage + (w * O::NI + q) * 1024), 16, o, 0, 0, 0);
  }
};

template <class G>
struct DlTile {
  DlOpTile<typename G::OA, G::BK> a;
  DlOpTile<typename G::OB, G::BK> b;
  int64_t K, kA, kB;  // k of the loop; k each operand holds
  int w;              // wave (uniform)

  __device__ __forceinline__ void init(const GemmArgs& g, int64_t m0, int64_t n0) {
    w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    K = g.K;
    // (g.K is rounded up to 8 when A is a zero-padded row-major copy)
    kA = G::OA::KC ? g.K : g.kB;
    kB = G::OB::KC ? g.K : g.kB;
    a.init(g.A, g.lda, m0, g.M - m0, w);
    b.init(g.B, g.ldb, n0, (G::OB::KC ? g.N : g.nB) - n0, w);
  }
};

// This wave's share of the loads of one k-block into one stage: NIA loads of
// A, then NIB loads of B, issued one at a time so that they can be spread
// between MFMAs. The blocks are taken in order from `kbeg` on; what a block
// has past the partition's end (the k tail, or a whole block past it) is out
// of range and read as zeros. A step to the next block is a few scalar
// additions: a wave issues one instruction at a time, and the MFMAs wait for
// whatever scalar work stands in front of them.
template <class G>
struct StageLoads {
  const char* pa;  // the block's first k of A's tile, and of B's
  const char* pb;
  int remA, remB;  // k of A and of B from there to the partition's end
  char* sA;
  char* sB;
  __device__ __forceinline__ void start(const DlTile<G>& t, int64_t kbeg, int64_t kstop) {
    pa = t.a.base + kbeg * t.a.kstep;
    pb = t.b.base + kbeg * t.b.kstep;
    remA = (int)(min(kstop, t.kA) - kbeg);
    remB = (int)(min(kstop, t.kB) - kbeg);
  }
  __device__ __forceinline__ void next(const DlTile<G>& t) {
    pa += G::BK * t.a.kstep;
    pb += G::BK * t.b.kstep;
    remA -= G::BK;
    remB -= G::BK;
  }
  // load q of this wave (0 .. NIA + NIB - 1; a compile-time index)
  __device__ __forceinline__ void issue(const DlTile<G>& t, int q) const {
    if (q < G::NIA)
      t.a.issue(pa, remA, sA, t.w, q);
    else
      t.b.issue(pb, remB, sB, t.w, q - G::NIA);
  }
};

// ---- loads through registers (any alignment, K >= 8 and N >= 8)
// The same chunks into the same LDS slots as the direct loads, fetched with
// 16-byte loads at any 2-byte address: a chunk that crosses the end of a
// row is loaded as the 16 bytes ending at the row end and shifted down in
// registers, with zeros past K (A columns, B rows) and past N (B columns).
// Rows past M re-read row M - 1 (their outputs are never stored).
template <class G>
struct DlTileU {
  const uint16_t* a;  // A + m0 * lda
  const uint16_t* B;
  int64_t ldb, K, N;
  uint32_t a_row[G::NIA];  // bytes: clamped row * lda * 2
  int32_t a_c[G::NIA];     // k of the chunk within the block
  int32_t b_kr[G::NIB];    // k-row of the chunk within the block
  uint32_t b_col[G::NIB];  // bytes: first column loaded (<= N - 8)
  int32_t b_cs[G::NIB];    // elements dropped at the N edge (0 .. 8)

  __device__ __forceinline__ void init(const GemmArgs& g, int64_t m0, int64_t n0) {
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    a = g.A + m0 * g.lda;
    B = g.B;
    ldb = g.ldb;
    K = g.K;
    N = g.N;
#pragma unroll
    for (int q = 0; q < G::NIA; ++q) {
      const int u = w * G::NIA + q;
      const int row = u * G::A_RPI + lane / G::A_LPR;
      const int c = (lane % G::A_LPR) ^ swz_a<G::BK>(row);
      a_row[q] = (uint32_t)((min(m0 + row, g.M - 1) - m0) * g.lda * 2);
      a_c[q] = c * 8;
    }
#pragma unroll
    for (int q = 0; q < G::NIB; ++q) {
      const int u = w * G::NIB + q;
      const int kr = u * G::B_RPI + lane / G::B_LPR;
      const int c = (lane % G::B_LPR) ^ swz_b(kr);
      const int64_t gn = n0 + c * 8, st = min(gn, g.N - 8);
      b_kr[q] = kr;
      b_col[q] = (uint32_t)(st * 2);
      b_cs[q] = (int32_t)min(gn - st, (int64_t)8);
    }
  }
};

template <class G>
struct RegLoads {
  u32x4 va[G::NIA], vb[G::NIB];
  uint32_t sha, shb;  // per chunk 4 bits: elements to drop (8 = all)
  const uint16_t* a0;  // A tile base at this block's k (elements: the chunk's start added per lane)
  const uint16_t* b0;  // B + min(k0, K - 1) * ldb
  int64_t k0, kb0;
  char* sA;
  char* sB;
  __device__ __forceinline__ void init(char* a_stage, char* b_stage, const DlTileU<G>& t, int64_t k) {
    k0 = k;
    kb0 = min(k, t.K - 1);
    b0 = t.B + kb0 * t.ldb;
    sA = a_stage;
    sB = b_stage;
    sha = shb = 0;
  }
  // global load q into registers (0 .. NIA + NIB - 1, a compile-time index)
  __device__ __forceinline__ void issue(const DlTileU<G>& t, int q) {
    if (q < G::NIA) {
      const int64_t e = k0 + t.a_c[q], st = min(e, t.K - 8);
      const uint32_t s = (uint32_t)min(e - st, (int64_t)8);
      va[q] = load16(reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(t.a) + t.a_row[q] + st * 2));
      sha |= s << (4 * q);
    } else {
      const int qb = q - G::NIA;
      const int64_t r = k0 + t.b_kr[qb];
      const int64_t rr = min(r, t.K - 1) - kb0;  // >= 0
      vb[qb] = load16(reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(b0) +
                                                         (uint32_t)(rr * t.ldb * 2) + t.b_col[qb]));
      const uint32_t s = r >= t.K ? 8u : (uint32_t)t.b_cs[qb];
      shb |= s << (4 * qb);
    }
  }
  // the shifted chunks into their LDS slots (after the loads landed)
  __device__ __forceinline__ void finish() {
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int q = 0; q < G::NIA; ++q)
      *reinterpret_cast<u32x4*>(sA + (w * G::NIA + q) * 1024 + lane * 16) = shift_down(va[q], (sha >> (4 * q)) & 15);
#pragma unroll
    for (int q = 0; q < G::NIB; ++q)
      *reinterpret_cast<u32x4*>(sB + (w * G::NIB + q) * 1024 + lane * 16) = shift_down(vb[q], (shb >> (4 * q)) & 15);
  }
};

// Byte offsets of a lane's fragment reads within a stage, computed once. KC:
// one per k-step (rows are ROW bytes apart, and the swizzle of row 32 i + l32
// is that of l32); else one per fragment (k-step and half are constant
// offsets: the swizzle only depends on the k-row mod 4). Opaque to the
// compiler: it may not take the sums apart into a chain of address steps, at
// whose end it no longer knows which stage is read and would wait for the
// loads into all of them.
template <class O, int BK, int T>
struct FragAddr {
  int at[O::KC ? BK / 16 : T];
  __device__ __forceinline__ void init(int e0) {  // e0: the wave's first row or column in the tile
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31, hi = lane >> 5, i16 = lane & 15, g = lane >> 4;
    if constexpr (O::KC) {
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) {
        const int ch = 2 * ks + hi;  // 8 consecutive k of the lane's k-group
        at[ks] = (e0 + l32) * O::ROW + ((ch ^ swz_a<BK>(l32)) << 4);
        asm("" : "+v"(at[ks]));
      }
    } else {
      // the transpose read of a 16-lane group covers 4 k-rows x 16 columns: lane
      // i16 addresses k-row i16 >> 2 and columns 4 * (i16 & 3) .. +3 and receives
      // column i16 of the 4 rows; groups 0 / 1 take columns 0-15 / 16-31 of the
      // fragment at the lane's k-group 0, groups 2 / 3 the same at k-group 1
      const int kr0 = 8 * (g >> 1) + (i16 >> 2);
#pragma unroll
      for (int j = 0; j < T; ++j) {
        const int col = e0 + 32 * j + 16 * (g & 1) + (i16 & 3) * 4;
        at[j] = kr0 * O::ROW + ((col >> 3) ^ swz_b(kr0)) * 16 + (col & 7) * 2;
        asm("" : "+v"(at[j]));
      }
    }
  }
  // fragment i of k-step ks (compile-time indices)
  __device__ __forceinline__ u32x4 read(const char* st, int ks, int i) const {
    if constexpr (O::KC) {
      return *reinterpret_cast<const u32x4*>(st + at[ks] + 32 * i * O::ROW);
    } else {
      uint32_t v[4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const tr16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_tr16x4*)(st + at[i] + (16 * ks + 4 * h) * O::ROW));
        const uint64_t bits = __builtin_bit_cast(uint64_t, r);
        v[2 * h] = (uint32_t)bits;
        v[2 * h + 1] = (uint32_t)(bits >> 32);
      }
      return u32x4{v[0], v[1], v[2], v[3]};
    }
  }
};

// Fragments of one k-step (16 k) of a stage.
template <class G>
struct Frags {
  u32x4 a[G::TM], b[G::TN];
};

template <class G>
struct FragAddrs {
  FragAddr<typename G::OA, G::BK, G::TM> a;
  FragAddr<typename G::OB, G::BK, G::TN> b;
};

template <class G>
__device__ __forceinline__ void read_frags(const char* sA, const char* sB, int ks, const FragAddrs<G>& at, Frags<G>& f) {
#pragma unroll
  for (int i = 0; i < G::TM; ++i) f.a[i] = at.a.read(sA, ks, i);
#pragma unroll
  for (int j = 0; j < G::TN; ++j) f.b[j] = at.b.read(sB, ks, j);
}

// What runs under the NMF MFMAs of one k-step: RD LDS reads (the next step's
// fragments), two to an MFMA from the first one on, and LD global loads one
// to an MFMA. A wave that stalls on a full LDS or load queue issues no MFMAs,
// so neither may leave in a burst.
template <int NMF, int RD, int LD>
__device__ __forceinline__ void interleave_step() {
  constexpr int RPM = 2 * NMF >= RD ? 2 : (RD + NMF - 1) / NMF, LPM = (LD + NMF - 1) / NMF;
#pragma unroll
  for (int m = 0; m < NMF; ++m) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                      // one MFMA
    if (m * RPM < RD) __builtin_amdgcn_sched_group_barrier(0x100, RPM, 0);  // LDS reads
    if ((m + 1) * LD / NMF > m * LD / NMF) __builtin_amdgcn_sched_group_barrier(0x020, LPM, 0);  // loads
  }
  __builtin_amdgcn_sched_barrier(0);
}

template <class G>
__device__ __forceinline__ void mfma_step(const Frags<G>& f, f32x16 (&acc)[G::TM][G::TN]) {
#pragma unroll
  for (int i = 0; i < G::TM; ++i)
#pragma unroll
    for (int j = 0; j < G::TN; ++j) acc[i][j] = mfma32(f.b[j], f.a[i], acc[i][j]);  // C^T: a lane holds a row of C
}

// One output tile (tile coordinates tm, tn) over K partition `split` of the
// plan's kper-block partitions.
template <int BM, int BN, int BK, int S, int OUT, bool RG, int LAY = 0>
__device__ __forceinline__ void dl_tile(const GemmArgs& g, int tm, int tn, int split) {
  typedef Dl<BM, BN, BK, S, LAY> G;
  typedef typename std::conditional<RG, DlTileU<G>, DlTile<G>>::type Tile;
  typedef typename std::conditional<RG, RegLoads<G>, StageLoads<G>>::type Loads;
  __shared__ __attribute__((aligned(1024))) char lA0[G::A_BYTES];
  __shared__ __attribute__((aligned(1024))) char lA1[G::A_BYTES];
  __shared__ __attribute__((aligned(1024))) char lA2[G::A_BYTES];
  __shared__ __attribute__((aligned(1024))) char lA3[G::A_BYTES];
  __shared__ __attribute__((aligned(1024))) char lA4[G::A_BYTES];
  __shared__ __attribute__((aligned(1024))) char lB0[G::B_BYTES];
  __shared__ __attribute__((aligned(1024))) char lB1[G::B_BYTES];
  __shared__ __attribute__((aligned(1024))) char lB2[G::B_BYTES];
  __shared__ __attribute__((aligned(1024))) char lB3[G::B_BYTES];
  __shared__ __attribute__((aligned(1024))) char lB4[G::B_BYTES];
  static_assert(S >= 2 && S <= 5, "stages");

  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  // the K partition: kper blocks of the plan's 64-deep granule, a whole
  // number of this kernel's k-blocks
  const int64_t kbeg = min((int64_t)split * g.kper * 64, g.K);
  const int64_t kend = min(kbeg + (int64_t)g.kper * 64, g.K);
  const int nk = (int)((kend - kbeg + G::BK - 1) / G::BK);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wr = wave / G::WN, wc = wave % G::WN;

  Tile t;
  t.init(g, m0, n0);

  f32x16 acc[G::TM][G::TN];
#pragma unroll
  for (int i = 0; i < G::TM; ++i)
#pragma unroll
    for (int j = 0; j < G::TN; ++j) acc[i][j] = f32x16{};

  // Stage I holds k-blocks I, I + S, I + 2S, ... of the partition. The
  // stage buffers are distinct variables so that the compiler's wait
  // before a read of one stage does not include the loads into the others.
  auto stA = [&](auto ic) -> char* {
    constexpr int I = decltype(ic)::value;
    return I == 0 ? lA0 : I == 1 ? lA1 : I == 2 ? lA2 : I == 3 ? lA3 : lA4;
  };
  auto stB = [&](auto ic) -> char* {
    constexpr int I = decltype(ic)::value;
    return I == 0 ? lB0 : I == 1 ? lB1 : I == 2 ? lB2 : I == 3 ? lB3 : lB4;
  };
  // k of block b of the partition; past its last block K, where every load
  // is out of range
  const int64_t kstop = kbeg + (int64_t)nk * G::BK;  // the partition's end, rounded up to a block
  auto kpos = [&](int b) { const int64_t k = kbeg + (int64_t)b * G::BK; return k < kstop ? k : t.K; };

  // The pipeline. A block's fragments are read one k-step ahead of their
  // MFMAs, also across blocks: before the last k-step of block kb the waves
  // meet (its fragments are in registers by then, and block kb + 1 has
  // landed), the first fragments of block kb + 1 are read under that step's
  // MFMAs, and block kb + S starts to load into the stage just freed. So no
  // MFMA waits for an LDS read issued after a barrier: with the reads at the
  // start of each block, after its barrier, the four waves' 32 KB of first
  // fragments (256 clocks of LDS time) were exposed per 2060 clocks of MFMAs
  // on the 256 x 256 x 64 tile.
  constexpr int KS = G::BK / 16, NMF = G::TM * G::TN;
  constexpr int RD = G::TM * G::OA::READS + G::TN * G::OB::READS;
  // loads of a block per k-step, from the barrier on: with two stages over the
  // first half of a block's MFMAs (they must land within the other half),
  // with more stages over all of them. 8192^3 on the 256 x 256 x 64 tile: all
  // in one step 855 us, over two 827, three 836, four 907. On eight shapes from
  // 4096 x 1536 x 4096 to 8192^3 (geometric means), all in one step takes 1.054x
  // the time on that tile, 1.05-1.11x on the 64-deep three-stage tiles and
  // 1.00-1.02x on the others; the other way round (two stages over all steps,
  // more over half) 1.10x, 0.99-1.02x, and 1.03-1.06x on the two-per-CU tiles.
  constexpr int LSTEPS = S == 2 ? (KS + 1) / 2 : KS;
  constexpr int LPS = RG ? G::LOADS : (G::LOADS + LSTEPS - 1) / LSTEPS;
  constexpr int REST = G::LOADS - LPS;  // loads left for the next block's k-steps
  FragAddrs<G> fa;
  fa.a.init(wr * G::WTM);
  fa.b.init(wc * G::WTN);
  Frags<G> f[2];
  Loads nxt;
  if (nk > 0) {
    if constexpr (RG) {
      Loads pro[S];
#pragma unroll
      for (int p = 0; p < S; ++p) {
        pro[p].init(p == 0 ? lA0 : p == 1 ? lA1 : p == 2 ? lA2 : p == 3 ? lA3 : lA4,
                    p == 0 ? lB0 : p == 1 ? lB1 : p == 2 ? lB2 : p == 3 ? lB3 : lB4, t, kpos(p));
#pragma unroll
        for (int q = 0; q < G::LOADS; ++q) pro[p].issue(t, q);
      }
#pragma unroll
      for (int p = 0; p < S; ++p) pro[p].finish();
      nxt.init(lA0, lB0, t, kpos(S));
#pragma unroll
      for (int q = 0; q < G::LOADS; ++q) nxt.issue(t, q);
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    } else {
      nxt.start(t, kbeg, kstop);
#pragma unroll
      for (int p = 0; p < S; ++p) {
        if (p > 0) nxt.next(t);
        nxt.sA = p == 0 ? lA0 : p == 1 ? lA1 : p == 2 ? lA2 : p == 3 ? lA3 : lA4;
        nxt.sB = p == 0 ? lB0 : p == 1 ? lB1 : p == 2 ? lB2 : p == 3 ? lB3 : lB4;
#pragma unroll
        for (int q = 0; q < (p == S - 1 ? LPS : G::LOADS); ++q) nxt.issue(t, q);
      }
      stage_barrier<(S - 1) * G::LOADS - REST>();
    }
    read_frags<G>(lA0, lB0, 0, fa, f[0]);
    __builtin_amdgcn_sched_barrier(0);
  }

  // k-steps 0 .. KS - 2 of the block in stage I; MORE: the rest of the loads
  // of the block issued last
  auto head = [&](auto ic, auto more) {
    if constexpr (decltype(more)::value && REST > 0) {
      // the stage they go to, as a constant: a pointer carried round the loop
      // would hide from the compiler which stage it is, and every read of
      // another stage would wait for these loads
      const std::integral_constant<int, (decltype(ic)::value + S - 1) % S> pv{};
      nxt.sA = stA(pv);
      nxt.sB = stB(pv);
    }
#pragma unroll
    for (int ks = 0; ks + 1 < KS; ++ks) {
      read_frags<G>(stA(ic), stB(ic), ks + 1, fa, f[(ks + 1) & 1]);
      mfma_step<G>(f[ks & 1], acc);
      if constexpr (decltype(more)::value && REST > 0) {
#pragma unroll
        for (int q = (ks + 1) * LPS; q < (ks + 2) * LPS && q < G::LOADS; ++q) nxt.issue(t, q);
        interleave_step<NMF, RD, LPS>();
      } else {
        interleave_step<NMF, RD, 0>();
      }
    }
  };
  // the barrier and the last k-step of block kb in stage I, with the first
  // reads of the next block and the first loads of block kb + S
  auto tail = [&](auto ic, int kb) {
    constexpr int I = decltype(ic)::value;
    const std::integral_constant<int, (I + 1) % S> nx{};
    if constexpr (RG) {
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      nxt.sA = stA(ic);
      nxt.sB = stB(ic);
      nxt.finish();  // block kb + S, loaded during the last block
      nxt.init(stA(ic), stB(ic), t, kpos(kb + S + 1));
    } else {
      stage_barrier<(S - 2) * G::LOADS>();
      nxt.next(t);
      nxt.sA = stA(ic);
      nxt.sB = stB(ic);
    }
    read_frags<G>(stA(nx), stB(nx), 0, fa, f[0]);
    mfma_step<G>(f[(KS - 1) & 1], acc);
#pragma unroll
    for (int q = 0; q < LPS; ++q) nxt.issue(t, q);
    interleave_step<NMF, RD, LPS>();
  };
  auto step = [&](auto ic, int kb) {
    head(ic, std::true_type{});
    tail(ic, kb);
  };
  // the last blocks (at most S, all loading or loaded): block I of them
  auto last = [&](auto ic, int left) {
    constexpr int I = decltype(ic)::value;
    if (I >= left) return;
    head(ic, std::integral_constant<bool, I == 0>{});
    if (I + 1 < left) {
      const std::integral_constant<int, (I + 1) % S> nx{};
      if constexpr (RG)
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      else
        stage_barrier<(S - 2 - I > 0 ? S - 2 - I : 0) * G::LOADS>();
      read_frags<G>(stA(nx), stB(nx), 0, fa, f[0]);
    }
    mfma_step<G>(f[(KS - 1) & 1], acc);
    __builtin_amdgcn_sched_barrier(0);
  };
  // groups of S blocks while more than S are left, then the rest
  int kb = 0;
  for (; nk - kb > S; kb += S) {
    step(std::integral_constant<int, 0>{}, kb);
    step(std::integral_constant<int, 1>{}, kb + 1);
    if constexpr (S > 2) step(std::integral_constant<int, 2>{}, kb + 2);
    if constexpr (S > 3) step(std::integral_constant<int, 3>{}, kb + 3);
    if constexpr (S > 4) step(std::integral_constant<int, 4>{}, kb + 4);
  }
  last(std::integral_constant<int, 0>{}, nk - kb);
  last(std::integral_constant<int, 1>{}, nk - kb);
  if constexpr (S > 2) last(std::integral_constant<int, 2>{}, nk - kb);
  if constexpr (S > 3) last(std::integral_constant<int, 3>{}, nk - kb);
  if constexpr (S > 4) last(std::integral_constant<int, 4>{}, nk - kb);

  // ---- epilogue
  const int64_t rbase = m0 + wr * G::WTM, cbase = n0 + wc * G::WTN;
  if constexpr (OUT == DL_BF16) {
    stage_barrier<0>();  // every wave's last reads of the stages are done, no load into them is in flight
    // the wave's slab: 32 rows x WTN bf16 in one of the stage buffers
    char* slab;
    if constexpr (G::SLAB_KIND == 0)
      slab = wave == 0 ? lA0 : wave == 1 ? lA1 : wave == 2 ? lB0 : lB1;
    else if constexpr (G::SLAB_KIND == 1)
      slab = wave == 0 ? lB0 : wave == 1 ? lB1 : wave == 2 ? lB2 : lB3;
    else if constexpr (G::SLAB_KIND == 3)
      slab = (wave < 2 ? lB0 : lB1) + (wave & 1) * G::SLAB;
    else
      slab = wave == 0 ? lA0 : wave == 1 ? lA1 : wave == 2 ? lA2 : lA3;
    uint16_t* ct = reinterpret_cast<uint16_t*>(slab);
    uint16_t* C = static_cast<uint16_t*>(g.C);
    constexpr int GPR = G::WTN / 8;  // 16-byte groups per slab row
#pragma unroll
    for (int i = 0; i < G::TM; ++i) {
      const int64_t row = rbase + 32 * i + (lane & 31);
#pragma unroll
      for (int j = 0; j < G::TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = 32 * j + (q << 3) + ((lane >> 5) << 2);  // acc elements 4q .. 4q+3: four columns
          float w[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          if (g.epi && row < g.M && cbase + c < g.N) epi_apply<true, 4>(g, w, row, cbase + c, g.N - cbase - c);
          const uint32_t lo = (uint32_t)to16(w[0]) | ((uint32_t)to16(w[1]) << 16);
          const uint32_t hi = (uint32_t)to16(w[2]) | ((uint32_t)to16(w[3]) << 16);
          *reinterpret_cast<uint64_t*>(ct + (lane & 31) * G::CT_LD + c) = (uint64_t)lo | ((uint64_t)hi << 32);
        }
      // the slab back as 16-byte row segments (the same wave: LDS is in order)
#pragma unroll
      for (int v = 0; v < 32 * GPR / 64; ++v) {
        const int u = lane + 64 * v, r = u / GPR, grp = u % GPR;
        const uint16_t* src = ct + r * G::CT_LD + grp * 8;
        const uint64_t a = *reinterpret_cast<const uint64_t*>(src);
        const uint64_t b = *reinterpret_cast<const uint64_t*>(src + 4);
        const int64_t gr = rbase + 32 * i + r, gc = cbase + grp * 8;
        if (gr < g.M && gc + 8 <= g.N) {
          const uint64_t vv[2] = {a, b};
          __builtin_memcpy(C + gr * g.ldc + gc, vv, 16);
        } else if (gr < g.M && gc < g.N) {  // the last, partial group of a row
          const uint16_t* e = src;
          for (int j = 0; j < (int)(g.N - gc); ++j) C[gr * g.ldc + gc + j] = e[j];
        }
      }
      __builtin_amdgcn_sched_barrier(0);  // slab by slab: bounded live registers
    }
  } else {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // no load into LDS outlives the workgroup
    float* dst = OUT == DL_PARTIAL ? g.ws + (size_t)split * (size_t)g.M * (size_t)g.ldw : static_cast<float*>(g.C);
    const int64_t ld = OUT == DL_PARTIAL ? g.ldw : g.ldc;
#pragma unroll
    for (int i = 0; i < G::TM; ++i) {
      const int64_t row = rbase + 32 * i + (lane & 31);
      if (row >= g.M) continue;
#pragma unroll
      for (int j = 0; j < G::TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t col = cbase + 32 * j + (q << 3) + ((lane >> 5) << 2);
          if (col >= g.N) continue;
          float w[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          if (OUT == DL_F32 && g.epi) epi_apply<false, 4>(g, w, row, col, g.N - col);
          if (col + 4 <= g.N) {
            const f32x4 vv = {w[0], w[1], w[2], w[3]};
            __builtin_memcpy(dst + row * ld + col, &vv, 16);
          } else {
            for (int e = 0; e < (int)(g.N - col); ++e) dst[row * ld + col + e] = w[e];
          }
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// a workgroup per output tile (blockIdx.x, in the plan's tile order) and K
// partition (blockIdx.y)
template <int BM, int BN, int BK, int S, int OUT, bool RG, int LAY = 0>
__device__ __forceinline__ void dl_kernel(const GemmArgs& g) {
  const int ntiles = g.tiles_m * g.tiles_n;
  int tile = blockIdx.x;
  if (g.swizzle) tile = xcd_remap(tile, ntiles);
  int tm, tn;
  tile_coords(tile, g.tiles_m, g.tiles_n, g.swizzle, tm, tn);
  // the division ran in vector registers: back to scalar ones, or the
  // operand pointers stay there and every load loops over its lanes' pointers
  tm = __builtin_amdgcn_readfirstlane(tm);
  tn = __builtin_amdgcn_readfirstlane(tn);
  dl_tile<BM, BN, BK, S, OUT, RG, LAY>(g, tm, tn, (int)blockIdx.y);
}

// the kernels: operand tiles loaded straight into LDS (k_dl), or through
// registers at any alignment (k_dlu)
template <int BM, int BN, int BK, int S, int OUT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Dl<BM, BN, BK, S>::WPE, Dl<BM, BN, BK, S>::WPE)))
void k_dl(GemmArgs g) {
  dl_kernel<BM, BN, BK, S, OUT, false>(g);
}
template <int BM, int BN, int BK, int S, int OUT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Dl<BM, BN, BK, S>::WPE, Dl<BM, BN, BK, S>::WPE)))
void k_dlu(GemmArgs g) {
  dl_kernel<BM, BN, BK, S, OUT, true>(g);
}

// the same with one operand column-major in memory, read in place (LAY 1: A,
// LAY 2: B): no transposed copy, the same bits
template <int BM, int BN, int BK, int S, int OUT, int LAY>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Dl<BM, BN, BK, S>::WPE, Dl<BM, BN, BK, S>::WPE)))
void k_dlc(GemmArgs g) {
  dl_kernel<BM, BN, BK, S, OUT, false, LAY>(g);
}

// Off-chip accumulation (the SingleCoreSplitK and HybridSplitK templates of
// Section 4.2; write volume of Eqs. 3 and 5): a workgroup owns a super-tile
// of two vertically adjacent tiles, 2BM x BN, whose fp32 accumulator does not
// fit the registers, and takes the plan's P_k k1-slices of K in order --
// all of them (gridDim.y = 1: SingleCoreSplitK) or its share of them
// (gridDim.y workgroups along K: HybridSplitK). For every slice it computes
// the upper tile, flushes its partial sums to the slice's fp32 partial buffer
// in the workspace, then the lower tile (whose B slice the upper one has just
// brought into the L2); the reduction kernel then adds the slices. Each tile
// of each slice is the direct-to-LDS tile kernel's own computation of that
// partition, so the result has the bits of the split-K plan with the same
// partitions.
template <int BM, int BN, int BK, int S>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Dl<BM, BN, BK, S>::WPE, Dl<BM, BN, BK, S>::WPE)))
void k_dl_sc(GemmArgs g) {
  const int sup = blockIdx.x;
  const int stm = __builtin_amdgcn_readfirstlane(sup / g.tiles_n), tn = sup - stm * g.tiles_n;
  const int per = g.pk / (int)gridDim.y;  // slices of this workgroup
  for (int q = 0; q < per; ++q) {
    const int split = (int)blockIdx.y * per + q;
#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
      const int tm = 2 * stm + h;
      if (tm >= g.tiles_m) break;
      // the previous tile's loads and stores are complete and no wave still
      // reads its LDS stages
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      __syncthreads();
      dl_tile<BM, BN, BK, S, DL_PARTIAL, false>(g, tm, tn, split);
    }
  }
}

// The grouped and strided-batch products on the direct-to-LDS tile (one tile
// of one group per workgroup, no K split): k_grouped's tiles and the same
// sums, so its bits, on operands whose every group has aligned rows.
//
// Tile order of a grouped product (swizzle): the tiles of a group run column
// panel by column panel, its row tiles one after the other (they share the
// panel's B), and the XCDs take GRP_CHUNK consecutive tiles in turn. Giving
// each XCD one contiguous eighth of the tiles, as for a plain product, left
// some XCDs with the heavy groups, whose tiles share B in the L2, and others
// with the light ones, each of whose tiles streams a panel of its own from
// HBM. 8192 rows over 64 groups of unequal load, K 4096, N 1536, 128 x 256
// tiles: register-staged 290 us, this kernel in that order 233, in chunks of
// one tile 242, 2: 221, 4: 214, 8: 209, 12: 212. On 30 products of 4 to 64
// groups (64-8192 rows, N and K 256-4096), chunks of 1, 4 and 16 take 1.118x,
// 1.019x and 1.016x the time of 8 in the geometric mean.
constexpr int GRP_CHUNK = 8;

template <int BM, int BN, int BK, int S, int OUT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Dl<BM, BN, BK, S>::WPE, Dl<BM, BN, BK, S>::WPE)))
void k_grouped_dl(GroupArgs a) {
  const int tiles_n = a.g.tiles_n;
  int t = blockIdx.x;
  int grp = 0, tm = 0, tn = 0;
  int64_t row0 = 0, rows_g = 0;
  if (a.counts == nullptr) {
    // strided batch: the grid is exactly groups x row tiles x column tiles
    if (a.g.swizzle) t = xcd_remap(t, (int)gridDim.x);
    const int slot = t / tiles_n;
    tn = t - slot * tiles_n;
    grp = slot / a.tiles_per_group;
    tm = slot - grp * a.tiles_per_group;
    rows_g = a.rows;
  } else {
    GroupChunk<BM> first;
    first.load(a, 0, 0);
    if (a.g.swizzle) {
      // over the tiles that exist: whole rounds of 8 chunks, the rest in order
      const int n = group_tiles_total<BM>(a, first) * tiles_n;
      if (t >= n) return;
      const int whole = n / (8 * GRP_CHUNK) * (8 * GRP_CHUNK);
      if (t < whole) {
        const int i = t >> 3;
        t = (i / GRP_CHUNK) * (8 * GRP_CHUNK) + (t & 7) * GRP_CHUNK + i % GRP_CHUNK;
      }
    }
    const int slot = t / tiles_n;
    if (!group_of_slot<BM>(a, first, slot, grp, row0, rows_g, tm)) return;
    // the group's tiles start at its first slot's
    const int in = t - (slot - tm) * tiles_n, rt = (int)((rows_g + BM - 1) / BM);
    tn = in / rt;
    tm = in - tn * rt;
  }
  // the same values in every lane: scalar for the address bases
  grp = __builtin_amdgcn_readfirstlane(grp);
  tm = __builtin_amdgcn_readfirstlane(tm);
  tn = __builtin_amdgcn_readfirstlane(tn);
  row0 = uniform64(row0);
  rows_g = uniform64(rows_g);

  GemmArgs g = a.g;
  g.A += row0 * g.lda + (int64_t)grp * a.stride_a;
  g.B += (int64_t)grp * a.stride_b;
  g.C = static_cast<char*>(g.C) + (row0 * g.ldc + (int64_t)grp * a.stride_c) * (OUT == DL_BF16 ? 2 : 4);
  if (g.epi && g.bias != nullptr) g.bias += (int64_t)grp * a.stride_bias;
  g.M = rows_g;
  dl_tile<BM, BN, BK, S, OUT, false>(g, tm, tn, 0);
}

template <int BM, int BN, int BK, int S, int OUT>
void start_dl(const GemmArgs& g, dim3 grid, hipStream_t st) {
  const dim3 block(256);
  if constexpr ((dl_col(BM, BN, BK, S) & 1) != 0)
    if (g.lay == 1) {
      hipLaunchKernelGGL((k_dlc<BM, BN, BK, S, OUT, 1>), grid, block, 0, st, g);
      return;
    }
  if constexpr ((dl_col(BM, BN, BK, S) & 2) != 0)
    if (g.lay == 2) {
      hipLaunchKernelGGL((k_dlc<BM, BN, BK, S, OUT, 2>), grid, block, 0, st, g);
      return;
    }
  hipLaunchKernelGGL((k_dl<BM, BN, BK, S, OUT>), grid, block, 0, st, g);
}

}  // namespace

// The launcher and the occupancy of one configuration. A configuration's
// kernels are compiled where these are instantiated: the file is compiled
// once per AC_DL_PART, each part with its configurations, so that the build
// runs in parallel.
template <int BM, int BN, int BK, int S>
hipError_t launch_dl(const Plan& p, const GemmArgs& g, hipStream_t st, bool obf) {
  const dim3 grid(p.grid_x, p.grid_y), block(256);
  if (g.lay != 0 && (p.unal || g.lay == 3 || (g.lay & ~dl_col(BM, BN, BK, S)) != 0)) return hipErrorInvalidValue;
  if (p.unal) {
    if constexpr (dl_has_unal(BM, BN, BK, S)) {
      if (p.pk > 1)
        hipLaunchKernelGGL((k_dlu<BM, BN, BK, S, DL_PARTIAL>), grid, block, 0, st, g);
      else if (obf)
        hipLaunchKernelGGL((k_dlu<BM, BN, BK, S, DL_BF16>), grid, block, 0, st, g);
      else
        hipLaunchKernelGGL((k_dlu<BM, BN, BK, S, DL_F32>), grid, block, 0, st, g);
    } else {
      return hipErrorInvalidValue;
    }
  } else if (p.pk > 1) {
    start_dl<BM, BN, BK, S, DL_PARTIAL>(g, grid, st);
  } else if (obf) {
    start_dl<BM, BN, BK, S, DL_BF16>(g, grid, st);
  } else {
    start_dl<BM, BN, BK, S, DL_F32>(g, grid, st);
  }
  return hipGetLastError();
}

// Workgroups per CU for the planner: the device's figure, but no more than
// the configuration is built for, which is what its costs were fitted with
// (28921 x 20011 x 59: a 128 x 128 x 32 tile priced at three per CU was taken
// at 320 us where the 64 x 512 one runs in 298).
template <int BM, int BN, int BK, int S>
int occ_dl() {
  int o = Dl<BM, BN, BK, S>::WPE;
  const void* ks[6] = {reinterpret_cast<const void*>(k_dl<BM, BN, BK, S, DL_F32>),
                       reinterpret_cast<const void*>(k_dl<BM, BN, BK, S, DL_BF16>),
                       reinterpret_cast<const void*>(k_dl<BM, BN, BK, S, DL_PARTIAL>), nullptr, nullptr, nullptr};
  if constexpr (dl_has_unal(BM, BN, BK, S)) {  // the register-load form: one occupancy for both
    ks[3] = reinterpret_cast<const void*>(k_dlu<BM, BN, BK, S, DL_F32>);
    ks[4] = reinterpret_cast<const void*>(k_dlu<BM, BN, BK, S, DL_BF16>);
    ks[5] = reinterpret_cast<const void*>(k_dlu<BM, BN, BK, S, DL_PARTIAL>);
  }
  for (const void* k : ks) {
    if (!k) continue;
    int a = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&a, k, 256, 0) != hipSuccess) a = 0;
    o = a < o ? a : o;
  }
  return o;
}

template <int BM, int BN, int BK, int S>
hipError_t launch_grouped_dl(const Plan& p, const GroupArgs& a, hipStream_t st, bool obf) {
  const dim3 grid(p.grid_x), block(256);
  if (obf)
    hipLaunchKernelGGL((k_grouped_dl<BM, BN, BK, S, DL_BF16>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((k_grouped_dl<BM, BN, BK, S, DL_F32>), grid, block, 0, st, a);
  return hipGetLastError();
}
#define GDL_INST(a, b, c, d) template hipError_t launch_grouped_dl<a, b, c, d>(const Plan&, const GroupArgs&, hipStream_t, bool);
#define GDL_EXT(a, b, c, d) extern GDL_INST(a, b, c, d)
#define DL_INST(a, b, c, d)                                                                   \
  template hipError_t launch_dl<a, b, c, d>(const Plan&, const GemmArgs&, hipStream_t, bool); \
  template int occ_dl<a, b, c, d>();
#define DL_EXT(a, b, c, d)                                                                           \
  extern template hipError_t launch_dl<a, b, c, d>(const Plan&, const GemmArgs&, hipStream_t, bool); \
  extern template int occ_dl<a, b, c, d>();
// (a configuration is in one part; the static assertion on DL_CFGS below and
// the linker hold the parts and the table together)
#if AC_DL_PART == 1
DL_INST(256, 256, 64, 2)
#elif AC_DL_PART == 2
DL_INST(256, 256, 32, 4)
DL_INST(256, 256, 32, 5)
#elif AC_DL_PART == 3
DL_INST(256, 128, 64, 3)
DL_INST(128, 256, 64, 3)
#elif AC_DL_PART == 4
DL_INST(256, 128, 32, 4)
DL_INST(128, 256, 32, 4)
DL_INST(128, 128, 64, 3)
#elif AC_DL_PART == 5
DL_INST(256, 128, 32, 2)
DL_INST(128, 128, 64, 2)
DL_INST(128, 128, 32, 2)
#elif AC_DL_PART == 6
DL_INST(32, 256, 64, 4)
DL_INST(64, 256, 64, 4)
DL_INST(32, 128, 64, 4)
DL_INST(64, 512, 32, 2)
#elif AC_DL_PART == 7
GDL_INST(256, 128, 64, 3)
GDL_INST(128, 256, 64, 3)
GDL_INST(128, 128, 64, 2)
GDL_INST(128, 128, 64, 3)
GDL_INST(64, 128, 64, 3)
#else
GDL_EXT(256, 128, 64, 3) GDL_EXT(128, 256, 64, 3) GDL_EXT(128, 128, 64, 2) GDL_EXT(128, 128, 64, 3)
GDL_EXT(64, 128, 64, 3)
DL_EXT(256, 256, 64, 2) DL_EXT(256, 256, 32, 4) DL_EXT(256, 256, 32, 5) DL_EXT(256, 128, 64, 3)
DL_EXT(128, 256, 64, 3) DL_EXT(256, 128, 32, 4) DL_EXT(128, 256, 32, 4) DL_EXT(128, 128, 64, 3)
DL_EXT(256, 128, 32, 2) DL_EXT(128, 128, 64, 2) DL_EXT(128, 128, 32, 2) DL_EXT(32, 256, 64, 4)
DL_EXT(64, 256, 64, 4) DL_EXT(32, 128, 64, 4) DL_EXT(64, 512, 32, 2)

namespace {
typedef hipError_t (*DlLaunchFn)(const Plan&, const GemmArgs&, hipStream_t, bool);
typedef int (*DlOccFn)();
#define DL_CFGS(X) X(256, 256, 64, 2), X(256, 128, 64, 3), X(128, 256, 64, 3), X(128, 128, 64, 3), X(256, 256, 32, 4), \
    X(256, 256, 32, 5), X(256, 128, 32, 4), X(128, 256, 32, 4), X(256, 128, 32, 2), X(128, 128, 64, 2),       \
    X(128, 128, 32, 2), X(32, 256, 64, 4), X(64, 256, 64, 4), X(32, 128, 64, 4), X(64, 512, 32, 2)
#define DL_L(a, b, c, d) &launch_dl<a, b, c, d>
#define DL_O(a, b, c, d) &occ_dl<a, b, c, d>
#define DL_C(a, b, c, d) {a, b, c, d}
const DlLaunchFn kDlFns[] = {DL_CFGS(DL_L)};
const DlOccFn kDlOcc[] = {DL_CFGS(DL_O)};
constexpr int kDlCheck[][4] = {DL_CFGS(DL_C)};
constexpr bool dl_match() {
  for (int i = 0; i < N_DL_CFG; ++i)
    if (kDlCheck[i][0] != kDlCfg[i].bm || kDlCheck[i][1] != kDlCfg[i].bn || kDlCheck[i][2] != kDlCfg[i].bk ||
        kDlCheck[i][3] != kDlCfg[i].stages)
      return false;
  return true;
}
static_assert(sizeof(kDlFns) / sizeof(kDlFns[0]) == N_DL_CFG && dl_match(), "kernels must follow kDlCfg");
#define DL_W(a, b, c, d) Dl<a, b, c, d>::WPE
constexpr int kDlWpe[] = {DL_CFGS(DL_W)};
constexpr bool dl_occ_match() {
  for (int i = 0; i < N_DL_CFG; ++i)
    if (kDlWpe[i] != kDlCfg[i].occ) return false;
  return true;
}
static_assert(dl_occ_match(), "the table's workgroups per CU must be those the kernels are built for");

// the off-chip accumulation kernels: super-tiles of the 256 x 256 tiles
// (DL configurations 0 and 4), whose 512 KiB fp32 accumulator exceeds the
// registers
template <int BM, int BN, int BK, int S>
hipError_t launch_dl_sc(const Plan& p, const GemmArgs& g, hipStream_t st) {
  hipLaunchKernelGGL((k_dl_sc<BM, BN, BK, S>), dim3(p.grid_x, p.grid_y), dim3(256), 0, st, g);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_dl_sc_main(const Plan& p, const GemmArgs& g, hipStream_t st) {
  const int cfg = p.cfg & 0xF, kc = 1 << (p.cfg >> 4);
  if (p.family != FAM_DLSC || (cfg != 0 && cfg != 4) || p.grid_y != kc || p.pk < 2 || p.pk % kc != 0 ||
      g.pk != p.pk || (int64_t)p.grid_x != (int64_t)((g.tiles_m + 1) / 2) * g.tiles_n || !ac::dl_operands_aligned(g))
    return hipErrorInvalidValue;
  return cfg == 0 ? launch_dl_sc<256, 256, 64, 2>(p, g, st) : launch_dl_sc<256, 256, 32, 4>(p, g, st);
}

hipError_t launch_dl_main(const Plan& p, const GemmArgs& g, hipStream_t st) {
  if (p.family != FAM_DL || p.cfg < 0 || p.cfg >= N_DL_CFG) return hipErrorInvalidValue;
  // the register-load form takes any alignment (K >= 8, N >= 8; two stages)
  if (p.unal ? (!kDlCfg[p.cfg].unal || g.K < 8 || g.N < 8) : !ac::dl_operands_aligned(g)) return hipErrorInvalidValue;
  if ((g.lay & ~kDlCfg[p.cfg].col) != 0) return hipErrorInvalidValue;
  return kDlFns[p.cfg](p, g, st, dtype_out16(p.s.dtype));
}

// The grouped kernel of a tile configuration in its direct-to-LDS form
// (where grouped_dl_runs; the register-staged one has the same bits).
hipError_t launch_grouped_dl_plan(const Plan& p, const GroupArgs& a, hipStream_t st) {
  if (!ac::grouped_dl_runs(p, a)) return hipErrorInvalidValue;
  const GemmArgs& g = a.g;
  GroupArgs b = a;
  b.g.kB = g.K;
  b.g.nB = g.N;
  const bool obf = dtype_out16(p.s.dtype);
  const TileCfg& t = kTileCfg[p.cfg];
  if (t.bm == 256 && t.bn == 128) return launch_grouped_dl<256, 128, 64, 3>(p, b, st, obf);
  if (t.bm == 128 && t.bn == 256) return launch_grouped_dl<128, 256, 64, 3>(p, b, st, obf);
  if (t.bm == 128 && t.bn == 128 && t.depth == 1) return launch_grouped_dl<128, 128, 64, 2>(p, b, st, obf);
  if (t.bm == 128 && t.bn == 128) return launch_grouped_dl<128, 128, 64, 3>(p, b, st, obf);
  if (t.bm == 64 && t.bn == 128) return launch_grouped_dl<64, 128, 64, 3>(p, b, st, obf);
  return hipErrorInvalidValue;
}

void query_occupancy_dl() {
  for (int i = 0; i < N_DL_CFG; ++i) set_runtime_occupancy(FAM_DL, i, kDlOcc[i]());
}

#endif  // AC_DL_PART

#if AC_INPUT_F16
}  // namespace f16
#elif AC_DL_PART == 0
bool dl_a_aligned(const void* A, int64_t lda, int64_t K) {
  return (reinterpret_cast<uintptr_t>(A) & 15) == 0 && (lda & 7) == 0 && (K & 7) == 0 && lda < DL_MAX_LD;
}
bool dl_b_aligned(const void* B, int64_t ldb, int64_t nB) {
  return (reinterpret_cast<uintptr_t>(B) & 15) == 0 && (ldb & 7) == 0 && (nB & 7) == 0 && ldb < DL_MAX_LD;
}
// Every group's operands must be aligned: the first one's, and the strides. A
// single k-block leaves nothing to pipeline: 96 products of 200 x 200 x 64 run
// in 6.5 us register-staged (128 x 64 tiles), 6.9 direct-to-LDS at best.
bool grouped_dl_aligned(const GroupArgs& a) {
  const GemmArgs& g = a.g;
  return g.K >= GROUPED_DL_MIN_K && dl_a_aligned(g.A, g.lda, g.K) && dl_b_aligned(g.B, g.ldb, g.N) &&
         (a.groups <= 1 || ((a.stride_a & 7) == 0 && (a.stride_b & 7) == 0));
}
bool grouped_dl_runs(const Plan& p, const GroupArgs& a) {
  return (p.family == FAM_GROUPED || p.family == FAM_BATCHED) && p.cfg >= 0 && p.cfg < N_TILE_CFG &&
         kGroupedDlStages[p.cfg] > 0 && grouped_dl_aligned(a);
}
// (an operand read in place column-major: rows of M, or of K)
bool dl_operands_aligned(const GemmArgs& g) {
  return ((g.lay & 1) ? dl_b_aligned(g.A, g.lda, g.M) : dl_a_aligned(g.A, g.lda, g.K)) &&
         ((g.lay & 2) ? dl_a_aligned(g.B, g.ldb, g.K) : dl_b_aligned(g.B, g.ldb, g.nB));
}

// ---- padding prologue (the Padding module of Table 2)
// dst (rows x ld_dst, ld_dst = cols rounded up to 8, 16-byte aligned) =
// src (rows x cols, row pitch ld_src, any 2-byte alignment), zeros in the pad
// columns: every row of the copy is a whole number of aligned 16-byte
// chunks. A thread moves one 16-byte group; x: groups of a row, y: rows.
__global__ __launch_bounds__(256) void k_pad16(const uint16_t* __restrict__ src, int64_t ld_src,
                                               uint16_t* __restrict__ dst, int64_t ld_dst, int64_t rows,
                                               int64_t cols) {
  const int64_t c = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (c >= ld_dst) return;
  for (int64_t r = blockIdx.y; r < rows; r += gridDim.y) {
    const uint16_t* s = src + r * ld_src + c;
    u32x4 v;
    if (c + 8 <= cols) {
      __builtin_memcpy(&v, s, 16);  // unaligned 16-byte load (gfx950 unaligned mode)
    } else {
      uint32_t h[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) h[e] = c + e < cols ? s[e] : 0u;
      v = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
    }
    __builtin_memcpy(dst + r * ld_dst + c, &v, 16);
  }
}

hipError_t launch_pad16(const uint16_t* src, int64_t ld_src, int64_t rows, int64_t cols, uint16_t* dst,
                        int64_t ld_dst, hipStream_t st) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if (ld_src < cols || ld_dst < cols || (ld_dst & 7) != 0 || ((uintptr_t)dst & 15) != 0) return hipErrorInvalidValue;
  const int64_t gx = (ld_dst / 8 + 255) / 256;
  if (gx > (1LL << 31) - 1) return hipErrorInvalidValue;
  const dim3 grid((unsigned)gx, (unsigned)(rows < 4096 ? rows : 4096)), block(256);
  hipLaunchKernelGGL(k_pad16, grid, block, 0, st, src, ld_src, dst, ld_dst, rows, cols);
  return hipGetLastError();
}
#endif
}  // namespace ac
