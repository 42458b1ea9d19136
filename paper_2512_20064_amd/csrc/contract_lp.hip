// Low-precision contraction of the MPS sampling sweep for gfx950: 16-bit
// MFMA operands with FP32 accumulation (Section 3.3.1, mixed precision).
//
// Forms
//   bf16x3  x = hi + lo with hi = bf16(x), lo = bf16(x - hi) for both the left
//           vectors and the site tensor; W = Lh*Bh + Lh*Bl + Ll*Bh on
//           v_mfma_f32_32x32x16_bf16 (the lo*lo term, ~2^-16 relative, is
//           dropped).  bf16 keeps FP32's exponent range, so no scaling is
//           needed beyond the per-sample renormalisation.
//   fp16    one product on v_mfma_f32_32x32x16_f16 with the left vector
//           renormalised per sample (|l_i| <= 1) and the site tensor's
//           entries bounded by 1 (orthonormal rows).
//   fp16f8  the fp16 product of the high parts, plus the two correction
//           products Lh*Bl and Ll*Bh in OCP FP8 E4M3 on the block-scaled
//           v_mfma_scale_f32_32x32x64_f8f6f4 (operand formats and scales in
//           sweep.h, kFp16F8).  One FP8 instruction takes 64 K values per
//           row and column: 32 real K values of each correction product,
//           so per 32 real K a 32x32 block costs two fp16 MFMAs (32 cycles
//           each) and one FP8 MFMA (64 cycles), against six 16-bit MFMAs
//           for bf16x3.
//   fp16f6  fp16f8 with the corrections in FP6 E2M3, one power-of-two scale
//           per 32-value lane record (sweep.h, kFp16F6): the FP6 instruction
//           runs at twice the FP8 rate, 96 cycles per 32 real K.
//
// Complex arithmetic uses the real embedding of the site tensor: real column
// (c, p) of branch i multiplies the interleaved left vector (re, im) by
// (Re a, -Im a) for p = 0 (real part of W) and (Im a, Re a) for p = 1
// (imaginary part).  Only the p = 0 rows are stored: pack_kernel writes one
// row per complex column, transposed so that K is contiguous ("NT" operands:
// both MFMA operands are 16-byte runs of K) and K-blocked (see kblk_off),
// each branch padded with zero columns to a multiple of the tile and K padded
// with zeros to a multiple of 64.  The p = 1 operand is the p = 0 one with
// every (re, im) pair of K values swapped and the new first member negated,
// which a lane does to its own registers (the turn functions below): exact,
// since fp16, bf16, E4M3 and E2M3 rounding are symmetric in sign.  The
// products do exactly the algorithmic 8 real flops per complex multiply-add.
//
// What bounds the plateau launches (65536 x 1024 x 4096 complex): the matrix
// cores at the clock the power limit leaves, then LDS: per slice a wave reads
// 64 rows and 64 columns of each plane.  With both rows of the embedding
// stored (half as much again read from LDS and L2, twice the packing) fp16f6
// took 3.55 ms per launch and bf16x3 4.95; now 3.1 and 4.5 (chi = 1024 chains,
// whole sweep: 48.5 -> 42.7 ms and 14.9 -> 13.9 ms).

#include "e2m3.h"
#include "lp_ops.h"
#include "sweep.h"
#include "tiling.h"

namespace mps {
namespace {

// ---------------------------------------------------------------- pack ----

constexpr int PK_L = 32;   // complex l per tile (64 real K)
constexpr int PK_C = 64;   // complex columns per tile
constexpr int PK_P = PK_C + 1;

template <typename T, int NPROD>
__global__ __launch_bounds__(256) void pack_kernel(const PackProb* probs, const int* blk_start, int nprob) {
  __shared__ float2 tile[PK_L][PK_P];
  const int p = find_problem(blk_start, nprob, blockIdx.x);
  const PackProb a = probs[p];
  const int lb = blockIdx.x - blk_start[p];
  const int ncb = a.CP / PK_C, nlb = a.Kp / (2 * PK_L);
  const int c0 = (lb % ncb) * PK_C;
  const int l0 = ((lb / ncb) % nlb) * PK_L;
  const int br = lb / (ncb * nlb);
  const int tid = threadIdx.x;
  const size_t pitch = (size_t)a.d * a.chi_r;
#pragma unroll
  for (int it = 0; it < PK_L * PK_C / 256; ++it) {
    const int idx = it * 256 + tid;
    const int l = idx / PK_C, c = idx % PK_C;
    const int gl = l0 + l, gc = c0 + c;
    tile[l][c] = (gl < a.K && gc < a.chi_r) ? a.A[(size_t)gl * pitch + (size_t)br * a.chi_r + gc]
                                            : make_float2(0.f, 0.f);
  }
  __syncthreads();
  // 64 output rows (the p = 0 row of every column) of 64 real K each, written
  // as 8 chunks of 8 elements.
  T* Bh = (T*)a.Bh;
  T* Bl = (T*)a.Bl;
#pragma unroll
  for (int it = 0; it < PK_C * 8 / 256; ++it) {
    const int idx = it * 256 + tid;
    const int c = idx >> 3, ch = idx & 7;
    float v[8];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const float2 z = tile[ch * 4 + m][c];
      v[m] = z.x;
      v[4 + m] = -z.y;
    }
    typename Vec8<T>::type h, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      h[e] = (T)v[e];
      lo[e] = (T)(v[e] - (float)h[e]);
    }
    const size_t orow = (size_t)br * a.CP + c0 + c;
    const size_t off = kblk_off(orow, 2 * l0 + ch * 8, a.Kp);
    *reinterpret_cast<typename Vec8<T>::type*>(Bh + off) = h;
    if (NPROD == 3) *reinterpret_cast<typename Vec8<T>::type*>(Bl + off) = lo;
  }
}

// ------------------------------------------------------------ contract ----

constexpr int BM = kLpBM;            // rows (samples) per workgroup
constexpr int BK = kLpBK;            // real K per pipeline stage
constexpr int ARR = BM * BK * 2;     // bytes of one left-vector tile in a stage (8 KiB)
static_assert(BM == 256 && BK == 16, "layout below assumes 256-row tiles and 16-K stages");

// Tile variants (sweep.h): NWC wave columns of 64 rows x 64 complex columns
// each, over 4 wave rows.  Wide: NWC = 2, a 256 x 128 complex tile of 8 waves;
// narrow: NWC = 1, 256 x 64, 4 waves.  Every wave runs the same code on the
// same 64 x 64 block shape, so both variants give the same bits.
template <int NWC>
struct LpTile {
  static constexpr int BN = 64 * NWC;             // complex columns (packed rows) per workgroup
  static constexpr int NTHR = 256 * NWC;          // 4 x NWC waves
  static constexpr int BARR = BN * BK * 2;        // bytes of one site-tensor tile in a stage
};

// s_waitcnt immediate: at most n vector-memory operations of this wave still
// outstanding, and every LDS read of this wave returned (lgkmcnt 0); expcnt
// is not waited on.
constexpr unsigned vmcnt_lgkm0_imm(unsigned n) { return (n & 0xF) | (0x7u << 4); }

// Load instruction idx (0 .. groups-1) of a slice: one KiB = 32 rows of one
// operand tile.  The NL left-vector tiles come first (8 row groups each),
// then the NB site-tensor tiles (BN/32 row groups each).
template <int NWC>
__device__ inline void load_slot(int idx, int NL, int& q, int& rg, int& ldst) {
  constexpr int GB = LpTile<NWC>::BN / 32;
  if (idx < NL * 8) {
    q = idx >> 3;
    rg = idx & 7;
    ldst = q * ARR + rg * 1024;
  } else {
    const int ib = idx - NL * 8;
    q = NL + ib / GB;
    rg = ib % GB;
    ldst = NL * ARR + (q - NL) * LpTile<NWC>::BARR + rg * 1024;
  }
}

// Partial branch weights of the tile (part_sum), one per wave column, staged
// in LDS and stored as one run of partials per row.
template <int NWC>
__device__ inline void store_partials(const floatx16 (&acc)[2][4], float* red, int wave, int wr, int half, int j,
                                      int tid, int m0, int rows, float* qpart, size_t qrow, int q0) {
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float s = part_sum(acc[rb][0][v], acc[rb][1][v], acc[rb][2][v], acc[rb][3][v]);
      const int r = wr + rb * 32 + (v >> 2) * 8 + half * 4 + (v & 3);
      if (j == 0) red[r * NWC + wave % NWC] = s;
    }
  }
  __syncthreads();
  if (tid < BM) {
    const int gr = m0 + tid;
    if (gr < rows) {
      float* dst = qpart + (size_t)gr * qrow + q0;
#pragma unroll
      for (int g = 0; g < NWC; ++g) dst[g] = red[tid * NWC + g];
    }
  }
}

// W element store (one complex): a global-memory (not flat) store marked
// nontemporal.  W is written once per launch and read back by the measurement
// only for the chosen branch, long after the 2 GiB of a plateau launch has
// left the caches, so its lines need not displace operand tiles in L2 (1-4 %
// per launch, standalone timing of the headline shape).
typedef float floatx2 __attribute__((ext_vector_type(2)));
__device__ inline void store_w(float2* p, float re, float im) {
  __builtin_nontemporal_store(floatx2{re, im}, (__attribute__((address_space(1))) floatx2*)p);
}

// W of a wave's block: output lane (j, half) of a 32x32 MFMA block holds its
// column's rows 8*(v/4) + 4*half + v%4.  Runs of 16 lanes store 128
// contiguous bytes of a row.
__device__ inline void store_w_block(const floatx16 (&acc)[2][4], float2* W, size_t ncols, int m0, int rows,
                                     size_t col0, int c0, int chi_r, int half, int j) {
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int cw = wave_col(b, j);
      if (c0 + cw < chi_r) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int gr = m0 + rb * 32 + (v >> 2) * 8 + half * 4 + (v & 3);
          if (gr < rows) store_w(W + (size_t)gr * ncols + col0 + cw, acc[rb][2 * b][v], acc[rb][2 * b + 1][v]);
        }
      }
    }
  }
}

// Pipeline: a stage is two 16-K slices (one barrier per 32 real K) and lives
// in LDS buffer (stage % NST).  Operand tiles go straight from memory into LDS
// (buffer loads to LDS: no staging registers and no LDS store phase), up to
// NST-1 stages ahead of the stage being read.  Ring: wide 144-160 KiB, one
// workgroup per CU; narrow at most 80 KiB and 256 registers, two workgroups
// per CU.
// (The body is a device function template with one plain kernel per variant
// below.)
template <typename T, int NPROD, int NWC>
__device__ inline void contract_lp_kernel(const ContractLpProb* probs, const int* tn_start, int nprob, int tn_total,
                                        int tiles_m, int per_xcd, int group_m, const ChunkArgs* chp) {
  typedef typename Vec8<T>::type V8;
  typedef LpTile<NWC> Tile;
  // Products per complex product: 3 = Lh*Bh + Lh*Bl + Ll*Bh (split form);
  // 2 = Lh*Bh + Ll*Bh (split left vectors, site tensor exact in T, so Bl = 0
  // and the omitted product adds exact zeros); 1 = Lh*Bh.
  constexpr int NL = NPROD >= 2 ? 2 : 1;    // left-vector tiles per stage: Ah, [Al]
  constexpr int NB = NPROD == 3 ? 2 : 1;    // site-tensor tiles per stage: Bh, [Bl]
  constexpr int SLICE = NL * ARR + NB * Tile::BARR;
  constexpr int STAGE = 2 * SLICE;
  constexpr int NST = (NWC == 2 ? 160 : 80) * 1024 / STAGE;
  constexpr int GROUPS = NL * 8 + NB * (Tile::BN / 32);  // 1 KiB load instructions per slice
  constexpr int NWAVE = 4 * NWC;
  constexpr int IPW = 2 * GROUPS / NWAVE;                // and per wave and stage
  static_assert(2 * GROUPS % NWAVE == 0, "loads must divide evenly over the waves");
  static_assert(NST >= 2 && NST <= 6 && (NST - 2) * IPW <= 15, "vmcnt immediates below");
  constexpr int BOFF = NL * ARR;             // offset of the Bh tile in a slice
  __shared__ __attribute__((aligned(16))) char lds[NST * STAGE];

  int tm, tng;
  if (!map_tile(blockIdx.x, tiles_m, tn_total, per_xcd, group_m, tm, tng)) return;
  const int rows = chp->rows;
  const int p = find_problem(tn_start, nprob, tng);
  const ContractLpProb a = probs[p];
  const int tn = tng - tn_start[p];
  const int TC = a.CP / Tile::BN;           // column tiles per branch
  const int branch = tn / TC;
  const int ct = tn - branch * TC;
  const int m0 = tm * BM;
  const int c0 = ct * Tile::BN;                              // first complex column within the branch
  const size_t prow = (size_t)branch * a.CP + c0;            // first packed row of the tile
  const size_t cblk = prow >> 8;                             // its 256-row block
  const int crow = (int)(prow & 255);                        // and row within the block (a multiple of BN)

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wr = (wave / NWC) * 64;
  const int wc = (wave % NWC) * 64;  // complex columns
  const int half = lane >> 5;
  const int j = lane & 31;

  // This wave's load instructions: slice u, tile q, row group rg (32 rows =
  // 1 KiB).  All are uniform over the wave, so each load goes through a buffer
  // descriptor (scalar registers) based at the tile's 256-row block; the K
  // position is a scalar offset and each lane keeps one 32-bit byte offset.
  const size_t kbs = (size_t)(a.Kp / BK) * 8192;  // bytes per 256-row block
  const int wv = __builtin_amdgcn_readfirstlane(wave);
  __amdgpu_buffer_rsrc_t rsrc[IPW];
  int voff[IPW], ldst[IPW], ksl[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    int q, rg, dst;
    const int slot = wv * IPW + i, u = slot / GROUPS;
    load_slot<NWC>(slot - u * GROUPS, NL, q, rg, dst);
    const bool is_b = q >= NL;
    const int qq = is_b ? q - NL : q;  // 0 = hi, 1 = lo
    const char* base = is_b ? (const char*)(qq ? a.Bl : a.Bh) + cblk * kbs
                            : (const char*)(qq ? a.Ll : a.Lh) + (size_t)tm * kbs;
    rsrc[i] = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)0xFFFFFFFF, 0x00020000);
    const int row = rg * 32 + (lane >> 1) + (is_b ? crow : 0);
    const int lc = (lane & 1) ^ swz(row);
    voff[i] = row * 32 + lc * 16;
    ldst[i] = u * SLICE + dst;
    ksl[i] = u * 8192;
  }
  auto issue = [&](int kt) {
    char* st = lds + (kt % NST) * STAGE;
#pragma unroll
    for (int i = 0; i < IPW; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc[i], (__attribute__((address_space(3))) void*)(st + ldst[i]), 16,
                                               voff[i], kt * 16384 + ksl[i], 0, 0);
  };

  floatx16 acc[2][4];
  const floatx16 zero = {};
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[rb][cb] = zero;

  // The operands of one slice, read from LDS into registers.  Two sets
  // alternate: while the MFMAs of one slice run on one set, the LDS reads of
  // the next fill the other, so LDS time hides behind MFMA time instead of
  // adding to it.
  struct Ops {
    V8 ah[2], al[2], bh[2], bl[2];
  };
  auto lds_read = [&](int kt, int u, Ops& o) {
    const char* st = lds + (kt % NST) * STAGE + u * SLICE;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const int row = wr + rb * 32 + j;
      o.ah[rb] = *reinterpret_cast<const V8*>(st + 0 * ARR + lds_off(row, half));
      if (NL == 2) o.al[rb] = *reinterpret_cast<const V8*>(st + 1 * ARR + lds_off(row, half));
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int row = wc + wave_col(b, j);
      o.bh[b] = *reinterpret_cast<const V8*>(st + BOFF + lds_off(row, half));
      if (NB == 2) o.bl[b] = *reinterpret_cast<const V8*>(st + BOFF + Tile::BARR + lds_off(row, half));
    }
  };
  auto mma = [&](const Ops& o) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      V8 bh = o.bh[b], bl;
      if (NB == 2) bl = o.bl[b];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        if (p == 1) {
          bh = turn(bh);
          if (NB == 2) bl = turn(bl);
        }
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          floatx16& c = acc[rb][2 * b + p];
          c = Vec8<T>::mfma(o.ah[rb], bh, c);
          if (NB == 2) c = Vec8<T>::mfma(o.ah[rb], bl, c);
          if (NL == 2) c = Vec8<T>::mfma(o.al[rb], bh, c);
        }
      }
    }
  };
  // Make stage s readable by every wave: wait for this wave's own loads of
  // stage s (the `issued - 1 - s` stages issued after it may stay in flight)
  // and for this wave's LDS reads, then one barrier; then issue the next
  // stage into the buffer of stage s - 1, whose LDS reads every wave has
  // finished (the LDS-read wait before the barrier; those reads were issued a
  // slice of MFMAs earlier).
  const int nst = a.Kp / (2 * BK);  // stages: at least 2 (Kp is a multiple of 64)
  int issued = 0;
  auto open_stage = [&](int s) {
    const int later = issued - 1 - s;
    if (later >= 4 && NST > 5) __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_imm(4 * IPW));
    else if (later == 3 && NST > 4) __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_imm(3 * IPW));
    else if (later == 2 && NST > 3) __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_imm(2 * IPW));
    else if (later == 1 && NST > 2) __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_imm(IPW));
    else __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_imm(0));
    asm volatile("s_barrier" ::: "memory");
    if (issued < nst) issue(issued++);
  };

#pragma unroll
  for (int i = 0; i < NST - 1; ++i)
    if (i < nst) issue(issued++);
  Ops o0, o1;
  open_stage(0);
  lds_read(0, 0, o0);
  // Steady state: `issued` = kt + NST at every step, so the wait keeps NST - 2
  // stages in flight and one stage is issued; as straight-line code (no
  // branch in the step) the compiler keeps the MFMAs ahead of the barrier.
  // The last stages take the general step below.
  int kt = 0;
  for (; kt + NST < nst; ++kt) {
    lds_read(kt, 1, o1);
    mma(o0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_imm((NST - 2) * IPW));
    asm volatile("s_barrier" ::: "memory");
    issue(issued++);
    __builtin_amdgcn_sched_barrier(0);
    lds_read(kt + 1, 0, o0);
    mma(o1);
    __builtin_amdgcn_sched_barrier(0);
  }
  for (; kt < nst; ++kt) {
    lds_read(kt, 1, o1);
    mma(o0);
    if (kt + 1 < nst) {
      open_stage(kt + 1);
      lds_read(kt + 1, 0, o0);
    }
    mma(o1);
  }
  __syncthreads();  // the stage buffers are reused below

  // Epilogue 1: W.
  store_w_block(acc, a.W, (size_t)a.d * a.chi_r, m0 + wr, rows, (size_t)branch * a.chi_r + c0 + wc, c0 + wc, a.chi_r,
                half, j);
  // Epilogue 2: partial weights per 64 complex columns; padded columns are
  // exact zeros.
  const int TP = a.CP / kPartCols;  // partials per branch
  store_partials<NWC>(acc, reinterpret_cast<float*>(lds), wave, wr, half, j, tid, m0, rows, a.qpart,
                      (size_t)a.d * TP, branch * TP + c0 / kPartCols);
}

#define MPS_LP_KERNEL(NAME, T, NPROD, NWC)                                                                        \
  __global__ __launch_bounds__(LpTile<NWC>::NTHR, 3 - NWC) void NAME(                                             \
      const ContractLpProb* probs, const int* tn_start, int nprob, int tn_total, int tiles_m, int per_xcd,        \
      int group_m, const ChunkArgs* chp) {                                                                        \
    contract_lp_kernel<T, NPROD, NWC>(probs, tn_start, nprob, tn_total, tiles_m, per_xcd, group_m, chp);            \
  }
MPS_LP_KERNEL(contract_bf16x3_wide, bf16_t, 3, 2)
MPS_LP_KERNEL(contract_bf16x3_narrow, bf16_t, 3, 1)
MPS_LP_KERNEL(contract_fp16x3_wide, f16_t, 3, 2)
MPS_LP_KERNEL(contract_fp16x3_narrow, f16_t, 3, 1)
MPS_LP_KERNEL(contract_fp16x2_wide, f16_t, 2, 2)
MPS_LP_KERNEL(contract_fp16x2_narrow, f16_t, 2, 1)
MPS_LP_KERNEL(contract_fp16_wide, f16_t, 1, 2)
MPS_LP_KERNEL(contract_fp16_narrow, f16_t, 1, 1)
#undef MPS_LP_KERNEL

// ------------------------------------------------------------ fp16f8 ----

// Smallest power of two s with amax / s <= 448 (the largest finite E4M3
// value), exponent clamped to the normal FP32 range; 1 for zero or a
// non-finite amax (which then shows as a non-finite S downstream).
__device__ inline float pow2_scale(float amax) {
  if (!(amax > 0.f) || isinf(amax)) return 1.f;
  int E;
  const float m = frexpf(amax, &E);  // amax = m * 2^E, m in [0.5, 1); 448 = 0.875 * 2^9
  int e = m <= 0.875f ? E - 9 : E - 8;
  e = e < -126 ? -126 : e;
  return ldexpf(1.f, e);
}

// Four floats to four E4M3 codes (round to nearest even), first in the low byte.
__device__ inline unsigned e4m3x4(float a, float b, float c, float d) {
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
  return (unsigned)w;
}

// Column maxima: one workgroup per (row block, branch, 64 complex columns);
// 4 row phases of 64 threads, maximum of |re| and |im| over the block's rows.
__global__ __launch_bounds__(256) void colmax_kernel(const PackProb* probs, const int* cm_start, int nprob) {
  __shared__ float part[4][64];
  const int p = find_problem(cm_start, nprob, blockIdx.x);
  const PackProb a = probs[p];
  const int ncb = a.CP / 64;
  const int wb = blockIdx.x - cm_start[p];
  const int rb = wb / (a.d * ncb);
  const int rest = wb - rb * (a.d * ncb);
  const int br = rest / ncb;
  const int c = (rest - br * ncb) * 64 + (threadIdx.x & 63);
  const int ph = threadIdx.x >> 6;
  const int RB = colmax_blocks(a.K);
  const int rpb = (a.K + RB - 1) / RB;
  const int l1 = min(a.K, (rb + 1) * rpb);
  float m = 0.f;
  if (c < a.chi_r) {
    const size_t pitch = (size_t)a.d * a.chi_r;
    const float2* col = a.A + (size_t)br * a.chi_r + c;
    for (int l = rb * rpb + ph; l < l1; l += 4) {
      const float2 z = col[(size_t)l * pitch];
      m = fmaxf(m, fmaxf(fabsf(z.x), fabsf(z.y)));
    }
  }
  part[ph][threadIdx.x & 63] = m;
  __syncthreads();
  if (threadIdx.x < 64) {
    const float mm = fmaxf(fmaxf(part[0][threadIdx.x], part[1][threadIdx.x]),
                           fmaxf(part[2][threadIdx.x], part[3][threadIdx.x]));
    a.colpart[(size_t)rb * a.d * a.CP + (size_t)br * a.CP + c] = mm;
  }
}

// Packing of the fp16f8 operands: the same tiles as pack_kernel; each real
// value v (column already divided by its scale) gives h = fp16(v) into the
// 16-bit plane and the codes e4m3(h), e4m3((v - h) * 2^11) into the pair
// plane (low part first: [B8l | B8h]).  F6 (fp16f6): the same two values per
// K as E2M3 codes of one 32-value record per packed row and 16-K slice
// (low parts codes 0..15, high parts 16..31), scaled by the record's
// power of two.
template <bool F6>
__global__ __launch_bounds__(256) void pack_f16f8_kernel(const PackProb* probs, const int* blk_start, int nprob) {
  __shared__ float2 tile[PK_L][PK_P];
  const int p = find_problem(blk_start, nprob, blockIdx.x);
  const PackProb a = probs[p];
  const int lb = blockIdx.x - blk_start[p];
  const int ncb = a.CP / PK_C, nlb = a.Kp / (2 * PK_L);
  const int c0 = (lb % ncb) * PK_C;
  const int l0 = ((lb / ncb) % nlb) * PK_L;
  const int br = lb / (ncb * nlb);
  const int tid = threadIdx.x;
  const size_t pitch = (size_t)a.d * a.chi_r;
#pragma unroll
  for (int it = 0; it < PK_L * PK_C / 256; ++it) {
    const int idx = it * 256 + tid;
    const int l = idx / PK_C, c = idx % PK_C;
    const int gl = l0 + l, gc = c0 + c;
    tile[l][c] = (gl < a.K && gc < a.chi_r) ? a.A[(size_t)gl * pitch + (size_t)br * a.chi_r + gc]
                                            : make_float2(0.f, 0.f);
  }
  // column scales of the tile's 64 columns from the row-block maxima; the
  // workgroups of the first K block also store them for the contraction
  __shared__ float inv_sh[PK_C];
  {
    __shared__ float mpart[4][PK_C];
    const int RB = colmax_blocks(a.K);
    const int c = tid & (PK_C - 1), ph = tid >> 6;
    const float* cp = a.colpart + (size_t)br * a.CP + c0 + c;
    float m = 0.f;
    for (int rb = ph; rb < RB; rb += 4) m = fmaxf(m, cp[(size_t)rb * a.d * a.CP]);
    mpart[ph][c] = m;
    __syncthreads();
    if (tid < PK_C) {
      const float s = pow2_scale(fmaxf(fmaxf(mpart[0][tid], mpart[1][tid]), fmaxf(mpart[2][tid], mpart[3][tid])));
      inv_sh[tid] = 1.f / s;  // exact: a power of two
      if (l0 == 0) a.colscale[(size_t)br * a.CP + c0 + tid] = s;
    }
  }
  __syncthreads();
  f16_t* Bh = (f16_t*)a.Bh;
  unsigned char* B8 = (unsigned char*)a.Bl;
#pragma unroll
  for (int it = 0; it < PK_C * 8 / 256; ++it) {
    const int idx = it * 256 + tid;
    const int c = idx >> 3, ch = idx & 7;
    const float inv = inv_sh[c];
    float v[8];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const float2 z = tile[ch * 4 + m][c];
      v[m] = z.x * inv;
      v[4 + m] = -z.y * inv;
    }
    f16x8 h;
    float hf[8], lo[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      h[e] = (f16_t)v[e];
      hf[e] = (float)h[e];
      lo[e] = (v[e] - hf[e]) * 2048.f;
    }
    const size_t orow = (size_t)br * a.CP + c0 + c;
    const int k = 2 * l0 + ch * 8;
    *reinterpret_cast<f16x8*>(Bh + kblk_off(orow, k, a.Kp)) = h;
    if constexpr (!F6) {
      unsigned char* d8 = B8 + pair_off(orow, k, a.Kp);
      *reinterpret_cast<uint2*>(d8) = make_uint2(e4m3x4(lo[0], lo[1], lo[2], lo[3]), e4m3x4(lo[4], lo[5], lo[6], lo[7]));
      *reinterpret_cast<uint2*>(d8 + 16) =
          make_uint2(e4m3x4(hf[0], hf[1], hf[2], hf[3]), e4m3x4(hf[4], hf[5], hf[6], hf[7]));
    } else {
      // The record of this packed row's 16-K slice: threads ch and ch^1
      // (adjacent lanes) hold its two halves; the scale is their common max.
      float m = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) m = fmaxf(m, fmaxf(fabsf(hf[e]), fabsf(lo[e])));
      m = fmaxf(m, __shfl_xor(m, 1));
      // (at least 2^-108, so that the stored scale code 127 + ke - 19 >= 0;
      // a record that small flushes to zero)
      const int ke = max(e2m3_scale_exp(m), -108);
      const float inv2 = ldexpf(1.f, -ke - 6);
      // this thread's codes, 4 of 6 bits each: low and high parts, re and im
      uint32_t c[4];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int e = 4 * i;
        c[2 * i] = e2m3x4(lo[e] * inv2, lo[e + 1] * inv2, lo[e + 2] * inv2, lo[e + 3] * inv2);
        c[2 * i + 1] = e2m3x4(hf[e] * inv2, hf[e + 1] * inv2, hf[e + 2] * inv2, hf[e + 3] * inv2);
      }
      // Site record: the 8 real parts' low codes, their high codes, then the
      // same of the imaginary parts; complex 0..3 of the slice from the
      // thread with (k & 8) == 0, 4..7 from its neighbour.  Both threads
      // assemble the 192 code bits and each stores one 16-byte half; byte 24
      // is the scale (the corrections' common 2^-19 rides on the site's
      // scale), zeros after.
      const int q = (k & 8) ? 1 : 0;
      uint32_t w[6];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint32_t lo_o = __shfl_xor(c[2 * i], 1), hi_o = __shfl_xor(c[2 * i + 1], 1);
        const uint32_t l0 = q ? lo_o : c[2 * i], l1 = q ? c[2 * i] : lo_o;
        const uint32_t h0 = q ? hi_o : c[2 * i + 1], h1 = q ? c[2 * i + 1] : hi_o;
        w[3 * i] = l0 | (l1 << 24);
        w[3 * i + 1] = (l1 >> 8) | (h0 << 16);
        w[3 * i + 2] = (h0 >> 16) | (h1 << 8);
      }
      unsigned char* rec = B8 + pair_off(orow, k & ~15, a.Kp);
      if (q == 0)
        *reinterpret_cast<uint4*>(rec) = make_uint4(w[0], w[1], w[2], w[3]);
      else
        *reinterpret_cast<uint4*>(rec + 16) = make_uint4(w[4], w[5], (uint32_t)(127 + ke - 19), 0u);
    }
  }
}

// The fp16f8 contraction.  Same tile (256 x 128 complex), waves, operand
// loading (global_load_lds into a 6-slice LDS ring) and epilogue as
// contract_lp_kernel; a slice holds 16 real K of [Lh | L8 | Bh | B8].  The FP8
// instruction takes 32 bytes per lane: lane half h of a row (column) reads
// its 32-byte row of the pair plane from slice 2m + h, so one instruction
// covers the slice pair (2m, 2m+1) and both correction products on it.  The
// slices are made readable a pair at a time (one barrier per 32 real K):
// while pair m is read and multiplied, slices 2m+2 .. 2m+5 are in flight,
// and the loads issued after the barrier of pair m+1 (slices 2m+6, 2m+7)
// refill the two buffers of pair m, whose LDS reads every wave has finished
// (LDS-read wait before the barrier).
// (The body is a device function template with one plain kernel per
// variant below.)
template <int NWC, bool F6>
__device__ inline void contract_f16f8_body(const ContractLpProb* probs, const int* tn_start, int nprob, int tn_total,
                                           int tiles_m, int per_xcd, int group_m, const ChunkArgs* chp) {
  typedef LpTile<NWC> Tile;
  constexpr int NST = 6;  // three slice pairs: one in use, two in flight
  constexpr int BOFF = 2 * ARR;  // stage: Lh, L8 (pair plane), Bh, B8 (pair plane)
  constexpr int STAGE = 2 * ARR + 2 * Tile::BARR;
  constexpr int GROUPS = 2 * 8 + 2 * (Tile::BN / 32);
  constexpr int IPW = GROUPS / (4 * NWC);
  static_assert(GROUPS % (4 * NWC) == 0 && 2 * IPW <= 15, "loads must divide evenly; vmcnt immediates");
  __shared__ __attribute__((aligned(16))) char lds[NST * STAGE];

  int tm, tng;
  if (!map_tile(blockIdx.x, tiles_m, tn_total, per_xcd, group_m, tm, tng)) return;
  const int rows = chp->rows;
  const int p = find_problem(tn_start, nprob, tng);
  const ContractLpProb a = probs[p];
  const int tn = tng - tn_start[p];
  const int TC = a.CP / Tile::BN;  // column tiles per branch
  const int branch = tn / TC;
  const int ct = tn - branch * TC;
  const int m0 = tm * BM;
  const int c0 = ct * Tile::BN;
  const size_t prow = (size_t)branch * a.CP + c0;  // first packed row of the tile
  const size_t cblk = prow >> 8;
  const int crow = (int)(prow & 255);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wr = (wave / NWC) * 64;
  const int wc = (wave % NWC) * 64;
  const int half = lane >> 5;
  const int j = lane & 31;

  // Loads: planes and pair planes are addressed alike (8 KiB per 256 rows
  // and 16 K).  Load i of a wave reads operand tile q (load_slot), a choice
  // that is uniform over the wave, through a buffer descriptor (scalar
  // registers) based at the tile's 256-row block; the slice is a scalar
  // offset and each lane keeps one 32-bit byte offset.
  const size_t kbs = (size_t)(a.Kp / BK) * 8192;  // bytes per 256-row block
  const int wv = __builtin_amdgcn_readfirstlane(wave);
  __amdgpu_buffer_rsrc_t rsrc[IPW];
  int voff[IPW], ldst[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    int q, rg, dst;
    load_slot<NWC>(wv * IPW + i, 2, q, rg, dst);  // q: 0 Lh, 1 L8, 2 Bh, 3 B8
    const char* base = q == 0 ? (const char*)a.Lh + (size_t)tm * kbs
                     : q == 1 ? (const char*)a.Ll + (size_t)tm * kbs
                     : q == 2 ? (const char*)a.Bh + cblk * kbs
                              : (const char*)a.Bl + cblk * kbs;
    rsrc[i] = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)0xFFFFFFFF, 0x00020000);
    const int row = rg * 32 + (lane >> 1) + (q >= 2 ? crow : 0);
    const int lc = (lane & 1) ^ swz(row);
    voff[i] = row * 32 + lc * 16;
    ldst[i] = dst;
  }
  auto issue = [&](int kt) {
    char* st = lds + (kt % NST) * STAGE;
#pragma unroll
    for (int i = 0; i < IPW; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc[i], (__attribute__((address_space(3))) void*)(st + ldst[i]), 16,
                                               voff[i], kt * 8192, 0, 0);
  };

  floatx16 acc[2][4];
  const floatx16 zero = {};
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[rb][cb] = zero;

  struct Ops16 {
    f16x8 a[2], b[2];
  };
  struct Ops8 {
    intx8 a[2], b[2];
  };
  // LDS read offsets.  Rows r, r + 16 and r + 32 have the same swizzle (it
  // depends on row bits 2 and 3 only), so one offset per operand and chunk
  // serves every block: row blocks 1 KiB apart, column blocks 16 rows (512
  // bytes) apart (immediate offsets).
  const int sj = swz(j);
  const int jc = wc + wave_col(0, j);
  const unsigned a_h = (unsigned)((wr + j) * 32 + ((half ^ sj) << 4));           // Lh, chunk `half`
  const unsigned b_h = (unsigned)(BOFF + jc * 32 + ((half ^ sj) << 4));           // Bh, chunk `half`
  const unsigned a8_0 = (unsigned)(ARR + (wr + j) * 32 + (sj << 4));              // L8, chunk 0
  const unsigned a8_1 = (unsigned)(ARR + (wr + j) * 32 + ((1 ^ sj) << 4));        // L8, chunk 1
  const unsigned b8_0 = (unsigned)(BOFF + Tile::BARR + jc * 32 + (sj << 4));        // B8, chunk 0
  const unsigned b8_1 = (unsigned)(BOFF + Tile::BARR + jc * 32 + ((1 ^ sj) << 4));  // B8, chunk 1
  auto read16 = [&](int kt, Ops16& o) {
    const char* st = lds + (kt % NST) * STAGE;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) o.a[rb] = *reinterpret_cast<const f16x8*>(st + a_h + rb * 1024);
#pragma unroll
    for (int b = 0; b < 2; ++b) o.b[b] = *reinterpret_cast<const f16x8*>(st + b_h + b * 512);
  };
  auto cat = [](intx4 x, intx4 y) -> intx8 { return __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7); };
  // FP6 records: dwords 0..5 codes, dword 6 scale, dword 7 zero (read as
  // two 16-byte chunks like the FP8 pairs: fewer LDS instructions than a
  // 16 + 8 + 4 byte split, and the kernel still fits without spills)
  auto rec6 = [](const char* q0, const char* q1) -> intx8 {
    const intx4 x = *reinterpret_cast<const intx4*>(q0);
    const intx4 y = *reinterpret_cast<const intx4*>(q1);
    return intx8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
  };
  auto read8 = [&](int m, Ops8& o) {
    const char* st = lds + ((2 * m + half) % NST) * STAGE;  // lane half h: slice 2m + h
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      if constexpr (F6)
        o.a[rb] = rec6(st + a8_0 + rb * 1024, st + a8_1 + rb * 1024);
      else
        o.a[rb] = cat(*reinterpret_cast<const intx4*>(st + a8_0 + rb * 1024),
                      *reinterpret_cast<const intx4*>(st + a8_1 + rb * 1024));
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if constexpr (F6)
        o.b[b] = rec6(st + b8_0 + b * 512, st + b8_1 + b * 512);
      else
        o.b[b] = cat(*reinterpret_cast<const intx4*>(st + b8_0 + b * 512),
                     *reinterpret_cast<const intx4*>(st + b8_1 + b * 512));
    }
  };
  // Per block of 32 columns: the real parts with the operand as read, then
  // the imaginary parts with it turned.
  auto mma16 = [&](const Ops16& o) {
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const f16x8 b = cb & 1 ? turn(o.b[cb >> 1]) : o.b[cb >> 1];
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
        acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(o.a[rb], b, acc[rb][cb], 0, 0, 0);
    }
  };
  // FP6: formats 2 (E2M3) on both sides; the first six dwords of a lane's
  // record are its 32 codes, the low byte of the seventh its scale.
  auto mma8 = [&](const Ops8& o) {
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const intx8 b = cb & 1 ? (F6 ? turn_e2m3(o.b[cb >> 1]) : turn_e4m3(o.b[cb >> 1])) : o.b[cb >> 1];
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        if constexpr (F6)
          acc[rb][cb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(o.a[rb], b, acc[rb][cb], 2, 2, 0, o.a[rb][6],
                                                                        0, b[6]);
        else
          acc[rb][cb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(o.a[rb], b, acc[rb][cb], 0, 0, 0, kScale8L, 0,
                                                                        kScale8B);
      }
    }
  };

  const int nkt = a.Kp / BK;  // a multiple of 4
  const int npair = nkt >> 1;
  int issued = 0;
  // Pair m readable: slices 2m and 2m+1 landed (pair m+1, issued after
  // them, may stay in flight), this wave's LDS reads done, one barrier; then
  // the next two slices are issued into the buffers of pair m-1.
  auto open_pair = [&](int m) {
    if (issued > 2 * m + 2) __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_imm(2 * IPW));
    else __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_imm(0));
    asm volatile("s_barrier" ::: "memory");
    if (issued < nkt) issue(issued++);
    if (issued < nkt) issue(issued++);
  };
#pragma unroll
  for (int i = 0; i < 4; ++i) issue(issued++);  // nkt >= 4
  // Operand registers: e (even slice, fp16), h (odd slice, fp16), f (FP8
  // operands of the pair); at most two of them are live at a time, each
  // read while the MFMAs of another run.
  Ops16 e, h;
  Ops8 f;
  open_pair(0);
  read16(0, e);
  read8(0, f);
  // (sched_barrier: the compiler keeps this order instead of hoisting the
  // next reads above the MFMAs, which would need a third register set)
  // Steady state, pairs 0 .. npair-4: every step opens the next pair and
  // issues two slices.  Straight-line code (no branch inside the step), so
  // that the MFMAs stay ahead of the barrier and the LDS-read waits before
  // mma16(h) cover the reads of h only; the last three pairs take the
  // general step below.
  int m = 0;
  // The FP8/FP6 operands of the next pair are read right after the barrier,
  // before mma16(h) (their registers are free once mma8(f) has issued), so
  // that they have the whole of mma16(h) and mma16(e') to arrive; the
  // reads of h may mix with the MFMAs of e.
  auto step = [&](int m) {
    mma16(e);
    read16(2 * m + 1, h);
    mma8(f);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_imm(2 * IPW));
    asm volatile("s_barrier" ::: "memory");
    issue(issued++);
    issue(issued++);
    __builtin_amdgcn_sched_barrier(0);
    read16(2 * m + 2, e);
    read8(m + 1, f);
    mma16(h);
    __builtin_amdgcn_sched_barrier(0);
  };
  for (; m + 4 < npair; m += 2) {
    step(m);
    step(m + 1);
  }
  for (; m < npair; ++m) {
    mma16(e);
    __builtin_amdgcn_sched_barrier(0);
    read16(2 * m + 1, h);
    mma8(f);
    __builtin_amdgcn_sched_barrier(0);
    if (m + 1 < npair) {
      open_pair(m + 1);
      read16(2 * m + 2, e);
    }
    mma16(h);
    __builtin_amdgcn_sched_barrier(0);
    if (m + 1 < npair) read8(m + 1, f);
  }
  __syncthreads();  // the stage buffers are reused below

  // Column scales: W[:, c] = s_c * acc (exact, a power of two).
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {
    const float sc = a.colscale[(size_t)branch * a.CP + c0 + wc + wave_col(cb >> 1, j)];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[rb][cb][v] *= sc;
  }

  store_w_block(acc, a.W, (size_t)a.d * a.chi_r, m0 + wr, rows, (size_t)branch * a.chi_r + c0 + wc, c0 + wc, a.chi_r,
                half, j);
  const int TP = a.CP / kPartCols;  // partials per branch
  store_partials<NWC>(acc, reinterpret_cast<float*>(lds), wave, wr, half, j, tid, m0, rows, a.qpart,
                      (size_t)a.d * TP, branch * TP + c0 / kPartCols);
}

__global__ __launch_bounds__(LpTile<2>::NTHR, 1) void contract_f16f8_wide(const ContractLpProb* probs,
                                                                          const int* tn_start, int nprob, int tn_total,
                                                                          int tiles_m, int per_xcd, int group_m,
                                                                          const ChunkArgs* chp) {
  contract_f16f8_body<2, false>(probs, tn_start, nprob, tn_total, tiles_m, per_xcd, group_m, chp);
}
__global__ __launch_bounds__(LpTile<1>::NTHR, 1) void contract_f16f8_narrow(const ContractLpProb* probs,
                                                                            const int* tn_start, int nprob,
                                                                            int tn_total, int tiles_m, int per_xcd,
                                                                            int group_m, const ChunkArgs* chp) {
  contract_f16f8_body<1, false>(probs, tn_start, nprob, tn_total, tiles_m, per_xcd, group_m, chp);
}
__global__ __launch_bounds__(LpTile<2>::NTHR, 1) void contract_f16f6_wide(const ContractLpProb* probs,
                                                                          const int* tn_start, int nprob, int tn_total,
                                                                          int tiles_m, int per_xcd, int group_m,
                                                                          const ChunkArgs* chp) {
  contract_f16f8_body<2, true>(probs, tn_start, nprob, tn_total, tiles_m, per_xcd, group_m, chp);
}
__global__ __launch_bounds__(LpTile<1>::NTHR, 1) void contract_f16f6_narrow(const ContractLpProb* probs,
                                                                            const int* tn_start, int nprob,
                                                                            int tn_total, int tiles_m, int per_xcd,
                                                                            int group_m, const ChunkArgs* chp) {
  contract_f16f8_body<1, true>(probs, tn_start, nprob, tn_total, tiles_m, per_xcd, group_m, chp);
}

template <typename T, int NPROD>
hipError_t launch_pack_t(const PackProb* probs, const int* blk_start, int nprob, int blk_total, hipStream_t s) {
  if (nprob <= 0 || blk_total <= 0) return hipSuccess;
  hipLaunchKernelGGL((pack_kernel<T, NPROD>), dim3(blk_total), dim3(256), 0, s, probs, blk_start, nprob);
  return hipGetLastError();
}

// Grid of a contraction launch: one workgroup per (row tile, column tile),
// dealt to the XCDs in contiguous runs (tiling.h).  The kernel is named in
// the launch itself so that its device code is instantiated.
#define MPS_CONTRACT_LAUNCH(KERNEL, NTHREADS)                                                                 \
  do {                                                                                                        \
    const int tiles_m = (grid_rows + BM - 1) / BM;                                                            \
    const long long ntiles = (long long)tiles_m * tn_total;                                                   \
    if (ntiles <= 0 || nprob <= 0) return hipSuccess;                                                         \
    const int per_xcd = (int)((ntiles + 7) / 8);                                                              \
    hipLaunchKernelGGL(KERNEL, dim3(per_xcd * 8), dim3(NTHREADS), 0, s, probs, tn_start, nprob, tn_total, tiles_m, \
                       per_xcd, group_m, ch);                                                                 \
    return hipGetLastError();                                                                                 \
  } while (0)

}  // namespace

hipError_t launch_colscale(const PackProb* probs, const int* cm_start, int nprob, int cm_total, hipStream_t s) {
  if (nprob <= 0 || cm_total <= 0) return hipSuccess;
  hipLaunchKernelGGL(colmax_kernel, dim3(cm_total), dim3(256), 0, s, probs, cm_start, nprob);
  return hipGetLastError();
}

hipError_t launch_pack_lp(int form, const PackProb* probs, const int* blk_start, int nprob, int blk_total,
                          hipStream_t s) {
  if (form == kFp16F6) {
    if (nprob <= 0 || blk_total <= 0) return hipSuccess;
    hipLaunchKernelGGL(pack_f16f8_kernel<true>, dim3(blk_total), dim3(256), 0, s, probs, blk_start, nprob);
    return hipGetLastError();
  }
  if (form == kFp16F8) {
    if (nprob <= 0 || blk_total <= 0) return hipSuccess;
    hipLaunchKernelGGL(pack_f16f8_kernel<false>, dim3(blk_total), dim3(256), 0, s, probs, blk_start, nprob);
    return hipGetLastError();
  }
  if (form == kBf16x3) return launch_pack_t<bf16_t, 3>(probs, blk_start, nprob, blk_total, s);
  if (form == kFp16x3) return launch_pack_t<f16_t, 3>(probs, blk_start, nprob, blk_total, s);
  return launch_pack_t<f16_t, 1>(probs, blk_start, nprob, blk_total, s);  // kFp16, kFp16x2: high parts only
}

hipError_t launch_contract_lp(int form, int tile, const ContractLpProb* probs, const int* tn_start, int nprob,
                              int tn_total, const ChunkArgs* ch, int grid_rows, int group_m, hipStream_t s) {
#define MPS_CONTRACT_FORM(NAME)                                                      \
  do {                                                                               \
    if (tile == kTileNarrow) MPS_CONTRACT_LAUNCH(NAME##_narrow, LpTile<1>::NTHR);    \
    MPS_CONTRACT_LAUNCH(NAME##_wide, LpTile<2>::NTHR);                               \
  } while (0)
  if (form == kFp16F8) MPS_CONTRACT_FORM(contract_f16f8);
  if (form == kFp16F6) MPS_CONTRACT_FORM(contract_f16f6);
  if (form == kBf16x3) MPS_CONTRACT_FORM(contract_bf16x3);
  if (form == kFp16x3) MPS_CONTRACT_FORM(contract_fp16x3);
  if (form == kFp16x2) MPS_CONTRACT_FORM(contract_fp16x2);
  MPS_CONTRACT_FORM(contract_fp16);
#undef MPS_CONTRACT_FORM
}

}  // namespace mps
