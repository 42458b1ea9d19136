// Persistent sweep for chains with small bonds (FP32): one workgroup takes 16
// samples of one chain through every site of the chain in a single launch,
// for every chain of the call at once (Section 3.1's data parallelism over
// samples, over chains, and over the sites of Section 2.2's sequential
// workflow without returning to memory between sites).
//
// Eligible chains have chi_k <= 32 and d_k <= 4 at every site: W of 16 samples
// then fits the LDS and registers of three workgroups per CU.  Per site the
// workgroup
//   1. contracts the site tensor with the 16 left vectors on
//      v_mfma_f32_16x16x4f32: W is 16 x (d * chi_r) complex, at most 8 groups
//      of 16 complex columns, two per wave.  A wave loads the columns that it
//      alone needs straight into registers, each value once (lane (i, g): row
//      4 q + g, one or two neighbouring columns), before the previous site's
//      measurement, which hides the latency; swaps of 16- and 32-lane rows
//      then give the lanes the rows of each MFMA step, and selects the real
//      embedding.  Every output is one chain of fused multiply-adds in order
//      of l, restarted every 16 l and added up (the two-level accumulation of
//      the FP32 contraction kernel: W is bit-identical to it);
//   2. writes W to LDS, then measures: 16 lanes per sample, 8 for two branches
//      each, form the branch weights (FP32 per lane, FP64 across 8 lanes in
//      a fixed butterfly on DPP), every lane of a quad takes one branch's
//      divisions and square root, and the renormalised chosen branch goes
//      back into the LDS left vectors.  The uniforms of 16 sites are drawn at
//      once, and their logarithms and outcomes leave at once.
// Left vectors and W never leave LDS; per site only the site tensor is read.
//
// What bounds it: the chain of one site's steps, ~8600 cycles at chi = 32, d = 4
// (3500 the matrix instructions, 2050 at their peak rate; 1700 the loads of
// the next site, 32 KiB per CU from L2; 2100 the measurement) when the samples
// are few, the FP32 matrix cores when the chip is full.  M = 32, d = 4,
// chi = 32, N = 4096: 163 us a call (the launch 116), against 497 us for
// 32-sample workgroups that staged the site tensor through LDS and kept every
// step of a sample's decision in line.  Spreading the loads over the measurement
// and placing the swaps between the matrix instructions by hand changed nothing.

#include "philox.h"
#include "sweep.h"
#include "tiling.h"

#include <math.h>

namespace mps {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int R = kSmallRows;   // samples per workgroup
constexpr int CHI = kSmallChi;  // largest bond
constexpr int DM = kSmallD;     // largest physical dimension
constexpr int NC = CHI * DM;    // largest d * chi_r (complex columns of W)
constexpr int NTHR = kSmallThreads;
constexpr int NG = NC / 16 / 4;  // column groups per wave
constexpr int NQ = CHI / 4;      // register quads of 4 complex l
constexpr int NSTEP = CHI / 2;   // K steps of 2 complex l
constexpr int SB = 16;           // sites whose uniforms, logarithms and outcomes go together
constexpr int WP = NC + 4;       // pitch of W: the 4 row groups of a store land in other banks
static_assert(R == 16 && DM == 4 && NTHR == R * SB, "lane roles below");

// Left vectors, K value k = 2 l + part of row r, as the MFMA reads them: step
// k / 4 holds 64 floats, one per lane, the rows rotated by the step so that
// the measurement's stores (16 l of one row) spread over the banks.
__device__ inline int l_off(int step, int k4, int row) { return step * 64 + k4 * 16 + ((row + step) & 15); }

template <int CTRL>
__device__ inline float dpp(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ inline double dpp(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (uint32_t)b, CTRL, 0xF, 0xF, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppRor8 = 0x128;

// LDS writes of this wave done, then every wave's; global loads and stores
// stay in flight.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), vmcnt and expcnt at their maxima
  asm volatile("s_barrier" ::: "memory");
}

__global__ __launch_bounds__(NTHR, 3) void sweep_small_kernel(const SmallChain* chains, const int* item_start,
                                                              int nchain, const ChunkArgs* chp, uint64_t seed,
                                                              int* nflag) {
  __shared__ float Ls[NSTEP * 64];
  __shared__ __attribute__((aligned(16))) float2 Ws[R * WP];  // W[row][c], c = i * chi_r + r
  __shared__ double us[SB][R];     // uniforms of the site block
  __shared__ double ratio[SB][R];  // q_s / S, then its logarithm
  __shared__ int oc[SB][R];        // outcomes

  const ChunkArgs ch = *chp;
  const int p = find_problem(item_start, nchain, blockIdx.x);
  const SmallChain c = chains[p];
  const int r0 = (blockIdx.x - item_start[p]) * R;
  if (r0 >= ch.rows) return;  // the whole workgroup: past the chunk
  // uniform tables, read through the scalar cache
  typedef const __attribute__((address_space(4))) int cint;
  typedef const __attribute__((address_space(4))) uint64_t cptr;
  cint* const chi = (cint*)(uintptr_t)c.chi;
  cint* const dims = (cint*)(uintptr_t)c.d;
  cptr* const sites = (cptr*)(uintptr_t)c.A;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15;  // MFMA row (left vectors) and column (site tensor)
  const int g = lane >> 4;  // its K value: part g & 1 of complex g >> 1 of the step
  const bool imag = g & 1;

  // chi_0 = 1: every left vector is [1]
  for (int e = tid; e < NSTEP * 64; e += NTHR) Ls[e] = e < R ? 1.f : 0.f;

  // measurement roles: 16 lanes per sample; lanes 0..7 branches 0 and 1, lanes
  // 8..15 branches 2 and 3; within 8 lanes, residue sl of r mod 8, placed so
  // that lane pairs (half mirror, xor 2, xor 1) are residues xor 4, 2, 1
  const int mrow = wave * 4 + g;
  const int ih = i >> 3, pos = i & 7;
  const int sl = pos < 4 ? pos : 11 - pos;
  const int grow = r0 + mrow;         // row within the chunk
  const bool valid = grow < ch.rows;
  const int64_t crow = ch.c0 + grow;  // row within the call
  const int hrow = tid >> 4, hs = tid & 15;  // site-block roles: row, site
  bool alive = true;
  double lp = 0.0;  // of row tid, threads 0..15

  // This wave's columns of a site tensor (K rows of ncols complex), zeros for
  // rows past K (the descriptor's size).  More than 64 columns: lanes take the
  // pair 32 wave + 2 i, else the column 16 wave + i.  Columns past ncols hold
  // other rows' values; their W is not read.  bq[q][0..1] and [2..3]: row
  // 4 q + g of the first and second column.
  float bq[NQ][4];
  auto load_site = [&](uint64_t A, int K, int ncols) {
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)A, (short)0, K * ncols * 8, 0x00020000);
    const bool two = ncols > 64;
    const unsigned off = (unsigned)(g * ncols + (two ? 32 * wave + 2 * i : 16 * wave + i)) * 8;
    if ((two ? 32 : 16) * wave >= ncols) return;
#pragma unroll
    for (int q = 0; q < NQ; q += 2) {
      if (4 * q < K) {
#pragma unroll
        for (int e = q; e < q + 2; ++e) {
          const unsigned o = off + (unsigned)(e * 4 * ncols * 8);
          if (two && (ncols & 1) == 0) {  // whole pairs: none is cut by the tensor's end
            const auto w = __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0);
#pragma unroll
            for (int x = 0; x < 4; ++x) bq[e][x] = __uint_as_float(w[x]);
          } else {
            const auto w = __builtin_amdgcn_raw_buffer_load_b64(rs, o, 0, 0);
            bq[e][0] = __uint_as_float(w[0]);
            bq[e][1] = __uint_as_float(w[1]);
            if (two) {
              const auto z = __builtin_amdgcn_raw_buffer_load_b64(rs, o + 8, 0, 0);
              bq[e][2] = __uint_as_float(z[0]);
              bq[e][3] = __uint_as_float(z[1]);
            }
          }
        }
      }
    }
  };
  // values of rows 4 q + (0, 1, 2, 3) in the four 16-lane rows -> two steps'
  // operands: rows (0, 0, 1, 1) and (2, 2, 3, 3)
  auto spread = [](float x, float& a, float& b) {
    const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const auto w = __builtin_amdgcn_permlane32_swap(h[0], h[1], false, false);
    a = __uint_as_float(w[0]);
    b = __uint_as_float(w[1]);
  };

  int K = chi[0], dk = dims[0], cr = chi[1];
  load_site(sites[0], K, dk * cr);
  for (int kb = 0; kb < c.M; kb += SB) {
    const int ns = min(SB, c.M - kb);
    if (hs < ns) us[hs][hrow] = draw_uniform((uint64_t)(ch.n_offset + ch.c0 + r0 + hrow), kb + hs, seed, c.mps_id);
    lds_barrier();
    for (int ks = 0; ks < ns; ++ks) {
      const int k = kb + ks;
      const int ncols = dk * cr;
      const bool more = k + 1 < c.M;
      const int kn = more ? k + 1 : k;
      const int dn = dims[kn], cn = chi[kn + 1];
      const uint64_t An = sites[kn];

      const bool two = ncols > 64;
      const bool busy = (two ? 32 : 16) * wave < ncols;
      if (busy) {
        float av[NSTEP];
#pragma unroll
        for (int st = 0; st < NSTEP; ++st) av[st] = Ls[l_off(st, g, i)];
        floatx4 tot[NG][2], blk[NG][2];
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) tot[gi][0] = tot[gi][1] = floatx4{};
#pragma unroll
        for (int l0 = 0; l0 < CHI; l0 += 16) {
          if (l0 < K) {
#pragma unroll
            for (int gi = 0; gi < NG; ++gi) blk[gi][0] = blk[gi][1] = floatx4{};
#pragma unroll
            for (int qb = l0 / 4; qb < l0 / 4 + 4; qb += 2) {
              if (4 * qb < K) {
#pragma unroll
                for (int q = qb; q < qb + 2; ++q) {
#pragma unroll
                  for (int gi = 0; gi < NG; ++gi) {
                    if (gi == 0 || two) {
                      float re[2], im[2];
                      spread(bq[q][2 * gi], re[0], re[1]);
                      spread(bq[q][2 * gi + 1], im[0], im[1]);
#pragma unroll
                      for (int h = 0; h < 2; ++h) {
                        const float a = av[2 * q + h];
                        blk[gi][0] =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(a, imag ? -im[h] : re[h], blk[gi][0], 0, 0, 0);
                        blk[gi][1] =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(a, imag ? re[h] : im[h], blk[gi][1], 0, 0, 0);
                      }
                    }
                  }
                }
              }
            }
#pragma unroll
            for (int gi = 0; gi < NG; ++gi) {
              tot[gi][0] += blk[gi][0];
              tot[gi][1] += blk[gi][1];
            }
          }
        }
        // W to LDS: lane (i, g) holds its columns' rows 4 g + v
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float2* const d = Ws + (4 * g + v) * WP + (two ? 32 * wave + 2 * i : 16 * wave + i);
          if (two)
            *reinterpret_cast<float4*>(d) = make_float4(tot[0][0][v], tot[0][1][v], tot[1][0][v], tot[1][1][v]);
          else
            *d = make_float2(tot[0][0][v], tot[0][1][v]);
        }
      }
      if (more) load_site(An, cr, dn * cn);
      lds_barrier();

      // measurement of sample mrow by its 16 lanes; columns past chi_r and
      // branches past d add zeros
      const float2* const Wr = Ws + mrow * WP;
      float2 w[2][CHI / 8];
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int t = 0; t < CHI / 8; ++t) {
          const int r = sl + 8 * t, br = 2 * ih + b;
          const bool in = r < cr && br < dk;
          const float2 z = Wr[in ? br * cr + r : 0];
          w[b][t] = in ? z : make_float2(0.f, 0.f);
        }
      float qa[2];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        qa[b] = 0.f;
#pragma unroll
        for (int t = 0; t < CHI / 8; ++t) qa[b] += __builtin_fmaf(w[b][t].x, w[b][t].x, w[b][t].y * w[b][t].y);
      }
      double v0 = (double)qa[0], v1 = (double)qa[1];
      v0 += dpp<kDppHalfMirror>(v0);
      v1 += dpp<kDppHalfMirror>(v1);
      v0 += dpp<kDppXor2>(v0);
      v1 += dpp<kDppXor2>(v1);
      v0 += dpp<kDppXor1>(v0);
      v1 += dpp<kDppXor1>(v1);
      const double o0 = dpp<kDppRor8>(v0), o1 = dpp<kDppRor8>(v1);
      const double q0 = ih ? o0 : v0, q1 = ih ? o1 : v1, q2 = ih ? v0 : o0, q3 = ih ? v1 : o1;
      const double P1 = q0 + q1, P2 = P1 + q2, S = P2 + q3;  // q_i = 0 past d
      // lane b of a quad takes branch b
      const int b = i & 3;
      const double Pb = b == 0 ? q0 : b == 1 ? P1 : b == 2 ? P2 : S;
      const double qb = b == 0 ? q0 : b == 1 ? q1 : b == 2 ? q2 : q3;
      const double u = us[ks][mrow];
      const float sc = (float)(1.0 / sqrt(qb));
      const double rat = qb / S;
      const uint64_t above = __ballot(b < dk && u > Pb / S);
      int s = min(__popc((unsigned)(above >> (16 * g)) & 0xFu), dk - 1);
      const double qs = s == 0 ? q0 : s == 1 ? q1 : s == 2 ? q2 : q3;
      const bool ok = alive && isfinite(S) && S > 0.0 && qs > 0.0;
      if (!ok) s = 0;
      const float s0 = dpp<0x00>(sc), s1 = dpp<0x55>(sc), s2 = dpp<0xAA>(sc), s3 = dpp<0xFF>(sc);
      const float scale = !ok ? 0.f : s == 0 ? s0 : s == 1 ? s1 : s == 2 ? s2 : s3;
      // the renormalised chosen branch becomes the sample's left vector;
      // values past chi_r stay finite ones of earlier sites, which the next
      // site multiplies by zeros
#pragma unroll
      for (int t = 0; t < CHI / 16; ++t) {
        const int r = i + 16 * t;
        if (r < cr) {
          const float2 z = Wr[s * cr + r];
          Ls[l_off(r >> 1, 2 * (r & 1), mrow)] = z.x * scale;
          Ls[l_off(r >> 1, 2 * (r & 1) + 1, mrow)] = z.y * scale;
        }
      }
      if (i == s) ratio[ks][mrow] = rat;
      if (i == 0) {
        oc[ks][mrow] = ok ? s : -1;
        if (valid) {
          if (alive && !ok) atomicAdd(nflag, 1);
          if (crow < c.emit_n) {
            if (c.emit_u) c.emit_u[(size_t)crow * c.M + k] = u;
            if (c.emit_probs) {
              double* ep = c.emit_probs + ((size_t)crow * c.M + k) * c.emit_dmax;
              const double q[DM] = {q0, q1, q2, q3};
#pragma unroll
              for (int e = 0; e < DM; ++e)
                if (e < dk && e < c.emit_dmax) ep[e] = ok ? q[e] / S : NAN;
            }
          }
        }
      }
      alive = ok;
      K = cr;
      dk = dn;
      cr = cn;
      lds_barrier();
    }
    // the block's logarithms and outcomes: thread (row, site)
    if (hs < ns) {
      ratio[hs][hrow] = log(ratio[hs][hrow]);
      if (r0 + hrow < ch.rows)
        c.outcomes[(size_t)(ch.c0 + r0 + hrow) * c.M + kb + hs] = oc[hs][hrow];
    }
    lds_barrier();
    if (tid < R)
      for (int e = 0; e < ns; ++e) lp = oc[e][tid] < 0 ? -INFINITY : lp + ratio[e][tid];
    lds_barrier();
  }
  if (c.logp && tid < R && r0 + tid < ch.rows) c.logp[ch.c0 + r0 + tid] = lp;
}

}  // namespace

hipError_t launch_sweep_small(const SmallChain* chains, const int* item_start, int nchain, int items,
                              const ChunkArgs* ch, uint64_t seed, int* nflag, hipStream_t s) {
  if (nchain <= 0 || items <= 0) return hipSuccess;
  hipLaunchKernelGGL(sweep_small_kernel, dim3(items), dim3(NTHR), 0, s, chains, item_start, nchain, ch, seed,
                     nflag);
  return hipGetLastError();
}

}  // namespace mps
