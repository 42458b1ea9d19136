// Persistent sweep for chains with medium bonds in FP32: one workgroup of 8
// waves takes 32 samples of one chain through every site of the chain in a
// single launch, for every such chain of the call at once (sweep_mid.hip does
// the same in the split forms and describes the steps).
//
// A wave contracts one unit of 32 complex columns (half a 64-column group of a
// branch; a site has at most 8) with the FP32 contraction kernel's
// instruction, order and two-level accumulation: W has its bits.  The site
// tensor is read as it lies in memory, one 4-byte word per lane, K step and
// column block, two units of 8 K steps ahead; left vectors sit in LDS as a
// real and an imaginary plane, and the chosen branch goes back into them from
// the registers that hold W.
//
// What bounds it: one workgroup per CU, whose matrix instructions (chi = 64,
// d = 4: 16000 cycles a site) and decision follow each other; with enough
// samples for the per-site tiles to fill the chip those are as fast
// (kMidRowsF32).  14 sites, 4096 samples, whole calls against per-site
// launches: chi = 64, d = 2 157 us against 422, d = 4 226 against 451;
// chi = 128, d = 2 271 against 504.  With up to four units per wave one after
// the other (W of chi = 256, d = 4 in registers) it lost from 16 units on
// (512 samples, chi = 100 and 128, d = 4: 546 us against 521, 692 against
// 547) and took 212 us where this takes 158 (chi = 64, d = 2); held to 128
// registers for two workgroups per CU it spills 692 bytes per lane (294 us).

#include "lp_ops.h"
#include "philox.h"
#include "sweep.h"
#include "tiling.h"

#include <math.h>

namespace mps {
namespace {

constexpr int R = kMidRows;
constexpr int NW = 8;
constexpr int NTHR = 64 * NW;
constexpr int LPR = NTHR / R;             // lanes per row in the decision; sites per block
constexpr int LP = R + 1;                 // pitch of the left-vector planes
constexpr int KU = 8;                     // K steps (complex l) per load unit
static_assert(R == 32 && LPR == 16 && NTHR == kMidThreads && kMidUnits == NW && kBK == 2 * KU,
              "lane roles and accumulation blocks below");

__device__ inline void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), vmcnt and expcnt at their maxima
  asm volatile("s_barrier" ::: "memory");
}

__global__ __launch_bounds__(NTHR, 2) void sweep_mid_f32(const MidChain* chains, const int* item_start, int nchain,
                                                         int plane, const ChunkArgs* chp, uint64_t seed, int* nflag) {
  __shared__ float qp[R][kMidUnits];
  __shared__ __attribute__((aligned(16))) double qd[R][LPR];
  __shared__ double us[LPR][R];
  __shared__ double ratio[LPR][R];
  __shared__ int oc[LPR][R];
  __shared__ __attribute__((aligned(16))) float2 pick[R];  // chosen branch (bits), 1 / sqrt(q_s)
  extern __shared__ __attribute__((aligned(16))) float Ls[];  // [part][l][row], then a dump slot per lane

  const ChunkArgs ch = *chp;
  const int p = find_problem(item_start, nchain, blockIdx.x);
  const MidChain c = chains[p];
  const int r0 = (blockIdx.x - item_start[p]) * R;
  if (r0 >= ch.rows) return;  // the whole workgroup: past the chunk
  typedef const __attribute__((address_space(4))) MidSite csite;
  csite* const sites = (csite*)(uintptr_t)c.sites;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5;
  const int j = lane & 31;
  const unsigned sgn = (half && !(j & 1)) ? 0x80000000u : 0u;
  const int drow = tid / LPR, db = tid % LPR;  // decision roles; site-block roles: row drow, site db
  const int grow = r0 + drow;
  const bool valid = grow < ch.rows;
  const int64_t crow = ch.c0 + grow;
  bool alive = true;
  double lp = 0.0;  // of row tid, threads 0..31

  // chi_0 = 1: every left vector is [1]; the planes start finite everywhere
  for (int e = tid; e < 2 * plane + 64; e += NTHR) Ls[e] = e < R ? 1.f : 0.f;

  // Unit u of a site: columns c0 .. c0 + 31 of branch br.
  struct Src {
    __amdgpu_buffer_rsrc_t rs;
    unsigned off[2];  // of this lane's word in row 0, per column block
    unsigned step;    // bytes per row
    int nk;           // load units
  };
  auto source = [&](int k, int u) {
    const int K = sites[k].K, d = sites[k].d, chr = sites[k].chi_r, T2 = sites[k].CP >> 5;
    const int br = u / T2, c0 = (u - br * T2) * 32;
    Src s;
    s.rs = __builtin_amdgcn_make_buffer_rsrc((void*)sites[k].Bh, (short)0, K * d * chr * 8, 0x00020000);
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      const int col = c0 + cb * 16 + (j >> 1);
      s.off[cb] = col < chr ? (unsigned)((br * chr + col) * 8 + ((j & 1) ^ half) * 4) : 0x80000000u;
    }
    s.step = (unsigned)(d * chr * 8);
    s.nk = (K + KU - 1) / KU;
    return s;
  };
  typedef float Unit[KU][2];
  auto load = [&](const Src& s, int n, Unit& o) {
#pragma unroll
    for (int l = 0; l < KU; ++l)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
        o[l][cb] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(s.rs, s.off[cb] + (unsigned)(n * KU + l) * s.step, 0, 0));
  };
  // units of a site that hold any column (the second half of a group may not)
  auto units = [&](int k) { return sites[k].d * (sites[k].CP >> 5); };

  Unit ring[2];
  bool primed = false;  // the ring holds the first units of this wave's next columns
  for (int kb = 0; kb < c.M; kb += LPR) {
    const int ns = min(LPR, c.M - kb);
    if (db < ns) us[db][drow] = draw_uniform((uint64_t)(ch.n_offset + crow), kb + db, seed, c.mps_id);
    lds_barrier();
    for (int ks = 0; ks < ns; ++ks) {
      const int k = kb + ks;
      const int d = sites[k].d, chr = sites[k].chi_r;
      const int T = sites[k].CP >> 6, U = units(k);
      const bool more = k + 1 < c.M;
      const int kn = more ? k + 1 : k;
      const int Un = units(kn);

      floatx16 tot[2];
      {
        if (wave < U) {
          const Src cur = source(k, wave);
          const bool then = more && wave < Un;
          const Src nxt = then ? source(kn, wave) : cur;
          const int nn = then ? nxt.nk : 0;
          if (!primed) {
            load(cur, 0, ring[0]);
            if (cur.nk > 1) load(cur, 1, ring[1]);
          }
#pragma unroll
          for (int cb = 0; cb < 2; ++cb) tot[cb] = floatx16{};
          // accumulation blocks of 16 l: two load units
          for (int n = 0; n < cur.nk; n += 2) {
            floatx16 blk[2] = {floatx16{}, floatx16{}};
            const bool last = n + 2 >= cur.nk;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              if (n + h < cur.nk) {
                const float* const av = Ls + half * plane + (n + h) * KU * LP + j;
#pragma unroll
                for (int l = 0; l < KU; ++l) {
                  const float a = av[l * LP];
#pragma unroll
                  for (int cb = 0; cb < 2; ++cb)
                    blk[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                        a, __uint_as_float(__float_as_uint(ring[h][l][cb]) ^ sgn), blk[cb], 0, 0, 0);
                }
              }
              if (n + h + 2 < cur.nk) load(cur, n + h + 2, ring[h]);
              else if (last && h < nn) load(nxt, h, ring[h]);
            }
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) tot[cb] += blk[cb];
          }
          primed = then;
          // partial weights of the unit's 64 real columns, as f32_epilogue adds
          // them: lane j < 16 of a half keeps that of row v = j
          float part = 0.f;
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            float s = __builtin_fmaf(tot[0][v], tot[0][v], tot[1][v] * tot[1][v]);
            const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(s), false, false);
            s = __uint_as_float(w[0]) + __uint_as_float(w[1]);
            s = add_ror<8>(s);
            s = add_ror<4>(s);
            s = add_ror<2>(s);
            s = add_ror<1>(s);
            part = j == v ? s : part;
          }
          if (j < 16) qp[(j >> 2) * 8 + half * 4 + (j & 3)][wave] = part;
        } else {
          primed = false;
        }
      }
      lds_barrier();

      // the decision of row drow: lane db takes branch db
      {
        double q = 0.0;
        if (db < d)
          for (int t = 0; t < T; ++t) q += (double)(qp[drow][2 * (db * T + t)] + qp[drow][2 * (db * T + t) + 1]);
        qd[drow][db] = q;
        __builtin_amdgcn_wave_barrier();  // a row's lanes are in one wave: its LDS operations are in order
        double S = 0.0, Pb = 0.0;
#pragma unroll
        for (int e = 0; e < LPR; ++e) {
          if (e < d) {
            S += qd[drow][e];  // P_e, left to right
            Pb = e == db ? S : Pb;
          }
        }
        const double u = us[ks][drow];
        const uint64_t above = __ballot(db < d && u > Pb / S);
        int s = min(__popcll((above >> (lane & ~(LPR - 1))) & ((1ull << LPR) - 1)), d - 1);
        const double qs = qd[drow][s];
        const bool ok = alive && isfinite(S) && S > 0.0 && qs > 0.0;
        if (!ok) s = 0;
        if (db == 0) {
          // (a flagged row's vector does not matter any more)
          pick[drow] = make_float2(__int_as_float(s), ok ? (float)(1.0 / sqrt(qs)) : 0.f);
          ratio[ks][drow] = qs / S;
          oc[ks][drow] = ok ? s : -1;
          if (valid && alive && !ok) atomicAdd(nflag, 1);
          if (valid && crow < c.emit_n && c.emit_u) c.emit_u[(size_t)crow * c.M + k] = u;
        }
        if (valid && crow < c.emit_n && c.emit_probs && db < d && db < c.emit_dmax)
          c.emit_probs[((size_t)crow * c.M + k) * c.emit_dmax + db] = ok ? q / S : NAN;
        alive = ok;
      }
      lds_barrier();

      if (more) {
        // The chosen branch of every row, scaled, into the planes; values of
        // other branches and past chi_r to a dump slot of the lane.  (Values
        // past chi_r in the planes stay finite and meet zeros.)
        {
          if (wave < U) {
            const int br = wave / (2 * T), c0 = (wave - br * 2 * T) * 32;
            const int dump = 2 * plane + lane;
#pragma unroll
            for (int v0 = 0; v0 < 16; v0 += 4) {
              const int row0 = (v0 >> 2) * 8 + half * 4;
              float4 pk[2];
              pk[0] = *reinterpret_cast<const float4*>(&pick[row0]);
              pk[1] = *reinterpret_cast<const float4*>(&pick[row0 + 2]);
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const bool mine = __float_as_int(e & 1 ? pk[e >> 1].z : pk[e >> 1].x) == br;
                const float sc = e & 1 ? pk[e >> 1].w : pk[e >> 1].y;
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                  const int col = c0 + cb * 16 + (j >> 1);
                  Ls[mine && col < chr ? (j & 1) * plane + col * LP + row0 + e : dump] =
                      __fmul_rn(tot[cb][v0 + e], sc);
                }
              }
            }
          }
        }
        lds_barrier();
      }
    }
    // the block's logarithms and outcomes: thread (row, site)
    lds_barrier();
    if (db < ns) {
      ratio[db][drow] = log(ratio[db][drow]);
      if (valid) c.outcomes[(size_t)crow * c.M + kb + db] = oc[db][drow];
    }
    lds_barrier();
    if (tid < R)
      for (int e = 0; e < ns; ++e) lp = oc[e][tid] < 0 ? -INFINITY : lp + ratio[e][tid];
    lds_barrier();
  }
  if (c.logp && tid < R && r0 + tid < ch.rows) c.logp[ch.c0 + r0 + tid] = lp;
}

}  // namespace

hipError_t launch_sweep_mid_f32(const MidChain* chains, const int* item_start, int nchain, int items, int chimax,
                                const ChunkArgs* ch, uint64_t seed, int* nflag, hipStream_t s) {
  if (nchain <= 0 || items <= 0) return hipSuccess;
  // whole load units of l; the planes half the banks apart
  const int plane = (((chimax + kBK - 1) / kBK * kBK * LP + 63) & ~63) + 32;
  hipLaunchKernelGGL(sweep_mid_f32, dim3(items), dim3(NTHR), (size_t)(2 * plane + 64) * sizeof(float), s, chains,
                     item_start, nchain, plane, ch, seed, nflag);
  return hipGetLastError();
}

}  // namespace mps
