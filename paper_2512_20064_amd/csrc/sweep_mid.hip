// Persistent sweep for chains with medium bonds in the split forms (bf16x3,
// fp16x3, fp16f8, fp16f6):
// one workgroup takes 32 samples of one chain through every site of the chain
// in a single launch, for every such chain of the call at once.  The site
// tensors have been packed once for the call (contract_lp.hip, 64-column
// tiles).
//
// A chain is eligible when every site has d * ceil(chi_r / 64) <= 16 groups of
// 64 complex columns: W of the workgroup's 32 rows then stays in registers (a
// wave holds one group, or two).  Per site
//   1. a wave contracts its groups: the left vectors' operand planes come from
//      LDS, its 64 packed rows straight from memory into registers (no other
//      wave of the workgroup needs them), four slices (two slice pairs) ahead,
//      across the end of the site: the next site's first slices arrive during
//      the measurement.  The MFMAs and their order per output are those of
//      the tile kernels, so W has the same bits;
//   2. partial weights (the same sums) go to LDS; the lanes of a row form the
//      branch weights, draw and normalise as the measurement kernel does, one
//      branch per lane; the waves that hold a row's chosen branch write it,
//      scaled, to LDS; all waves split it into the next site's operand planes.
// W and the left vectors never leave the CU; the uniforms of 8 or 16 sites are
// drawn at once, and their logarithms and outcomes leave at once.
//
// What bounds it: at few samples the chain of a site's steps (chi = 64, d = 4,
// fp16f6: 16000 cycles, of them 5600 the contraction, whose matrix
// instructions take 1500: its operands come at 64 B per clock and CU from L2);
// when the chip is full the matrix cores and that operand stream, 8 bytes per
// complex entry of the site tensor and 32 samples.  The per-site launches
// need four launches of 5 to 25 us a site and take W through memory.  Whole
// calls, persistent against per-site launches with the same packing:
//   chi = 64, d = 4, 24 sites, 512 samples, fp16f6     210 us against  900
//   chi = 100, d = 3, 40 sites, 2999 samples, bf16x3   428 us against 1515
//   chi = 128, d = 4, 14 sites, 65536 samples, fp16f6 1.48 ms against 1.86
//   chi = 256, d = 4, 14 sites, 65536 samples, fp16f6 3.40 ms against 3.91
// At every size measured (chi 64 .. 256, d 2 and 4, 512 .. 65536 samples,
// fp16f6 and bf16x3) it was the faster one, by 1.11 to 3.6 times, so it is
// taken wherever W fits the registers; above that the tile kernels' reuse of
// the operands over 256 rows is needed.  Operands 6 slices ahead instead of 4
// spill (227 us against 211).

#include "lp_ops.h"
#include "philox.h"
#include "sweep.h"
#include "tiling.h"

#include <math.h>

#include <type_traits>

namespace mps {
namespace {

constexpr int R = kMidRows;
constexpr int NGMAX = kMidGroups;
static_assert(R == 32 && NGMAX == 16, "one MFMA row block; lane roles below");

// LDS writes of this wave done, then every wave's; global loads and stores
// stay in flight.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), vmcnt and expcnt at their maxima
  asm volatile("s_barrier" ::: "memory");
}

// Operands of a wave's 64 columns for UK slices of 16 K (two column blocks).
template <int FORM>
struct MidOps {  // 16-bit forms: one slice
  static constexpr int UK = 1;
  typedef typename Vec8<typename std::conditional<FORM == kBf16x3, bf16_t, f16_t>::type>::type V8;
  V8 h[2], l[2];
};
struct MidOps8 {  // fp16f8, fp16f6: a slice pair
  static constexpr int UK = 2;
  f16x8 e[2], h[2];
  intx8 f[2];
};
template <>
struct MidOps<kFp16F8> : MidOps8 {};
template <>
struct MidOps<kFp16F6> : MidOps8 {};

template <int FORM, int NW, int GPW>
__device__ inline void sweep_mid_body(const MidChain* chains, const int* item_start, int nchain, int slices, int sp,
                                      const ChunkArgs* chp, uint64_t seed, int* nflag) {
  constexpr int NTHR = 64 * NW;
  static_assert(NTHR <= kMidThreads, "the host plans launches with the largest workgroup");
  constexpr int LPR = NTHR / R;  // lanes per row in the decision; sites per block
  constexpr bool F8F6 = FORM == kFp16F8 || FORM == kFp16F6;
  typedef MidOps<FORM> Ops;
  constexpr int UK = Ops::UK;
  // units in flight: 4 slices with one W group per wave (6 spill), else 2
  constexpr int DEPTH = (GPW == 1 ? 4 : 2) / UK;
  __shared__ float qp[R][NGMAX];
  __shared__ __attribute__((aligned(16))) double qd[R][LPR];
  __shared__ double us[LPR][R];
  __shared__ double ratio[LPR][R];
  __shared__ int oc[LPR][R];
  __shared__ __attribute__((aligned(16))) float2 pick[R];  // chosen branch (bits), 1 / sqrt(q_s)
  extern __shared__ __attribute__((aligned(16))) char dyn[];  // planes [slices][32 rows][32 B], then the branch rows
  char* const lh = dyn;
  char* const ll = dyn + slices * 1024;
  float2* const br_sh = reinterpret_cast<float2*>(dyn + 2 * slices * 1024);

  const ChunkArgs ch = *chp;
  const int p = find_problem(item_start, nchain, blockIdx.x);
  const MidChain c = chains[p];
  const int r0 = (blockIdx.x - item_start[p]) * R;
  if (r0 >= ch.rows) return;  // the whole workgroup: past the chunk
  // uniform tables, read through the scalar cache
  typedef const __attribute__((address_space(4))) MidSite csite;
  csite* const sites = (csite*)(uintptr_t)c.sites;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5;
  const int j = lane & 31;
  // decision roles: LPR lanes per row, lane b of them branch b; site-block
  // roles: row hrow, site hs
  const int drow = tid / LPR, db = tid % LPR;
  const int grow = r0 + drow;
  const bool valid = grow < ch.rows;
  const int64_t crow = ch.c0 + grow;
  const int hrow = tid / LPR, hs = tid % LPR;
  bool alive = true;
  double lp = 0.0;  // of row tid, threads 0..31

  const unsigned a16 = (unsigned)lds_off(j, half);  // a slice's chunk `half` of row j
  const unsigned a8_0 = (unsigned)lds_off(j, 0), a8_1 = (unsigned)lds_off(j, 1);

  // Group g of a site: 64 packed rows in one 256-row block.
  struct Src {
    __amdgpu_buffer_rsrc_t h, l;
    int nk;  // units of UK slices that hold any of the K values (the others add zeros)
  };
  const unsigned v16 = (unsigned)(wave_col(0, j) * 32 + half * 16);           // 16-bit plane: chunk `half`
  const unsigned v8 = (unsigned)(wave_col(0, j) * 32 + half * 8192);          // pair plane: slice `half` of a pair
  auto source = [&](int k, int g) {
    const size_t row = (size_t)g * 64;
    const int Kp = sites[k].Kp;
    const size_t off = (row >> 8) * ((size_t)(Kp >> 4) * 8192) + (row & 255) * 32;
    Src s;
    s.h = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)sites[k].Bh + off), (short)0, (int)0xFFFFFFFF, 0x00020000);
    s.l = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)sites[k].Bl + off), (short)0,
                                            (int)0xFFFFFFFF, 0x00020000);
    s.nk = (2 * sites[k].K + 16 * UK - 1) / (16 * UK);
    return s;
  };
  auto load = [&](const Src& s, int n, Ops& o) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if constexpr (F8F6) {
        const int so = n * 2 * 8192;
        o.e[b] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(s.h, v16 + b * 512, so, 0));
        o.h[b] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(s.h, v16 + b * 512, so + 8192, 0));
        const intx4 x = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(s.l, v8 + b * 512, so, 0));
        const intx4 y = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(s.l, v8 + b * 512 + 16, so, 0));
        o.f[b] = __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7);
      } else {
        typedef typename Ops::V8 V8;
        const int so = n * 8192;
        o.h[b] = __builtin_bit_cast(V8, __builtin_amdgcn_raw_buffer_load_b128(s.h, v16 + b * 512, so, 0));
        o.l[b] = __builtin_bit_cast(V8, __builtin_amdgcn_raw_buffer_load_b128(s.l, v16 + b * 512, so, 0));
      }
    }
  };
  // one unit: acc[2 b + p], p = 0 with the operand as read, p = 1 turned
  auto mma = [&](int n, const Ops& o, floatx16 (&acc)[4]) {
    if constexpr (F8F6) {
      const char* const q = lh + n * 2048;
      const char* const q8 = ll + (2 * n + half) * 1024;
      const f16x8 ae = *reinterpret_cast<const f16x8*>(q + a16);
      const f16x8 ah = *reinterpret_cast<const f16x8*>(q + 1024 + a16);
      const intx4 x = *reinterpret_cast<const intx4*>(q8 + a8_0), y = *reinterpret_cast<const intx4*>(q8 + a8_1);
      const intx8 af = __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
        acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ae, cb & 1 ? turn(o.e[cb >> 1]) : o.e[cb >> 1], acc[cb], 0, 0, 0);
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const intx8 b = cb & 1 ? (FORM == kFp16F6 ? turn_e2m3(o.f[cb >> 1]) : turn_e4m3(o.f[cb >> 1])) : o.f[cb >> 1];
        if constexpr (FORM == kFp16F6)
          acc[cb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(af, b, acc[cb], 2, 2, 0, af[6], 0, b[6]);
        else
          acc[cb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(af, b, acc[cb], 0, 0, 0, kScale8L, 0, kScale8B);
      }
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
        acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, cb & 1 ? turn(o.h[cb >> 1]) : o.h[cb >> 1], acc[cb], 0, 0, 0);
    } else {
      typedef typename Ops::V8 V8;
      typedef Vec8<typename std::conditional<FORM == kBf16x3, bf16_t, f16_t>::type> M;
      const V8 ah = *reinterpret_cast<const V8*>(lh + n * 1024 + a16);
      const V8 al = *reinterpret_cast<const V8*>(ll + n * 1024 + a16);
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const V8 bh = cb & 1 ? turn(o.h[cb >> 1]) : o.h[cb >> 1];
        const V8 bl = cb & 1 ? turn(o.l[cb >> 1]) : o.l[cb >> 1];
        acc[cb] = M::mfma(ah, bh, acc[cb]);
        acc[cb] = M::mfma(ah, bl, acc[cb]);
        acc[cb] = M::mfma(al, bh, acc[cb]);
      }
    }
  };
  // 8 complex of a row (a slice) into the operand planes
  auto store_slice = [&](int row, int sl, const float2 (&v)[8]) {
    uint32_t h[8], w[8];
    if constexpr (FORM == kFp16F6) {
      split8_e2m3(v, h, w);
    } else {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float2 v4[4] = {v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        uint32_t h4[4];
        if constexpr (FORM == kFp16F8) {
          uint32_t hc[2], lc[2];
          split4_e4m3(v4, h4, hc, lc);
          w[2 * q] = hc[0];
          w[2 * q + 1] = hc[1];
          w[4 + 2 * q] = lc[0];
          w[4 + 2 * q + 1] = lc[1];
        } else {
          uint32_t l4[4];
          split4<typename std::conditional<FORM == kBf16x3, bf16_t, f16_t>::type>(v4, h4, l4);
#pragma unroll
          for (int e = 0; e < 4; ++e) w[4 * q + e] = l4[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) h[4 * q + e] = h4[e];
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      *reinterpret_cast<uint4*>(lh + sl * 1024 + lds_off(row, q)) =
          make_uint4(h[4 * q], h[4 * q + 1], h[4 * q + 2], h[4 * q + 3]);
      *reinterpret_cast<uint4*>(ll + sl * 1024 + lds_off(row, q)) =
            make_uint4(w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]);
    }
  };

  // chi_0 = 1: every left vector is [1]
  for (int e = tid; e < R * (lp_pad_k(1) >> 4); e += NTHR) {
    float2 v[8] = {};
    if (e < R) v[0].x = 1.f;
    store_slice(e & (R - 1), e / R, v);
  }

  Ops ring[DEPTH];
  bool primed = false;  // the ring holds the first units of this wave's next group
  auto prime = [&](const Src& s) {
#pragma unroll
    for (int u = 0; u < DEPTH; ++u)
      if (u < s.nk) load(s, u, ring[u]);
  };
  for (int kb = 0; kb < c.M; kb += LPR) {
    const int ns = min(LPR, c.M - kb);
    if (hs < ns) us[hs][hrow] = draw_uniform((uint64_t)(ch.n_offset + ch.c0 + r0 + hrow), kb + hs, seed, c.mps_id);
    lds_barrier();
    for (int ks = 0; ks < ns; ++ks) {
      const int k = kb + ks;
      const int d = sites[k].d, chr = sites[k].chi_r, CP = sites[k].CP;
      const int T = CP >> 6, G = d * T;
      const bool more = k + 1 < c.M;
      const int kn = more ? k + 1 : k;
      const int Gn = sites[kn].d * (sites[kn].CP >> 6);

      floatx16 acc[GPW][4];
#pragma unroll
      for (int t = 0; t < GPW; ++t) {
        const int g = wave + NW * t;
        if (g < G) {
          const Src cur = source(k, g);
          const bool same = t + 1 < GPW && g + NW < G;   // another group of this site follows
          const bool then = same || (more && wave < Gn);  // a group follows
          const Src nxt = then ? (same ? source(k, g + NW) : source(kn, wave)) : cur;
          float cs[2] = {1.f, 1.f};
          if constexpr (F8F6) {
            cs[0] = sites[k].cs[g * 64 + wave_col(0, j)];
            cs[1] = sites[k].cs[g * 64 + wave_col(1, j)];
          }
          if (!primed) prime(cur);
#pragma unroll
          for (int cb = 0; cb < 4; ++cb) acc[t][cb] = floatx16{};
          // Unit n sits in slot n % DEPTH; a slot done with this group takes
          // the next group's unit of its number.
          int n = 0;
          for (; n + 2 * DEPTH <= cur.nk; n += DEPTH) {
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
              mma(n + u, ring[u], acc[t]);
              load(cur, n + u + DEPTH, ring[u]);
            }
          }
          const int nn = then ? nxt.nk : 0;
          for (; n < cur.nk; n += DEPTH) {
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
              if (n + u < cur.nk) mma(n + u, ring[u], acc[t]);
              if (n + u + DEPTH < cur.nk) load(cur, n + u + DEPTH, ring[u]);
              else if (n + DEPTH >= cur.nk && u < nn) load(nxt, u, ring[u]);
            }
          }
          primed = then;
          if constexpr (F8F6) {
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
              for (int v = 0; v < 16; ++v) acc[t][cb][v] *= cs[cb >> 1];
          }
          float part = 0.f;  // lane j < 16 of a half keeps the partial of row v = j
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const float s = part_sum(acc[t][0][v], acc[t][1][v], acc[t][2][v], acc[t][3][v]);
            part = j == v ? s : part;
          }
          if (j < 16) qp[(j >> 2) * 8 + half * 4 + (j & 3)][g] = part;
        } else if (t == 0) {
          primed = false;
        }
      }
      lds_barrier();

      // the decision of row drow: lane db takes branch db
      {
        double q = 0.0;
        if (db < d)
          for (int t = 0; t < T; ++t) q += (double)qp[drow][db * T + t];
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
        // The chosen branch of every row, scaled.  Every wave stores all its
        // values, those of other branches to a dump slot of the lane: no
        // divergent code.
#pragma unroll
        for (int t = 0; t < GPW; ++t) {
          const int g = wave + NW * t;
          if (g < G) {
            const int br = g / T, c0 = (g - br * T) * 64;
            const int off[2] = {c0 + wave_col(0, j) < chr ? c0 + wave_col(0, j) : -1,
                                c0 + wave_col(1, j) < chr ? c0 + wave_col(1, j) : -1};
            const int dump = R * sp + lane;
#pragma unroll
            for (int v0 = 0; v0 < 16; v0 += 4) {
              const int row0 = (v0 >> 2) * 8 + half * 4;
              float4 pk[2];
              pk[0] = *reinterpret_cast<const float4*>(&pick[row0]);
              pk[1] = *reinterpret_cast<const float4*>(&pick[row0 + 2]);
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int v = v0 + e;
                const bool mine = __float_as_int(e & 1 ? pk[e >> 1].z : pk[e >> 1].x) == br;
                const float sc = e & 1 ? pk[e >> 1].w : pk[e >> 1].y;
#pragma unroll
                for (int b = 0; b < 2; ++b)
                  br_sh[mine && off[b] >= 0 ? (row0 + e) * sp + off[b] : dump] =
                      make_float2(__fmul_rn(acc[t][2 * b][v], sc), __fmul_rn(acc[t][2 * b + 1][v], sc));
              }
            }
          }
        }
        lds_barrier();
        // its operand planes, a slice of a row at a time
        const int nsl = lp_pad_k(chr) >> 4;
        for (int e = tid; e < R * nsl; e += NTHR) {
          const int row = e & (R - 1), sl = e / R;
          const float2* const src = br_sh + row * sp + 8 * sl;
          float2 v[8];
          if (8 * sl + 8 <= chr) {
#pragma unroll
            for (int x = 0; x < 8; x += 2) {
              const float4 z = *reinterpret_cast<const float4*>(src + x);
              v[x] = make_float2(z.x, z.y);
              v[x + 1] = make_float2(z.z, z.w);
            }
          } else {
#pragma unroll
            for (int x = 0; x < 8; ++x) v[x] = 8 * sl + x < chr ? src[x] : make_float2(0.f, 0.f);
          }
          store_slice(row, sl, v);
        }
        lds_barrier();
      }
    }
    // the block's logarithms and outcomes: thread (row, site)
    lds_barrier();
    if (hs < ns) {
      ratio[hs][hrow] = log(ratio[hs][hrow]);
      if (r0 + hrow < ch.rows) c.outcomes[(size_t)(ch.c0 + r0 + hrow) * c.M + kb + hs] = oc[hs][hrow];
    }
    lds_barrier();
    if (tid < R)
      for (int e = 0; e < ns; ++e) lp = oc[e][tid] < 0 ? -INFINITY : lp + ratio[e][tid];
    lds_barrier();
  }
  if (c.logp && tid < R && r0 + tid < ch.rows) c.logp[ch.c0 + r0 + tid] = lp;
}

#define MPS_MID_KERNEL1(NAME, FORM, G, NW, GPW)                                                                      \
  __global__ __launch_bounds__(64 * NW, 8 / NW) void sweep_mid_##NAME##_##G(                                         \
      const MidChain* chains, const int* item_start, int nchain, int slices, int sp, const ChunkArgs* chp,           \
      uint64_t seed, int* nflag) {                                                                                   \
    sweep_mid_body<FORM, NW, GPW>(chains, item_start, nchain, slices, sp, chp, seed, nflag);                         \
  }
#define MPS_MID_KERNEL(NAME, FORM)       \
  MPS_MID_KERNEL1(NAME, FORM, 4, 4, 1)   \
  MPS_MID_KERNEL1(NAME, FORM, 8, 8, 1)   \
  MPS_MID_KERNEL1(NAME, FORM, 16, 8, 2)
MPS_MID_KERNEL(bf16x3, kBf16x3)
MPS_MID_KERNEL(fp16x3, kFp16x3)
MPS_MID_KERNEL(f16f8, kFp16F8)
MPS_MID_KERNEL(f16f6, kFp16F6)
#undef MPS_MID_KERNEL
#undef MPS_MID_KERNEL1

}  // namespace

hipError_t launch_sweep_mid(int form, int groups, const MidChain* chains, const int* item_start, int nchain, int items,
                            int chimax, const ChunkArgs* ch, uint64_t seed, int* nflag, hipStream_t s) {
  if (nchain <= 0 || items <= 0) return hipSuccess;
  const int slices = lp_pad_k(chimax) >> 4;
  const int sp = mid_row_pitch(chimax);
  const size_t lds = mid_lds_bytes(chimax);
#define MPS_MID_LAUNCH1(KERNEL, NTHREADS)                                                                       \
  hipLaunchKernelGGL(KERNEL, dim3(items), dim3(NTHREADS), lds, s, chains, item_start, nchain, slices, sp, ch, seed, \
                     nflag)
#define MPS_MID_LAUNCH(NAME)                                            \
  do {                                                                  \
    if (groups <= 4) MPS_MID_LAUNCH1(sweep_mid_##NAME##_4, 256);        \
    else if (groups <= 8) MPS_MID_LAUNCH1(sweep_mid_##NAME##_8, 512);   \
    else MPS_MID_LAUNCH1(sweep_mid_##NAME##_16, 512);                   \
    return hipGetLastError();                                           \
  } while (0)
  if (form == kBf16x3) MPS_MID_LAUNCH(bf16x3);
  if (form == kFp16x3) MPS_MID_LAUNCH(fp16x3);
  if (form == kFp16F8) MPS_MID_LAUNCH(f16f8);
  if (form == kFp16F6) MPS_MID_LAUNCH(f16f6);
  return hipErrorInvalidValue;
#undef MPS_MID_LAUNCH
#undef MPS_MID_LAUNCH1
}

}  // namespace mps
