// Streaming list forward on the matrix cores, for lists with linears of up to
// 64 tokens (Proposition 1, Eq. proposition1; both paths summed as in Eq.
// final_weight_approx_res), in three kinds of launch whatever the list's
// length, with no workgroup waiting for another:
//   S1  one workgroup per (linear, path, group of latent tiles, run of d_in):
//       D[k][t] = sum_j (s(V_p[j][k]) g_p[j]) x[t][j] over the run with
//       v_mfma_f32_16x16x32_bf16; the bf16 terms of the run's g are cut once
//       into LDS, the 4 waves split the group's latent tiles; the partial sums
//       go to the workspace in accumulator order (one launch per token tile
//       count, 1..4);
//   R   one thread per (linear, path, token tile, 32 latents, lane): w = l (.) z
//       from the runs' partials in ascending run order, cut into bf16 terms and
//       stored as stage 2's B operand;
//   S2  one workgroup per (linear, 128 to 512 output rows): the B operands of both
//       paths stream through LDS, shared by the 4 waves, each 32-latent block's
//       A operand (U signs) is built once per row tile and serves every token
//       tile, y = h_0 u_0 + h_1 u_1 rounded once (one launch per token tile
//       count).
// Operands as in the single-launch matrix-core kernel: g and x are cut into
// exact bf16 terms (1, 2 or 3 per value for bf16, f16, fp32), so every product
// is exact and the sums are fp32; w is cut into 2 bf16 terms (3 for fp32
// outputs), which carries 16 (24) significant bits into stage 2.
//
// Inputs of this path: x and g read as aligned groups of four (d_in a
// multiple of 4, x and g aligned to four elements).
#include <algorithm>
#include <cstring>
#include <vector>

#include "device_common.h"
#include "lb_few.h"
#include "stream_plan.h"

namespace lb {

namespace {

using splan::align256;
using splan::has_work;
using splan::kHdrCounts;
using splan::kHdrFp;
using splan::kHdrN;
using splan::packed_bytes64;
using splan::plan_ok;
using splan::StreamLinear;

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kGroups = 4;  // one linear: groups of 4 waves taking turns over the blocks of a reduction
constexpr int kMaxTok = 64;
constexpr int kMaxRank = 1024;
constexpr int kMaxRuns = 511;   // S1 map code: 9 bits of run
constexpr int kMaxBpr = 64;     // most 32-input blocks per run (its g terms are held in LDS)
constexpr int kMinBpr = 8;      // fewest, for lists too short to fill the chip with longer runs
constexpr int kWantWg1 = 1024;  // S1 workgroups below which runs get shorter

// 16-latent tiles a wave holds: the smallest class that takes the linear in
// the fewest groups (4 accumulator registers per tile and token tile)
constexpr int kMtClasses = 4;
__host__ __device__ constexpr int mt_cls(int tt, int c) {
  return c == 0 ? 2 : (c == 1 ? 3 : (c == 2 ? 5 : (tt <= 2 ? 8 : 6)));
}

using SmGeom = FewPlan;  // cls: launch of S1, (tt - 1) kMtClasses + class

// bpr: 32-input blocks per run wanted
SmGeom sm_geometry(const ForwardArgs& a, int bpr) {
  SmGeom g{};
  g.tt = (a.T + 15) / 16;
  g.nmf = (a.r + 15) / 16;
  const int most = kWaves * mt_cls(g.tt, kMtClasses - 1);
  g.ng = (g.nmf + most - 1) / most;
  const int need = (g.nmf + kWaves * g.ng - 1) / (kWaves * g.ng);
  int c = 0;
  while (mt_cls(g.tt, c) < need) ++c;
  g.mt = need;
  g.cls = (g.tt - 1) * kMtClasses + c;
  const int nbt = nblocks32(a.d_in);
  g.bpr = std::min(kMaxBpr, std::max(bpr, (nbt + kMaxRuns - 1) / kMaxRuns));
  g.s1d = (nbt + g.bpr - 1) / g.bpr;
  return g;
}

// partial sums of one linear: [2][s1d][nmf][tt][64 lanes][4] floats
size_t part_bytes(const SmGeom& g) { return static_cast<size_t>(2) * g.s1d * g.nmf * g.tt * 1024; }

// ---------------------------------------------------------------------------
// S1
// ---------------------------------------------------------------------------
// low (high) halves of a and b as one register: a's in the low half
__device__ __forceinline__ uint32_t lo16s(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t hi16s(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

typedef __attribute__((address_space(3))) void* lds_ptr;

// at most VM vector-memory operations of this wave outstanding and its LDS
// accesses done, then the barrier; LDS accesses stay on their side of it
template <int VM>
__device__ __forceinline__ void wait_barrier() {
  static_assert(VM >= 0 && VM < 64, "vmcnt range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | (7 << 4));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Wave w of a group holds latent tiles t0 + (0 .. mt - 1), t0 = (4 grp + w) mt.
// x (shared by the waves) and each wave's V words stream through a ring of
// LDS buffers of CB blocks, filled by global-to-LDS loads kBuf - 1 chunks ahead:
// loads into registers had cost the occupancy that was to hide their latency.
// What bounds it then: building the A operands, 13 VALU instructions per tile
// and block with f16 scales (2 terms) for 2 matrix instructions per token tile,
// so up to 16 tokens the VALU, from 32 tokens on the matrix cores.  The g terms
// are cut once per workgroup (a wave that cut its own spent 40 instructions a
// block on them), partial sums leave as 16-byte stores, and the waves split the
// latents, not the blocks, so no sum crosses waves.
constexpr int kBuf1 = 3;         // lists: several workgroups a CU hide the rest of the latency
constexpr size_t kOneLds = 150 * 1024;  // one linear: about one workgroup a CU, so as deep as its LDS goes
constexpr int kOneBuf = 8;
__host__ __device__ constexpr int cb_of(int tt, int act) { return tt >= 3 && act == kDtF32 ? 1 : 2; }

// LDS of S1: the run's g terms, the x and V-word buffers, the tail block's
// words.  One array: of several the compiler would follow each buffer's loads
// and wait for the newest before every read.
template <int TT, int MT, int ACT, int SC, bool ONE = false>
struct S1Lds {
  static constexpr int XC = ACT == kDtF32 ? 2 : 1;
  static constexpr int G = ONE ? kGroups : 1, NWV = G * kWaves;  // wave groups, waves
  static constexpr int CB = ONE ? G : cb_of(TT, ACT);
  static constexpr int XI = (CB * TT * XC + NWV - 1) / NWV;  // x fragments per wave and chunk
  static constexpr int NV = (MT + 3) / 4;
  static constexpr int kXbuf = (TT == 1 ? CB * XC : XI * NWV) * 1024;
  static constexpr int kXs = kMaxBpr * 4 * nterms<SC>() * 16;
  static constexpr int kVbuf = CB * kWaves * NV * 256;
  // most vector-memory operations of a wave per chunk, of at most 63 in flight
  static constexpr int kXops = TT == 1 ? CB * XC / G : 4 * XI, kVops = CB / G * NV;
  static constexpr int kOps = kXops + kVops;
  static constexpr int kDeep = static_cast<int>((kOneLds - kXs) / (kXbuf + kVbuf));
  static constexpr int kDeepOps = 2 + 63 / kOps;
  static constexpr int kBuf =
      !ONE ? kBuf1
           : (kDeep < kOneBuf ? (kDeep < kDeepOps ? kDeep : kDeepOps) : (kOneBuf < kDeepOps ? kOneBuf : kDeepOps));
  static constexpr int kVs = kXs + kBuf * kXbuf;
  static constexpr int kVt = kVs + kBuf * kVbuf;
  static constexpr int kRed = 2 * kWaves * MT * TT * 1024;  // ONE: two groups' sums, in place of the ring
  static constexpr int kRing = kVt + NWV * NV * 256;
  static constexpr int kBytes = ONE && kRed > kRing ? kRed : kRing;
  static_assert(kBuf >= 2 && kBytes <= (ONE ? 160 * 1024 : 65536), "ring depth; S1's lists raise no LDS limit");
};

template <int TT, int MT, int ACT, int SC, bool ONE>
__device__ __forceinline__ void sm_s1_body(const StreamLinear& L, int p, int grp, int c) {
  constexpr int NG = nterms<SC>(), NX = nterms<ACT>();
  constexpr int EX = ACT == kDtF32 ? 4 : 2;
  constexpr int CB = ONE ? kGroups : cb_of(TT, ACT);
  constexpr int XC = EX / 2;                       // 16-byte pieces of a lane's 8 inputs
  constexpr int kXf = CB * TT * XC;                  // x fragments (1 KB) of a chunk
  constexpr int XI = S1Lds<TT, MT, ACT, SC, ONE>::XI;  // of them per wave
  constexpr int NV = (MT + 3) / 4;                   // word loads (64 latents) per wave and block
  using Lds = S1Lds<TT, MT, ACT, SC, ONE>;
  constexpr int kBuf = Lds::kBuf, G = Lds::G, NWV = Lds::NWV;
  extern __shared__ __attribute__((aligned(16))) char sm_lds[];
  u32x4* gt = reinterpret_cast<u32x4*>(sm_lds);
  auto xs = [&](int buf) { return reinterpret_cast<u32x4*>(sm_lds + Lds::kXs + buf * Lds::kXbuf); };
  auto vs = [&](int buf, int bl, int w) {
    return reinterpret_cast<uint32_t*>(sm_lds + Lds::kVs + ((buf * CB + bl) * kWaves + w) * NV * 256);
  };
  uint32_t* vt = reinterpret_cast<uint32_t*>(sm_lds + Lds::kVt) + (threadIdx.x >> 6) * NV * 64;  // this wave's tail words
  const int T = L.T, r = L.r, d_in = L.d_in, mt = L.mt;
  const int tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int grp4 = wv / kWaves, wave = wv % kWaves;  // group of 4 waves; the wave's role in it
  const int n16 = lane & 15, gq = lane >> 4;
  const rsrc_t vr = make_rsrc_uniform(p ? L.V[1] : L.V[0], L.v_bytes);
  const rsrc_t gr = make_rsrc_uniform(p ? L.g[1] : L.g[0], L.g_bytes);
  const rsrc_t xr = make_rsrc_uniform(L.x, L.x_bytes);
  const int nbt = nblocks32(d_in), nbv = d_in >> 5, tailv = d_in & 31;
  const int b0 = c * L.bpr;
  const int b1 = min(nbt, b0 + L.bpr);
  const int nch = (b1 - b0 + CB - 1) / CB;
  const int nmf = (r + 15) >> 4;
  const int t0 = (kWaves * grp + wave) * mt;
  const int mts = min(mt, nmf - t0);  // this wave's tiles (<= 0: none)
  const bool xv = d_in % (16 / EX) == 0 && reinterpret_cast<uintptr_t>(L.x) % 16 == 0;
  const bool tail16 = tailv != 0 && tailv <= 16 && b1 > nbv;  // 16-bit tail words

  // loads of chunk ch into its buffer: x fragments as 16-byte pieces of rows
  // (4-byte ones when rows are not whole pieces; up to 16 tokens always, each
  // wave a quarter of every fragment) and NV CB word loads per wave.  x is zero
  // past d_in and past T; words past r or past the run are whatever is there
  // (zero past the buffer): no product of theirs is kept.
  const uint32_t xlane = static_cast<uint32_t>(n16) * d_in + 8 * gq;
  auto load_x4 = [&](char* dst, int tt, int j, int d, bool on) {
    // dword lane + 64 d of the fragment: lane (lane + 64 d) / 4 of the 16-byte form, dword % 4 of its piece
    const int ln = (lane >> 2) + 16 * d;
    const int e = j + 8 * (ln >> 4) + (lane & 3) * (4 / EX);
    const uint32_t off = (static_cast<uint32_t>(16 * tt + (ln & 15)) * d_in + e) * EX;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_ptr)(dst + 256 * d), 4, on && e < d_in ? off : kOob, 0, 0, 0);
  };
  const uint32_t vlane = 16 * t0 + lane;
  auto load = [&](int ch, int buf) {
    const int bb = b0 + ch * CB;
    if constexpr (TT == 1) {
#pragma unroll
      for (int f = 0; f < CB * XC; ++f)
        if (f / XC % G == grp4)
          load_x4(reinterpret_cast<char*>(xs(buf) + f * 64), 0, 32 * (bb + f / XC) + 4 * (f % XC), wave, true);
    } else {
#pragma unroll
      for (int i = 0; i < XI; ++i) {
        const int f = wv + NWV * i;  // (block, token tile, piece), piece fastest
        const int pc = f % XC, tt = (f / XC) % TT, bl = f / (XC * TT);
        char* dst = reinterpret_cast<char*>(xs(buf) + f * 64);
        const int j = 32 * (bb + bl) + 4 * pc;  // piece pc of lane group gq: inputs j + 8 gq ..
        if (xv) {
          const uint32_t off = (static_cast<uint32_t>(16 * tt) * d_in + j + xlane) * EX;
          __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_ptr)dst, 16, f < kXf && j + 8 * gq < d_in ? off : kOob, 0,
                                                   0, 0);
        } else {
#pragma unroll
          for (int d = 0; d < 4; ++d) load_x4(dst, tt, j, d, f < kXf);
        }
      }
    }
#pragma unroll
    for (int b = 0; b < CB / G; ++b)
#pragma unroll
      for (int d = 0; d < NV; ++d) {
        const int bl = G * b + grp4;
        // (32-bit tail entries sit where a full word would)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, (lds_ptr)(vs(buf, bl, wave) + 64 * d), 4,
                                                 (static_cast<uint32_t>(bb + bl) * r + vlane + 64 * d) * 4u, 0, 0, 0);
      }
  };
#pragma unroll
  for (int ch = 0; ch < kBuf - 1; ++ch) load(ch, ch);

  if (tail16)
#pragma unroll
    for (int d = 0; d < NV; ++d) {
      const int k = 16 * t0 + 64 * d + lane;
      vt[64 * d + lane] = static_cast<uint16_t>(
          __builtin_amdgcn_raw_buffer_load_b16(vr, k < r ? 4u * nbv * r + 2u * k : kOob, 0, 0));
    }
  // the run's g terms (zero past d_in): [block][lane group][term]
  for (int it = tid; it < (b1 - b0) * 4; it += NWV * 64) {
    const uint32_t j0 = 32 * (b0 + (it >> 2)) + 4 * (it & 3);
    uint32_t raw[2][4];
    bload4<SC, true>(gr, j0, true, raw[0]);
    bload4<SC, true>(gr, j0 + 16, true, raw[1]);
    u32x4 d[NG];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      uint32_t lo[NG], hi[NG];
      split_exact<NG>(raw4_elem<SC, true>(raw[0], v), lo);
      split_exact<NG>(raw4_elem<SC, true>(raw[1], v), hi);
#pragma unroll
      for (int s = 0; s < NG; ++s) d[s][v] = lo[s] | (hi[s] << 16);
    }
#pragma unroll
    for (int s = 0; s < NG; ++s) gt[it * NG + s] = d[s];
  }

  floatx4 acc[MT][TT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) acc[m][tt] = floatx4{0.f, 0.f, 0.f, 0.f};

  // products of block b.  All MT tiles, whether this wave has them or not: a
  // branch per tile had kept the tiles' operands from overlapping.
  auto block = [&](int b, int buf, int bl) {
    u32x4 g[NG];
#pragma unroll
    for (int s = 0; s < NG; ++s) g[s] = gt[((b - b0) * 4 + gq) * NG + s];
    const uint32_t* wp = tail16 && b == nbv ? vt : vs(buf, bl, wave);
    uint32_t words[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) words[m] = wp[16 * m + n16];
    u32x4 X[TT][NX];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const u32x4* xf = xs(buf) + (bl * TT + tt) * XC * 64;
      // inputs 4 gq .. + 3 and the same + 16: halves of the pieces of lane groups gq / 2 and gq / 2 + 2
      uint32_t ra[4] = {0u, 0u, 0u, 0u}, rd[4] = {0u, 0u, 0u, 0u};
      if constexpr (XC == 1) {
        const u32x2* x2 = reinterpret_cast<const u32x2*>(xf) + ((gq >> 1) * 16 + n16) * 2 + (gq & 1);
        const u32x2 a = x2[0], d = x2[64];
        ra[0] = a[0], ra[1] = a[1], rd[0] = d[0], rd[1] = d[1];
      } else {
        const u32x4 a = xf[(gq & 1) * 64 + (gq >> 1) * 16 + n16], d = xf[(gq & 1) * 64 + ((gq >> 1) + 2) * 16 + n16];
#pragma unroll
        for (int v = 0; v < 4; ++v) ra[v] = a[v], rd[v] = d[v];
      }
      if constexpr (NX == 1) {
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          X[tt][0][2 * v] = lo16s(ra[v], rd[v]);
          X[tt][0][2 * v + 1] = hi16s(ra[v], rd[v]);
        }
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          uint32_t lo[NX], hi[NX];
          split_exact<NX>(raw4_elem<ACT, true>(ra, v), lo);
          split_exact<NX>(raw4_elem<ACT, true>(rd, v), hi);
#pragma unroll
          for (int e = 0; e < NX; ++e) X[tt][e][v] = lo[e] | (hi[e] << 16);
        }
      }
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const uint32_t ws = words[m] >> (4 * gq);
      u32x4 sg;
#pragma unroll
      for (int v = 0; v < 4; ++v) sg[v] = (ws << (15 - v)) & 0x80008000u;
#pragma unroll
      for (int s = 0; s < NG; ++s) {
        const u32x4 A = sg ^ g[s];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
          for (int e = 0; e < NX; ++e) acc[m][tt] = mfma(A, X[tt][e], acc[m][tt]);
      }
    }
  };
  // fp32 inputs: the sums of kFold blocks are added apart, so that a run of 64
  // blocks does not add 576 products' rounding to one accumulator.  Error
  // against 64 bits (unfolded; folds of 4, 8 and 16 blocks for 1, 2 and more token
  // tiles; these; runs of 4 to 16 blocks an accumulator split over four waves): 70B
  // at 0.55 bits, 64 tokens 5.9e-7, 5.0e-7, 4.4e-7, 4.9e-7; 13B at 0.55, 31 tokens
  // -, 4.04e-7, 3.80e-7, 4.02e-7; 13B at 0.1, 16 tokens -, 2.6e-7, 2.2e-7, 2.5e-7.
  // They cost 1-2% of a pass, 4% at 17 to 32 tokens.  bf16 and f16 lists of 4 to 64
  // tokens lie as far from the 64-bit result without folds as with ones of 2 to 8
  // blocks (to 6 digits; those took 1-8% longer): their outputs' rounding is far
  // above that of the sums.
  constexpr int kFold = ACT == kDtF32 && !ONE ? (TT == 1 ? 2 : (TT == 2 ? 6 : 12)) : 0;
  floatx4 tot[kFold > 0 ? MT * TT : 1] = {};
  constexpr int kAhead = kBuf - 2;  // chunks still in flight when one is used
  int buf = 0;
  for (int ch = 0; ch < nch; ++ch) {
    // chunk ch has landed (each wave waits for its own loads, the barrier for
    // everyone's) and every wave is done with the buffer of chunk ch - 1
    if (TT == 1)
      wait_barrier<kAhead * Lds::kOps>();
    else if (xv)
      wait_barrier<kAhead * (XI + Lds::kVops)>();
    else
      wait_barrier<kAhead * Lds::kOps>();
    load(ch + kBuf - 1, buf == 0 ? kBuf - 1 : buf - 1);
    if (mts > 0) {
#pragma unroll
      for (int i = 0; i < CB / G; ++i) {
        const int bl = G * i + grp4, b = b0 + ch * CB + bl;
        if (b < b1) block(b, buf, bl);
      }
    }
    buf = buf == kBuf - 1 ? 0 : buf + 1;
    if constexpr (kFold > 0)
      if ((ch + 1) % (kFold / CB) == 0) {
#pragma unroll
        for (int m = 0; m < MT * TT; ++m) {
          tot[m] += acc[m / TT][m % TT];
          acc[m / TT][m % TT] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
      }
  }
  if constexpr (kFold > 0)
#pragma unroll
    for (int m = 0; m < MT * TT; ++m) acc[m / TT][m % TT] += tot[m];
  // global-to-LDS loads past the run are still in flight: none may land after
  // the workgroup's LDS is given away
  __builtin_amdgcn_s_waitcnt(0);
  if constexpr (ONE) {
    // the groups' sums, (0 + 2) + (1 + 3), through LDS
    static_assert(kGroups == 4, "two steps");
    floatx4* red = reinterpret_cast<floatx4*>(sm_lds) + wave * MT * TT * 64 + lane;
#pragma unroll
    for (int n = 2; n >= 1; n >>= 1) {
      __syncthreads();
      if (grp4 >= n && grp4 < 2 * n)
#pragma unroll
        for (int m = 0; m < MT * TT; ++m) red[((grp4 - n) * kWaves * MT * TT + m) * 64] = acc[m / TT][m % TT];
      __syncthreads();
      if (grp4 < n)
#pragma unroll
        for (int m = 0; m < MT * TT; ++m) acc[m / TT][m % TT] += red[(grp4 * kWaves * MT * TT + m) * 64];
    }
    if (grp4 > 0) return;
  }
  if (mts <= 0) return;
  float* out = L.part + (static_cast<int64_t>(p * L.s1d + c) * nmf + t0) * TT * 256 + lane * 4;
#pragma unroll
  for (int m = 0; m < MT; ++m)
    if (m < mts)
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) *reinterpret_cast<floatx4*>(out + (m * TT + tt) * 256) = acc[m][tt];
}

template <int TT, int MT, int ACT, int SC>
__global__ void __launch_bounds__(kThreads) sm_s1_kernel(const uint32_t* __restrict__ hdr,
                                                         const StreamLinear* __restrict__ descs,
                                                         const uint32_t* __restrict__ map, uint64_t fp) {
  if (!plan_ok(hdr, fp)) return;
  const uint32_t code = map[blockIdx.x];
  sm_s1_body<TT, MT, ACT, SC, false>(descs[code >> 16], (code >> 15) & 1, (code >> 9) & 63, code & 511);
}

// ---------------------------------------------------------------------------
// R: w = l (.) z, the runs' partial sums in ascending run order, written as NW
// bf16 terms straight into the matrix-core B fragments of stage 2: for path p,
// 32-latent block kb, token tile tt and term a, one u32x4 per lane, lane (n16,
// gq) register v holding the term of w at token 16 tt + n16 and latents 32 kb +
// 4 gq + v (low half) and + 16 (high half); latents past r are zero.  The two
// accumulator tiles of a block are read as S1's lanes wrote them, so loads and
// stores are whole 1 KB lines (one element per thread, with 2-byte stores,
// took 143 us in the 7B, 0.55 bits per weight, 64-token list).
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int nw_of(int act) { return act == kDtF32 ? 3 : 2; }

__host__ __device__ inline size_t frag_bytes(int T, int r, int nw) {
  return static_cast<size_t>(2) * ((T + 15) / 16) * nblocks32(r) * nw * 1024;
}
// threads of R for one linear
__host__ __device__ inline int r_items(int T, int r) { return 2 * ((T + 15) / 16) * nblocks32(r) * 64; }

// SPLIT (few fragments): a workgroup's waves share a fragment, each adding a
// share of the runs, and the shares are added in order: the sum is
// one round of loads instead of four (6.5 us at 16 runs).
template <int NW, int SC, int SPLIT>
__device__ __forceinline__ void sm_r_body(const StreamLinear& L, int e) {
  const int T = L.T, r = L.r, s1d = L.s1d;
  if (e >= r_items(T, r)) return;
  const int tt_n = (T + 15) / 16, nkb = nblocks32(r), nmf = (r + 15) >> 4;
  const int lane = e & 63, gq = lane >> 4;
  const int f = e >> 6;  // (p, kb, tt), tt fastest
  const int tt = f % tt_n, pk = f / tt_n;
  const int p = pk >= nkb ? 1 : 0, kb = pk - p * nkb;
  const bool two = 2 * kb + 1 < nmf;
  const float* src = L.part + ((static_cast<int64_t>(p) * s1d * nmf + 2 * kb) * tt_n + tt) * 256 + lane * 4;
  const int64_t cs = static_cast<int64_t>(nmf) * tt_n * 256;
  const int64_t hs = two ? tt_n * 256 : 0;
  const rsrc_t lr = make_rsrc(p ? L.l[1] : L.l[0], L.l_bytes);
  floatx4 l0, l1;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int k = 32 * kb + 4 * gq + v;
    l0[v] = bits_to_f32<SC>(bload<SC>(lr, k, k < r));
    l1[v] = bits_to_f32<SC>(bload<SC>(lr, k + 16, k + 16 < r));
  }
  floatx4 z0 = {0.f, 0.f, 0.f, 0.f}, z1 = z0;
  const int wave = threadIdx.x >> 6;
  const int per = (s1d + SPLIT - 1) / SPLIT;
  const int c0 = SPLIT > 1 ? min(s1d, wave * per) : 0, c1 = SPLIT > 1 ? min(s1d, c0 + per) : s1d;
#pragma unroll 8
  for (int c = c0; c < c1; ++c) {
    z0 += *reinterpret_cast<const floatx4*>(src + c * cs);
    z1 += *reinterpret_cast<const floatx4*>(src + c * cs + hs);
  }
  if constexpr (SPLIT > 1) {
    __shared__ floatx4 part[SPLIT - 1][2][64];
    if (wave > 0) {
      part[wave - 1][0][lane] = z0;
      part[wave - 1][1][lane] = z1;
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < SPLIT - 1; ++w) {
      z0 += part[w][0][lane];
      z1 += part[w][1][lane];
    }
  }
  uint32_t lo[4][NW], hi[4][NW];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int k = 32 * kb + 4 * gq + v;
    split_round<NW>(k < r ? z0[v] * l0[v] : 0.0f, lo[v]);
    split_round<NW>(k + 16 < r ? z1[v] * l1[v] : 0.0f, hi[v]);
  }
  u32x4* frag = reinterpret_cast<u32x4*>(L.wlat) + static_cast<int64_t>(f) * NW * 64 + lane;
#pragma unroll
  for (int a = 0; a < NW; ++a)
    frag[a * 64] = u32x4{lo[0][a] | (hi[0][a] << 16), lo[1][a] | (hi[1][a] << 16), lo[2][a] | (hi[2][a] << 16),
                         lo[3][a] | (hi[3][a] << 16)};
}

// SPLIT = kWaves: a fragment per workgroup; 1: one per wave
template <int NW, int SC, int SPLIT>
__global__ void __launch_bounds__(kThreads) sm_r_kernel(const uint32_t* __restrict__ hdr,
                                                        const StreamLinear* __restrict__ descs,
                                                        const uint32_t* __restrict__ map, uint64_t fp) {
  if (!plan_ok(hdr, fp)) return;
  const uint32_t code = map[blockIdx.x];
  const int j = static_cast<int>(code & 0xffffu);
  sm_r_body<NW, SC, SPLIT>(descs[code >> 16],
                           SPLIT > 1 ? j * 64 + (threadIdx.x & 63) : j * kThreads + static_cast<int>(threadIdx.x));
}

// the bits st<DT> would store (16-bit dtypes)
template <int DT>
__device__ __forceinline__ uint32_t round16(float v) {
  if constexpr (DT == kDtBF16) {
    return f32_to_bf16_bits(v);
  } else {
    asm volatile("" : "+v"(v));  // the fp32 value is formed first, as in st<>
    return __half_as_ushort(__float2half_rn(v));
  }
}

// ---------------------------------------------------------------------------
// S2: 64 RB output rows of one linear, every token, both paths.  Wave w holds
// row tiles RB w .. RB w + RB - 1 of 16 rows for every token tile.  The B
// fragments (shared by the waves) and each wave's U words stream through
// a ring of LDS buffers in chunks of kCk 32-latent blocks (path 0, then path 1),
// filled by global-to-LDS loads kBuf - 1 chunks ahead, one barrier a chunk.
// Up to 16 tokens the A operands bound it (9 VALU instructions for 2 matrix
// instructions), from 32 on the matrix cores.
// ---------------------------------------------------------------------------
constexpr int kBuf2 = 3;
constexpr int kCk = 2;
// row tiles per wave of the list kernels: 4, and up to 16 tokens, where a row
// tile takes 8 registers (32 from 49 tokens), 8, or 2 in short lists
__host__ __device__ constexpr int rb_of(int tt, bool shrt) { return tt == 1 ? (shrt ? 2 : 8) : 4; }

// LDS of S2 (one array, as in S1): the fragment and U-word buffers, the 16-bit
// tail words
template <int TT, int RB, int ACT, bool ONE = false>
struct S2Lds {
  static constexpr int G = ONE ? kGroups : 1, NWV = G * kWaves, CK = ONE ? G : kCk;
  static constexpr int FI = (CK * TT * nw_of(ACT) + NWV - 1) / NWV;
  static constexpr int NV = (RB + 3) / 4;
  static constexpr int kBbuf = FI * NWV * 1024;
  static constexpr int kUbuf = CK * kWaves * NV * 256;
  static constexpr int kDeep = static_cast<int>(kOneLds / (kBbuf + kUbuf));
  static constexpr int kBuf = !ONE ? kBuf2 : (kDeep < kOneBuf ? kDeep : kOneBuf);
  static constexpr int kUs = kBuf * kBbuf;
  static constexpr int kUt = kUs + kBuf * kUbuf;
  static constexpr int kRed = 2 * kWaves * RB * TT * 1024;
  static constexpr int kRing = kUt + 2 * kWaves * NV * 256;
  static constexpr int kBytes = ONE && kRed > kRing ? kRed : kRing;
};

template <int TT, int RB, int ACT, int SC, bool ONE>
__device__ __forceinline__ void sm_s2_body(const StreamLinear& L, int q) {
  constexpr int NW = nw_of(ACT);
  constexpr int NV = (RB + 3) / 4;                 // word loads (64 rows) per wave and block
  using Lds = S2Lds<TT, RB, ACT, ONE>;
  constexpr int kBuf = Lds::kBuf, G = Lds::G, NWV = Lds::NWV, CK = Lds::CK;
  constexpr int FI = Lds::FI;                      // fragments (1 KB) of a chunk per wave
  extern __shared__ __attribute__((aligned(16))) char sm_lds[];
  auto bs = [&](int buf) { return reinterpret_cast<u32x4*>(sm_lds + buf * Lds::kBbuf); };
  auto us = [&](int buf, int u, int w) {
    return reinterpret_cast<uint32_t*>(sm_lds + Lds::kUs + ((buf * CK + u) * kWaves + w) * NV * 256);
  };
  auto ut = [&](int pp, int w) {  // 16-bit tail words
    return reinterpret_cast<uint32_t*>(sm_lds + Lds::kUt + (pp * kWaves + w) * NV * 256);
  };
  const int T = L.T, r = L.r, d_out = L.d_out;
  const int tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int grp4 = wv / kWaves, wave = wv % kWaves;  // group of 4 waves; the wave's role in it
  const int n16 = lane & 15, gq = lane >> 4;
  const int nkb = nblocks32(r), nbu = r >> 5, tailu = r & 31;
  const int nch = (nkb + CK - 1) / CK;  // chunks per path
  const int row0 = (q * kWaves + wave) * 16 * RB;
  const bool active = row0 < d_out;  // a wave past the last row only loads and keeps the barriers
  const bool tail16 = tailu != 0 && tailu <= 16;
  const rsrc_t fr = make_rsrc_uniform(L.wlat, static_cast<uint32_t>(frag_bytes(T, r, NW)));
  const rsrc_t ur0 = make_rsrc_uniform(L.U[0], L.u_bytes), ur1 = make_rsrc_uniform(L.U[1], L.u_bytes);
  // chunk ci (path ci / nch): FI fragment and NV CK word loads per wave.
  // Fragments past a path's blocks and words past a block's rows are whatever
  // is there (zero past the buffers): no product of theirs is kept.
  const uint32_t flane = wv * 1024u + lane * 16u, ulane = row0 + lane;
  auto load = [&](int ci, int buf) {
    const int p = ci >= nch ? 1 : 0, kb0 = (ci - p * nch) * CK;
    const uint32_t f0 = static_cast<uint32_t>((p * nkb + kb0) * TT * NW) * 1024u + flane;
#pragma unroll
    for (int i = 0; i < FI; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(fr, (lds_ptr)(bs(buf) + (wv + NWV * i) * 64), 16,
                                               f0 + NWV * i * 1024u, 0, 0, 0);
    const rsrc_t ur = p ? ur1 : ur0;
#pragma unroll
    for (int i = 0; i < CK / G; ++i)
#pragma unroll
      for (int d = 0; d < NV; ++d) {
        const int u = G * i + grp4;
        // (32-bit tail entries sit where a full word would)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ur, (lds_ptr)(us(buf, u, wave) + 64 * d), 4,
                                                 (static_cast<uint32_t>(kb0 + u) * d_out + ulane + 64 * d) * 4u, 0, 0,
                                                 0);
      }
  };
#pragma unroll
  for (int ci = 0; ci < kBuf - 1; ++ci) load(ci, ci);
  if (tail16 && grp4 == 0)
#pragma unroll
    for (int pp = 0; pp < 2; ++pp)
#pragma unroll
      for (int d = 0; d < NV; ++d) {
        const int row = row0 + 64 * d + lane;
        ut(pp, wave)[64 * d + lane] = static_cast<uint16_t>(__builtin_amdgcn_raw_buffer_load_b16(
            pp ? ur1 : ur0, row < d_out ? 4u * nbu * d_out + 2u * row : kOob, 0, 0));
      }
  uint32_t sgn_m = 0x80008000u, one_b = 0x3F803F80u;  // in registers: one VALU op per operand register
  asm volatile("" : "+v"(sgn_m), "+v"(one_b));
  floatx4 acc[RB][TT], yv[RB][TT];
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int j = 0; j < TT; ++j) acc[b][j] = yv[b][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  // y += h_p acc, acc = 0 (rows row0 + 16 b + 4 gq + e)
  auto fold = [&](int p) {
    const rsrc_t hr = make_rsrc_uniform(p ? L.h[1] : L.h[0], L.h_bytes);
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float hv = bits_to_f32<SC>(bload<SC>(hr, row0 + 16 * b + 4 * gq + e));
#pragma unroll
        for (int j = 0; j < TT; ++j) {
          yv[b][j][e] += hv * acc[b][j][e];
          acc[b][j][e] = 0.0f;
        }
      }
  };
  int buf = 0;
#pragma unroll 1
  for (int ci = 0; ci < 2 * nch; ++ci, buf = buf == kBuf - 1 ? 0 : buf + 1) {
    // chunk ci has landed (each wave waits for its own loads, the barrier for
    // everyone's) and every wave is done with the buffer of chunk ci - 1
    wait_barrier<(kBuf - 2) * (FI + NV * CK / G)>();
    load(ci + kBuf - 1, buf == 0 ? kBuf - 1 : buf - 1);
    if (!active) continue;
    const int p = ci >= nch ? 1 : 0, kb0 = (ci - p * nch) * CK;
    if (ci == nch) fold(0);
#pragma unroll
    for (int i = 0; i < CK / G; ++i) {
      const int u = G * i + grp4, kb = kb0 + u;
      if (kb >= nkb) break;
      const uint32_t* wp = tail16 && kb == nbu ? ut(p, wave) : us(buf, u, wave);
      uint32_t words[RB];
#pragma unroll
      for (int b = 0; b < RB; ++b) words[b] = wp[16 * b + n16] >> (4 * gq);
      u32x4 B[TT][NW];
#pragma unroll
      for (int j = 0; j < TT; ++j)
#pragma unroll
        for (int a = 0; a < NW; ++a) B[j][a] = bs(buf)[((u * TT + j) * NW + a) * 64 + lane];
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        u32x4 A;
#pragma unroll
        for (int v = 0; v < 4; ++v) A[v] = ((words[b] << (15 - v)) & sgn_m) | (one_b & ~sgn_m);
#pragma unroll
        for (int a = 0; a < NW; ++a)
#pragma unroll
          for (int j = 0; j < TT; ++j) acc[b][j] = mfma(A, B[j][a], acc[b][j]);
      }
    }
  }
  // global-to-LDS loads past the end are still in flight: none may land after
  // the workgroup's LDS is given away
  __builtin_amdgcn_s_waitcnt(0);
  if (active) fold(1);
  if constexpr (ONE) {
    // the groups' shares of y, (0 + 2) + (1 + 3), through LDS
    floatx4* red = reinterpret_cast<floatx4*>(sm_lds) + wave * RB * TT * 64 + lane;
#pragma unroll
    for (int n = 2; n >= 1; n >>= 1) {
      __syncthreads();
      if (grp4 >= n && grp4 < 2 * n)
#pragma unroll
        for (int m = 0; m < RB * TT; ++m) red[((grp4 - n) * kWaves * RB * TT + m) * 64] = yv[m / TT][m % TT];
      __syncthreads();
      if (grp4 < n)
#pragma unroll
        for (int m = 0; m < RB * TT; ++m) yv[m / TT][m % TT] += red[(grp4 * kWaves * RB * TT + m) * 64];
    }
    if (grp4 > 0) return;
  }
  if (!active) return;
  // 4 consecutive outputs per lane and token
  const bool vec = d_out % 4 == 0 && reinterpret_cast<uintptr_t>(L.y) % (ACT == kDtF32 ? 16 : 8) == 0;
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const int i = row0 + 16 * b + 4 * gq;
#pragma unroll
    for (int j = 0; j < TT; ++j) {
      const int t = 16 * j + n16;
      if (t >= T) continue;
      const int64_t o = static_cast<int64_t>(t) * d_out + i;
      if (vec) {
        if (i >= d_out) continue;
        if constexpr (ACT == kDtF32) {
          *reinterpret_cast<floatx4*>(static_cast<float*>(L.y) + o) = yv[b][j];
        } else {
          uint32_t h[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) h[e] = round16<ACT>(yv[b][j][e]);
          *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(L.y) + o) =
              u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (i + e < d_out) st<ACT>(L.y, o + e, yv[b][j][e]);
      }
    }
  }
}

template <int TT, int RB, int ACT, int SC>
__global__ void __launch_bounds__(kThreads) sm_s2_kernel(const uint32_t* __restrict__ hdr,
                                                         const StreamLinear* __restrict__ descs,
                                                         const uint32_t* __restrict__ map, uint64_t fp) {
  if (!plan_ok(hdr, fp)) return;
  const uint32_t code = map[blockIdx.x];
  sm_s2_body<TT, RB, ACT, SC, false>(descs[code >> 16], static_cast<int>(code & 0xffffu));
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
void fill_desc(StreamLinear& L, const ForwardArgs& f, const SmGeom& g) {
  L.x = f.x;
  L.y = f.y;
  for (int p = 0; p < 2; ++p) {
    L.U[p] = f.U[p];
    L.V[p] = f.V[p];
    L.h[p] = f.h[p];
    L.g[p] = f.g[p];
    L.l[p] = f.l[p];
  }
  L.T = f.T;
  L.d_in = f.d_in;
  L.d_out = f.d_out;
  L.r = f.r;
  L.s1d = g.s1d;
  L.bpr = g.bpr;
  L.mt = g.mt;
  const int64_t ex = f.act_dt == kDtF32 ? 4 : 2, es = f.sc_dt == kDtF32 ? 4 : 2;
  L.x_bytes = static_cast<uint32_t>(static_cast<int64_t>(f.T) * f.d_in * ex);
  L.g_bytes = static_cast<uint32_t>(f.d_in * es);
  L.h_bytes = static_cast<uint32_t>(f.d_out * es);
  L.l_bytes = static_cast<uint32_t>(f.r * es);
  L.v_bytes = static_cast<uint32_t>(packed_bytes64(f.r, f.d_in));
  L.u_bytes = static_cast<uint32_t>(packed_bytes64(f.d_out, f.r));
}

// Lists too short to fill the chip with the workgroups that serve long ones best
// (us a pass of 3 tokens, none of the three rules below -> all of them; 128-row
// workgroups and one thread a latent, as before these stages, in brackets: a 7B
// block 23.8 -> 15.7 (20.0), three 13B blocks 40.4 -> 29.0 (28.9), a 70B block 46.0 ->
// 30.0 (27.9), two 54.5 -> 37.5 (41.1); 16 tokens, a 70B block 46.7 -> 30.1 (32.9)):
//   S1  one launch per class of latent tiles is one after the other, and short
//       ones leave the chip partly idle: below kOneClassWg1 workgroups they go out
//       as one, of the largest class, unless that is over twice the tiles or more than
//       kOneClassTiles idle ones over the blocks (16 70B blocks, 49000: 167 -> 156 us
//       at 16 tokens; 32 7B blocks at 0.55 bits, 196000: f16 377 -> 397);
//   S2  below kShortWg2 workgroups of 8 row tiles a wave, 2 row tiles (16 tokens);
//   R   below kShortFrag fragments, four waves on each: a fragment's runs are read
//       one after the other, 112 of them in a 70B down projection.
constexpr int kOneClassWg1 = 4 * kWantWg1;
constexpr int kOneClassTiles = 65536;
constexpr int kShortWg2 = 512;
constexpr int kShortFrag = 2048;

struct PlanLayout {
  int bpr = kMaxBpr;
  bool one_cls = false;  // one launch of S1 per token tile count, of its linears' largest class
  bool short2 = false;   // S2 of 2 row tiles a wave (up to 16 tokens)
  bool shortr = false;   // R of kWaves waves a fragment
  int cls[4] = {};       // one_cls: that class
  int n1 = 0, nr = 0, n2 = 0;
  int n1_cls[4 * kMtClasses + 1] = {};  // S1 items of classes < k are map entries [0, n1_cls[k])
  int n2_cls[5] = {0, 0, 0, 0, 0};  // the same for S2 items
  size_t desc_off = 0, map1_off = 0, mapr_off = 0, map2_off = 0, data_off = 0, bytes = 0;
};

int r_groups(const ForwardArgs& a, bool shrt) {
  const int n = shrt ? 64 : kThreads;
  return (r_items(a.T, a.r) + n - 1) / n;
}
int s2_groups(const ForwardArgs& a, bool shrt) {
  const int rw = 16 * kWaves * rb_of((a.T + 15) / 16, shrt);
  return (a.d_out + rw - 1) / rw;
}
// launch of S1: (tt - 1) kMtClasses + class
int s1_launch(const PlanLayout& P, const SmGeom& g) { return P.one_cls ? (g.tt - 1) * kMtClasses + P.cls[g.tt - 1] : g.cls; }

PlanLayout plan_layout(const ForwardArgs* a, int n) {
  PlanLayout P;
  // the longest runs (fewest partial sums) that still give kWantWg1 workgroups
  for (;; P.bpr /= 2) {
    int64_t n1 = 0, n2 = 0, nf = 0, by_cls[4 * kMtClasses] = {};
    for (int i = 0; i < n; ++i)
      if (has_work(a[i])) {
        const SmGeom g = sm_geometry(a[i], P.bpr);
        n1 += 2 * g.ng * g.s1d;
        by_cls[g.cls] += 2 * g.ng * g.s1d;
        n2 += s2_groups(a[i], false);
        nf += r_items(a[i].T, a[i].r) / 64;
      }
    if (n1 < kWantWg1 && P.bpr > kMinBpr) continue;
    int64_t tiles = 0, tiles_one = 0;  // over S1's workgroups
    for (int t = 0; t < 4; ++t) {
      const int64_t* m = by_cls + t * kMtClasses;
      for (int c = 0; c < kMtClasses; ++c)
        if (m[c] > 0) P.cls[t] = c;
      for (int c = 0; c < kMtClasses; ++c) {
        tiles += m[c] * mt_cls(t + 1, c);
        tiles_one += m[c] * mt_cls(t + 1, P.cls[t]);
      }
    }
    P.one_cls = n1 < kOneClassWg1 && tiles_one <= 2 * tiles && (tiles_one - tiles) * P.bpr <= kOneClassTiles;
    P.short2 = n2 < kShortWg2;
    P.shortr = nf < kShortFrag;
    break;
  }
  size_t data = 0;
  for (int i = 0; i < n; ++i) {
    if (!has_work(a[i])) continue;
    const SmGeom g = sm_geometry(a[i], P.bpr);
    P.n1 += 2 * g.ng * g.s1d;
    P.n1_cls[s1_launch(P, g) + 1] += 2 * g.ng * g.s1d;
    P.nr += r_groups(a[i], P.shortr);
    P.n2 += s2_groups(a[i], P.short2);
    P.n2_cls[g.tt] += s2_groups(a[i], P.short2);
    data += align256(part_bytes(g)) + align256(frag_bytes(a[i].T, a[i].r, nw_of(a[i].act_dt)));
  }
  for (int k = 1; k <= 4 * kMtClasses; ++k) P.n1_cls[k] += P.n1_cls[k - 1];
  for (int k = 1; k < 5; ++k) P.n2_cls[k] += P.n2_cls[k - 1];
  P.desc_off = kCtrlBytes;
  P.map1_off = P.desc_off + align256(sizeof(StreamLinear) * static_cast<size_t>(n));
  P.mapr_off = P.map1_off + align256(4 * static_cast<size_t>(P.n1));
  P.map2_off = P.mapr_off + align256(4 * static_cast<size_t>(P.nr));
  P.data_off = P.map2_off + align256(4 * static_cast<size_t>(P.n2));
  P.bytes = P.data_off + data;
  return P;
}

template <int TT, int C, int ACT, int SC>
void launch_s1(const char* b, const PlanLayout& P, uint64_t fp, hipStream_t stream) {
  constexpr int MT = mt_cls(TT, C), k = (TT - 1) * kMtClasses + C;
  const int n = P.n1_cls[k + 1] - P.n1_cls[k];
  if (n == 0) return;
  hipLaunchKernelGGL((sm_s1_kernel<TT, MT, ACT, SC>), dim3(n), dim3(kThreads), (S1Lds<TT, MT, ACT, SC>::kBytes),
                     stream, reinterpret_cast<const uint32_t*>(b),
                     reinterpret_cast<const StreamLinear*>(b + P.desc_off),
                     reinterpret_cast<const uint32_t*>(b + P.map1_off) + P.n1_cls[k], fp);
}
template <int TT, int ACT, int SC>
void launch_s1(const char* b, const PlanLayout& P, uint64_t fp, hipStream_t stream) {
  launch_s1<TT, 0, ACT, SC>(b, P, fp, stream);
  launch_s1<TT, 1, ACT, SC>(b, P, fp, stream);
  launch_s1<TT, 2, ACT, SC>(b, P, fp, stream);
  launch_s1<TT, 3, ACT, SC>(b, P, fp, stream);
}

template <int TT, int RB, int ACT, int SC>
void launch_s2_rb(const char* b, const PlanLayout& P, uint64_t fp, hipStream_t stream) {
  const int n = P.n2_cls[TT] - P.n2_cls[TT - 1];
  if (n == 0) return;
  // (past 64 KB for 33 to 64 tokens in fp32; a failure is left to hipGetLastError)
  constexpr int bytes = S2Lds<TT, RB, ACT>::kBytes;
  static LdsLimit limit;
  (void)raise_lds(reinterpret_cast<const void*>(&sm_s2_kernel<TT, RB, ACT, SC>), bytes, limit);
  hipLaunchKernelGGL((sm_s2_kernel<TT, RB, ACT, SC>), dim3(n), dim3(kThreads), bytes, stream,
                     reinterpret_cast<const uint32_t*>(b), reinterpret_cast<const StreamLinear*>(b + P.desc_off),
                     reinterpret_cast<const uint32_t*>(b + P.map2_off) + P.n2_cls[TT - 1], fp);
}
template <int TT, int ACT, int SC>
void launch_s2(const char* b, const PlanLayout& P, uint64_t fp, hipStream_t stream) {
  if (TT == 1 && P.short2)
    launch_s2_rb<TT, rb_of(TT, TT == 1), ACT, SC>(b, P, fp, stream);
  else
    launch_s2_rb<TT, rb_of(TT, false), ACT, SC>(b, P, fp, stream);
}
template <int NW, int SC, int SPLIT>
void launch_r(const char* b, const PlanLayout& P, uint64_t fp, hipStream_t stream) {
  hipLaunchKernelGGL((sm_r_kernel<NW, SC, SPLIT>), dim3(P.nr), dim3(kThreads), 0, stream,
                     reinterpret_cast<const uint32_t*>(b), reinterpret_cast<const StreamLinear*>(b + P.desc_off),
                     reinterpret_cast<const uint32_t*>(b + P.mapr_off), fp);
}

template <int ACT, int SC>
void launch_all(const void* ws, const PlanLayout& P, uint64_t fp, hipStream_t stream) {
  const char* b = static_cast<const char*>(ws);
  launch_s1<1, ACT, SC>(b, P, fp, stream);
  launch_s1<2, ACT, SC>(b, P, fp, stream);
  launch_s1<3, ACT, SC>(b, P, fp, stream);
  launch_s1<4, ACT, SC>(b, P, fp, stream);
  if (P.shortr)
    launch_r<nw_of(ACT), SC, kWaves>(b, P, fp, stream);
  else
    launch_r<nw_of(ACT), SC, 1>(b, P, fp, stream);
  launch_s2<1, ACT, SC>(b, P, fp, stream);
  launch_s2<2, ACT, SC>(b, P, fp, stream);
  launch_s2<3, ACT, SC>(b, P, fp, stream);
  launch_s2<4, ACT, SC>(b, P, fp, stream);
}

template <int ACT>
void launch_act(const void* ws, const PlanLayout& P, int sc_dt, uint64_t fp, hipStream_t stream) {
  switch (sc_dt) {
    case kDtF32: launch_all<ACT, kDtF32>(ws, P, fp, stream); break;
    case kDtF16: launch_all<ACT, kDtF16>(ws, P, fp, stream); break;
    default: launch_all<ACT, kDtBF16>(ws, P, fp, stream); break;
  }
}

}  // namespace

bool stream_mma_supports(const ForwardArgs& a) {
  if (!has_work(a)) return true;
  if (a.T > kMaxTok || a.r > kMaxRank) return false;
  const int64_t ex = a.act_dt == kDtF32 ? 4 : 2, es = a.sc_dt == kDtF32 ? 4 : 2;
  // x and g as aligned groups of four elements
  if (a.d_in % 4 != 0 || reinterpret_cast<uintptr_t>(a.x) % (4 * ex) != 0 ||
      reinterpret_cast<uintptr_t>(a.g[0]) % (4 * es) != 0 || reinterpret_cast<uintptr_t>(a.g[1]) % (4 * es) != 0)
    return false;
  // 32-bit buffer offsets: the (up to 16 ceil(T / 16)) token rows read, the packed signs
  const int64_t lim = int64_t(1) << 31;
  const int64_t rows = 16 * ((a.T + 15) / 16);
  if ((rows + 1) * a.d_in * ex >= lim || packed_bytes64(a.d_out, a.r) >= lim || packed_bytes64(a.r, a.d_in) >= lim)
    return false;
  // d_in: 511 runs of 16, 32 or 64 blocks by token tiles (the plan's runs, of up
  // to 64 blocks whatever the tiles, need less)
  const int tt = (a.T + 15) / 16;
  if (nblocks32(a.d_in) > kMaxRuns * (tt == 1 ? 16 : (tt == 2 ? 32 : 64))) return false;
  // map codes: 16 bits of work index per linear
  if (2 * 16 * tt * 32 * nblocks32(a.r) > 65535 * kThreads || a.d_out > 65535 * 64) return false;
  return true;
}

size_t stream_mma_workspace_bytes(const ForwardArgs* a, int n) { return plan_layout(a, n).bytes; }

hipError_t stream_mma_init(const ForwardArgs* a, int n, uint64_t fp, void* ws, hipStream_t stream) {
  const PlanLayout P = plan_layout(a, n);
  std::vector<char> host(P.data_off, 0);
  uint32_t* hdr = reinterpret_cast<uint32_t*>(host.data());
  hdr[kHdrFp] = static_cast<uint32_t>(fp);
  hdr[kHdrFp + 1] = static_cast<uint32_t>(fp >> 32);
  hdr[kHdrN] = static_cast<uint32_t>(n);
  hdr[kHdrCounts + 0] = static_cast<uint32_t>(P.n1);
  hdr[kHdrCounts + 1] = static_cast<uint32_t>(P.nr);
  hdr[kHdrCounts + 2] = static_cast<uint32_t>(P.n2);
  StreamLinear* D = reinterpret_cast<StreamLinear*>(host.data() + P.desc_off);
  uint32_t* m1 = reinterpret_cast<uint32_t*>(host.data() + P.map1_off);
  uint32_t* mr = reinterpret_cast<uint32_t*>(host.data() + P.mapr_off);
  uint32_t* m2 = reinterpret_cast<uint32_t*>(host.data() + P.map2_off);
  char* data = static_cast<char*>(ws) + P.data_off;
  int i1[4 * kMtClasses], ir = 0;
  std::copy(P.n1_cls, P.n1_cls + 4 * kMtClasses, i1);
  int i2[4] = {P.n2_cls[0], P.n2_cls[1], P.n2_cls[2], P.n2_cls[3]};
  for (int i = 0; i < n; ++i) {
    StreamLinear& L = D[i];
    const ForwardArgs& f = a[i];
    if (!has_work(f)) continue;
    const SmGeom g = sm_geometry(f, P.bpr);
    fill_desc(L, f, g);
    L.part = reinterpret_cast<float*>(data);
    data += align256(part_bytes(g));
    L.wlat = reinterpret_cast<float*>(data);  // the B fragments of stage 2
    data += align256(frag_bytes(f.T, f.r, nw_of(f.act_dt)));
    // S1 items grouped by class, S2 items by token-tile count (one launch each)
    for (int p = 0; p < 2; ++p)
      for (int gr = 0; gr < g.ng; ++gr)
        for (int c = 0; c < g.s1d; ++c)
          m1[i1[s1_launch(P, g)]++] = (static_cast<uint32_t>(i) << 16) | (p << 15) | (gr << 9) | c;
    const int nrb = r_groups(f, P.shortr);
    for (int j = 0; j < nrb; ++j) mr[ir++] = (static_cast<uint32_t>(i) << 16) | j;
    const int nrow = s2_groups(f, P.short2);
    for (int j = 0; j < nrow; ++j) m2[i2[g.tt - 1]++] = (static_cast<uint32_t>(i) << 16) | j;
  }
  hipError_t e = hipMemcpyAsync(ws, host.data(), host.size(), hipMemcpyHostToDevice, stream);
  if (e != hipSuccess) return e;
  return hipStreamSynchronize(stream);
}

hipError_t stream_mma_forward(const ForwardArgs* a, int n, uint64_t fp, void* ws, hipStream_t stream) {
  const PlanLayout P = plan_layout(a, n);
  if (P.n1 == 0) return hipSuccess;
  int act = -1, sc = -1;
  for (int i = 0; i < n; ++i)
    if (has_work(a[i])) {
      act = a[i].act_dt;
      sc = a[i].sc_dt;
      break;
    }
  switch (act) {
    case kDtF32: launch_act<kDtF32>(ws, P, sc, fp, stream); break;
    case kDtF16: launch_act<kDtF16>(ws, P, sc, fp, stream); break;
    default: launch_act<kDtBF16>(ws, P, sc, fp, stream); break;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// One linear of up to 64 tokens, or a few of one token tile count: the same
// three stages, the descriptors as a kernel argument (grid y: the linear).  A
// linear's runs and wave groups do not depend on the others, so its result has
// the same bits alone and among others.
// ---------------------------------------------------------------------------
namespace {

constexpr int kOneThreads = kGroups * kThreads;

struct FewArgs {
  StreamLinear l[kFewMaxBatch];
};

template <int TT, int MT, int ACT, int SC>
__global__ void __launch_bounds__(kOneThreads) sm_one_s1_kernel(FewArgs A) {
  const StreamLinear& L = A.l[blockIdx.y];
  const int rest = blockIdx.x / L.s1d;
  if ((rest >> 1) * kWaves * L.mt >= (L.r + 15) >> 4) return;  // past this linear's groups
  sm_s1_body<TT, MT, ACT, SC, true>(L, rest & 1, rest >> 1, blockIdx.x - rest * L.s1d);
}
template <int NW, int SC>
__global__ void __launch_bounds__(kThreads) sm_one_r_kernel(FewArgs A) {
  const StreamLinear& L = A.l[blockIdx.y];
  sm_r_body<NW, SC, kWaves>(L, blockIdx.x * 64 + (threadIdx.x & 63));
}
template <int TT, int ACT, int SC>
__global__ void __launch_bounds__(kOneThreads) sm_one_s2_kernel(FewArgs A) {
  const StreamLinear& L = A.l[blockIdx.y];
  if (static_cast<int>(blockIdx.x) * 16 * kWaves >= L.d_out) return;
  sm_s2_body<TT, 1, ACT, SC, true>(L, blockIdx.x);
}

constexpr int kOneWantWg = 192;  // S1 workgroups wanted
constexpr int kOneMaxRuns = 16;  // runs at most: R adds them
constexpr int kOneMinBpr = 8;    // 32-input blocks of a run at least: two per wave group
// largest tile class: 3 tiles a wave (from r = 961 and 16 runs; more tiles never give kOneWantWg)
constexpr int kOneMaxCls = 1;
static_assert(2 * ((kMaxRank / 16 + kWaves * mt_cls(1, 2) - 1) / (kWaves * mt_cls(1, 2))) * kOneMaxRuns < kOneWantWg,
              "a larger class would be chosen");

// the plan of one linear in ws_bytes of workspace (bpr 0: none fits): as many
// runs as give kOneWantWg workgroups, fewer tiles a wave when they do not
SmGeom one_geometry(const ForwardArgs& a, size_t ws_bytes) {
  SmGeom g = sm_geometry(a, kMaxBpr);
  const int nbt = nblocks32(a.d_in);
  const size_t room = ws_bytes - kScratchOff;
  const size_t frag = align256(frag_bytes(a.T, a.r, nw_of(a.act_dt)));
  const int max_runs = std::max(1, std::min(kOneMaxRuns, nbt / kOneMinBpr));
  int c = kOneMaxCls;
  for (;; --c) {
    g.ng = (g.nmf + kWaves * mt_cls(g.tt, c) - 1) / (kWaves * mt_cls(g.tt, c));
    if (c == 0 || 2 * g.ng * max_runs >= kOneWantWg) break;
  }
  g.mt = (g.nmf + kWaves * g.ng - 1) / (kWaves * g.ng);
  g.cls = (g.tt - 1) * kMtClasses + c;
  int runs = std::max(1, std::min(max_runs, (kOneWantWg + 2 * g.ng - 1) / (2 * g.ng)));
  runs = std::max(runs, (nbt + kMaxBpr - 1) / kMaxBpr);
  for (;; --runs) {
    g.bpr = (nbt + runs - 1) / runs;
    g.s1d = (nbt + g.bpr - 1) / g.bpr;
    if (g.bpr > kMaxBpr) {
      g.bpr = 0;  // no room
      return g;
    }
    if (align256(part_bytes(g)) + frag <= room) return g;
    if (runs == 1) {
      g.bpr = 0;
      return g;
    }
  }
}

template <int TT, int C, int ACT, int SC>
hipError_t one_s1(const FewArgs& A, int n, int n1, hipStream_t stream) {
  constexpr int MT = mt_cls(TT, C), bytes = S1Lds<TT, MT, ACT, SC, true>::kBytes;
  static LdsLimit limit;
  const hipError_t e = raise_lds(reinterpret_cast<const void*>(&sm_one_s1_kernel<TT, MT, ACT, SC>), bytes, limit);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((sm_one_s1_kernel<TT, MT, ACT, SC>), dim3(n1, n), dim3(kOneThreads), bytes, stream, A);
  return hipGetLastError();
}
template <int TT, int ACT, int SC>
hipError_t one_launch(const FewArgs& A, int n, int c, int n1, int nr, int n2, hipStream_t stream) {
  constexpr int bytes = S2Lds<TT, 1, ACT, true>::kBytes;
  static LdsLimit limit;
  hipError_t e = raise_lds(reinterpret_cast<const void*>(&sm_one_s2_kernel<TT, ACT, SC>), bytes, limit);
  if (e != hipSuccess) return e;
  e = c == 0 ? one_s1<TT, 0, ACT, SC>(A, n, n1, stream) : one_s1<TT, kOneMaxCls, ACT, SC>(A, n, n1, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((sm_one_r_kernel<nw_of(ACT), SC>), dim3(nr, n), dim3(kThreads), 0, stream, A);
  hipLaunchKernelGGL((sm_one_s2_kernel<TT, ACT, SC>), dim3(n2, n), dim3(kOneThreads), bytes, stream, A);
  return hipGetLastError();
}
template <int ACT, int SC>
hipError_t one_tt(const FewArgs& A, int n, int tt, int c, int n1, int nr, int n2, hipStream_t stream) {
  switch (tt) {
    case 1: return one_launch<1, ACT, SC>(A, n, c, n1, nr, n2, stream);
    case 2: return one_launch<2, ACT, SC>(A, n, c, n1, nr, n2, stream);
    case 3: return one_launch<3, ACT, SC>(A, n, c, n1, nr, n2, stream);
    default: return one_launch<4, ACT, SC>(A, n, c, n1, nr, n2, stream);
  }
}
template <int ACT>
hipError_t one_sc(int sc_dt, const FewArgs& A, int n, int tt, int c, int n1, int nr, int n2, hipStream_t stream) {
  switch (sc_dt) {
    case kDtF32: return one_tt<ACT, kDtF32>(A, n, tt, c, n1, nr, n2, stream);
    case kDtF16: return one_tt<ACT, kDtF16>(A, n, tt, c, n1, nr, n2, stream);
    default: return one_tt<ACT, kDtBF16>(A, n, tt, c, n1, nr, n2, stream);
  }
}

}  // namespace

bool few_tokens_plan(const ForwardArgs& a, size_t ws_bytes, FewPlan& g) {
  if (!stream_mma_supports(a) || !has_work(a) || ws_bytes <= kScratchOff) return false;
  g = one_geometry(a, ws_bytes);
  return g.bpr > 0;
}

hipError_t launch_few_tokens(const ForwardArgs* a, const FewPlan* plans, int n, hipStream_t stream) {
  if (n < 1 || n > kFewMaxBatch) return hipErrorInvalidValue;
  FewArgs A{};
  const int tt = (a[0].T + 15) / 16;
  int c = 0, n1 = 0, nr = 0, n2 = 0;  // the largest tile class and grids
  for (int i = 0; i < n; ++i) {
    if ((a[i].T + 15) / 16 != tt || a[i].act_dt != a[0].act_dt || a[i].sc_dt != a[0].sc_dt) return hipErrorInvalidValue;
    const FewPlan& g = plans[i];
    StreamLinear& L = A.l[i];
    fill_desc(L, a[i], g);
    char* data = static_cast<char*>(a[i].ws) + kScratchOff;
    L.part = reinterpret_cast<float*>(data);
    L.wlat = reinterpret_cast<float*>(data + align256(part_bytes(g)));
    c = std::max(c, g.cls % kMtClasses);
    n1 = std::max(n1, 2 * g.ng * g.s1d);
    nr = std::max(nr, r_items(L.T, L.r) / 64);
    n2 = std::max(n2, (L.d_out + 16 * kWaves - 1) / (16 * kWaves));
  }
  switch (a[0].act_dt) {
    case kDtF32: return one_sc<kDtF32>(a[0].sc_dt, A, n, tt, c, n1, nr, n2, stream);
    case kDtF16: return one_sc<kDtF16>(a[0].sc_dt, A, n, tt, c, n1, nr, n2, stream);
    default: return one_sc<kDtBF16>(a[0].sc_dt, A, n, tt, c, n1, nr, n2, stream);
  }
}

}  // namespace lb
