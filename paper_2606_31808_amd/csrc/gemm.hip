// W4A16 GEMM for gfx950: C = A . deq(W)^T with A fp16 [M][K] (tokens x
// features), W int4 [N][K] with one fp16 scale per 32 input features, fp32
// accumulation on MFMA 16x16x32 f16.  The same body serves FP8 weights (OCP
// E4M3 codes, one fp32 scale per output column: the FP8 checkpoint layout).
// The LM head (fp16 weight) is a kernel of its own at the end of the file.
//
// Tiling.  The packed weight is kept in strips of 16 columns, contiguous
// along K.  A workgroup's waves stand side by side along N; a wave owns all
// 16*MI tokens of the tile and FJ strips, so each weight fragment is
// dequantised once per workgroup and feeds MI MFMAs.  K advances in stages of
// KP panels of 64 features through an LDS ring filled by direct global->LDS
// loads (global_load_lds_dwordx4, 1 KB per wave instruction).
//   A panel: 128-byte rows, 16-byte chunks XOR-swizzled by row so that one
//           fragment load (16 rows) is free of LDS bank conflicts.
//   codes and scales: copied verbatim from the packed layout; lane 16g + c
//           holds the codes of column c, features 8g .. 8g+7 of both halves.
// Each wave dequantises its own weight fragments in registers (nibble |
// 0x6400 = 1024 + u in fp16, minus 1032 gives the exact code, times the fp16
// scale: one rounding).
//
// What bounds it.  A wave issues in order, and on this chip an MFMA of 16
// cycles hides two VALU instructions behind it, no third, and no wait: a loop
// that loads, waits, converts and then multiplies leaves the matrix core idle
// for most of a step unless a second wave fills in (one wave per SIMD: 2,200
// cycles for a step of 64 MFMAs).  So the loop is a software pipeline over
// phases of KK steps of 32 features, in a schedule pinned MFMA by MFMA: while
// the MFMAs of one phase run, the next phase's activation fragments are read
// from LDS into registers and its weight fragments are dequantised, two VALU
// instructions to an MFMA, and the global->LDS loads of a later stage are
// spread over the whole stage (issued in one go they held up a wave for 30 ns
// each).  One barrier per stage, before its last phase: by then every
// fragment of the stage is in registers, so its slot is free, and the next
// stage has landed.  Small tiles have short phases; they take KK > 1 (a phase
// longer than an LDS access) and read codes two phases ahead.
//
// Measured against the loop before (wait, read, convert, multiply; token
// tiles of 128, 64 and 32 rows by 256 columns), same card, weights from
// memory, the shape that the rule picks (up to 16 tokens mostly the kernel for
// few tokens below), us per launch:
//   K = 4096, N = 4096 (O):      9 tokens 36.4 -> 6.5, 60: 37.4 -> 9.8,
//     160: 38.2 -> 17.3, 500: 39.0 -> 25.7, 1000: 52.0 -> 41.4, 2048: 79.8 -> 75.4
//   K = 14336, N = 4096 (down):  9: 120.7 -> 15.0, 60: 122.5 -> 26.1,
//     160: 122.6 -> 51.1, 500: 123.9 -> 77.3, 1000: 162.6 -> 130, 2048: 244 -> 211
//   K = 4096, N = 28672 (gate/up): 9: 36.4 -> 16.1, 60: 38.1 -> 23.3,
//     160: 62.3 -> 54.8, 1000: 201 -> 200, 2048: 382 -> 368, 16384: 2947 -> 2868
// A layer's four projections together are faster at every size measured (1 to
// 16384 tokens, 8B and 1B widths, both formats); single ones of 1,500 to 4,096
// tokens are up to 7% slower (QKV of 1500: 87 -> 91-94, down of 3000: 310 -> 325).
// At 16384 tokens the card's power limit bounds it (1.2-1.4 PFLOP/s on such
// weights; the fp16 library product reaches 1.46).  Below a few hundred tokens
// MFMAs and conversion are less than half of a launch: a 64x128 tile alone on
// a CU takes 330 ns per panel of 16 MFMAs a wave (107 ns) with the VALU mostly
// behind them; what the rest is has not been measured.
//
// The MFMA takes the weight fragment as its A operand and the activations
// as its B operand, so the accumulator holds C^T: every lane owns 4
// consecutive output columns of one token, which makes the epilogue's
// stores 8-byte (fp16) or 16-byte (fp32) vectors.
//
// FP8 weights: twice the int4 bytes per strip.  A lane's 8 codes convert to
// fp16 exactly with four v_cvt_scalef32_pk_f16_fp8 (every E4M3 value is an
// fp16 value); the per-column scale multiplies the fp32 accumulator before
// the epilogue.
//
// Workgroups are mapped to tiles XCD-aware: the hardware deals workgroups to
// the 8 XCDs round-robin, so each XCD is given one contiguous range of
// tiles, ordered in groups of GM token tiles so that concurrently running
// tiles on an XCD share A and W panels in that XCD's L2.
#include "common.h"
#include "gemm_ring.h"
#include "gemm_tiles.h"
#include "kernels.h"
#include "lds_dma.h"

#include <type_traits>
#include <utility>

namespace lmop {

namespace {

// Dequantisation of a word of 8 biased codes to 8 fp16 weights (nibble p
// holds feature 2p for p < 4 and 2(p-4)+1 otherwise), in two halves of three
// steps of two VALU instructions each, which the main loop places between
// MFMAs.  Masking nibbles p and p+4 and or-ing in 0x6400 makes fp16 1024 + u,
// minus 1032 gives the exact code; masking the next nibble pair in place
// makes 1024 + 16u, and one fma by 1/16 with -72 gives the exact code as
// well, so the second half needs one shift by 8.  Times the scale: one
// rounding.  `mask` and `magic` arrive in registers the compiler cannot see
// through, so (x & mask) | magic becomes one v_and_or.
struct DeqTmp {
  uint32_t t0, t1;
  f16x2 h0, h1;
};
template <int STEP>
LMOP_DEVICE void dequant_step(uint32_t w, int half, f16x2 s2, uint32_t mask, uint32_t magic,
                              DeqTmp& d) {
  if constexpr (STEP == 0) {
    const uint32_t x = half ? w >> 8 : w;
    d.t0 = (x & mask) | magic;
    d.t1 = (x & (mask << 4)) | magic;
  } else if constexpr (STEP == 1) {
    d.h0 = __builtin_bit_cast(f16x2, d.t0) - f16x2{(f16)1032.0f, (f16)1032.0f};
    d.h1 = __builtin_elementwise_fma(__builtin_bit_cast(f16x2, d.t1),
                                     f16x2{(f16)0.0625f, (f16)0.0625f},
                                     f16x2{(f16)-72.0f, (f16)-72.0f});
  } else {
    d.h0 = d.h0 * s2;
    d.h1 = d.h1 * s2;
  }
}

// The 4 E4M3 codes of a word (byte 0 first) as fp16, exactly: every E4M3
// value is an fp16 value, so a unit scale changes nothing.
LMOP_DEVICE f16x4 fp8x4(uint32_t d) {
  const f16x2 a = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(d, 1.0f, false);
  const f16x2 b = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(d, 1.0f, true);
  return f16x4{a.x, a.y, b.x, b.y};
}

// fp16 of a product that has first been rounded to fp32: without the empty
// asm the compiler turns some of these into one instruction that rounds once,
// in some tile shapes and not in others
LMOP_DEVICE f16 f16_of(float x) {
  asm("" : "+v"(x));
  return (f16)x;
}

LMOP_DEVICE float silu(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// 16-byte chunk swizzle of a 128-byte LDS row; with it a fragment load (16
// rows x 4 chunks) is free of bank conflicts on gfx950 (measured with the
// SQ_LDS_BANK_CONFLICT counter)
LMOP_DEVICE int swz(int row) { return row & 7; }

constexpr int GM = 4;      // token tiles per L2 group

// weight formats of the kernel's weight operand
constexpr int WF_INT4 = 1;  // int4, one fp16 scale per 32 features
constexpr int WF_FP8 = 2;   // OCP E4M3, one fp32 scale per output column

// ---------------------------------------------------------------- epilogues
// X[m][n .. n+3] += v
LMOP_DEVICE void add_residual(const GemmArgs& p, int m, int n, f32x4 v) {
  if (m >= p.M || n >= p.n_out) return;
  float4* xp = (float4*)(p.X + (size_t)m * p.ldx + n);
  float4 x = *xp;
  x.x += v[0];
  x.y += v[1];
  x.z += v[2];
  x.w += v[3];
  *xp = x;
}

// token m, lane group g: the strips 2 pair, 2 pair + 1 of the packed columns
// (rows 4g .. 4g+3 of each)
template <int EPI>
LMOP_DEVICE void store_pair(const GemmArgs& p, int m, int g, f32x4 x1, f32x4 x2, int pair) {
  if (m >= p.M) return;
  if constexpr (EPI == EPI_SWIGLU) {
    // 16 gate columns and the matching up columns
    const int col = pair * 16 + 4 * g;
    if (col < p.n_out)
      *(f16x4*)((f16*)p.C + (size_t)m * p.ldc + col) =
          f16x4{f16_of(silu(x1[0]) * x2[0]), f16_of(silu(x1[1]) * x2[1]),
                f16_of(silu(x1[2]) * x2[2]), f16_of(silu(x1[3]) * x2[3])};
  } else {
    static_assert(EPI == EPI_QKV, "paired epilogues");
    const int half = p.hd >> 1;
    const int pph = p.hd >> 5;  // strip pairs per head
    const int nqp = p.nq * pph, nkp = p.nkv * pph;
    pair += p.pair0;
    if (pair >= p.pair_end) return;
    const int sec = pair < nqp ? 0 : (pair < nqp + nkp ? 1 : 2);
    const int hp = pair - (sec == 0 ? 0 : (sec == 1 ? nqp : nqp + nkp));
    const int head = hp / pph, sub = hp - head * pph;
    if (sec < 2) {
      const float2* cs = p.rope + (size_t)p.pos[m] * half;
      f16* dst = sec == 0 ? (f16*)p.qout + (size_t)m * p.nq * p.hd + head * p.hd
                          : (f16*)p.kc + (size_t)p.slot[m] * (p.nkv * p.hd) + head * p.hd;
      const int d = 16 * sub + 4 * g;
      const float4 c01 = *(const float4*)(cs + d);
      const float4 c23 = *(const float4*)(cs + d + 2);
      const float cr[4] = {c01.x, c01.z, c23.x, c23.z};
      const float sr[4] = {c01.y, c01.w, c23.y, c23.w};
      f16x4 y1, y2;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        y1[r] = (f16)(x1[r] * cr[r] - x2[r] * sr[r]);
        y2[r] = (f16)(x1[r] * sr[r] + x2[r] * cr[r]);
      }
      *(f16x4*)(dst + d) = y1;
      *(f16x4*)(dst + half + d) = y2;
    } else {
      f16* vt = (f16*)p.vt + (size_t)head * p.hd * p.cap + p.slot[m];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        vt[(size_t)(32 * sub + 4 * g + r) * p.cap] = (f16)x1[r];
        vt[(size_t)(32 * sub + 16 + 4 * g + r) * p.cap] = (f16)x2[r];
      }
    }
  }
}

// Tile of a workgroup: 16*MI tokens x 16*FJ*NW columns, KP panels of 64
// features per ring stage, OCC workgroups per CU; NW waves side by side along
// N, each with all the tokens and FJ strips of 16 columns.
template <int MI, int WF, int FJ, int NW, int KP, int OCC>
struct Cfg {
  static constexpr int BM = 16 * MI, BN = 16 * FJ * NW;
  static constexpr int PANEL = BM * 128;                   // 64 features of BM tokens
  static constexpr int WB = WF == WF_INT4 ? 512 : 1024;    // codes of 16 columns x 64 features
  static constexpr int A_BYTES = KP * PANEL;
  static constexpr int W_WAVE = FJ * KP * WB;              // one wave's codes
  static constexpr int S_WAVE = WF == WF_INT4 ? FJ * KP * 64 : 0;  // and scales
  static constexpr int STAGE = A_BYTES + NW * (W_WAVE + S_WAVE);
  static_assert(STAGE % 128 == 0, "stages keep the alignment the swizzle assumes");
  // int4 residual-add tiles prefetch the residual rows into an unread LDS
  // area (1 KB per wave), only so that they are in the caches by the epilogue
  static constexpr int PF = WF == WF_INT4 && BN <= 256 && MI >= 4 ? 1024 * NW : 0;
  // ring stages: what OCC workgroups' rings leave of a CU's LDS, at most 6
  static constexpr int FIT = (160 * 1024 / OCC - PF) / STAGE;
  static constexpr int NS = FIT < 6 ? FIT : 6;
  static_assert(NS >= 2, "a stage in use and one in flight");
  // with 4 stages or more, a stage has landed one stage before it is used, so
  // that its codes can be read two phases before their fragments are
  static constexpr int AHEAD = NS >= 4 ? 1 : 0;
  static constexpr int LDS = NS * STAGE + PF;
  // global->LDS instructions one wave issues per stage (activations, codes, scales)
  static constexpr int A_INSTR = KP * BM / 8;              // of the workgroup
  static constexpr int A_LOADS = (A_INSTR + NW - 1) / NW;
  static constexpr int W_LOADS = (W_WAVE + 1023) / 1024;
  static constexpr int LOADS = A_LOADS + W_LOADS + (WF == WF_INT4 ? 1 : 0);
  static_assert(LOADS + 1 < 64, "a stage's loads fit the vmcnt counter");
};

// One wave's share of one strip's codes and scales of a 64-feature panel:
// [kk] = the 32-feature half
template <int WF>
struct Codes;
template <>
struct Codes<WF_INT4> {
  uint2 w;
  f16x2 s;
};
template <>
struct Codes<WF_FP8> {
  uint4 w;
};

template <int MI, int WF, int EPI, int FJ, int NW, int KP, int KK, int OCC>
__global__ __launch_bounds__((64 * NW), ((OCC * NW + 3) / 4)) void gemm_kernel(const GemmArgs p) {
  using C = Cfg<MI, WF, FJ, NW, KP, OCC>;
  constexpr int BM = C::BM, BN = C::BN, NS = C::NS;
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  // the wave index is uniform; saying so keeps LDS addresses in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;

  // ---- XCD-aware tile mapping
  const int ntm = (p.M + BM - 1) / BM, ntn = (p.N + BN - 1) / BN;
  const int total = ntm * ntn;
  const int b = blockIdx.x;
  const int xcd = b & 7, j = b >> 3;
  const int per = total >> 3, rem = total & 7;
  const int logical = xcd * per + (xcd < rem ? xcd : rem) + j;
  const int grp = logical / (GM * ntn);
  const int within = logical - grp * GM * ntn;
  const int gsz = (ntm - grp * GM) < GM ? (ntm - grp * GM) : GM;
  const int mt = grp * GM + within % gsz;
  const int nt = within / gsz;
  const int m0 = mt * BM, n0 = nt * BN;

  const int K64 = p.K >> 6;     // 64-feature panels
  const int KT = K64 / KP;      // ring stages
  const f16* A = (const f16*)p.A;
  // stages whose issue also prefetches residual rows (1 KB = RPI rows of the
  // tile per wave); PFW stages cover the tile
  constexpr int RPI = C::PF > 0 ? 256 / BN : 1;
  constexpr int PF_ALL = C::PF > 0 && EPI == EPI_ADD_F32 ? BM / (RPI * NW) : 0;
  const int PFW = KT < PF_ALL ? KT : PF_ALL;

  // ---- global -> LDS issue of one stage; every wave issues exactly C::LOADS
  // instructions, which the vmcnt waits below rely on.  Each load is a base
  // in scalar registers (moved by the stage) plus a per-lane 32-bit byte
  // offset computed once, and an LDS destination in a scalar register.
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)smem;
  uint32_t aoff[C::A_LOADS], woff[C::W_LOADS], soff = 0;
#pragma unroll
  for (int i = 0; i < C::A_LOADS; ++i) {
    int q = wave + NW * i;  // 8 rows of one panel per instruction
    if (q >= C::A_INSTR) q = C::A_INSTR - 1;  // surplus waves repeat the last rows
    const int r = (q % (BM / 8)) * 8 + (lane >> 3);
    const int chunk = (lane & 7) ^ swz(r);
    const int gm = m0 + r < p.M ? r : p.M - 1 - m0;  // row within the tile, clamped
    aoff[i] = (uint32_t)(gm * p.lda + (q / (BM / 8)) * 64 + chunk * 8) * 2u;
  }
  const char* abase = (const char*)(A + (size_t)m0 * p.lda);
  const size_t strip0 = (size_t)(n0 >> 4) + wave * FJ;  // this wave's first strip
  const char* wbase = (const char*)p.bq + strip0 * K64 * C::WB;
  const char* sbase = (const char*)p.bs + strip0 * K64 * 64;
#pragma unroll
  for (int i = 0; i < C::W_LOADS; ++i) {
    const int o = (i * 64 + lane) * 16;  // byte of the wave's codes: [strip][panel][WB]
    const int piece = o / C::WB;
    woff[i] = (uint32_t)(((piece / KP) * K64 + piece % KP) * C::WB + o % C::WB);
  }
  if constexpr (WF == WF_INT4) {
    const int piece = lane >> 2;
    soff = (uint32_t)(((piece / KP) * K64 + piece % KP) * 64 + (lane & 3) * 16);
  }
  // instruction n of a stage's loads: activations, codes, scales
  auto issue_one = [&](int n, uint32_t sA, int kt) {
    if (n < C::A_LOADS) {
      int q = wave + NW * n;
      if (q >= C::A_INSTR) q = C::A_INSTR - 1;
      g2l16_m0(abase + (size_t)kt * (KP * 128), aoff[n], sA + (uint32_t)q * 1024u);
    } else if (n < C::A_LOADS + C::W_LOADS) {
      const int i = n - C::A_LOADS;
      const uint32_t sW = sA + C::A_BYTES + (uint32_t)(wave * C::W_WAVE) + (uint32_t)i * 1024u;
      if (C::W_WAVE >= (i + 1) * 1024)
        g2l16_m0(wbase + (size_t)kt * (KP * C::WB), woff[i], sW);
      else
        g2l16_m0_lanes<(C::W_WAVE % 1024) / 16>(wbase + (size_t)kt * (KP * C::WB), woff[i], sW);
    } else if constexpr (WF == WF_INT4) {
      const uint32_t sS = sA + C::A_BYTES + NW * C::W_WAVE + (uint32_t)(wave * C::S_WAVE);
      g2l16_m0_lanes<C::S_WAVE / 16>(sbase + (size_t)kt * (KP * 64), soff, sS);
    }
  };
  // residual rows for the epilogue, after a stage's own loads so the waits
  // below can count them
  auto issue_pf = [&](int kt) {
    if constexpr (PF_ALL > 0) {
      if (kt >= KT - PFW) {
        const int r = ((kt - (KT - PFW)) * NW + wave) * RPI + lane / (BN / 4);
        int gm = m0 + (r < BM ? r : BM - 1);
        gm = gm < p.M ? gm : p.M - 1;
        int col = n0 + (lane % (BN / 4)) * 4;
        col = col + 4 <= p.n_out ? col : p.n_out - 4;
        g2l16_m0((const char*)(p.X + (size_t)m0 * p.ldx), (uint32_t)((gm - m0) * p.ldx + col) * 4u,
                 lds0 + (uint32_t)(NS * C::STAGE + wave * 1024));
      }
    }
  };

  // dequant constants kept opaque to the optimiser (see dequant_step)
  uint32_t dq_mask = 0x000F000Fu, dq_magic = 0x64006400u;
  asm volatile("" : "+s"(dq_mask));
  asm volatile("" : "+v"(dq_magic));

  f32x4 acc[FJ][MI];
#pragma unroll
  for (int f = 0; f < FJ; ++f)
#pragma unroll
    for (int i = 0; i < MI; ++i) acc[f][i] = f32x4{0.f, 0.f, 0.f, 0.f};

  // ---- software pipeline over phases of 32 features.  While the MFMAs of
  // one phase run, the next phase's activation fragments are read from LDS
  // and its weight fragments are dequantised.
  const uint32_t a_lane[2] = {(uint32_t)(c * 128 + ((g ^ swz(c)) * 16)),
                              (uint32_t)(c * 128 + (((4 + g) ^ swz(c)) * 16))};
  const uint32_t w_lane = (uint32_t)(C::A_BYTES + wave * C::W_WAVE + lane * (C::WB / 64));
  const uint32_t s_lane = (uint32_t)(C::A_BYTES + NW * C::W_WAVE + wave * C::S_WAVE + c * 4);
  // token group i of the stage's 32-feature step ks
  auto read_a = [&](uint32_t st, int ks, int i) {
    return *(const f16x8*)(smem + st + a_lane[ks & 1] + (ks >> 1) * C::PANEL + i * 2048);
  };
  auto read_codes = [&](uint32_t st, int panel, Codes<WF>* cd) {
#pragma unroll
    for (int f = 0; f < FJ; ++f) {
      if constexpr (WF == WF_INT4) {
        cd[f].w = *(const uint2*)(smem + st + w_lane + (f * KP + panel) * C::WB);
        cd[f].s = *(const f16x2*)(smem + st + s_lane + (f * KP + panel) * 64);
      } else {
        cd[f].w = *(const uint4*)(smem + st + w_lane + (f * KP + panel) * C::WB);
      }
    }
  };
  constexpr int PH = 2 * KP / KK;      // phases of a stage, KK steps of 32 features each
  constexpr int SLOTS = KK * MI * FJ;  // MFMAs of a phase
  constexpr int LOADS = C::LOADS, AHEAD = C::AHEAD;
  static_assert((2 * KP) % KK == 0 && PH >= 2, "a stage is freed while its last phase runs");
  // panels whose codes a phase needs (with KK = 1 two phases share a panel)
  constexpr int NPC = KK == 1 ? 1 : KK / 2;
  // dequantisation of one phase's KK * FJ weight fragments in DP pieces of
  // about two VALU instructions; step0 = the phase's first step in its stage
  constexpr int PW = WF == WF_INT4 ? 6 : 4;  // pieces per fragment
  constexpr int DP = PW * FJ * KK;
  DeqTmp dt;
  auto deq = [&](int n, const Codes<WF>* cds, int step0, f16x8* wv) {
    const int fi = n / PW, q = n % PW;
    const int half_k = (step0 + fi / FJ) & 1;
    const Codes<WF>& cf = cds[(KK == 1 ? 0 : fi / FJ / 2) * FJ + fi % FJ];
    f16x8& o = wv[fi];
    if constexpr (WF == WF_INT4) {
      const uint32_t word = half_k ? cf.w.y : cf.w.x;
      const f16x2 s2 = half_k ? __builtin_shufflevector(cf.s, cf.s, 1, 1)
                              : __builtin_shufflevector(cf.s, cf.s, 0, 0);
      const int half = q / 3;
      if (q % 3 == 0) dequant_step<0>(word, half, s2, dq_mask, dq_magic, dt);
      if (q % 3 == 1) dequant_step<1>(word, half, s2, dq_mask, dq_magic, dt);
      if (q % 3 == 2) {
        dequant_step<2>(word, half, s2, dq_mask, dq_magic, dt);
        if (half == 0)
          o = f16x8{dt.h0.x, dt.h0.y, dt.h1.x, dt.h1.y, 0, 0, 0, 0};
        else
          o = f16x8{o[0], o[1], o[2], o[3], dt.h0.x, dt.h0.y, dt.h1.x, dt.h1.y};
      }
    } else {
      const uint32_t word =
          half_k ? (q >> 1 ? cf.w.w : cf.w.z) : (q >> 1 ? cf.w.y : cf.w.x);
      const f16x2 v = (q & 1) ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(word, 1.0f, true)
                              : __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(word, 1.0f, false);
      if (q == 0) o = f16x8{v.x, v.y, 0, 0, 0, 0, 0, 0};
      if (q == 1) o = f16x8{o[0], o[1], v.x, v.y, 0, 0, 0, 0};
      if (q == 2) o = f16x8{o[0], o[1], o[2], o[3], v.x, v.y, 0, 0};
      if (q == 3) o = f16x8{o[0], o[1], o[2], o[3], o[4], o[5], v.x, v.y};
    }
  };
  // A stage's loads are issued over the PH phases that follow the barrier
  // that frees its slot, evenly (issued at once they hold up the MFMAs): load
  // n goes with slot n * TS / LOADS of those phases' TS slots.
  constexpr int TS = PH * SLOTS;
  auto issue_part = [&](int at, uint32_t st, int kt) {
#pragma unroll
    for (int n = (at * LOADS + TS - 1) / TS; n < ((at + 1) * LOADS + TS - 1) / TS; ++n)
      issue_one(n, lds0 + st, kt);
    if (at == TS - 1) issue_pf(kt);
  };

#pragma unroll
  for (int st = 0; st < NS - 1; ++st)
    if (st < KT) {
#pragma unroll
      for (int n = 0; n < LOADS; ++n) issue_one(n, lds0 + (uint32_t)(st * C::STAGE), st);
      issue_pf(st);
    }
  // a PF load more per stage only waits for more than is needed here
  if (KT >= NS - 1)
    wait_vmcnt<(NS - 2 - AHEAD) * LOADS>();
  else
    wait_vmcnt<0>();
  barrier();
  // cd: codes of the phase dequantised next, cdn: of the one after it
  Codes<WF> cd[NPC * FJ], cdn[NPC * FJ];
  f16x8 a[KK * MI], w[KK * FJ];
  // codes of phase ph (KK >= 2), or of phase ph's panel
  auto read_phase_codes = [&](uint32_t st, int ph, Codes<WF>* c_) {
#pragma unroll
    for (int q = 0; q < NPC; ++q) read_codes(st, KK == 1 ? ph / 2 : ph * NPC + q, c_ + q * FJ);
  };
  read_phase_codes(0, 0, cd);
#pragma unroll
  for (int r = 0; r < KK * MI; ++r) a[r] = read_a(0, r / MI, r % MI);
  if (AHEAD && KK > 1) read_phase_codes(0, 1, cdn);
#pragma unroll
  for (int n = 0; n < DP; ++n) deq(n, cd, 0, w);
  if (NS - 1 < KT) {
#pragma unroll
    for (int sl = 0; sl < SLOTS; ++sl) issue_part(sl, (uint32_t)((NS - 1) * C::STAGE), NS - 1);
  }
  uint32_t st_cur = 0, st_prev = (uint32_t)((NS - 1) * C::STAGE);  // byte offsets of stages
  // MORE: 2 = stages kt + NS - 1 and kt + NS exist, 1 = only the first, 0 = neither
  auto stage = [&](int kt, auto more_) {
    constexpr int MORE = decltype(more_)::value;
    const uint32_t st_next = st_cur + C::STAGE == NS * C::STAGE ? 0u : st_cur + C::STAGE;
#pragma unroll
    for (int ph = 0; ph < PH; ++ph) {
      const bool last = ph == PH - 1;
      if (last && (MORE || kt + 1 < KT)) {
        // every fragment of this stage is in registers, so its slot is free
        // once all waves are here; stage kt + 1 + AHEAD has landed once at
        // most the later ones are in flight
        if (MORE) {
          constexpr int FLY = NS - 2 - AHEAD;
          if (PF_ALL > 0 && all_carry_prefetch(kt + NS - 1, FLY, KT, PFW))
            wait_vmcnt_lgkm0<FLY * (LOADS + 1)>();
          else
            wait_vmcnt_lgkm0<FLY * LOADS>();
        } else {
          wait_vmcnt_lgkm0<0>();
        }
        barrier();
      }
      const uint32_t nst = last ? st_next : st_cur;
      const int nph = last ? 0 : ph + 1;  // the next phase
      f16x8 an[KK * MI], wn[KK * FJ];
      if constexpr (KK == 1) {
        if (AHEAD && (nph & 1) == 1)  // the next phase but one's codes
          read_phase_codes(ph == PH - 2 ? st_next : st_cur, ph == PH - 2 ? 0 : ph + 2, cdn);
        if (AHEAD && (nph & 1) == 0)
#pragma unroll
          for (int f = 0; f < FJ; ++f) cd[f] = cdn[f];
        if (!AHEAD && (nph & 1) == 0) read_phase_codes(nst, nph, cd);
      } else if constexpr (AHEAD) {
#pragma unroll
        for (int q = 0; q < NPC * FJ; ++q) cd[q] = cdn[q];
        read_phase_codes(ph + 2 >= PH ? st_next : st_cur, (ph + 2) % PH, cdn);
      } else {
        read_phase_codes(nst, nph, cd);
      }
      constexpr int R = KK * MI;  // activation fragments of a phase
      an[0] = read_a(nst, nph * KK, 0);
      if constexpr (R > 1) an[1] = read_a(nst, nph * KK + 1 / MI, 1 % MI);
      __builtin_amdgcn_sched_barrier(0);
      // the phase's slots: one MFMA, then a share of the next phase's reads,
      // of its dequantisation (not before its codes can have arrived) and of
      // a later stage's loads
      const int skip = (KK > 1 || (nph & 1) == 0) && !AHEAD ? (SLOTS >= 16 ? 6 : SLOTS / 4) : 0;
#pragma unroll
      for (int sl = 0; sl < SLOTS; ++sl) {
        const int r = sl / FJ, f = sl % FJ;
        acc[f][r % MI] = mfma16x16x32(w[(r / MI) * FJ + f], a[r], acc[f][r % MI]);
        if (f == FJ - 1 && r + 2 < R)
          an[r + 2] = read_a(nst, nph * KK + (r + 2) / MI, (r + 2) % MI);
        const int d0 = sl < skip ? 0 : (sl - skip) * DP / (SLOTS - skip);
        const int d1 = sl < skip ? 0 : (sl + 1 - skip) * DP / (SLOTS - skip);
#pragma unroll
        for (int n = d0; n < d1; ++n) {
          deq(n, cd, nph * KK, wn);
          if ((n + 1) % PW == 0)  // computed here, not where it is used
            asm volatile("" : "+v"(wn[n / PW]));
        }
        if (MORE == 2 && last) issue_part(sl, st_cur, kt + NS);
        if (MORE >= 1 && !last) issue_part((ph + 1) * SLOTS + sl, st_prev, kt + NS - 1);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) a[r] = an[r];
#pragma unroll
      for (int q = 0; q < KK * FJ; ++q) w[q] = wn[q];
    }
    st_prev = st_cur;
    st_cur = st_next;
  };
  int kt = 0;
  for (; kt + NS < KT; ++kt) stage(kt, std::integral_constant<int, 2>{});
  if (kt + NS - 1 < KT) stage(kt++, std::integral_constant<int, 1>{});
  for (; kt < KT; ++kt) stage(kt, std::integral_constant<int, 0>{});

  // ------------------------------------------------------------ epilogue
  // acc[f][i][r] = C[m][n], m = m0 + 16i + c, n = ncol + 16f + r
  const int mrow = m0 + c;
  const int ncol = n0 + wave * 16 * FJ + 4 * g;
  if constexpr (WF == WF_FP8) {
    // the FP8 weight's per-column scale
#pragma unroll
    for (int f = 0; f < FJ; ++f) {
      const float4 sc = *(const float4*)(p.bsc + ncol + 16 * f);
#pragma unroll
      for (int i = 0; i < MI; ++i) acc[f][i] = acc[f][i] * f32x4{sc.x, sc.y, sc.z, sc.w};
    }
  }
  if constexpr (EPI == EPI_ADD_F32) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int f = 0; f < FJ; ++f) add_residual(p, mrow + 16 * i, ncol + 16 * f, acc[f][i]);
  } else {
    // strips 2t, 2t + 1 belong together: f(i, x1, x2, pair) with pair = their
    // index in the packed columns.  With one strip per wave, waves 2t and
    // 2t + 1 swap accumulators through the ring's LDS and share the tokens.
    auto for_pairs = [&](auto&& fn) {
      const int pair0 = (n0 >> 5) + (wave * FJ >> 1);
      if constexpr (FJ == 1) {
        static_assert(FJ > 1 || NW * MI * 1024 <= C::LDS, "the accumulators fit the ring");
        f32x4* ex = (f32x4*)smem;
        // the ring's last reads are done in every wave, and no load is in flight
        wait_vmcnt_lgkm0<0>();
        barrier();
#pragma unroll
        for (int i = 0; i < MI; ++i) ex[(wave * MI + i) * 64 + lane] = acc[0][i];
        wait_vmcnt_lgkm0<0>();
        barrier();
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          if (MI > 1 ? (i & 1) != (wave & 1) : (wave & 1) != 0) continue;
          const f32x4 o = ex[((wave ^ 1) * MI + i) * 64 + lane];
          const bool odd = (wave & 1) != 0;
          fn(i, odd ? o : acc[0][i], odd ? acc[0][i] : o, pair0);
        }
      } else {
#pragma unroll
        for (int t = 0; t < FJ / 2; ++t)
#pragma unroll
          for (int i = 0; i < MI; ++i) fn(i, acc[2 * t][i], acc[2 * t + 1][i], pair0 + t);
      }
    };
    for_pairs([&](int i, f32x4 x1, f32x4 x2, int pair) {
      store_pair<EPI>(p, mrow + 16 * i, g, x1, x2, pair);
    });
  }
}

// ---------------------------------------------------------------- few tokens
// The same product for few tokens, where dequantising is most of the work and
// the strips alone do not fill the SIMDs (256 strips for N = 4096): a
// workgroup of 16 tokens x FJ strips has 3 waves that only issue loads (a
// wave that also converts is held up by each load), 8 that dequantise a
// share of each stage's weight fragments each into LDS, and one that only
// multiplies (in the same order as above).
// One barrier per stage of KP panels: while stage kt is multiplied, stage
// kt + 1 is converted and later ones are loaded.
// Measured at 9 tokens (us, against the best shape of gemm_kernel): K 4096, N
// 4096 9.8 -> 6.8; K 14336 24.3 -> 14.8; QKV (K 4096, N 6144) 9.8 -> 8.2.  A
// stage of 512 features takes about 1,000 cycles: the converters' read,
// convert and write chain and the barrier, then LDS traffic.
template <int WF, int FJ, int KP>
struct SplitCfg {
  static constexpr int BM = 16, BN = 16 * FJ, NP = 8, NLA = 2;
  static constexpr int WAVES = 1 + NLA + NP + 1;
  static constexpr int PANEL = BM * 128;
  static constexpr int WB = WF == WF_INT4 ? 512 : 1024;
  static constexpr int A_BYTES = KP * PANEL, C_BYTES = FJ * KP * WB;
  // codes, then scales (FJ * KP * 64 bytes, padded to a load of 1 KB)
  static constexpr int W_BYTES = C_BYTES + (WF == WF_INT4 ? 1024 : 0);
  static constexpr int FRAGS = 2 * FJ * KP;  // weight fragments (1 KB) of a stage
  static constexpr int FB = FRAGS * 1024;
  // load instructions of a stage
  static constexpr int A_LOADS = A_BYTES / 1024 / NLA, W_LOADS = W_BYTES / 1024;  // of a loader
  static_assert(A_BYTES % (1024 * NLA) == 0, "the same for every loader");
  // A ring of activation stages (from L2) and a deeper one of weight stages
  // (from memory: with three stages in flight its latency of about 1.6 us was
  // the whole time of a stage)
  static constexpr int NSA = 4;
  static constexpr int FIT = (160 * 1024 - 2 * FB - NSA * A_BYTES) / W_BYTES;
  static constexpr int CNT = 63 / W_LOADS + 1;  // loads in flight fit the vmcnt counter
  static constexpr int NSW = FIT < CNT ? (FIT < 12 ? FIT : 12) : (CNT < 12 ? CNT : 12);
  static_assert(NSW >= 4 && (NSA - 2) * A_LOADS < 64 && (NSW - 1) * W_LOADS < 64, "rings");
  static_assert(FJ * KP * 64 <= 1024 && FRAGS % (2 * NP) == 0, "whole panels per converter");
  static constexpr int LDS = NSA * A_BYTES + NSW * W_BYTES + 2 * FB;
};

// waits until at most n stages of L loads each are in flight (n <= MAX)
template <int L, int MAX>
LMOP_DEVICE void wait_stages(int n) {
  if constexpr (MAX == 0) {
    wait_vmcnt<0>();
  } else {
    if (n >= MAX)
      wait_vmcnt<MAX * L>();
    else
      wait_stages<L, MAX - 1>(n);
  }
}

template <int WF, int EPI, int FJ, int KP>
__global__ __launch_bounds__((64 * SplitCfg<WF, FJ, KP>::WAVES), 3) void gemm_split_kernel(const GemmArgs p) {
  using C = SplitCfg<WF, FJ, KP>;
  constexpr int BM = C::BM, BN = C::BN, NP = C::NP, NLA = C::NLA, NSA = C::NSA, NSW = C::NSW;
  static_assert(EPI == EPI_ADD_F32 || FJ % 2 == 0, "pairs in one wave");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  // XCD-aware tile order as in gemm_kernel
  const int ntm = (p.M + BM - 1) / BM, ntn = p.N / BN;
  const int total = ntm * ntn;
  const int b = blockIdx.x;
  const int xcd = b & 7, j = b >> 3;
  const int per = total >> 3, rem = total & 7;
  const int logical = xcd * per + (xcd < rem ? xcd : rem) + j;
  const int grp = logical / (GM * ntn);
  const int within = logical - grp * GM * ntn;
  const int gsz = (ntm - grp * GM) < GM ? (ntm - grp * GM) : GM;
  const int mt = grp * GM + within % gsz;
  const int nt = within / gsz;
  const int m0 = mt * BM, n0 = nt * BN;
  const int K64 = p.K >> 6, KT = K64 / KP;
  char* const wring = smem + NSA * C::A_BYTES;
  char* const fb = wring + NSW * C::W_BYTES;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)smem;

  if (wave == 0) {
    // ---- loader of the weight stages
    const size_t strip0 = (size_t)(n0 >> 4);
    constexpr int CL = C::C_BYTES / 1024;  // loads of codes
    uint32_t voff[C::W_LOADS];
#pragma unroll
    for (int n = 0; n < C::W_LOADS; ++n) {
      if (n < CL) {
        const int o = (n * 64 + lane) * 16;  // [strip][panel][WB]
        const int piece = o / C::WB;
        voff[n] = (uint32_t)(((piece / KP) * K64 + piece % KP) * C::WB + o % C::WB);
      } else {
        // scales; lanes past them repeat the last piece into the padding
        const int piece = (lane >> 2) < FJ * KP ? lane >> 2 : FJ * KP - 1;
        voff[n] = (uint32_t)(((piece / KP) * K64 + piece % KP) * 64 + (lane & 3) * 16);
      }
    }
    const char* qb = (const char*)p.bq + strip0 * K64 * C::WB;
    const char* sb = (const char*)p.bs + strip0 * K64 * 64;
    auto issue = [&](int slot, int kt) {
      const uint32_t d = lds0 + (uint32_t)(NSA * C::A_BYTES + slot * C::W_BYTES);
#pragma unroll
      for (int n = 0; n < C::W_LOADS; ++n)
        g2l16_m0(n < CL ? qb + (size_t)kt * (KP * C::WB) : sb + (size_t)kt * (KP * 64), voff[n],
                 d + (uint32_t)n * 1024u);
    };
    const int first = NSW < KT ? NSW : KT;
    for (int st = 0; st < first; ++st) issue(st, st);
    wait_stages<C::W_LOADS, NSW - 1>(first - 1);  // stage 0
    barrier();
    wait_stages<C::W_LOADS, NSW - 1>(first - 2);  // stage 1
    int slot = 0;
    for (int kt = 0; kt < KT; ++kt) {
      // stage kt is converted, so its slot is free
      barrier();
      if (kt + NSW < KT) issue(slot, kt + NSW);
      // stage kt + 2, with those up to kt + NSW in flight
      const int issued = kt + NSW < KT ? kt + NSW : KT - 1;
      wait_stages<C::W_LOADS, NSW - 2>(issued - (kt + 2));
      slot = slot == NSW - 1 ? 0 : slot + 1;
    }
    return;
  }
  if (wave <= NLA) {
    // ---- loader of a share of the activation stages
    uint32_t voff[C::A_LOADS];
#pragma unroll
    for (int n = 0; n < C::A_LOADS; ++n) {
      const int q = (wave - 1) * C::A_LOADS + n;
      const int r = (q % (BM / 8)) * 8 + (lane >> 3);  // 8 rows of panel q / (BM / 8)
      const int gm = m0 + r < p.M ? r : p.M - 1 - m0;
      voff[n] = (uint32_t)(gm * p.lda + (q / (BM / 8)) * 64 + ((lane & 7) ^ swz(r)) * 8) * 2u;
    }
    const char* ab = (const char*)((const f16*)p.A + (size_t)m0 * p.lda);
    auto issue = [&](int slot, int kt) {
#pragma unroll
      for (int n = 0; n < C::A_LOADS; ++n)
        g2l16_m0(ab + (size_t)kt * (KP * 128), voff[n],
                 lds0 + (uint32_t)(slot * C::A_BYTES + ((wave - 1) * C::A_LOADS + n) * 1024));
    };
    const int first = NSA - 1 < KT ? NSA - 1 : KT;
    for (int st = 0; st < first; ++st) issue(st, st);
    barrier();
    wait_stages<C::A_LOADS, NSA - 2>(first - 1);  // stage 0
    int slot = NSA - 1;
    for (int kt = 0; kt < KT; ++kt) {
      // stage kt - 1 is multiplied, so its slot is free
      barrier();
      if (kt + NSA - 1 < KT) issue(slot, kt + NSA - 1);
      // stage kt + 1, with those up to kt + NSA - 1 in flight
      const int issued = kt + NSA - 1 < KT ? kt + NSA - 1 : KT - 1;
      wait_stages<C::A_LOADS, NSA - 2>(issued - (kt + 1));
      slot = slot == NSA - 1 ? 0 : slot + 1;
    }
    return;
  }
  if (wave < 1 + NLA + NP) {
    // ---- converter
    const int cw = wave - 1 - NLA;
    uint32_t dq_mask = 0x000F000Fu, dq_magic = 0x64006400u;
    asm volatile("" : "+s"(dq_mask));
    asm volatile("" : "+v"(dq_magic));
    // (strip, panel) pairs cw, cw + NP, ...: both fragments of the panel
    auto convert = [&](uint32_t st, int buf) {
      constexpr int Q = C::FRAGS / 2 / NP;
      uint4 w[Q];
      f16x2 sc[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int piece = cw + NP * q;
        const char* src = wring + st + piece * C::WB + lane * (C::WB / 64);
        if constexpr (WF == WF_INT4) {
          const uint2 x = *(const uint2*)src;
          w[q] = make_uint4(x.x, x.y, 0u, 0u);
          sc[q] = *(const f16x2*)(wring + st + C::C_BYTES + piece * 64 + c * 4);
        } else {
          w[q] = *(const uint4*)src;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        char* out = fb + buf * C::FB + (cw + NP * q) * 2048 + lane * 16;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          f16x8 v;
          if constexpr (WF == WF_INT4) {
            const f16x2 s2 = kk ? __builtin_shufflevector(sc[q], sc[q], 1, 1)
                                : __builtin_shufflevector(sc[q], sc[q], 0, 0);
            const uint32_t word = kk ? w[q].y : w[q].x;
            DeqTmp d0, d1;
            dequant_step<0>(word, 0, s2, dq_mask, dq_magic, d0);
            dequant_step<0>(word, 1, s2, dq_mask, dq_magic, d1);
            dequant_step<1>(word, 0, s2, dq_mask, dq_magic, d0);
            dequant_step<1>(word, 1, s2, dq_mask, dq_magic, d1);
            dequant_step<2>(word, 0, s2, dq_mask, dq_magic, d0);
            dequant_step<2>(word, 1, s2, dq_mask, dq_magic, d1);
            v = f16x8{d0.h0.x, d0.h0.y, d0.h1.x, d0.h1.y, d1.h0.x, d1.h0.y, d1.h1.x, d1.h1.y};
          } else {
            const uint32_t lo = kk ? w[q].z : w[q].x, hi = kk ? w[q].w : w[q].y;
            const f16x2 x0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 1.0f, false);
            const f16x2 x1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 1.0f, true);
            const f16x2 x2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 1.0f, false);
            const f16x2 x3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 1.0f, true);
            v = f16x8{x0.x, x0.y, x1.x, x1.y, x2.x, x2.y, x3.x, x3.y};
          }
          *(f16x8*)(out + kk * 1024) = v;
        }
      }
    };
    barrier();
    convert(0u, 0);
    uint32_t st_next = C::W_BYTES;
    for (int kt = 0; kt < KT; ++kt) {
      wait_vmcnt_lgkm0<0>();  // stage kt's fragments are written
      barrier();
      if (kt + 1 < KT) convert(st_next, (kt + 1) & 1);
      st_next = st_next + C::W_BYTES == NSW * C::W_BYTES ? 0u : st_next + C::W_BYTES;
    }
    return;
  }

  // ---- consumer
  const uint32_t a_lane[2] = {(uint32_t)(c * 128 + ((g ^ swz(c)) * 16)),
                              (uint32_t)(c * 128 + (((4 + g) ^ swz(c)) * 16))};
  f32x4 acc[FJ];
#pragma unroll
  for (int f = 0; f < FJ; ++f) acc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  barrier();
  uint32_t st = 0;
  for (int kt = 0; kt < KT; ++kt) {
    barrier();
    const char* fr = fb + (kt & 1) * C::FB + lane * 16;
    // (strip f, panel)'s fragments are at ((f * KP + panel) * 2 + kk) KB
    f16x8 a[2 * KP], w[2 * KP][FJ];
#pragma unroll
    for (int ks = 0; ks < 2 * KP; ++ks) {
#pragma unroll
      for (int f = 0; f < FJ; ++f)
        w[ks][f] = *(const f16x8*)(fr + ((f * KP + (ks >> 1)) * 2 + (ks & 1)) * 1024);
      a[ks] = *(const f16x8*)(smem + st + a_lane[ks & 1] + (ks >> 1) * C::PANEL);
    }
    // all reads before the first MFMA (the compiler would read, wait and
    // multiply step by step)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2 * KP; ++ks)
#pragma unroll
      for (int f = 0; f < FJ; ++f) acc[f] = mfma16x16x32(w[ks][f], a[ks], acc[f]);
    wait_vmcnt_lgkm0<0>();  // this stage is read, also where an MFMA was moved past the barrier
    st = st + C::A_BYTES == NSA * C::A_BYTES ? 0u : st + C::A_BYTES;
  }
  const int m = m0 + c, ncol = n0 + 4 * g;
  if constexpr (WF == WF_FP8) {
#pragma unroll
    for (int f = 0; f < FJ; ++f) {
      const float4 sc = *(const float4*)(p.bsc + ncol + 16 * f);
      acc[f] = acc[f] * f32x4{sc.x, sc.y, sc.z, sc.w};
    }
  }
  if constexpr (EPI == EPI_ADD_F32) {
#pragma unroll
    for (int f = 0; f < FJ; ++f) add_residual(p, m, ncol + 16 * f, acc[f]);
  } else {
#pragma unroll
    for (int t = 0; t < FJ / 2; ++t)
      store_pair<EPI>(p, m, g, acc[2 * t], acc[2 * t + 1], (n0 >> 5) + t);
  }
}

template <int WF, int EPI, int FJ, int KP>
hipError_t launch_split(hipStream_t s, const GemmArgs& a) {
  using C = SplitCfg<WF, FJ, KP>;
  const int tiles = ((a.M + C::BM - 1) / C::BM) * (a.N / C::BN);
  if (tiles == 0) return hipSuccess;
  static const hipError_t attr = hipFuncSetAttribute(
      (const void*)gemm_split_kernel<WF, EPI, FJ, KP>,
      hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((gemm_split_kernel<WF, EPI, FJ, KP>), dim3(tiles),
                     dim3(64 * C::WAVES), C::LDS, s, a);
  return hipGetLastError();
}
template <int MI, int WF, int EPI, int FJ, int NW, int KP, int KK, int OCC>
hipError_t launch_cfg(hipStream_t s, const GemmArgs& a) {
  using C = Cfg<MI, WF, FJ, NW, KP, OCC>;
  const int tiles = ((a.M + C::BM - 1) / C::BM) * ((a.N + C::BN - 1) / C::BN);
  if (tiles == 0) return hipSuccess;
  // set once per instantiation (a function-local static is initialised once,
  // also when several threads launch)
  static const hipError_t attr = hipFuncSetAttribute(
      (const void*)gemm_kernel<MI, WF, EPI, FJ, NW, KP, KK, OCC>,
      hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((gemm_kernel<MI, WF, EPI, FJ, NW, KP, KK, OCC>), dim3(tiles), dim3(64 * NW), C::LDS, s,
                     a);
  return hipGetLastError();
}

template <int WF, int EPI, int I>
hipError_t launch_tile(hipStream_t s, const GemmArgs& a) {
  constexpr GemmTile t = kGemmTiles[I];
  if constexpr (!t.offered(WF == WF_FP8, EPI == EPI_ADD_F32))
    return hipErrorInvalidValue;  // never picked
  else if constexpr (t.kk == 0)
    return launch_split<WF, EPI, t.fj, t.kp>(s, a);
  else
    return launch_cfg<t.mi, WF, EPI, t.fj, t.nw, t.kp, t.kk, t.occ>(s, a);
}

template <int WF, int EPI, int... I>
hipError_t launch_picked(hipStream_t s, const GemmArgs& a, std::integer_sequence<int, I...>) {
  const int pick = pick_gemm_tile(WF == WF_FP8, EPI == EPI_ADD_F32, a.M, a.N, a.K);
  hipError_t e = hipErrorInvalidValue;
  (void)((pick == I && (e = launch_tile<WF, EPI, I>(s, a), true)) || ...);
  return e;
}

template <int WF, int EPI>
hipError_t launch_epi(hipStream_t s, const GemmArgs& a) {
  return launch_picked<WF, EPI>(s, a, std::make_integer_sequence<int, kNumGemmTiles>{});
}

// ---------------------------------------------------------------- LM head
// 16-byte chunk swizzle of a 64-byte LDS row: the 8 lanes a ds_read_b128
// serves together (rows c .. c+7 of a fragment, one chunk) fall on 8
// distinct 16-byte bank groups of a 128-byte window
LMOP_DEVICE int swz64(int row) { return (row >> 1) & 3; }

// ---------------------------------------------------------------- LM head
// z = W_lm . h for R token rows: the head weight W_lm fp16 (tiled, see
// kHeadTileRows) is the vocabulary operand (M), the final-normalised rows h
// fp16 [R][K] the token operand (N); both stream through an LDS ring by
// direct global->LDS loads, 32 features per step in 64-byte LDS rows.  A
// workgroup of 8 waves holds two vocabulary tiles (256 rows) and 64*F token
// rows: wave w computes vocabulary tile w / 4 of the pair for token-row
// group w % 4 (16*F rows).  The two tiles share the token rows in LDS, so
// token rows cross from L2 once per 256 vocabulary rows, and one workgroup
// per CU affords a ring of NS stages (four: three steps of loads in flight).
// Per token and 128-entry vocabulary chunk the epilogue writes (max, sum
// exp) and the allowed tokens' logits; the chunking never depends on the
// tile or the number of rows, so a row's log-probabilities do not depend on
// how rows are batched.  (One 128-row vocabulary tile per 4-wave workgroup,
// two workgroups per CU, ran 12-14% longer; token rows loaded straight into
// registers ran ~35% longer than through the ring.)
template <int F_, int NS_>
struct Head2Cfg {
  static constexpr int F = F_, NS = NS_, NW = 8, BK = 32, MI = 8;
  static constexpr int BM = 2 * kHeadTileRows, BN = 4 * 16 * F;
  static constexpr int A_BYTES = BM * 64, T_BYTES = BN * 64;
  static constexpr int STAGE = A_BYTES + T_BYTES;
  static constexpr int LDS = NS * STAGE;
  static_assert(NS >= 2 && LDS <= 160 * 1024, "LDS of one CU");
  static constexpr int T_BLOCKS = BN / 16;
  static constexpr int T_MAX = (T_BLOCKS + NW - 1) / NW;  // token blocks of the first waves
  static constexpr int T_FULL = T_BLOCKS % NW == 0 ? NW : T_BLOCKS % NW;  // waves with T_MAX
  static constexpr int LOADS_HI = 2 + T_MAX, LOADS_LO = 2 + T_MAX - 1;
  static_assert((NS - 2) * LOADS_HI <= 63, "loads in flight fit the vmcnt counter");
};

template <int F, int NS_>
__global__ __launch_bounds__(512, 1) void head2_kernel(const GemmArgs p) {
  using C = Head2Cfg<F, NS_>;
  constexpr int BK = C::BK, BM = C::BM, BN = C::BN, NS = C::NS, MI = C::MI;
  constexpr int A_BYTES = C::A_BYTES, STAGE = C::STAGE;
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int half = wave >> 2, grp_t = wave & 3;

  // XCD-aware tile order as in gemm_kernel
  const int ntm = (p.M + BM - 1) / BM, ntn = (p.N + BN - 1) / BN;
  const int total = ntm * ntn;
  const int b = blockIdx.x;
  const int xcd = b & 7, j = b >> 3;
  const int per = total >> 3, rem = total & 7;
  const int logical = xcd * per + (xcd < rem ? xcd : rem) + j;
  const int grp = logical / (GM * ntn);
  const int within = logical - grp * GM * ntn;
  const int gsz = (ntm - grp * GM) < GM ? (ntm - grp * GM) : GM;
  const int mt = grp * GM + within % gsz;
  const int nt = within / gsz;
  const int n0 = nt * BN;
  const int w0 = n0 + grp_t * 16 * F;  // this wave's first token row
  const int KT = p.K / BK;
  const int n_tiles = (p.M + kHeadTileRows - 1) / kHeadTileRows;
  const f16* W = (const f16*)p.A;
  const f16* H = (const f16*)p.bh;

  // loads: wave w fetches 16-row block w of both vocabulary tiles (the
  // second clamped to the last tile of the weight) and token blocks w, w+8,
  // ...; the first T_FULL waves have one token block more, so the waits
  // take one of two compile-time counts
  const int rr = lane >> 2, pc = lane & 3;
  const int ra = wave * 16 + rr;
  const uint32_t aoff = (uint32_t)(ra * 64 + (pc ^ swz64(ra)) * 16);
  const char* wbase[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int t = 2 * mt + h < n_tiles ? 2 * mt + h : n_tiles - 1;
    wbase[h] = (const char*)(W + (size_t)t * KT * (kHeadTileRows * 32));
  }
  uint32_t toff[C::T_MAX];
#pragma unroll
  for (int i = 0; i < C::T_MAX; ++i) {
    int q = wave + 8 * i;
    if (q >= C::T_BLOCKS) q = C::T_BLOCKS - 1;
    const int r = q * 16 + rr;
    const int gn = n0 + r < p.N ? r : p.N - 1 - n0;
    toff[i] = (uint32_t)(gn * p.ldb + (pc ^ swz64(r)) * 8) * 2u;
  }
  const char* hbase = (const char*)(H + (size_t)n0 * p.ldb);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)smem;
  const bool t_hi = wave < C::T_FULL;
  auto issue = [&](int st, int kt) {
    const uint32_t sA = lds0 + (uint32_t)(st * STAGE);
    const uint32_t sT = sA + A_BYTES;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      g2l16_m0(wbase[h] + (size_t)kt * (kHeadTileRows * 64), aoff,
               sA + (uint32_t)(h * kHeadTileRows * 64 + wave * 1024));
#pragma unroll
    for (int i = 0; i < C::T_MAX; ++i)
      if (i < C::T_MAX - 1 || t_hi)
        g2l16_m0(hbase + kt * BK * 2, toff[i], sT + (uint32_t)(wave + 8 * i) * 1024u);
  };

  f32x4 acc[F][MI];
#pragma unroll
  for (int f = 0; f < F; ++f)
#pragma unroll
    for (int i = 0; i < MI; ++i) acc[f][i] = f32x4{0.f, 0.f, 0.f, 0.f};

  const bool wave_active = w0 < p.N;
#pragma unroll
  for (int st = 0; st < NS - 1; ++st)
    if (st < KT) issue(st, st);
  for (int kt = 0; kt < KT; ++kt) {
    // this step's stage is complete once at most the later steps' loads
    // (NS - 2 stages of them) are in flight; near the end, none
    if (kt + NS - 2 < KT) {
      if (t_hi)
        wait_vmcnt<(NS - 2) * C::LOADS_HI>();
      else
        wait_vmcnt<(NS - 2) * C::LOADS_LO>();
    } else {
      wait_vmcnt<0>();
    }
    barrier();
    if (kt + NS - 1 < KT) issue((kt + NS - 1) % NS, kt + NS - 1);
    if (wave_active) {
      const char* sA = smem + (kt % NS) * STAGE + half * (kHeadTileRows * 64);
      const char* sT = smem + (kt % NS) * STAGE + A_BYTES;
      f16x8 a[MI], t[F];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int r = 16 * i + c;
        a[i] = *(const f16x8*)(sA + r * 64 + ((g ^ swz64(r)) * 16));
      }
#pragma unroll
      for (int f = 0; f < F; ++f) {
        const int r = grp_t * 16 * F + 16 * f + c;
        t[f] = *(const f16x8*)(sT + r * 64 + ((g ^ swz64(r)) * 16));
      }
#pragma unroll
      for (int f = 0; f < F; ++f)
#pragma unroll
        for (int i = 0; i < MI; ++i) acc[f][i] = mfma16x16x32(t[f], a[i], acc[f][i]);
    }
  }

  // acc[f][i][r] = z[vocabulary m0 + 16i + c][token w0 + 16f + 4g + r]
  const int chunk = 2 * mt + half;
  const int n_chunks = n_tiles;
  if (chunk >= n_chunks) return;  // a pair's second tile past the vocabulary
  const int mrow = chunk * kHeadTileRows + c;
  const int ncol = w0 + 4 * g;
#pragma unroll
  for (int f = 0; f < F; ++f)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int n = ncol + 16 * f + r;  // token
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < MI; ++i)
        if (mrow + 16 * i < p.M) mx = fmaxf(mx, acc[f][i][r]);
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) mx = fmaxf(mx, shfl_xor(mx, o));
      float sm = 0.f;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int v = mrow + 16 * i;  // vocabulary entry
        if (v < p.M) {
          const float z = acc[f][i][r];
          sm += __expf(z - mx);
          if (n < p.N) {
            const int si = p.sel[v];
            if (si >= 0) p.zsel[(size_t)n * p.n_sel + si] = z;
            if (p.dump) p.dump[(size_t)n * p.ld_dump + v] = z;
          }
        }
      }
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) sm += shfl_xor(sm, o);
      if (c == 0 && n < p.N) p.part[(size_t)n * n_chunks + chunk] = make_float2(mx, sm);
    }
}

template <int F, int NS>
hipError_t launch_head2(hipStream_t s, const GemmArgs& a) {
  using C = Head2Cfg<F, NS>;
  const int tiles = ((a.M + C::BM - 1) / C::BM) * ((a.N + C::BN - 1) / C::BN);
  if (tiles == 0) return hipSuccess;
  static const hipError_t attr = hipFuncSetAttribute(
      (const void*)head2_kernel<F, NS>, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((head2_kernel<F, NS>), dim3(tiles), dim3(512), C::LDS, s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------- LM head, few rows
// The same for at most 64 rows (see head_streams), where the head is a stream
// over its weight (1.05 GB for V = 128256, d = 4096) and the ring's barriers
// and its 256 token rows of loads keep it at 5.0 TB/s.  One wave per vocabulary tile with
// all rows (F groups of 16): the weight goes straight from memory to
// registers, D steps of 8 KB ahead per wave and no barrier anywhere, and the
// token rows come from L2.  Every logit is accumulated in the same order as
// above.  Measured (us, d 4096 / d 2048, against the ring): 9 rows 213 ->
// 155 / 132 -> 82 (6.8 TB/s at d 4096, what a read of this card's memory
// reaches), 32 rows 219 -> 160 / 137 -> 85, 64 rows 232 -> 212 / 150 -> 115.
template <int F, int D>
__global__ __launch_bounds__(256, 2) void head_few_kernel(const GemmArgs p) {
  constexpr int MI = 8;
  const int lane = threadIdx.x & 63;
  const int chunk = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_chunks = (p.M + kHeadTileRows - 1) / kHeadTileRows;
  if (chunk >= n_chunks) return;
  const int g = lane >> 4, c = lane & 15;
  const int KT = p.K / 32;
  // lane 16g + c: vocabulary row 16i + c (or token row 16f + c), features 8g ..
  const f16* W = (const f16*)p.A + (size_t)chunk * KT * (kHeadTileRows * 32) + c * 32 + g * 8;
  const f16* H[F];
#pragma unroll
  for (int f = 0; f < F; ++f) {
    const int n = 16 * f + c < p.N ? 16 * f + c : p.N - 1;
    H[f] = (const f16*)p.bh + (size_t)n * p.ldb + g * 8;
  }
  f32x4 acc[F][MI];
#pragma unroll
  for (int f = 0; f < F; ++f)
#pragma unroll
    for (int i = 0; i < MI; ++i) acc[f][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  f16x8 a[D][MI], t[D][F];
  auto load = [&](int kt, f16x8* av, f16x8* tv) {
    kt = kt < KT ? kt : KT - 1;  // past the end: read again, never used
#pragma unroll
    for (int f = 0; f < F; ++f) tv[f] = *(const f16x8*)(H[f] + kt * 32);
#pragma unroll
    for (int i = 0; i < MI; ++i)
      av[i] = __builtin_nontemporal_load((const f16x8*)(W + (size_t)kt * (kHeadTileRows * 32) + i * 512));
  };
#pragma unroll
  for (int d = 0; d < D; ++d) load(d, a[d], t[d]);
  for (int kt = 0; kt < KT; kt += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (kt + d < KT) {
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
          for (int i = 0; i < MI; ++i) acc[f][i] = mfma16x16x32(t[d][f], a[d][i], acc[f][i]);
      }
      load(kt + d + D, a[d], t[d]);
    }
  }
  // acc[f][i][r] = z[vocabulary 128 chunk + 16i + c][token 16f + 4g + r]
  const int v0 = chunk * kHeadTileRows + c;
  int si[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i) si[i] = v0 + 16 * i < p.M ? p.sel[v0 + 16 * i] : -1;
#pragma unroll
  for (int f = 0; f < F; ++f)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int n = 16 * f + 4 * g + r;
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < MI; ++i)
        if (v0 + 16 * i < p.M) mx = fmaxf(mx, acc[f][i][r]);
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) mx = fmaxf(mx, shfl_xor(mx, o));
      float sm = 0.f;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int v = v0 + 16 * i;
        if (v < p.M) {
          const float z = acc[f][i][r];
          sm += __expf(z - mx);
          if (n < p.N) {
            if (si[i] >= 0) p.zsel[(size_t)n * p.n_sel + si[i]] = z;
            if (p.dump) p.dump[(size_t)n * p.ld_dump + v] = z;
          }
        }
      }
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) sm += shfl_xor(sm, o);
      if (c == 0 && n < p.N) p.part[(size_t)n * n_chunks + chunk] = make_float2(mx, sm);
    }
}

template <int F, int D>
hipError_t launch_head_few(hipStream_t s, const GemmArgs& a) {
  const int n_chunks = (a.M + kHeadTileRows - 1) / kHeadTileRows;
  if (n_chunks == 0 || a.N == 0) return hipSuccess;
  hipLaunchKernelGGL((head_few_kernel<F, D>), dim3((n_chunks + 3) / 4), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_f16(hipStream_t s, const GemmArgs& a, int epi) {
  using H256 = Head2Cfg<4, 4>;  // 256-token tile
  using H320 = Head2Cfg<5, 4>;  // 320-token tile
  static_assert(kHeadTileRows == kHeadVocabChunk, "partials per vocabulary chunk");
  if (a.K % 32 != 0 || epi != EPI_HEAD || a.ldb % 8 != 0)
    return hipErrorInvalidValue;
  // per-lane token-row offsets are 32-bit byte offsets within one tile's rows
  if ((size_t)512 * a.ldb * 2 >= (size_t(1) << 31)) return hipErrorInvalidValue;
  if (head_streams(a.N, a.M)) {
    if (a.N <= 16) return launch_head_few<1, 4>(s, a);
    if (a.N <= 32) return launch_head_few<2, 3>(s, a);
    return launch_head_few<4, 2>(s, a);
  }
  // A workgroup's time barely depends on how many of its token rows are
  // real, so the tile that needs fewer token tiles wins; a full 320-token
  // tile runs about 10% longer than a full 256-token one.  Each logit's
  // accumulation order is the same in both, so the choice never changes a bit.
  const int t256 = (a.N + H256::BN - 1) / H256::BN, t320 = (a.N + H320::BN - 1) / H320::BN;
  if (10 * t256 > 11 * t320) return launch_head2<5, 4>(s, a);
  return launch_head2<4, 4>(s, a);
}

hipError_t launch_gemm_w4(hipStream_t s, const GemmArgs& a, int epi) {
  // the packed weight is padded to 256 columns so every tile shape divides it
  if (a.K % 64 != 0 || a.N % 256 != 0) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_ADD_F32: return launch_epi<WF_INT4, EPI_ADD_F32>(s, a);
    case EPI_SWIGLU: return launch_epi<WF_INT4, EPI_SWIGLU>(s, a);
    case EPI_QKV: return launch_epi<WF_INT4, EPI_QKV>(s, a);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm_w8(hipStream_t s, const GemmArgs& a, int epi) {
  // the packed weight is padded to 256 columns (and its scales with it)
  if (a.K % 64 != 0 || a.N % 256 != 0 || !a.bsc) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_ADD_F32: return launch_epi<WF_FP8, EPI_ADD_F32>(s, a);
    case EPI_SWIGLU: return launch_epi<WF_FP8, EPI_SWIGLU>(s, a);
    case EPI_QKV: return launch_epi<WF_FP8, EPI_QKV>(s, a);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lmop
