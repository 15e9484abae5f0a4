// Ternary matrix times 2..8 activation rows on the matrix cores (Eq. 10 with
// one group and zero bias, plus the Eq. 11 residual), for every problem of a
// plan in one persistent launch, or for one problem on its own.
//
// The product runs on v_mfma_scale_f32_16x16x128_f8f6f4 with exact operands:
//
//   B (128 columns x 16 rows of W): the ternary codes as FP4 (-1, 0, +1).
//     One LDS read per packed byte gives its five codes as five nibbles of a
//     dword (a table of 243 dwords, 32 copies so that a half-wave's reads hit
//     distinct banks); the dword is one pack's share of the operand as it is,
//     its last three nibbles zero.  A lane's four dwords are four packs: one
//     instruction takes 16 packs of each of 16 rows (80 of its 128 columns).
//   A (16 x 128 columns): a_j = v_j x[b][j] (exact in fp32) in fixed point,
//     split into six base-32 digits -16..15.  A digit d is the FP6 (E2M3)
//     value d / 8, so with q_j = rint(a_j 2^(154 - E)), |q_j| <= 2^28, E the biased
//     exponent of the largest |a| of a block of 20 columns, digit l of the
//     block has the block scale 2^(E + 5 l - 151): the instruction's E8M0
//     scale operand (one per 32 operand columns, which is one block).  An
//     a_j (22 bits) down to 2^-6 of its block's power of two is represented
//     exactly, the others to 2^-28 of that.  Where that matters (an outlier
//     among small columns: tern_rest) two more digits hold what is left, to
//     2^-37 of it.  A block with an a_j that is not finite takes the NaN
//     scale: every output of that batch row is then NaN.
//
// Each digit has its own row of the 16 x 16 result, so the digits' sums are
// sums of small integers (exact in fp32 as long as the blocks' scales stay
// within a few powers of two) and are rounded when they are added, lowest
// digit first, at the end of a panel part: y = alpha_r sum + residual.
//
// Result rows (of the 16 NB): batch row b = kg + 4 j owns lane group kg's
// result registers 6 j .. 6 j + 5 (NB = 2: batch 2..4, the two more digits in
// its registers 6 and 7; NB = 3: 5..8, those digits as a result block of their
// own, which only the slices that have some multiply).
//
// Why this form.  The kernel of grouped_mma.hip decodes a byte to fp16 codes
// with two LDS reads (10 bytes) and about 5.6 VALU.  Here it is one 4-byte LDS
// read and 1.5 VALU, the instruction (16 cycles of a SIMD's matrix pipe, four
// per result block and 1024 packed bytes) takes five times as many codes, and
// the decode table is 31 KB instead of 93.  What it pays for is the digits:
// about 240 VALU per batch row and slice.  Relative L2 error against 64 bits
// 4e-8 to 7e-8 at K = 4096 (fp16 halves: 7e-8 to 1.4e-7), with or without
// outliers of 100 to 60000 among N(0, 1) activations.  What bounds it: VALU issue (the
// 8B stack at batch 4 takes 385 us per call, 327 without the digits' build,
// 344 without the residual, 262 without decode too: the weight stream).
// A form at batch 1 (one result block, 64-row tiles on 16 waves or 256-row
// tiles on 4, digits of four slices built together) took 290 to 340 us per
// token of the 8B stack against the table kernel's 255: there the digits
// cost as much as the tables, and the sums have no batch to share them.
//
// Work unit = (problem, panel, K slice of 4 sixteen-pack groups = 320
// columns); a wave owns TW 64-row tiles of the panel, each four 16-row tiles:
// tile q holds rows 32 (q / 2) + 8 (q mod 2) + {0..7, 16..23}, so that one load
// instruction covers whole 128-byte lines (rows 16 m + 4 q + s, which need
// no select below, halve every line: 20 to 35 us more per 8B-stack token).  Byte i
// of row r is pack (i + r) mod 16 of its group: of the rotation's dword part
// (r / 4 mod 4) the upper bit is the tile's (register choice) and the lower
// the lane's (a select per dword), and the byte part takes one v_perm per dword.
// The digit images of a slice are built one unit ahead in LDS (two buffers),
// so a unit needs one barrier.  Every weight register is refilled with the
// next unit's bytes as soon as it has been decoded.
//
// Residual.  The activations of the salient columns are gathered by rank
// into a ring in LDS as their slices are staged; whenever 32 of the panel
// part's salient columns are there (or the part ends) they are multiplied:
// v_mfma_f32_16x16x32_f16 with a K index (column, position of the row in its
// four-row group) and one result row per (batch row, position), so a
// residual value enters as one 64-bit word, its fp16 bits shifted to its
// position, and no value is masked or expanded per row.  The values and
// position words of the next 32 columns are already in flight.
#include <type_traits>

#include "tern_common.h"

namespace qtea_grouped {
namespace {

// batch rows of the kernel with NB result blocks, at most
constexpr int tern_bm(int NB) { return NB == 2 ? 4 : 8; }
constexpr int kRest = 2;  // digits of a second set

template <int NB, int WAVES, int TW>
struct TLds {
  static constexpr int BM = tern_bm(NB);
  static constexpr int IMG = kTab;                          // [2 buffers] of digit images
  static constexpr int IMG1 = kUnitMfma * NB * 64 * 16;     // first 16 bytes of every lane's operand
  static constexpr int IMGB = kUnitMfma * NB * 64 * 24;     // one buffer: those, then the last 8 bytes
  static constexpr int SC = IMG + 2 * IMGB;                 // u32 [2][NB][64]: E8M0 scales, byte i for instruction i
  // NB = 3: the second sets' operands and scales, [2 buffers], for the batch
  // rows marked in RFLAG, u32 [2 buffers][8]
  static constexpr int RIMG = SC + 2 * NB * 256;
  static constexpr int RIMGB = kUnitMfma * 64 * 24 + 256;
  static constexpr int RFLAG = RIMG + (NB == 3 ? 2 * RIMGB : 0);
  static constexpr int BYTES = RFLAG + (NB == 3 ? 64 : 0);
  // In the holes: the ring of the salient activations, u16 [batch row][32
  // RING ranks], and the staging areas.  A unit's waves read ring chunks of 32
  // ranks from the one holding the unit's first salient column (less up to 31
  // left over) on, while the next unit's are gathered: 22 chunks at most.
  static constexpr int RING = 24;
  static_assert(31 + 2 * kSliceCols + 31 <= 32 * (RING - 1), "unread and newly gathered ranks do not meet");
  static constexpr int RINGB = RING * 64 * BM;
  static_assert(RINGB % 128 == 0 && RINGB + WAVES * TW * kStage <= kHoleBytes, "small areas fit the holes");
};

// F8: residual values are E4M3 bytes (layout 3), else fp16 (layout 2).
// ONE: a single problem launched on its own (GOne, no plan and no queue):
// workgroup g takes the units [g U / G, (g + 1) U / G).
template <int NB, int WAVES, int TW, bool F8, bool ONE>
__global__ __launch_bounds__(WAVES * 64, WAVES / 4) void tern_mfma_kernel(const uint8_t* __restrict__ plan,
                                                                          float* __restrict__ part, const GOne one) {
  using L = TLds<NB, WAVES, TW>;
  constexpr int kT = WAVES * 64, RP = kT * TW;  // threads; rows per panel (TW 64-row tiles per wave)
  constexpr int RBK = L::BM / 4;                // result blocks of the residual
  const GPlanHeader* H = reinterpret_cast<const GPlanHeader*>(plan);
  const GProblem* P = reinterpret_cast<const GProblem*>(plan + kPlanProblemsOff);
  auto PR = [&](int m) -> const GProblem& {
    if constexpr (ONE) return one.pr;
    else return P[m];
  };
  const int g = blockIdx.x;
  const int B = ONE ? one.batch : H->batch;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n16 = lane & 15, kg = lane >> 4;  // row within a 16-row tile (or result row), column group of the slice
  const uint32_t lane_tab = 4u * uint32_t(lane & 31);
  const uint32_t sel_rot = 0x07060504u - 0x01010101u * uint32_t(n16 & 3);

  // this workgroup's run of units
  int u, ue;
  Cursor cur;
  if constexpr (ONE) {
    const int G = int(gridDim.x);
    u = int(one_first(g, one.n_units, G));
    ue = int(one_first(g + 1, one.n_units, G));
    cur = Cursor{0, u / one.pr.n_slices, u % one.pr.n_slices};
  } else {
    if (g >= H->n_chunks) return;
    const GChunk rec = reinterpret_cast<const GChunk*>(plan + H->off_chunks)[g];
    u = rec.ub;
    ue = rec.ue;
    cur = Cursor{rec.m, rec.panel, rec.slice};
  }

  // --- loads of a unit's weights -------------------------------------------
  // byte offset of this lane's 16-byte unit within a 64-row tile's group 0
  auto trit_rsrc = [&](const GProblem& pr) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(pr.trits), 0,
                                             int(uint32_t(pr.n_pad >> 6) * uint32_t(pr.n_groups) * (kTileRows * kGroupPacks)),
                                             kBufferWord3);
  };
  auto tile_of = [&](const Cursor cc, const GProblem& pr, int tw) -> int {
    return min(cc.panel * (RP / 64) + w * TW + tw, int(pr.n_pad >> 6) - 1);
  };
  const uint32_t lane_row = uint32_t(16 * (n16 >> 3) + (n16 & 7)) * kGroupPacks;
  auto q_row = [](int q) -> int { return 32 * (q >> 1) + 8 * (q & 1); };  // first row of 16-row tile q
  auto lane_off = [&](const Cursor cc, const GProblem& pr) -> uint32_t {
    return uint32_t(min(cc.slice * kSliceGroups + kg, pr.n_groups - 1)) * (kTileRows * kGroupPacks) + lane_row;
  };
  auto tile_off = [&](const Cursor cc, const GProblem& pr, int tw) -> uint32_t {
    return uint32_t(tile_of(cc, pr, tw)) * uint32_t(pr.n_groups) * (kTileRows * kGroupPacks);
  };
  u32x4 W[TW][4];
  {
    const GProblem& pr = PR(cur.m);
    const __amdgpu_buffer_rsrc_t rs = trit_rsrc(pr);
    const uint32_t lo = lane_off(cur, pr);
#pragma unroll
    for (int tw = 0; tw < TW; ++tw)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        W[tw][q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, int(lo + q_row(q) * kGroupPacks),
                                                                                    int(tile_off(cur, pr, tw)), kAuxNT));
  }

  // --- digit images ---------------------------------------------------------
  // A task is one batch row over the slice's 64 packs, one pack per lane; wave
  // w runs task w.  (Waves w and w + 4 share a SIMD: fewer, whole tasks cost
  // it less than the same digits split over both, since every task converts
  // and scales its activations.)
  static_assert(L::BM <= WAVES, "a wave per batch row");
  uint32_t xr[5], vr[5];
  // (columns past the last and batch rows past the launch's read zero)
  auto load_xv = [&](const Cursor cc) {
    const GProblem& pr = PR(cc.m);
    const int lane = fresh(tid & 63);
    const __amdgpu_buffer_rsrc_t vres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t*>(pr.vs), 0, int(4 * uint32_t(pr.n_groups) * kGroupCols), kBufferWord3);
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(pr.x) + int64_t(min(w, B - 1)) * pr.K, 0, w < B ? int(2 * uint32_t(pr.K)) : 0, kBufferWord3);
    const int col0 = cc.slice * kSliceCols + 5 * lane;
    const u32x4 v4 = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(vres, 4 * col0, 0, 0));
    vr[0] = v4.x;
    vr[1] = v4.y;
    vr[2] = v4.z;
    vr[3] = v4.w;
    vr[4] = __builtin_amdgcn_raw_buffer_load_b32(vres, 4 * col0 + 16, 0, 0);
#pragma unroll
    for (int i = 0; i < 5; ++i) xr[i] = __builtin_amdgcn_raw_buffer_load_b16(xres, 2 * col0 + 2 * i, 0, 0);
  };
  // images of the loaded slice into buffer bb; its salient activations into
  // the ring, the first xb ranks after the first of chunk rc0
  // NB = 2: the second sets have the batch rows' last two result rows, which
  // hold zeros in the slices without one.  clear_rest: zeros there, in buffer bb,
  // for this wave's batch row (lanes 0..31: instruction, column group, row).
  auto clear_rest = [&](int bb, int lane) {
    if (lane >= 32) return;
    const uint32_t pi = uint32_t(lane) & 3u, m = 4u * uint32_t(w) + 2u + uint32_t(lane >> 4) + 16u * (uint32_t(lane >> 2) & 3u);
    const uint32_t rec = (pi * NB + 1u) * 64u + (m ^ pi), img = uint32_t(L::IMG + bb * L::IMGB);
    lds_write<u32x4>(img + rec * 16u, u32x4{0u, 0u, 0u, 0u});
    lds_write<u32x2>(img + uint32_t(L::IMG1) + rec * 8u, u32x2{0u, 0u});
    lds_write<uint32_t>(uint32_t(L::SC + bb * NB * 256) + (64u + m) * 4u, 0u);
  };
  uint32_t used = 0;  // bit bb: buffer bb holds a second set
  auto build = [&](int bb, int rc0, int xb) {
    if (w >= B) return;  // uniform
    const int lane = fresh(tid & 63), kg = lane >> 4, b = w;
    const uint32_t pi = uint32_t(lane >> 2) & 3u, pp = uint32_t(lane) & 3u;  // instruction and dword group of the pack
    const uint32_t img = uint32_t(L::IMG + bb * L::IMGB), img2 = img + uint32_t(L::IMG1);
    const uint32_t sc = uint32_t(L::SC + bb * NB * 256);
    float a[5], f[5];
    uint32_t ex, mx, top = 0;
    // (opaque, in 32 bits: the compiler packed x's values in pairs where they
    // were loaded, behind a wait for them)
#pragma unroll
    for (int i = 0; i < 5; ++i) asm volatile("" : "+v"(xr[i]));
    tern_products(vr, xr, a);
    tern_fixed(a, f, ex, mx);
    // A quad of lanes holds the four packs of one instruction, column group
    // and digit: 30-bit codes at bits 0, 48, 96, 144 of the operand.  Its
    // first lane writes the first four dwords, its last lane the other two.
    // Digit l goes to the operand record that row(l) names (address of its
    // first 16 bytes, of its last 8, of its scales).
    auto put = [&](auto nd, auto row, auto scale) {
      constexpr int ND = decltype(nd)::value;
      uint32_t P[ND], P1[ND], P2[ND];
      tern_digits<ND>(f, P);
      top = P[ND - 1];
#pragma unroll
      for (int l = 0; l < ND; ++l) {
        P1[l] = quad_next(P[l]);
        P2[l] = quad_next2(P[l]);
      }
      if (pp == 0u) {
#pragma unroll
        for (int l = 0; l < ND; ++l) {
          uint32_t at16, at8, at_scale;
          row(l, at16, at8, at_scale);
          lds_write<u32x4>(at16, u32x4{P[l], P1[l] << 16, P1[l] >> 16, P2[l]});
          lds_write<uint8_t>(at_scale + pi, scale(l));
        }
      }
      if (pp == 3u) {
#pragma unroll
        for (int l = 0; l < ND; ++l) {
          uint32_t at16, at8, at_scale;
          row(l, at16, at8, at_scale);
          lds_write<u32x2>(at8, u32x2{P[l] << 16, P[l] >> 16});
        }
      }
    };
    // slot s of batch row b: result row 4 (b mod 4) + s mod 4 of block s / 4
    auto slot = [&](uint32_t s, uint32_t& at16, uint32_t& at8, uint32_t& at_scale) {
      const uint32_t nb = s >> 2, m = 4u * uint32_t(b & 3) + (s & 3u) + 16u * uint32_t(kg);
      const uint32_t rec = (pi * NB + nb) * 64u + (m ^ pi);
      at16 = img + rec * 16u;
      at8 = img2 + rec * 8u;
      at_scale = sc + (nb * 64u + m) * 4u;
    };
    put(std::integral_constant<int, kDigits>{},
        [&](int l, uint32_t& r, uint32_t& r2, uint32_t& rs) { slot(uint32_t(kDigits * (b >> 2) + l), r, r2, rs); },
        [&](int l) { return tern_scale(ex, mx, l); });
    const bool rest = tern_rest<kRest>(a, f, ex, top);
    constexpr std::integral_constant<int, kRest> nr{};
    if constexpr (NB == 2) {
      if (rest) {
        put(
            nr, [&](int l, uint32_t& r, uint32_t& r2, uint32_t& rs) { slot(uint32_t(kDigits + l), r, r2, rs); },
            [&](int l) { return tern_rest_scale<kRest>(ex, mx, l); });
        used |= 1u << bb;
      } else if ((used >> bb) & 1u) {
        clear_rest(bb, lane);
        used &= ~(1u << bb);
      }
    } else {
      if (rest)
        put(
            nr,
            [&](int l, uint32_t& r, uint32_t& r2, uint32_t& rs) {
              const uint32_t m = 4u * uint32_t(b & 3) + uint32_t(2 * (b >> 2) + l) + 16u * uint32_t(kg);
              const uint32_t rec = pi * 64u + (m ^ pi), rimg = uint32_t(L::RIMG + bb * L::RIMGB);
              r = rimg + rec * 16u;
              r2 = rimg + uint32_t(kUnitMfma * 64 * 16) + rec * 8u;
              rs = rimg + uint32_t(kUnitMfma * 64 * 24) + 4u * m;
            },
            [&](int l) { return tern_rest_scale<kRest>(ex, mx, l); });
      lds_write<uint32_t>(uint32_t(L::RFLAG + 32 * bb + 4 * b), rest ? 1u : 0u);
    }
    // the batch row's salient activations
    const uint32_t first = uint32_t(32 * rc0 - 1 + xb);
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const uint32_t rk = vr[i] >> 16;
      if (rk != 0u) {
        const uint32_t pos = first + rk, wrapped = min(pos, pos - uint32_t(32 * L::RING));
        lds_write<uint16_t>(hole(uint32_t(b) * uint32_t(L::RING * 64) + 2u * wrapped), uint16_t(xr[i]));
      }
    }
  };

  // --- residual -------------------------------------------------------------
  // the wave's staging areas: rows of 128 bytes, 256 apart
  const uint32_t stg = hole(uint32_t(L::RINGB + w * TW * kStage));
  constexpr uint32_t SR = 256, ST = kStage / 128 * SR;  // distance of the rows, of the tiles' areas
  u32x4 rvq[TW];
  uint32_t ris[(TW + 1) / 2];
  // values and position words of the 32 salient columns from rank s on, for
  // this wave's tiles (past the matrix's last: zeros)
  auto load_res = [&](const Cursor cc, int s) {
    const GProblem& pr = PR(cc.m);
    const int lane = fresh(tid & 63);
    constexpr uint32_t VB = F8 ? 16u : 32u;
    const uint32_t nS = uint32_t(pr.nS), nt = uint32_t(pr.n_pad >> 6);
    const __amdgpu_buffer_rsrc_t vres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(pr.rval), 0, int(nt * nS * VB), kBufferWord3);
    const __amdgpu_buffer_rsrc_t ires =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(pr.ridx), 0, int(nt * nS * 4u), kBufferWord3);
#pragma unroll
    for (int tw = 0; tw < TW; ++tw) {
      const uint32_t first = uint32_t(tile_of(cc, pr, tw)) * nS + uint32_t(s);
      if constexpr (F8) {
        const u32x2 t = __builtin_bit_cast(
            u32x2, __builtin_amdgcn_raw_buffer_load_b64(vres, int(8u * uint32_t(lane)), int(first * VB), 0));
        rvq[tw] = u32x4{t.x, t.y, 0u, 0u};
      } else {
        rvq[tw] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(vres, int(16u * uint32_t(lane)), int(first * VB), 0));
      }
    }
    // lanes 0..31 an even tile's words, 32..63 the next one's
#pragma unroll
    for (int tp = 0; tp < TW; tp += 2) {
      const uint32_t f0 = uint32_t(tile_of(cc, pr, tp)) * nS, f1 = uint32_t(tile_of(cc, pr, min(tp + 1, TW - 1))) * nS;
      ris[tp / 2] = __builtin_amdgcn_raw_buffer_load_b32(
          ires, int(4u * ((lane < 32 ? f0 : f1) + uint32_t(s) + uint32_t(lane & 31))), 0, 0);
    }
  };
  f32x4 racc[TW][RBK];
  // chunk `ch` of the ring holds the activations of the columns in rvq, ris;
  // n of its 32 columns belong to the part
  auto residual = [&](int ch, int n) {
    const int lane = fresh(tid & 63), n16 = lane & 15, kg = lane >> 4;
    // selectors that put an activation's fp16 bits at the position of this
    // lane's result row (position n16 & 3) in a 64-bit word
    const uint32_t p4 = uint32_t(n16) & 3u, zz = 0x0c0c0c0cu;
    const uint32_t se = (p4 & 1u) ? 0x01000c0cu : 0x0c0c0100u, so = (p4 & 1u) ? 0x03020c0cu : 0x0c0c0302u;
    const uint32_t se0 = p4 < 2u ? se : zz, se1 = p4 < 2u ? zz : se, so0 = p4 < 2u ? so : zz, so1 = p4 < 2u ? zz : so;
    u32x4 X[RBK];
#pragma unroll
    for (int jb = 0; jb < RBK; ++jb) {
      // (a batch row past the launch's feeds result rows that are not stored)
      const uint32_t b = min(uint32_t(4 * jb + (n16 >> 2)), uint32_t(L::BM - 1));
      X[jb] = lds_read<u32x4>(hole(b * uint32_t(L::RING * 64) + uint32_t(ch) * 64u + uint32_t(kg) * 16u));
      if (n < 32) {  // uniform: the last columns of a part; what the ring holds past them may be anything
        const int have = n - 8 * kg;
#pragma unroll
        for (int d = 0; d < 4; ++d) X[jb][d] &= have >= 2 * d + 2 ? 0xffffffffu : (have == 2 * d + 1 ? 0xffffu : 0u);
      }
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int tw = 0; tw < TW; ++tw) {
      if constexpr (F8)
        lds_write<u32x2>(stg + tw * ST + uint32_t(lane >> 4) * SR + uint32_t(lane & 15) * 8u, u32x2{rvq[tw].x, rvq[tw].y});
      else
        lds_write<u32x4>(stg + tw * ST + uint32_t(lane >> 3) * SR + uint32_t(lane & 7) * 16u, rvq[tw]);
    }
#pragma unroll
    for (int tp = 0; tp < (TW + 1) / 2; ++tp)  // (with one tile both halves write the same words)
      lds_write<uint32_t>(stg + (TW == 1 ? 0u : uint32_t(2 * tp + (lane >> 5)) * ST) + 8u * SR + 4u * uint32_t(lane & 31), ris[tp]);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int tw = 0; tw < TW; ++tw) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const u32x2 pw = lds_read<u32x2>(stg + tw * ST + 8u * SR + 32u * uint32_t(kg) + 8u * j);
        uint32_t bw[4];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          const int h = 2 * j + hh;
          uint32_t rb;
          if constexpr (F8) {
            // the magnitude bits at bits 7..13 are the fp16 bits of value * 2^-8
            const uint32_t t = lds_read<uint8_t>(stg + tw * ST + uint32_t(kg) * SR + 16u * h + uint32_t(n16));
            const _Float16 v8 = __builtin_bit_cast(_Float16, uint16_t(((t & 0x7fu) << 7) | ((t & 0x80u) << 8)));
            rb = __builtin_bit_cast(uint16_t, _Float16(v8 * _Float16(256.0f)));
          } else {
            rb = lds_read<uint16_t>(stg + tw * ST + uint32_t(kg) * 2u * SR + uint32_t(h >> 2) * SR + uint32_t(h & 3) * 32u +
                                    2u * uint32_t(n16));
          }
          const uint32_t pos = __builtin_amdgcn_ubfe(hh ? pw.y : pw.x, 2u * uint32_t(n16), 2);
          const uint64_t v = uint64_t(rb) << (pos << 4);
          bw[2 * hh] = uint32_t(v);
          bw[2 * hh + 1] = uint32_t(v >> 32);
        }
        const half8 Bv = as_half8(bw[0], bw[1], bw[2], bw[3]);
#pragma unroll
        for (int jb = 0; jb < RBK; ++jb) {
          const uint32_t x2 = X[jb][j];
          const half8 A = as_half8(__builtin_amdgcn_perm(0u, x2, se0), __builtin_amdgcn_perm(0u, x2, se1),
                                   __builtin_amdgcn_perm(0u, x2, so0), __builtin_amdgcn_perm(0u, x2, so1));
          racc[tw][jb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, Bv, racc[tw][jb], 0, 0, 0);
        }
      }
    }
    asm volatile("" ::: "memory");
  };

  // --- start ----------------------------------------------------------------
  // range of salient ranks of a slice: lane 0 reads the first bound, the
  // others the second (a scalar load would hold every LDS wait until it is
  // back from memory)
  auto load_spos = [&](const Cursor cc) -> int {
    const GProblem& pr = PR(cc.m);
    const int g0 = cc.slice * kSliceGroups;
    return gptr(pr.spos)[(tid & 63) == 0 ? g0 : min(g0 + kSliceGroups, pr.n_groups)];
  };
  load_xv(cur);
  int spv = load_spos(cur);
  // decode table: 32 copies of every entry, four per store
  for (int e = tid; e < kTabRows * 8; e += kT) {
    const uint32_t v = (e >> 3) < kCodes ? tern_entry(uint32_t(e >> 3)) : 0u;
    lds_write<u32x4>(uint32_t(e >> 3) * 256u + uint32_t(e & 7) * 16u, u32x4{v, v, v, v});
  }
  // result rows no digit uses: zero operands (their results are not read;
  // zeros keep the matrix pipe's inputs quiet)
  if constexpr (!ONE) {
    for (int e = tid; e < 2 * L::IMGB / 16; e += kT) lds_write<u32x4>(uint32_t(L::IMG + 16 * e), u32x4{0u, 0u, 0u, 0u});
    for (int e = tid; e < 2 * NB * 64; e += kT) lds_write<uint32_t>(uint32_t(L::SC + 4 * e), 0u);
    __syncthreads();
  } else if (NB == 2 && w < B) {
    // (behind the first loads and the table: in front of them it held the
    // launch's start, 28672 x 4096 at batch 4 18.2 instead of 17.4 us)
    clear_rest(0, lane);
    clear_rest(1, lane);
  }
  int ring = 0;  // ring chunk of column s0
  // first salient column of the part not yet multiplied; end of the unit's
  int s0 = __builtin_amdgcn_readlane(spv, 0), s_hi = __builtin_amdgcn_readlane(spv, 1);
  load_res(cur, s0);
  build(0, ring, 0);
  __syncthreads();

  const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
  f32x4 C[TW][4][NB], R3[NB == 3 ? 4 : 1];
#pragma unroll
  for (f32x4& r : R3) r = zero4;
#pragma unroll
  for (int tw = 0; tw < TW; ++tw) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) C[tw][q][nb] = zero4;
#pragma unroll
    for (int jb = 0; jb < RBK; ++jb) racc[tw][jb] = zero4;
  }
#ifdef QTEA_DEBUG
  uint32_t bad = 0;  // bit 4 tw + q: a byte of the lane's row of that tile is no code
#endif
  int pstart_slice = cur.slice;
  bool part_first = true;  // the open panel part began at the run's first unit

  for (int it = 0, first = u; u < ue; ++it, ++u) {
    const GProblem& pr = PR(cur.m);
    const bool has_next = u + 1 < ue;
    const bool pend = cur.slice == pr.n_slices - 1 || !has_next;
    if (cur.slice == 0 || u == first) {
      pstart_slice = cur.slice;
      part_first = u == first;
    }
    Cursor nxt = cur;  // (stays on the run's last unit)
    if (has_next && ++nxt.slice == pr.n_slices) {
      nxt.slice = 0;
      if (++nxt.panel == pr.n_panels) {
        nxt.panel = 0;
        ++nxt.m;
      }
    }
    const GProblem& pn = PR(nxt.m);
    const int sb = it & 1;

    // 1. residual: the part's salient columns staged so far, 32 at a time,
    // all of them at the part's end; then the next columns' loads
    while (s0 + 32 <= s_hi || (pend && s0 < s_hi)) {
      residual(ring, s_hi - s0);
      s0 += 32;
      ring = ring + 1 < L::RING ? ring + 1 : 0;
      if (!pend || s0 < s_hi) load_res(cur, s0);
    }

    // 2. the next unit's activations and salient ranks
    if (!ONE || has_next) {
      load_xv(nxt);
      spv = load_spos(nxt);
    }

    // 3. the unit's products
    {
      const int lane = fresh(tid & 63), n16 = lane & 15;
      const __amdgpu_buffer_rsrc_t wres = trit_rsrc(pn);
      const uint32_t mask = has_next ? 0xffffffffu : 0u;
      const uint32_t n_lo = lane_off(nxt, pn) & mask;
      const uint32_t img = uint32_t(L::IMG + sb * L::IMGB) + 16u * uint32_t(lane);
      const uint32_t img2 = img + uint32_t(L::IMG1) - 8u * uint32_t(lane);
      uint32_t scv[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        scv[nb] = lds_read<uint32_t>(uint32_t(L::SC + (sb * NB + nb) * 256) + 4u * uint32_t(lane));
      auto digits = [&](int i, int nb, u32x4& d, u32x2& d2) {
        const uint32_t o = uint32_t((i * NB + nb) * 64);
        d = lds_read<u32x4>((img ^ (16u * uint32_t(i))) + 16u * o);
        d2 = lds_read<u32x2>((img2 ^ (8u * uint32_t(i))) + 8u * o);
      };
      // The rotation of tile (tw, q)'s bytes: the lane's dword part undone in
      // place, then the tile's dword part and the byte part as dword i (packs
      // 4 i .. 4 i + 3) is taken.
      auto turn = [&](int tw, int q) {
        const u32x4 o = W[tw][q];
#pragma unroll
        for (int k = 0; k < 4; ++k) W[tw][q][k] = (n16 & 4) ? o[(k + 3) & 3] : o[k];
      };
      auto packs = [&](int tw, int q, int i) -> uint32_t {
        const int c = 2 * (q & 1);
        const uint32_t U = __builtin_amdgcn_perm(W[tw][q][(i - c) & 3], W[tw][q][(i - c - 1) & 3], sel_rot);
#ifdef QTEA_DEBUG
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (((U >> (8 * k)) & 255u) >= uint32_t(kCodes)) bad |= 1u << (4 * tw + q);
#endif
        return U;
      };
      auto unrotate = [&](int tw, int q, uint32_t (&U)[4]) {
        turn(tw, q);
#pragma unroll
        for (int i = 0; i < 4; ++i) U[i] = packs(tw, q, i);
      };
      auto decode = [&](uint32_t U, uint32_t (&e)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          e[k] = lds_read<uint32_t>(__builtin_amdgcn_perm(lane_tab, U, 0x0C0C0004u | (uint32_t(k) << 8)));
      };
      // the next unit's bytes into the registers just read (after the run's
      // last unit every lane reads the matrix's first bytes)
      auto refill = [&](int tw, int q) {
        if (!ONE || has_next)
          W[tw][q] = __builtin_bit_cast(
              u32x4, __builtin_amdgcn_raw_buffer_load_b128(wres, int(n_lo + q_row(q) * kGroupPacks),
                                                           int(tile_off(nxt, pn, tw) & mask), kAuxNT));
      };
      auto product = [&](auto ic, int tw, int q, int nb, const u32x4 d, const u32x2 d2, const uint32_t (&e)[4]) {
        C[tw][q][nb] = tern_mfma<decltype(ic)::value>(d, d2, e, C[tw][q][nb], scv[nb]);
        // a use in this block: without one the compiler sinks the products
        // below the image build and holds every decoded dword in registers
        asm volatile("" : "+v"(C[tw][q][nb]));
      };
      // NB = 3: the second sets' products (result rows of batch rows without
      // one: whatever their operands hold is masked)
      uint32_t rest = 0, flag = 0;
      if constexpr (NB == 3) flag = lds_read<uint32_t>(uint32_t(L::RFLAG + 32 * sb) + 4u * uint32_t(lane & 7));
      auto product_rest = [&](auto ic, const uint32_t (&e)[4][4]) {
        constexpr int i = decltype(ic)::value;
        if (i == 0) rest = uint32_t(__ballot(lane < B && flag != 0u));
        if (rest == 0u) return;  // uniform
        const int lane = fresh(tid & 63), n16 = lane & 15;
        const uint32_t rimg = uint32_t(L::RIMG + sb * L::RIMGB), rec = uint32_t(64 * i + (lane ^ i));
        u32x4 d = lds_read<u32x4>(rimg + 16u * rec);
        u32x2 d2 = lds_read<u32x2>(rimg + uint32_t(kUnitMfma * 64 * 16) + 8u * rec);
        uint32_t sc = lds_read<uint32_t>(rimg + uint32_t(kUnitMfma * 64 * 24) + 4u * uint32_t(lane));
        const uint32_t have = 0u - ((rest >> ((n16 >> 2) + 4 * ((n16 >> 1) & 1))) & 1u);
        d &= have;
        d2 &= have;
        sc &= have;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          R3[q] = tern_mfma<i>(d, d2, e[q], R3[q], sc);
          asm volatile("" : "+v"(R3[q]));
        }
      };
      constexpr std::integral_constant<int, 0> i0{};
      constexpr std::integral_constant<int, 1> i1{};
      constexpr std::integral_constant<int, 2> i2{};
      constexpr std::integral_constant<int, 3> i3{};
      if constexpr (NB > 2) {
        // (the registers hold no second copy of the packs or of the digits)
        auto step = [&](int tw, auto ic) {
          constexpr int i = decltype(ic)::value;
          uint32_t e[4][4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (i == 0) turn(tw, q);
            decode(packs(tw, q, i), e[q]);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (i == 3) {
#pragma unroll
            for (int q = 0; q < 4; ++q) refill(tw, q);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            u32x4 d;
            u32x2 d2;
            digits(i, nb, d, d2);
#pragma unroll
            for (int q = 0; q < 4; ++q) product(ic, tw, q, nb, d, d2, e[q]);
          }
          product_rest(ic, e);
          __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int tw = 0; tw < TW; ++tw) {
          step(tw, i0);
          step(tw, i1);
          step(tw, i2);
          step(tw, i3);
        }
      } else {
        // Steps (tile tw, instruction i) in a row, each decoding the next
        // step's packs and reading its digits ahead of its own products.
        uint32_t U[4][4], e[2][4][4];
        u32x4 d[2][NB];
        u32x2 d2[2][NB];
        auto open_tile = [&](int tw) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            unrotate(tw, q, U[q]);
            __builtin_amdgcn_sched_barrier(0);
            refill(tw, q);
            __builtin_amdgcn_sched_barrier(0);
          }
        };
        auto fetch = [&](int i, int buf) {
#pragma unroll
          for (int q = 0; q < 4; ++q) decode(U[q][i], e[buf][q]);
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) digits(i, nb, d[buf][nb], d2[buf][nb]);
        };
        auto step = [&](auto twc, auto ic) {
          constexpr int tw = decltype(twc)::value, i = decltype(ic)::value;
          if constexpr (i == 3 && tw + 1 < TW) open_tile(tw + 1);
          if constexpr (i < 3 || tw + 1 < TW) fetch((i + 1) & 3, (i + 1) & 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int q = 0; q < 4; ++q) product(ic, tw, q, nb, d[i & 1][nb], d2[i & 1][nb], e[i & 1][q]);
          __builtin_amdgcn_sched_barrier(0);
        };
        open_tile(0);
        fetch(0, 0);
        constexpr std::integral_constant<int, 1> t1{};
        step(i0, i0);
        step(i0, i1);
        step(i0, i2);
        step(i0, i3);
        if constexpr (TW > 1) {
          step(t1, i0);
          step(t1, i1);
          step(t1, i2);
          step(t1, i3);
        }
        static_assert(TW == 1 || TW == 2, "one or two tiles per wave");
      }
    }

    // 4. the next unit's digit images into the other buffer
    const int sn_lo = __builtin_amdgcn_readlane(spv, 0), sn_hi = __builtin_amdgcn_readlane(spv, 1);
    if (pend) {  // the next unit starts a new part
      s0 = sn_lo;
      if (has_next) load_res(nxt, s0);
    }
    if (has_next) build(sb ^ 1, ring, sn_lo - s0);

    // 5. part end: y = alpha * sum + residual (or a partial of a split panel).
    // The digit sums go through the wave's staging area to the layout of the
    // residual sums: lane group kg holds batch row 4 jb + kg, rows 4 n16 ..
    // 4 n16 + 3 of the wave's tile.
    if (pend) {
      const int lane = fresh(tid & 63), n16 = lane & 15, kg = lane >> 4;
      const bool owned = pstart_slice == 0 && cur.slice == pr.n_slices - 1;
      float* dst = part + (2 * int64_t(g) + (part_first ? 0 : 1)) * int64_t(RP) * B;
#ifdef QTEA_DEBUG
      bad |= uint32_t(__shfl_xor(int(bad), 16));
      bad |= uint32_t(__shfl_xor(int(bad), 32));
#endif
#pragma unroll
      for (int tw = 0; tw < TW; ++tw) {
        const int64_t row0 = int64_t(cur.panel) * RP + int64_t(w * TW + tw) * 64;
        // row scales of rows 4 n16 .. 4 n16 + 3 of the tile
        const u32x2 al2 = *reinterpret_cast<gu32x2*>(gptr(pr.alpha) + tile_of(cur, pr, tw) * 64 + 4 * n16);
#pragma unroll
        for (int jb = 0; jb < RBK; ++jb) {
          asm volatile("" ::: "memory");
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4(&Cq)[NB] = C[tw][q];
            float s = 0.0f;
#pragma unroll
            for (int d = 0; d < kRest; ++d) s += NB == 2 ? Cq[1][2 + d] : R3[q][2 * jb + d];
#pragma unroll
            for (int d = 0; d < kDigits; ++d) s += Cq[(kDigits * jb + d) >> 2][(kDigits * jb + d) & 3];
#ifdef QTEA_DEBUG
            if ((bad >> (4 * tw + q)) & 1u) s = __builtin_nanf("");
#endif
            const uint32_t row = uint32_t(q_row(q) + 16 * (n16 >> 3) + (n16 & 7));
            lds_write<float>(stg + uint32_t(kg) * 2u * SR + (row >> 5) * SR + (row & 31u) * 4u, s);
          }
          asm volatile("" ::: "memory");
          const f32x4 t = lds_read<f32x4>(stg + uint32_t(kg) * 2u * SR + uint32_t(n16 >> 3) * SR + uint32_t(n16 & 7) * 16u);
          asm volatile("" ::: "memory");
          f32x4 yv;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float rv = racc[tw][jb][v];
            const float tv = t[v];
            const float al = h2f(uint16_t((v & 1) ? al2[v >> 1] >> 16 : al2[v >> 1] & 0xffffu));
            yv[v] = al * tv + rv;
          }
          const int b = 4 * jb + kg;
          if (b < B) {
            if (owned) {
              if (row0 + 4 * n16 < pr.N)  // N % 4 == 0: the four rows are all in or all out
                *(gf32x4u*)(pr.y + int64_t(b) * pr.N + row0 + 4 * n16) = yv;
            } else {
              *reinterpret_cast<f32x4*>(dst + int64_t(b) * RP + (w * TW + tw) * 64 + 4 * n16) = yv;
            }
          }
          racc[tw][jb] = zero4;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) C[tw][q][nb] = zero4;
      }
#pragma unroll
      for (f32x4& r : R3) r = zero4;
#ifdef QTEA_DEBUG
      bad = 0;
#endif
    }
    __syncthreads();  // the next unit's images are complete; this unit's are free
    s_hi = sn_hi;
    cur = nxt;
  }
}

template <int NB, int WAVES, int TW, bool F8, bool ONE>
hipError_t launch(const uint8_t* plan, int grid, float* part, const GOne& one, hipStream_t st) {
  using L = TLds<NB, WAVES, TW>;
  static_assert(L::BYTES <= 160 * 1024, "LDS of one workgroup");
  static std::atomic<int> done[kMaxDevices];
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(&tern_mfma_kernel<NB, WAVES, TW, F8, ONE>), L::BYTES, done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((tern_mfma_kernel<NB, WAVES, TW, F8, ONE>), dim3(grid), dim3(WAVES * 64), L::BYTES, st, plan, part, one);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_grouped_tern(const uint8_t* plan, int grid, bool f8, float* part, hipStream_t st) {
  const GOne none{};
  return f8 ? launch<2, 8, 2, true, false>(plan, grid, part, none, st)
            : launch<2, 8, 2, false, false>(plan, grid, part, none, st);
}

hipError_t launch_one_tern(const GOne& one, int grid, bool f8, float* part, hipStream_t st) {
  if (one.batch <= 4)
    return f8 ? launch<2, 8, 1, true, true>(nullptr, grid, part, one, st)
              : launch<2, 8, 1, false, true>(nullptr, grid, part, one, st);
  return f8 ? launch<3, 8, 1, true, true>(nullptr, grid, part, one, st)
            : launch<3, 8, 1, false, true>(nullptr, grid, part, one, st);
}

}  // namespace qtea_grouped
