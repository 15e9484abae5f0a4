// One matrix times one activation row on the FP4 matrix-core path (Eq. 10 with
// one group and zero bias, plus the Eq. 11 residual): qtea_gemv and
// qtea_gemm_lowbatch at batch 1, layouts 2 and 3, where solo_shape takes it (the
// table kernel is faster for few slices of many tiles and for parts of few tiles).
//
// What bounds it is latency: the bytes of these matrices stream in 0.5 to 4 us
// and a launch on other units (512-row panels x 320-column slices) spent its
// 8 to 14 us on building a 62 KB table per unit and on summing 13 to 45 parts
// per panel across workgroups.  Here a task is one 320-column slice of the
// matrix, or 32 to 96 of its salient columns; a workgroup's 16 waves take up to 16
// tasks, one each, for the whole launch, and walk over 64-row tiles together:
//
//   - a wave splits its slice's activations into digits once (tern_common.h)
//     and keeps the four instructions' operands in registers, or gathers the
//     activations of its salient columns; neither needs another wave;
//   - per tile a wave decodes its 4 KB of packed bytes, sixteen instructions,
//     and writes the tile's 64 row sums to LDS; one wave (another each tile)
//     adds the 16 rows of sums in task order, scales by alpha and stores y,
//     while the others are at the next tile, whose bytes were already loading;
//   - up to 16 tasks (4096 columns with 5 % salient ones) nothing crosses
//     workgroups.  A longer matrix is cut in parts of at most 16 tasks, one
//     part per workgroup; a tile's part sums (64 floats each) are added in
//     part order by the last part to arrive (a counter per tile).
//
// An activation that is not finite makes every output NaN.
//
// us per launch (graph of 20), the table kernel's in brackets, 2 % salient: 4096 x
// 4096 6.8 (7.4), 6144 x 4096 6.9 (7.3), 28672 x 4096 10.5 (13.1), 128256 x 2048
// 17.5 (21.5), 512 x 700 3.7 (6.3); 4096 x 14336 with 5 %, four parts, 10.3 (10.5).
// Whole 64-row tiles at 4096 x 4096: 7.6.  Relative L2 error against 64 bits 8e-8 to 1.1e-7 (table
// sums: 1e-7 to 1.3e-7), with or without outliers of 100 to 60000 among N(0, 1)
// activations: a slice that has some takes four more digits (tern_rest), in
// result rows that are there anyway.  Looking for them costs 0.1 us (0.2 with their
// code in line with the rest, where every launch fetched it), a launch that
// finds some 0.5 to 1.
#include <type_traits>

#include "tern_common.h"

namespace qtea_grouped {
namespace {

constexpr int kSoloWaves = kSoloTasks;                // one task per wave
constexpr int kSoloImg1 = kUnitMfma * 32 * 16;        // a wave's digit operands: first 16 bytes of 32 records
constexpr int kSoloImg = kUnitMfma * 32 * 24;         // (result rows 0..7, 4 column groups) per instruction
constexpr int kSoloArea = kSoloImg + 128;             // and their scales, u32 per record
static_assert(kSoloArea >= kStage, "a residual wave stages its values in the same area");
constexpr int kSoloRed = kTab + kSoloWaves * kSoloArea;          // fp32 [2][task][64] row sums
constexpr int kSoloRest = 4;                          // digits of a second set
constexpr int kSoloBytes = kSoloRed + 2 * kSoloWaves * 64 * 4;

// QN: 16-row tiles (of a 64-row tile's four) that the workgroups walk over
template <bool F8, int QN>
__global__ __launch_bounds__(kSoloWaves * 64, 4) void tern_solo_kernel(const GProblem pr, const int parts, const int cr,
                                                                       float* __restrict__ part,
                                                                       uint32_t* __restrict__ counters) {
  extern __shared__ float smem[];
  (void)smem;
  const int tid = threadIdx.x, lane = tid & 63, n16 = lane & 15, kg = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int p = blockIdx.x % parts, G = int(gridDim.x) / parts, t0 = blockIdx.x / parts;
  constexpr int SPLIT = 4 / QN;  // pieces of a 64-row tile
  const int n_tiles = int(pr.n_pad >> 6), n_pieces = n_tiles * SPLIT, nS = pr.nS;
  const int T = pr.n_slices + (nS + 32 * cr - 1) / (32 * cr);
  const int task = p * kSoloTasks + w, n_here = min(T - p * kSoloTasks, kSoloTasks);
  const bool slice_task = task < pr.n_slices, res_task = !slice_task && task < T;  // uniform per wave
  // tasks of this part that are slices (the first ones)
  const int n_sl = max(0, min(pr.n_slices - p * kSoloTasks, n_here));
  const uint32_t area = uint32_t(kTab + w * kSoloArea);
  const uint32_t lane_tab = 4u * uint32_t(lane & 31);
  const uint32_t sel_rot = 0x07060504u - 0x01010101u * uint32_t(n16 & 3);
  auto q_row = [](int q) -> int { return 32 * (q >> 1) + 8 * (q & 1); };  // first row of 16-row tile q

  const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
  auto table = [&]() {
    for (int e = tid; e < kTabRows * 8; e += kSoloWaves * 64) {
      const uint32_t v = (e >> 3) < kCodes ? tern_entry(uint32_t(e >> 3)) : 0u;
      lds_write<u32x4>(uint32_t(e >> 3) * 256u + uint32_t(e & 7) * 16u, u32x4{v, v, v, v});
    }
  };
  // Every wave walks over the workgroup's tiles: sums(t, tn, red) leaves the
  // wave's 64 sums of tile t at red (tn: the next tile; after the last one its
  // bytes are loaded for nothing), then one wave adds the tasks' sums.
  // Lane = row of the 64-row tile; the rows of the piece's 16-row tiles:
  auto mine = [&](int t) -> bool { return (2 * (lane >> 5) + ((lane >> 3) & 1)) / QN == t % SPLIT; };
  auto walk = [&](auto sums) {
    for (int t = t0, it = 0; t < n_pieces; t += G, ++it) {
      const uint32_t red = uint32_t(kSoloRed + (it & 1) * kSoloWaves * 256);
      const bool adds = (it & (kSoloWaves - 1)) == w;
      uint16_t al = 0;
      if (adds) al = gptr(pr.alpha)[t / SPLIT * 64 + lane];
      sums(t, min(t + G, n_pieces - 1), red + uint32_t(w) * 256u);
      __syncthreads();  // the tile's sums are complete (the next tile's go to the other buffer)
      if (!adds) continue;
      float s = 0.0f, rs = 0.0f;
      for (int k = 0; k < n_sl; ++k) s += lds_read<float>(red + uint32_t(k) * 256u + 4u * uint32_t(lane));
      for (int k = n_sl; k < n_here; ++k) rs += lds_read<float>(red + uint32_t(k) * 256u + 4u * uint32_t(lane));
      const float y = h2f(al) * s + rs;
      const int64_t row = int64_t(t / SPLIT) * 64 + lane;
      if (parts > 1)
        store_coherent(part + (int64_t(t) * parts + p) * 64 + lane, y);  // its arrival is counted after the last tile
      else if (row < pr.N && mine(t))
        ((gf32*)pr.y)[row] = y;
    }
  };
  if (slice_task) {
    // weights of a tile: 16-byte units as in tern_mfma.hip
    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(pr.trits), 0, int(uint32_t(n_tiles) * uint32_t(pr.n_groups) * (kTileRows * kGroupPacks)),
        kBufferWord3);
    const uint32_t tile_bytes = uint32_t(pr.n_groups) * (kTileRows * kGroupPacks);
    const uint32_t w_lo = uint32_t(min(task * kSliceGroups + kg, pr.n_groups - 1)) * (kTileRows * kGroupPacks) +
                          uint32_t(16 * (n16 >> 3) + (n16 & 7)) * kGroupPacks;
    u32x4 W[QN];
    auto load_w = [&](int q, int t) {  // q: of the piece
      W[q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wres, int(w_lo),
                                                                              int(uint32_t(t / SPLIT) * tile_bytes) + q_row(t % SPLIT * QN + q) * kGroupPacks, kAuxNT));
    };
    uint32_t xr[5], vr[5];
#pragma unroll
    for (int q = 0; q < QN; ++q) load_w(q, t0);
    // columns past the last read zero
    const __amdgpu_buffer_rsrc_t vsr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t*>(pr.vs), 0, int(4 * uint32_t(pr.n_groups) * kGroupCols), kBufferWord3);
    const __amdgpu_buffer_rsrc_t xsr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(pr.x), 0, int(2 * uint32_t(pr.K)), kBufferWord3);
    const int col0 = task * kSliceCols + 5 * lane;
    const u32x4 v4 = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(vsr, 4 * col0, 0, 0));
    vr[0] = v4.x;
    vr[1] = v4.y;
    vr[2] = v4.z;
    vr[3] = v4.w;
    vr[4] = __builtin_amdgcn_raw_buffer_load_b32(vsr, 4 * col0 + 16, 0, 0);
#pragma unroll
    for (int i = 0; i < 5; ++i) xr[i] = __builtin_amdgcn_raw_buffer_load_b16(xsr, 2 * col0 + 2 * i, 0, 0);
    table();
    // the digits' operands, which stay for the launch
    u32x4 D[4];
    u32x2 D2[4];
    uint32_t scv;
    float a[5], f[5];
    uint32_t ex, mx, top = 0;
    // (result rows 6 and 7 hold no digit: not read)
    const uint32_t r0 = uint32_t(n16 & 7) + 8u * uint32_t(kg);
    // the digits of f as the operands of the lanes that take them, through the wave's area
    auto operands = [&](auto nd, bool take, auto scale) {
      constexpr int ND = decltype(nd)::value;
      uint32_t P[ND], P1[ND], P2[ND];
      tern_digits<ND>(f, P);
      top = P[ND - 1];
      const uint32_t pi = uint32_t(lane >> 2) & 3u, pp = uint32_t(lane) & 3u;  // instruction and dword group of the pack
#pragma unroll
      for (int l = 0; l < ND; ++l) {
        P1[l] = quad_next(P[l]);
        P2[l] = quad_next2(P[l]);
      }
      // digit l is result row l; record (row, column group) of instruction i at (row + 8 group) ^ i
      if (pp == 0u) {
#pragma unroll
        for (int l = 0; l < ND; ++l) {
          const uint32_t rec = pi * 32u + ((uint32_t(l) + 8u * uint32_t(kg)) ^ pi);
          lds_write<u32x4>(area + rec * 16u, u32x4{P[l], P1[l] << 16, P1[l] >> 16, P2[l]});
          lds_write<uint8_t>(area + uint32_t(kSoloImg) + (uint32_t(l) + 8u * uint32_t(kg)) * 4u + pi, scale(l));
        }
      }
      if (pp == 3u) {
#pragma unroll
        for (int l = 0; l < ND; ++l) {
          const uint32_t rec = pi * 32u + ((uint32_t(l) + 8u * uint32_t(kg)) ^ pi);
          lds_write<u32x2>(area + uint32_t(kSoloImg1) + rec * 8u, u32x2{P[l] << 16, P[l] >> 16});
        }
      }
      asm volatile("" ::: "memory");  // (this wave's own area: in order)
      if (take) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t rec = uint32_t(i) * 32u + (r0 ^ uint32_t(i));
          D[i] = lds_read<u32x4>(area + rec * 16u);
          D2[i] = lds_read<u32x2>(area + uint32_t(kSoloImg1) + rec * 8u);
        }
        scv = lds_read<uint32_t>(area + uint32_t(kSoloImg) + r0 * 4u);
      }
      asm volatile("" ::: "memory");
    };
    tern_products(vr, xr, a);
    tern_fixed(a, f, ex, mx);
    operands(std::integral_constant<int, kDigits>{}, true, [&](int l) { return tern_scale(ex, mx, l); });  // result rows 8..15 repeat 0..7 ...
    const bool rest = tern_rest<kSoloRest>(a, f, ex, top);
    if (__builtin_expect(rest, 0))
      operands(std::integral_constant<int, kSoloRest>{}, n16 >= 8, [&](int l) { return tern_rest_scale<kSoloRest>(ex, mx, l); });  // ... or are the second set's
    __syncthreads();  // the decode table is complete
    walk([&](int t, int tn, uint32_t out) {
      (void)t;
      f32x4 C[QN];
#ifdef QTEA_DEBUG
      uint32_t bad = 0;
#endif
#pragma unroll
      for (int q = 0; q < QN; ++q) {
        const u32x4 o = W[q];
        uint32_t r[4], e[4][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = (n16 & 4) ? o[(k + 3) & 3] : o[k];
        if (QN == 1 && (t & 1)) {  // uniform
          const uint32_t r0 = r[0], r1 = r[1];
          r[0] = r[2];
          r[1] = r[3];
          r[2] = r0;
          r[3] = r1;
        }
        const int c = QN == 1 ? 0 : 2 * (q & 1);
        uint32_t U[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (QN == 1)  // an odd tile's dword rotation (by 2) was undone with the lane's
            U[i] = __builtin_amdgcn_perm(r[i], r[(i - 1) & 3], sel_rot);
          else
            U[i] = __builtin_amdgcn_perm(r[(i - c) & 3], r[(i - c - 1) & 3], sel_rot);
#ifdef QTEA_DEBUG
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (((U[i] >> (8 * k)) & 255u) >= uint32_t(kCodes)) bad |= 1u << q;
#endif
        }
        __builtin_amdgcn_sched_barrier(0);
        load_w(q, tn);  // in place, after the last read of the old bytes
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int k = 0; k < 4; ++k)
            e[i][k] = lds_read<uint32_t>(__builtin_amdgcn_perm(lane_tab, U[i], 0x0C0C0004u | (uint32_t(k) << 8)));
        C[q] = tern_mfma<0>(D[0], D2[0], e[0], zero4, scv);
        C[q] = tern_mfma<1>(D[1], D2[1], e[1], C[q], scv);
        C[q] = tern_mfma<2>(D[2], D2[2], e[2], C[q], scv);
        C[q] = tern_mfma<3>(D[3], D2[3], e[3], C[q], scv);
        asm volatile("" : "+v"(C[q]));  // (a use here: else the products sink and every decoded dword is held)
        __builtin_amdgcn_sched_barrier(0);
      }
#ifdef QTEA_DEBUG
      bad |= uint32_t(__shfl_xor(int(bad), 16));
      bad |= uint32_t(__shfl_xor(int(bad), 32));
#endif
#pragma unroll
      for (int q = 0; q < QN; ++q) {
        // lane group 0 holds digits 0..3, group 1 digits 4 and 5, group 2 the second set's
        const float s4 = C[q][0] + C[q][1];
        const float s6 = (s4 + C[q][2]) + C[q][3];
        const float mine = (kg & 1) ? s4 : s6;
        float s = mine + __shfl_xor(mine, 16);
        if (__builtin_expect(rest, 0)) s += __shfl(s6, lane | 32);  // (uniform; lane group 0's is stored)
#ifdef QTEA_DEBUG
        if ((bad >> q) & 1u) s = __builtin_nanf("");
#endif
        if (kg == 0) lds_write<float>(out + 4u * uint32_t(q_row(t % SPLIT * QN + q) + 16 * (n16 >> 3) + (n16 & 7)), s);
      }
    });
  } else if (res_task) {
    // its chunks of 32 columns: values and position words of a tile, and the
    // activations, which stay for the launch
    constexpr uint32_t VB = F8 ? 16u : 32u;
    const int s0 = (task - pr.n_slices) * 32 * cr;
    const int n_ch = min(cr, (nS - s0 + 31) / 32);
    const __amdgpu_buffer_rsrc_t vres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(pr.rval), 0, int(uint32_t(n_tiles) * uint32_t(nS) * VB), kBufferWord3);
    const __amdgpu_buffer_rsrc_t ires = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t*>(pr.ridx), 0, int(uint32_t(n_tiles) * uint32_t(nS) * 4u), kBufferWord3);
    u32x4 rvq[kSoloChunks] = {};
    uint32_t ris[kSoloChunks] = {};
    auto load_res = [&](int c, int t) {
      const uint32_t first = uint32_t(t) * uint32_t(nS) + uint32_t(s0 + 32 * c);
      if constexpr (F8) {
        const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(vres, 8 * lane, int(first * VB), 0));
        rvq[c] = u32x4{v.x, v.y, 0u, 0u};
      } else {
        rvq[c] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(vres, 16 * lane, int(first * VB), 0));
      }
      ris[c] = __builtin_amdgcn_raw_buffer_load_b32(ires, 4 * (lane & 31), int(4u * first), 0);
    };
    int scol[kSoloChunks][8];
#pragma unroll
    for (int c = 0; c < kSoloChunks; ++c)
      if (c < n_ch) {
        load_res(c, t0 / SPLIT);
#pragma unroll
        for (int h = 0; h < 8; ++h) scol[c][h] = gptr(pr.S)[min(s0 + 32 * c + 8 * kg + h, nS - 1)];
      }
    table();
    uint32_t X[kSoloChunks][4] = {};
    // selectors that put an activation's fp16 bits at the result row's position of a 64-bit word
    const uint32_t p4 = uint32_t(n16) & 3u, zz = 0x0c0c0c0cu;
    const uint32_t se = (p4 & 1u) ? 0x01000c0cu : 0x0c0c0100u, so = (p4 & 1u) ? 0x03020c0cu : 0x0c0c0302u;
    const uint32_t se0 = p4 < 2u ? se : zz, se1 = p4 < 2u ? zz : se, so0 = p4 < 2u ? so : zz, so1 = p4 < 2u ? zz : so;
#pragma unroll
    for (int c = 0; c < kSoloChunks; ++c)
      if (c < n_ch) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int s = s0 + 32 * c + 8 * kg + 2 * j;
          const uint32_t x0 = s < nS ? uint32_t(gptr(pr.x)[scol[c][2 * j]]) : 0u;
          const uint32_t x1 = s + 1 < nS ? uint32_t(gptr(pr.x)[scol[c][2 * j + 1]]) : 0u;
          X[c][j] = x0 | (x1 << 16);
        }
      }
    __syncthreads();
    walk([&](int, int tn, uint32_t out) {
      f32x4 acc = zero4;
#pragma unroll
      for (int c = 0; c < kSoloChunks; ++c) {
        if (c >= n_ch) break;  // uniform
        asm volatile("" ::: "memory");
        if constexpr (F8)
          lds_write<u32x2>(area + 8u * uint32_t(lane), u32x2{rvq[c].x, rvq[c].y});
        else
          lds_write<u32x4>(area + 16u * uint32_t(lane), rvq[c]);
        if (lane < 32) lds_write<uint32_t>(area + 1024u + 4u * uint32_t(lane), ris[c]);
        asm volatile("" ::: "memory");
        load_res(c, tn / SPLIT);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const u32x2 pw = lds_read<u32x2>(area + 1024u + 32u * uint32_t(kg) + 8u * j);
          uint32_t bw[4];
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            const uint32_t col = 8u * uint32_t(kg) + 2u * j + hh;
            uint32_t rb;
            if constexpr (F8) {
              // the magnitude bits at bits 7..13 are the fp16 bits of value * 2^-8
              const uint32_t v = lds_read<uint8_t>(area + 16u * col + uint32_t(n16));
              const _Float16 v8 = __builtin_bit_cast(_Float16, uint16_t(((v & 0x7fu) << 7) | ((v & 0x80u) << 8)));
              rb = __builtin_bit_cast(uint16_t, _Float16(v8 * _Float16(256.0f)));
            } else {
              rb = lds_read<uint16_t>(area + 32u * col + 2u * uint32_t(n16));
            }
            const uint32_t pos = __builtin_amdgcn_ubfe(hh ? pw.y : pw.x, 2u * uint32_t(n16), 2);
            const uint64_t v = uint64_t(rb) << (pos << 4);
            bw[2 * hh] = uint32_t(v);
            bw[2 * hh + 1] = uint32_t(v >> 32);
          }
          const uint32_t x2 = X[c][j];
          acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(
              as_half8(__builtin_amdgcn_perm(0u, x2, se0), __builtin_amdgcn_perm(0u, x2, se1),
                       __builtin_amdgcn_perm(0u, x2, so0), __builtin_amdgcn_perm(0u, x2, so1)),
              as_half8(bw[0], bw[1], bw[2], bw[3]), acc, 0, 0, 0);
        }
        asm volatile("" ::: "memory");
      }
      // result rows 0..3 (positions): lane n16 of group 0 holds rows 4 n16 .. 4 n16 + 3
      if (kg == 0) lds_write<f32x4>(out + 16u * uint32_t(n16), acc);
    });
  } else {  // no task: this wave only adds
    table();
    __syncthreads();
    walk([](int, int, uint32_t) {});
  }
  if (parts == 1) return;
  // the tiles this wave added: count the part's arrival, and add a tile's
  // parts where it is the last (not in the loop above: an atomic's round trip
  // would hold the next tile's barrier)
  __builtin_amdgcn_s_waitcnt(0);  // the parts are complete before their arrivals are counted
  for (int t = t0 + w * G; t < n_pieces; t += kSoloWaves * G) {
    uint32_t before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(counters + t, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    before = uint32_t(__builtin_amdgcn_readfirstlane(int(before)));
    if (before != uint32_t(parts - 1)) continue;
    if (lane == 0) __hip_atomic_store(counters + t, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    float v[8], sum = 0.0f;
    for (int k0 = 0; k0 < parts; k0 += 8) {
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = load_coherent(part + (int64_t(t) * parts + min(k0 + k, parts - 1)) * 64 + lane);
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k0 + k < parts) sum += v[k];
    }
    const int64_t row = int64_t(t / SPLIT) * 64 + lane;
    if (row < pr.N && mine(t)) ((gf32*)pr.y)[row] = sum;
  }
}

template <bool F8, int QN>
hipError_t launch(const GProblem& pr, const SoloShape& s, int max_wg, float* part, uint32_t* counters, hipStream_t st) {
  static std::atomic<int> done[kMaxDevices];
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(&tern_solo_kernel<F8, QN>), kSoloBytes, done);
  if (e != hipSuccess) return e;
  const int pieces = int(pr.n_pad >> 6) * s.split, G = std::max(1, std::min(pieces, max_wg / s.parts));
  hipLaunchKernelGGL((tern_solo_kernel<F8, QN>), dim3(uint32_t(G * s.parts)), dim3(kSoloWaves * 64), kSoloBytes, st, pr,
                     s.parts, s.chunks, part, counters);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_solo(const GProblem& pr, const SoloShape& s, int max_wg, bool f8, float* part, uint32_t* counters,
                       hipStream_t st) {
  if (s.split == 4)
    return f8 ? launch<true, 1>(pr, s, max_wg, part, counters, st) : launch<false, 1>(pr, s, max_wg, part, counters, st);
  if (s.split == 2)
    return f8 ? launch<true, 2>(pr, s, max_wg, part, counters, st) : launch<false, 2>(pr, s, max_wg, part, counters, st);
  return f8 ? launch<true, 4>(pr, s, max_wg, part, counters, st) : launch<false, 4>(pr, s, max_wg, part, counters, st);
}

}  // namespace qtea_grouped
