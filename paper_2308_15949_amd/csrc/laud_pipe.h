// The convolutions of the block as gathered implicit GEMMs for many rows, on gfx950 MFMA: k_pipe<MODE, ET, BM, BN, WM, WN, KS, NS>
// computes a BM x BN output tile; modes and arguments are those of laud_gemm.h.
//
// These launches are short (tens of microseconds) and their operands come out of the L2, so what bounds them is how many
// bytes a compute unit keeps in flight: both operands reach LDS with LDS-direct 16-byte loads -- no registers hold a slice on
// its way -- into a ring of NS slices of 128 bytes a row, NS - 1 of them under way.  A chunk that must read as zero (outside the
// image, past K, past the last row) has the top bit of its offset set, which lies outside the operand's descriptor.
//   Chunk c of row r lies at position c ^ (r & 7) ^ ((r >> 3) & 1) of the row's eight: fragment reads are free of bank
// conflicts; the swizzle is applied to the global address.  One barrier per slice, in the middle of its MFMAs: behind it every
// wave's part of the next slice has landed and everyone is done with the slice before, whose place is refilled.  Fragments are
// read one K step ahead of their MFMAs, across slices too.
//   The MFMAs compute the transposed tile (weights first): a lane holds 4 x 4 consecutive channels of one row, so that after one
// lane swap per register pair results leave, and residuals come, in 32-byte pieces without a transpose through LDS; from the large tiles
// they go through LDS (TURN).
//   KS = 2: the waves form two groups that share the slices and take two of a slice's four K steps each; their sums meet in LDS
// (first group plus second, always).
//
// Vector-memory waits: the LDS-direct loads are issued from inline assembly, so every wait for them is explicit; it counts the
// loads a wave issued behind the ones needed (loads return in order).
#pragma once

#include "laud_common.h"
#include "laud_gemm.h"
#include "laud_tail_pack.h"
#include "laud_tile_util.h"

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace laud {

struct PipeArgs {
  GemmArgs g;
  int ring;  // bytes of the ring: NS slices, or all there are (1x1s only)
  FastDiv ct, tpg, s, ss, pps, wp, howo, wo, grp;
};

namespace pipe {
constexpr unsigned kOob = 0x80000000u;
constexpr int kMaxGroups = 1024;  // channel-skip decisions per sample the kernels can hold in LDS
template <int BM, int BN, int NS> __host__ __device__ constexpr int ring_bytes() { return NS * (BM + BN) * 128; }
// behind the ring: scale, shift [BN] floats; offset, unreadable taps, output row [BM]; then per mode: SD1 inactive [BM], channel
// skipping the kept groups, DENSE1 the masker's weights [K to whole slices]
template <int MODE, int BM, int BN, int NS> __host__ __device__ constexpr int lds_bytes() {
  return ring_bytes<BM, BN, NS>() + 2 * BN * 4 + 3 * BM * 4 + (MODE == M_SD1 ? BM * 4 : 0) +
         (MODE >= M_CS1 && MODE <= M_CS3 ? kMaxGroups * 4 + 16 : 0);
}
// A 1x1 of fewer than NS slices takes the LDS of those: such launches are bound by memory, and what a compute unit keeps in flight goes
// with the workgroups it holds, tiles and copies alike.  Last 1x1 with the whole ring / here: 128 images of 56 x 56 x 64, one slice, out of
// place at 0.15 77.7 / 49.8 us; stage 2 of 128 images, two slices, in place at 0.5 29.0 / 26.5 us; float32 stage 1 of 32 images out of
// place at 0.86 67.8 / 54.4.
template <int MODE, int KS> __host__ __device__ constexpr bool short_ring() {
  return KS == 1 && (MODE == M_CONV1 || MODE == M_CONV3 || MODE == M_DENSE1 || MODE == M_SD1 || MODE == M_SD3);
}
// ... the masker's weights: K floats to whole slices, brought in pieces of 64
constexpr int kMaxMaskerK = 4096;
template <typename ET> __host__ __device__ constexpr int masker_bytes(int K) {
  return ((K + 8 * elem<ET>::per16 - 1) / (8 * elem<ET>::per16) * (8 * elem<ET>::per16) + 63) / 64 * 256;
}
}  // namespace pipe

// Waits until all but the `behind` slices requested last (0 .. MOST of them, L loads each, and RL loads more behind those) have landed.
template <int MOST, int L, int RL>
__device__ __forceinline__ void wait_tail(int behind) {
  if constexpr (MOST <= 0) {
    vm_wait<RL>();
  } else {
    if (behind >= MOST) vm_wait<MOST * L + RL>();
    else wait_tail<MOST - 1, L, RL>(behind);
  }
}

template <int MODE, typename ET, int BM, int BN, int WM, int WN, int KS, int NS>
__global__ __launch_bounds__(64 * WM * WN * KS) void k_pipe(const PipeArgs ka) {
  using namespace pipe;
  prefetch_args<sizeof(PipeArgs)>();
  const GemmArgs& a = ka.g;
  constexpr int NW = WM * WN * KS, NT = 64 * NW;
  constexpr int EPC = elem<ET>::per16, ES = (int)sizeof(ET), BKE = 8 * EPC;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32, NB = TM * TN;
  constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW, L = LA + LB;  // LDS-direct instructions per wave and slice (8 rows each)
  constexpr int KG = 4 / KS;                                      // K steps of a slice one wave takes
  constexpr int STAGE = (BM + BN) * 128;
  static_assert(NW % 2 == 0 && LA >= 1 && LB >= 1 && TM >= 1 && TN >= 1 && NT >= BM && NS >= 3, "tile and waves do not fit");
  static_assert(KS == 1 || (KS == 2 && NB % 2 == 0), "the two K groups share the result blocks");
  static_assert(MODE != M_DENSE1 || KS == 1, "the K groups' exchange would overwrite the projection's partial sums while other waves read them");
  constexpr bool TAPS = (MODE == M_CONV2 || MODE == M_CS2 || MODE == M_U2 || MODE == M_SD2 || MODE == M_G2);
  constexpr bool CS = (MODE >= M_CS1 && MODE <= M_CS3);
  constexpr bool RES = (MODE == M_CONV3 || MODE == M_CS3 || MODE == M_SD3);
  // Results of the tiles that have a compute unit to themselves pass through LDS on their way to memory, and residuals come the way they
  // leave: four lanes on 64 bytes of a row.  Straight from the accumulators a lane holds 32 bytes of a row of its own, and the compute
  // unit's path takes 16 bytes a cycle of those: ResNet stage 4 of 128 images, first block's 1x1s 37.6 / 36.2 -> 35.4 / 34.7 us, its 3x3
  // 39.6 -> 37.1, last 1x1 26.3 -> 25.2, an identity block's 3x3 27.5 -> 26.0 (a dozen passes; without a pause and on changing inputs,
  // where the clock is lower and the input cold, 45.1 / 43.2 -> 44.1 / 43.0, 42.5 -> 42.0).  Smaller tiles, several a compute unit, hide it, and
  // the round through LDS costs them (channel skipping of stage 1, last 1x1: 54.1 -> 55.4).
  constexpr bool TURN = ES == 2 && NT == 512 && !(MODE >= M_U1 && MODE <= M_U3);
  constexpr bool LISTED = (MODE == M_CONV1 || MODE == M_CONV2 || MODE == M_CONV3 || MODE == M_G2 || MODE == M_U1 || MODE == M_U2 || MODE == M_U3);
  extern __shared__ __align__(16) unsigned char smem[];
  const int tab = short_ring<MODE, KS>() ? ka.ring : ring_bytes<BM, BN, NS>();
  float* const s_scale = reinterpret_cast<float*>(smem + tab);
  float* const s_shift = s_scale + BN;
  unsigned* const s_voff = reinterpret_cast<unsigned*>(s_shift + BN);
  unsigned* const s_bad = s_voff + BM;
  int* const s_row = reinterpret_cast<int*>(s_bad + BM);
  int* const s_extra = s_row + BM;
  float* const s_wm = reinterpret_cast<float*>(s_extra);  // DENSE1
  const int wm_off = tab + 2 * BN * 4 + 3 * BM * 4;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, lhi = lane >> 5, l8 = lane >> 3, l7 = lane & 7;
  const int ks = wave / (WM * WN), wv = wave % (WM * WN), wm = wv / WN, wn = wv % WN;
  if constexpr (MODE == M_CONV1 || MODE == M_DENSE1) {
    if (a.pk_out != nullptr && (int)blockIdx.x >= a.pk_first_block) {
      const int nextra = (int)gridDim.x - a.pk_first_block;
      for (int idx = ((int)blockIdx.x - a.pk_first_block) * NT + tid; idx < a.pk_chunks; idx += nextra * NT)
        tail_pack_chunk(idx, (const uint4*)a.pk_w2, (const uint4*)a.pk_w3, (uint4*)a.pk_out);
      return;
    }
  }
  if constexpr (MODE == M_CONV3) {
    if (a.cp.nblocks && (int)blockIdx.x >= a.cp.first) {
      copy_inactive_part<NT>(a.cp, blockIdx.x - a.cp.first, a.cp.nblocks, smem);
      return;
    }
  }
  // ---- which tile ---------------------------------------------------------------------------
  int rt, ct, sample = 0, M;
  const int32_t* listp = a.list;
  if constexpr (!CS) {
    // consecutive workgroup ids go round-robin over the 8 XCDs: the column tiles of one row tile (same rows of A) are given to
    // the same XCD, one after the other
    const int s = blockIdx.x >> 3, r8 = fast_div(s, ka.ct);
    rt = r8 * 8 + (blockIdx.x & 7);
    ct = s - r8 * a.col_tiles;
    if (rt >= a.row_tiles) return;
    if constexpr (MODE == M_CONV1) {
      // the dilated pixel lists are per group of samples: tile -> (group, tile within the group)
      const int g = fast_div(rt, ka.tpg);
      rt -= g * a.tiles_per_group;
      listp += (size_t)g * a.group_rows;
      M = a.count[g] * (a.hw ? a.hw : 1);
    } else if constexpr (LISTED) {
      M = *a.count * (MODE == M_U1 ? (a.S + 2) * (a.S + 2) : a.S * a.S);
    } else {
      M = a.m_rows;
    }
  } else {
    ct = blockIdx.x / a.row_tiles;
    rt = blockIdx.x - ct * a.row_tiles;
    sample = blockIdx.y;
    M = a.H * a.W;
  }
  const int row0 = rt * BM, col0 = ct * BN;
  if (row0 >= M) return;

  // ---- channel skipping: kept-group list of this sample (ballot + prefix, one wave) ----------
  int ncols = a.Ncols, keff = a.K;
  if constexpr (CS) {
    if (wave == 0) {
      int base = 0;
      for (int g0 = 0; g0 < a.D; g0 += kWave) {
        const int g = g0 + lane;
        const bool f = g < a.D && a.cmask[(size_t)sample * a.D + g] != 0;
        const unsigned long long b = __ballot(f);
        if (f) s_extra[base + ballot_prefix(b)] = g;
        base += __popcll(b);
      }
      if (lane == 0) s_extra[kMaxGroups] = base;
    }
    __syncthreads();
    const int kw = __builtin_amdgcn_readfirstlane(s_extra[kMaxGroups]) * a.G;
    if (MODE != M_CS3) ncols = kw;
    if (MODE != M_CS1) keff = kw;
    if (col0 >= ncols) return;
  }
  auto kept = [&](int c) __attribute__((always_inline)) -> int {  // channel of position c among the kept ones
    const int g = fast_div(c, ka.grp);
    return s_extra[g] * a.G + (c - g * a.G);
  };
  // group convolution: the reduction runs over the input channels col0 .. col0+BN-1 (the groups of this tile's output channels;
  // a tile holds whole groups)
  if constexpr (MODE == M_G2) keff = min(BN, a.K - col0);

  // ---- operands -------------------------------------------------------------------------------
  // Instruction i of wave w loads rows 8 (w + NW i) .. +7 of a slice of either operand, lane l position l % 8 of row .. + l / 8.
  // The taps reach one row and one pixel back: A's descriptor starts that far before it.
  const int rowW = MODE == M_U2 ? a.S + 2 : a.W;
  const long long ashift = TAPS ? (long long)(rowW + 1) * a.lda * ES : 0;
  const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(reinterpret_cast<const char*>(a.A)) - ashift, 0, (int)kOob, 0x00020000);
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.Wt), 0, (int)kOob, 0x00020000);
  const int chunk = l7 ^ l8 ^ (wave & 1);
  const unsigned ldsw = (unsigned)wave * 1024u;
  const int kchunks = (keff + BKE - 1) / BKE;
  const int KT = (TAPS ? 9 : 1) * kchunks;
  const unsigned lastbad = (kchunks - 1) * BKE + chunk * EPC < keff ? 0u : kOob;  // only a tap's last slice can be partial

  // affine of the tile's columns (columns past the end: zeros), masker weights
  for (int p = wave; p < 2 * BN / 64; p += NW) {
    const int c = (p % (BN / 64)) * 64 + lane, col = col0 + c;
    int ch = col;
    if constexpr (MODE == M_CS1 || MODE == M_CS2) ch = col < ncols ? kept(col) : 0;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(p < BN / 64 ? a.scale : a.shift), 0, a.Ncols * 4, 0x00020000);
    dma4(rs, col < ncols ? (unsigned)ch * 4u : kOob, 0, (unsigned)(tab + p * 256));
  }
  const bool do_proj = MODE == M_DENSE1 && ct == 0 && a.wmask != nullptr;
  if constexpr (MODE == M_DENSE1) {
    if (do_proj) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.wmask), 0, a.K * 4, 0x00020000);
      for (int p = wave; p < (kchunks * BKE + 63) / 64; p += NW) dma4(rs, (unsigned)(p * 64 + lane) * 4u, 0, (unsigned)(wm_off + p * 256));
    }
  }

  // ---- weight rows ----------------------------------------------------------------------------
  unsigned voffW[LB];
  int wrel[LB];
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    const int c = col0 + 8 * (wave + NW * i) + l8;
    int wr = c < ncols ? c : col0;  // a column past the end re-reads the tile's first row: its result is dropped
    wrel[i] = 0;
    if constexpr (MODE == M_CS1 || MODE == M_CS2) wr = kept(wr);
    if constexpr (MODE == M_G2) {
      wrel[i] = col0 + chunk * EPC - (wr & ~(a.gw - 1));  // chunk's first channel inside the row's group (widths are powers of two)
      voffW[i] = (unsigned)(wr * a.ldw * ES);
    } else if constexpr (MODE == M_CS2 || MODE == M_CS3) {
      voffW[i] = (unsigned)(wr * a.ldw * ES);
    } else {
      voffW[i] = (unsigned)(wr * a.ldw * ES + chunk * 16);
    }
  }
  // Slices in order: K chunk after K chunk, tap after tap.  A wave issues a dozen scalar and vector instructions a slice beside its
  // loads, and these stand between its MFMAs: what changes from tap to tap only is worked out there.
  constexpr bool WLANE = (MODE == M_G2 || MODE == M_CS2 || MODE == M_CS3);  // the position inside a tap goes into the per-lane offset
  const bool ragged = __builtin_amdgcn_readfirstlane(keff % BKE) != 0;
  const int pix_b = a.lda * ES, back_b = (kchunks - 1) * 128;  // from a tap's last slice back to its first
  const int a_pixjump = pix_b - back_b, a_rowjump = (rowW - 2) * pix_b - back_b;
  const int w_tapjump = WLANE ? (MODE == M_G2 ? a.gw : a.K) * ES : a.K * ES - back_b;
  int ld_kc = 0, ld_tap = 0, ld_kx = 0;
  unsigned a_off = 0, w_off = 0, to = 0;         // of the next slice to request: in A, in the weights, its stage
  unsigned voffA[LA], abad[LA], vA[LA], vW[LB];  // abad: bit t set = tap t reads as zero (bit 0 outside the tap modes)
  auto set_weights = [&]() __attribute__((always_inline)) {
    const unsigned kbad = ld_kc == kchunks - 1 ? lastbad : 0u;
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      vW[i] = voffW[i] | kbad;
      if constexpr (MODE == M_CS2 || MODE == M_CS3) {
        vW[i] = (voffW[i] + (unsigned)kept(max(min(ld_kc * BKE + chunk * EPC, keff - EPC), 0)) * (unsigned)ES) | kbad;
      } else if constexpr (MODE == M_G2) {
        const int rel = wrel[i] + ld_kc * BKE;
        vW[i] = (voffW[i] + (unsigned)(rel * ES)) | ((unsigned)(rel | (a.gw - 1 - rel)) & kOob) | kbad;
      }
    }
  };
  auto set_rows = [&]() __attribute__((always_inline)) {
    const unsigned kbad = ld_kc == kchunks - 1 ? lastbad : 0u;
#pragma unroll
    for (int i = 0; i < LA; ++i) vA[i] = voffA[i] | kbad | ((abad[i] << (31 - (TAPS ? ld_tap : 0))) & kOob);
  };
  auto issue_W = [&]() __attribute__((always_inline)) {
    const unsigned dst = __builtin_amdgcn_readfirstlane(to + ldsw + BM * 128), src = __builtin_amdgcn_readfirstlane(w_off);
#pragma unroll
    for (int i = 0; i < LB; ++i) dma16(wrsrc, vW[i], src, dst + NW * i * 1024);
  };
  auto issue_A = [&]() __attribute__((always_inline)) {
    const unsigned dst = __builtin_amdgcn_readfirstlane(to + ldsw), src = __builtin_amdgcn_readfirstlane(a_off);
#pragma unroll
    for (int i = 0; i < LA; ++i) dma16(arsrc, vA[i], src, dst + NW * i * 1024);
  };
  auto advance = [&]() __attribute__((always_inline)) {  // (all but the stage)
    ++ld_kc;
    a_off += 128;
    if constexpr (!WLANE) w_off += 128;
    if (TAPS && ld_kc == kchunks) {
      ld_kc = 0;
      ++ld_tap;
      const bool rowwrap = ld_kx == 2;
      ld_kx = rowwrap ? 0 : ld_kx + 1;
      a_off += (rowwrap ? a_rowjump : a_pixjump) - 128;
      w_off += w_tapjump - (WLANE ? 0 : 128);
      set_rows();
      if (ragged || (WLANE && kchunks > 1)) set_weights();
    } else if (ragged || (WLANE && MODE != M_G2) || (MODE == M_G2 && kchunks > 1)) {
      set_rows();
      set_weights();
    }
  };
  set_weights();
  if (KT > 0) issue_W();  // (the weights of the first slice: they depend on nothing but the tile)

  // ---- rows: one thread looks a row up for the workgroup ----------------------------------------
  if (tid < BM) {
    const int rho = row0 + tid;
    const bool live = rho < M;
    const int Hp = fast_div(a.stride > 1 ? a.Ho : a.H, ka.s), Wp = fast_div(a.stride > 1 ? a.Wo : a.W, ka.s);
    int y = 0, x = 0, o = rho, inact = 1;
    unsigned pix = (unsigned)rho;
    if (live) {
      if constexpr (MODE == M_CONV1) {
        if (a.hw) {
          const int p = fast_div(rho, ka.howo);
          o = a.list[p] * a.hw + (rho - p * a.hw);
        } else {
          o = listp[rho];
        }
        pix = (unsigned)o;
      } else if constexpr (MODE == M_CONV2 || MODE == M_G2 || MODE == M_CONV3) {
        const int p = fast_div(rho, ka.ss), j = rho - p * (a.S * a.S), q = a.list[p];
        const int n = fast_div(q, ka.pps), r2 = q - n * (Hp * Wp), py = fast_div(r2, ka.wp), px = r2 - py * Wp, jy = fast_div(j, ka.s);
        const int yo = py * a.S + jy, xo = px * a.S + (j - jy * a.S);
        if constexpr (MODE == M_CONV3) {
          o = (n * (a.stride > 1 ? a.Ho : a.H) + yo) * (a.stride > 1 ? a.Wo : a.W) + xo;
        } else {
          const int sy = a.stride > 1 ? a.stride : 1;
          y = yo * sy;  // centre of the 3x3 on the input grid
          x = xo * sy;
          pix = (unsigned)((n * a.H + y) * a.W + x);
        }
      } else if constexpr (MODE == M_SD1 || MODE == M_SD2) {
        const int n = fast_div(rho, ka.howo), r2 = rho - n * (a.Ho * a.Wo), yo = fast_div(r2, ka.wo), xo = r2 - yo * a.Wo;
        y = yo * a.stride;
        x = xo * a.stride;
        pix = (unsigned)((n * a.H + y) * a.W + x);
        if constexpr (MODE == M_SD1) {
          // shortcut of a dynamic first block: the activation is applied here only where the branch will not be added
          // (inactive patches); active rows get it in the last conv's epilogue
          if (a.list != nullptr) {
            const int q = (n * Hp + fast_div(yo, ka.s)) * Wp + fast_div(xo, ka.s);
            const int cnt = *a.count;
            const int pos = lower_bound_dev(a.list, cnt, q);
            inact = !(pos < cnt && a.list[pos] == q);
          }
        }
      } else {
        pix = (unsigned)source_row<MODE>(a, rho, sample, y, x);
        o = output_row<MODE>(a, rho, sample, Hp, Wp);
      }
    }
    unsigned mk = ~0u;
    if constexpr (TAPS && MODE != M_U2)
      mk = ((y > 0 ? 0x7u : 0u) | 0x38u | (y < a.H - 1 ? 0x1c0u : 0u)) & ((x > 0 ? 0x49u : 0u) | 0x92u | (x < a.W - 1 ? 0x124u : 0u));
    s_voff[tid] = live ? (pix * (unsigned)a.lda + (unsigned)(MODE == M_G2 ? col0 : 0)) * (unsigned)ES : 0u;
    s_bad[tid] = live ? ~mk : ~0u;
    s_row[tid] = live ? o : -1;
    if constexpr (MODE == M_SD1) s_extra[tid] = inact;
  }
  lds_wait();
  wg_barrier();
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = 8 * (wave + NW * i) + l8;
    voffA[i] = s_voff[r] + (unsigned)chunk * 16u;
    abad[i] = s_bad[r];
  }
  set_rows();
  // the residual of this wave's blocks is requested right behind the last slice (ahead of the slices it would delay them)
  constexpr int NBO = NB / KS;             // blocks a wave finishes
  constexpr int RPB = ES == 4 ? 4 : 2;     // 16-byte pieces of a block per lane
  constexpr int RL = RES ? NBO * RPB : 0;  // loads that stand behind the last slice's
  uint4 res[RES ? NBO * RPB : 1];
  auto load_res = [&]() __attribute__((always_inline)) {
    if constexpr (RES) {
#pragma unroll
      for (int bb = 0; bb < NBO; ++bb) {
        const int i = (ks * NBO + bb) / TN, j = (ks * NBO + bb) % TN;
#pragma unroll
        for (int u = 0; u < RPB; ++u) {  // (columns past the end read valid ones; nothing is stored there)
          const int rl = wm * (BM / WM) + 32 * i + (TURN ? 16 * u + (lane >> 2) : l31);
          const int col = col0 + wn * (BN / WN) + 32 * j + (TURN ? 8 * (lane & 3) : ES == 4 ? 8 * u + 4 * lhi : 16 * lhi + 8 * u);
          res[bb * RPB + u] = *reinterpret_cast<const uint4*>((const ET*)a.Res + (size_t)max(s_row[rl], 0) * a.ldo + min(col, ncols - EPC));
        }
      }
    }
  };
  if (KT > 0) {
    issue_A();
    advance();
  }
#pragma unroll
  for (int s = 1; s < NS - 1; ++s)
    if (s < KT) {
      to = s * STAGE;
      issue_W();
      issue_A();
      advance();
    }
  if (KT <= NS - 1) load_res();

  // ---- fragments: row lane % 32 of a 32-row block, chunk 2 kg + lane / 32, swizzled -------------------------------------
  unsigned pa[KG], pb[KG];  // addresses inside a stage
#pragma unroll
  for (int kk = 0; kk < KG; ++kk) {
    const unsigned swz = (unsigned)l31 * 128u + (((unsigned)(2 * (ks * KG + kk) + lhi) ^ (unsigned)(l31 & 7) ^ ((unsigned)(l31 >> 3) & 1u)) << 4);
    pa[kk] = swz + wm * (BM / WM) * 128;
    pb[kk] = swz + BM * 128 + wn * (BN / WN) * 128;
  }
  f32x16 acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[b][e] = 0.f;
  float psum[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) psum[i] = 0.f;
  uint4 fa[2][TM], fb[2][TN];
  auto read_frags = [&](int buf, unsigned stage, int kk) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[buf][j] = *reinterpret_cast<const uint4*>(smem + (stage + pb[kk]) + j * 4096);
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[buf][i] = *reinterpret_cast<const uint4*>(smem + (stage + pa[kk]) + i * 4096);
  };
  if (KT > NS - 1) vm_wait<(NS - 2) * L>();
  else wait_tail<NS - 2, L, RL>(KT - 1);
  wg_barrier();
  unsigned stage = 0;  // of the slice at hand; the one before it (at first: the last) is the next to be refilled
  to = (NS - 1) * STAGE;
  read_frags(0, 0, 0);
  // One slice; FULL: another one is requested.
  auto slice = [&](int s, auto full) __attribute__((always_inline)) {
    constexpr bool FULL = decltype(full)::value;
    const bool wrap = stage == (NS - 1) * STAGE || (short_ring<MODE, KS>() && !FULL && s + 1 == KT);
    const unsigned next = wrap ? 0u : stage + STAGE;
#pragma unroll
    for (int kk = 0; kk < KG; ++kk) {
      const int buf = kk & 1;
      if (kk < KG - 1) read_frags(buf ^ 1, stage, kk + 1);
      else read_frags(buf ^ 1, next, 0);  // (behind the last slice: read and not used)
      __builtin_amdgcn_sched_barrier(0);  // the next step's fragment reads stay ahead of this step's MFMAs
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) mma16<ET>(acc[i * TN + j], fb[buf][j], fa[buf][i]);
      if constexpr (MODE == M_DENSE1) {
        // the masker projection, from the fragments at hand: of the WN waves that hold these rows one takes this K step
        if (do_proj && kk % WN == wn) {
          const float* wk = s_wm + s * BKE + (2 * (ks * KG + kk) + lhi) * EPC;
          float wf[EPC];
#pragma unroll
          for (int u = 0; u < EPC / 4; ++u) {
            const float4 t4 = reinterpret_cast<const float4*>(wk)[u];
            wf[4 * u] = t4.x; wf[4 * u + 1] = t4.y; wf[4 * u + 2] = t4.z; wf[4 * u + 3] = t4.w;
          }
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            ET xe[EPC];
            __builtin_memcpy(xe, &fa[buf][i], 16);
#pragma unroll
            for (int e = 0; e < EPC; ++e) psum[i] += elem<ET>::load(&xe[e]) * wf[e];
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (kk == KG / 2 - 1) {
        // slice s + 1 is needed from the end of this one on; those requested behind it, up to s + NS - 2, are younger
        if constexpr (FULL) vm_wait<(NS - 3) * L>();
        else wait_tail<NS - 3, L, RL>(KT - 2 - s);
        wg_barrier();
        if constexpr (FULL) issue_A();
      }
      if (FULL && kk == KG / 2) {
        issue_W();
        advance();
      }
    }
    to = stage;
    stage = next;
  };
  int s = 0;
  for (; s + NS - 1 < KT; ++s) slice(s, std::true_type{});
  if (KT > NS - 1) load_res();
  for (; s < KT; ++s) slice(s, std::false_type{});

  if (TURN || do_proj || KS == 2) {
    lds_wait();
    wg_barrier();  // everyone is done with the slices
  }

  // ---- the masker projection: two K halves of a row in lanes l and l + 32, then the waves that share the rows -----------
  if constexpr (MODE == M_DENSE1) {
    if (do_proj) {
      float* const s_part = reinterpret_cast<float*>(smem);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const float v = psum[i] + __shfl_xor(psum[i], 32, kWave);
        if (lhi == 0) s_part[(ks * WN + wn) * BM + wm * (BM / WM) + 32 * i + l31] = v;
      }
      lds_wait();
      wg_barrier();
      if (tid < BM && row0 + tid < M) {
        float p = 0.f;
#pragma unroll
        for (int w = 0; w < WN * KS; ++w) p += s_part[w * BM + tid];
        a.proj[row0 + tid] = p;
      }
    }
  }
  // ---- KS = 2: each group hands the other the blocks that one finishes --------------------------------------------------
  if constexpr (KS == 2) {
    uint4* const xch = reinterpret_cast<uint4*>(smem) + (size_t)wv * (NBO * 4 * 64) + lane;
    constexpr int GRP = WM * WN * NBO * 4 * 64;
#pragma unroll
    for (int b = 0; b < NBO; ++b)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        uint4 t;
        if (ks == 0) __builtin_memcpy(&t, reinterpret_cast<const char*>(&acc[NBO + b]) + 16 * u, 16);
        else __builtin_memcpy(&t, reinterpret_cast<const char*>(&acc[b]) + 16 * u, 16);
        xch[ks * GRP + (b * 4 + u) * 64] = t;
      }
    lds_wait();
    wg_barrier();
#pragma unroll
    for (int b = 0; b < NBO; ++b)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint4 t = xch[(ks ^ 1) * GRP + (b * 4 + u) * 64];
        const float f[4] = {__uint_as_float(t.x), __uint_as_float(t.y), __uint_as_float(t.z), __uint_as_float(t.w)};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float mine = ks == 0 ? acc[b][4 * u + e] : acc[NBO + b][4 * u + e];
          acc[b][4 * u + e] = mine + f[e];
        }
      }
  }

  // ---- epilogue ---------------------------------------------------------------------------------
  const float floor_ = act_floor(a.relu);
#pragma unroll
  for (int bb = 0; bb < NBO; ++bb) {
    const int i = (ks * NBO + bb) / TN, j = (ks * NBO + bb) % TN;
    const int rl = wm * (BM / WM) + 32 * i + l31, cb = wn * (BN / WN) + 32 * j;
    int orow = s_row[rl];
    bool zero_row = false;
    if constexpr (MODE == M_U1) {
      if (orow <= -2) { orow = -2 - orow; zero_row = true; }
    }
    float v[16];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 sc = *reinterpret_cast<const float4*>(s_scale + cb + 8 * g + 4 * lhi);
      const float4 sh = *reinterpret_cast<const float4*>(s_shift + cb + 8 * g + 4 * lhi);
      v[4 * g + 0] = acc[bb][4 * g + 0] * sc.x + sh.x;
      v[4 * g + 1] = acc[bb][4 * g + 1] * sc.y + sh.y;
      v[4 * g + 2] = acc[bb][4 * g + 2] * sc.z + sh.z;
      v[4 * g + 3] = acc[bb][4 * g + 3] * sc.w + sh.w;
    }
    if constexpr (MODE == M_SD1) {
      if (a.relu && s_extra[rl]) {
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = fmaxf(v[e], 0.f);
      }
    } else if constexpr (!RES && MODE != M_U3) {
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = fmaxf(v[e], 0.f);
    }
    if (zero_row) {
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = 0.f;
    }
    if constexpr (ES == 4 || MODE == M_U3) {  // (the unfused schedule's branch output stays float32)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int col = col0 + cb + 8 * g + 4 * lhi;
        if (orow >= 0 && col < ncols) {
          float4 o = make_float4(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]);
          const size_t off = (size_t)orow * a.ldo + col;
          if constexpr (RES) {
            const uint4 r = res[bb * RPB + g];
            o.x += __uint_as_float(r.x); o.y += __uint_as_float(r.y); o.z += __uint_as_float(r.z); o.w += __uint_as_float(r.w);
            if (a.relu) { o.x = fmaxf(o.x, 0.f); o.y = fmaxf(o.y, 0.f); o.z = fmaxf(o.z, 0.f); o.w = fmaxf(o.w, 0.f); }
          }
          *reinterpret_cast<float4*>((float*)a.Out + off) = o;
        }
      }
    } else if constexpr (TURN) {
      // through LDS of the wave's own (its operations stay in order), in the ring's bytes: four lanes then hold 64 bytes of a row
      constexpr int kBuf = RES ? kTurnBytes : kTurnBytes / 2;
      constexpr int kTurnOff = KS == 2 ? 2 * WM * WN * NBO * 4096 : MODE == M_DENSE1 ? 4096 : 0;  // (behind the exchange, the partial sums)
      static_assert(kTurnOff + NW * kBuf <= (short_ring<MODE, KS>() ? 1 : NS) * STAGE && (MODE != M_DENSE1 || WN * BM * 4 <= kTurnOff), "the turning buffers");
      unsigned char* const turn = smem + kTurnOff + wave * kBuf;
      const int col = col0 + cb + 8 * (lane & 3);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if constexpr (RES) {
          *reinterpret_cast<float4*>(turn + turn_put(lane, g)) = make_float4(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]);
        } else {
          *reinterpret_cast<u32x2*>(turn + row_put(lane, g)) = u32x2{pack_bf16(v[4 * g], v[4 * g + 1]), pack_bf16(v[4 * g + 2], v[4 * g + 3])};
        }
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        u32x4 o;
        if constexpr (RES) {
          const uint4 r = res[bb * RPB + q];
          const unsigned ru[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const float4 x = *reinterpret_cast<const float4*>(turn + turn_get(lane, q, h));
            o[2 * h] = pack_bf16(fmaxf(x.x + __uint_as_float(ru[2 * h] << 16), floor_), fmaxf(x.y + __uint_as_float(ru[2 * h] & 0xffff0000u), floor_));
            o[2 * h + 1] = pack_bf16(fmaxf(x.z + __uint_as_float(ru[2 * h + 1] << 16), floor_), fmaxf(x.w + __uint_as_float(ru[2 * h + 1] & 0xffff0000u), floor_));
          }
        } else {
          o = *reinterpret_cast<const u32x4*>(turn + row_get(lane, q));
        }
        const int row = s_row[wm * (BM / WM) + 32 * i + 16 * q + (lane >> 2)];
        if (row >= 0 && col < ncols) *reinterpret_cast<u32x4*>((ET*)a.Out + (size_t)row * a.ldo + col) = o;
      }
    } else {
      to_consecutive_channels(v);  // 0-3, 8-11, 4-7, 12-15: channels 16 lhi + 0 .. 15
      const float yv[16] = {v[0], v[1], v[2], v[3], v[8], v[9], v[10], v[11], v[4], v[5], v[6], v[7], v[12], v[13], v[14], v[15]};
      const int col = col0 + cb + 16 * lhi;
      const size_t off = (size_t)max(orow, 0) * a.ldo + col;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (orow >= 0 && col + 8 * h < ncols) {
          unsigned pk[4];
          uint4 r = make_uint4(0, 0, 0, 0);
          if constexpr (RES) r = res[bb * RPB + h];
          const unsigned ru[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            float lo = yv[8 * h + 2 * d], hi = yv[8 * h + 2 * d + 1];
            if constexpr (RES) {
              lo += __uint_as_float(ru[d] << 16);
              hi += __uint_as_float(ru[d] & 0xffff0000u);
              if (a.relu) { lo = fmaxf(lo, 0.f); hi = fmaxf(hi, 0.f); }
            }
            pk[d] = pack_bf16(lo, hi);
          }
          *reinterpret_cast<uint4*>((ET*)a.Out + off + 8 * h) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        }
      }
    }
  }
}

// ---- host side ------------------------------------------------------------------------------------------------------
// More than 64 KB of dynamic LDS has to be requested once per kernel and device.  The request is idempotent, so threads that
// race on a first call only repeat it; laud_init() makes it for every kernel up front.
template <int MODE, typename ET, int BM, int BN, int WM, int WN, int KS, int NS>
static int pipe_request_lds() {
  static std::atomic<unsigned> done{0};  // one bit per device ordinal (ordinals >= 32 repeat the request)
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return LAUD_ERR_HIP;
  const unsigned bit = dev >= 0 && dev < 32 ? 1u << dev : 0u;
  if (bit && (done.load(std::memory_order_acquire) & bit)) return LAUD_OK;
  constexpr int kLds = pipe::lds_bytes<MODE, BM, BN, NS>() + (MODE == M_DENSE1 ? pipe::masker_bytes<ET>(pipe::kMaxMaskerK) : 0);
  static_assert(kLds <= 160 * 1024, "LDS");
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pipe<MODE, ET, BM, BN, WM, WN, KS, NS>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, kLds) != hipSuccess)
    return LAUD_ERR_HIP;
  done.fetch_or(bit, std::memory_order_release);
  return LAUD_OK;
}

// cap_rows < 0: only make the request
template <int MODE, typename ET, int BM, int BN, int WM, int WN, int KS, int NS>
static int launch_pipe_t(const GemmArgs& args, long long cap_rows, int nsamples, hipStream_t st) {
  const int rc = pipe_request_lds<MODE, ET, BM, BN, WM, WN, KS, NS>();
  if (rc != LAUD_OK || cap_rows < 0) return rc;
  constexpr bool CS = (MODE >= M_CS1 && MODE <= M_CS3);
  constexpr int NT = 64 * WM * WN * KS;
  PipeArgs k{};
  k.g = args;
  GemmArgs& a = k.g;
  a.row_tiles = (int)((cap_rows + BM - 1) / BM);
  if constexpr (MODE == M_CONV1) {  // cap_rows = rows per group of samples, nsamples = number of groups
    a.tiles_per_group = a.row_tiles;
    a.row_tiles *= nsamples;
  }
  a.col_tiles = (a.Ncols + BN - 1) / BN;
  dim3 grid = CS ? dim3((unsigned)(a.row_tiles * a.col_tiles), (unsigned)nsamples)
                 : dim3((unsigned)(((a.row_tiles + 7) / 8) * 8 * a.col_tiles));
  if constexpr (MODE == M_CONV1 || MODE == M_DENSE1) {
    if (a.pk_out != nullptr) {  // spare workgroups for the weight re-ordering: one chunk per thread
      a.pk_first_block = (int)grid.x;
      grid.x += (unsigned)((a.pk_chunks + NT - 1) / NT);
    }
  }
  if constexpr (MODE == M_CONV3) {
    if (NT == 256) a.cp.nblocks = std::min(a.cp.npatch * a.cp.S, 2 * a.cp.nblocks);  // (shares for workgroups of half as many threads)
    a.cp.first = (int)grid.x;
    grid.x += (unsigned)a.cp.nblocks;
  }
  const int oH = a.stride > 1 ? a.Ho : a.H, oW = a.stride > 1 ? a.Wo : a.W;
  k.ct = make_fast_div(a.col_tiles); k.tpg = make_fast_div(std::max(a.tiles_per_group, 1));
  k.s = make_fast_div(a.S); k.ss = make_fast_div(a.S * a.S);
  k.pps = make_fast_div(std::max((oH / a.S) * (oW / a.S), 1)); k.wp = make_fast_div(std::max(oW / a.S, 1));
  k.howo = make_fast_div(std::max(MODE == M_CONV1 ? a.hw : a.Ho * a.Wo, 1)); k.wo = make_fast_div(std::max(a.Wo, 1)); k.grp = make_fast_div(std::max(a.G, 1));
  constexpr int kRing = pipe::ring_bytes<BM, BN, NS>(), BKE = 8 * elem<ET>::per16;
  k.ring = pipe::short_ring<MODE, KS>() ? std::min(NS, (a.K + BKE - 1) / BKE) * (kRing / NS) : kRing;
  const int lds = pipe::lds_bytes<MODE, BM, BN, NS>() - kRing + k.ring + (MODE == M_DENSE1 && a.wmask ? pipe::masker_bytes<ET>(a.K) : 0);
  hipLaunchKernelGGL((k_pipe<MODE, ET, BM, BN, WM, WN, KS, NS>), grid, dim3(NT), lds, st, k);
  return check_launch();
}


// The tiles.  A launch lasts (tiles per compute unit) x (slices x time of a slice + start and end), and a slice's time goes with
// the bytes of its rows, so large tiles move fewer bytes for the same product and small ones fill the chip and hide each
// other's start and end.  (256 below: the compute units of an MI355X.)  us a slice and start + end, measured on ResNet stages 2 to 4:
//   128 x  64  two workgroups a compute unit: 0.52 for both, 0.48 for one alone
//    64 x 128  the K steps split, six slices deep: 0.285, 4.5: shortest chain, for launches that fill the chip once
//   128 x 128  0.48, 4.5      256 x 128 and 128 x 256  0.75 (1x1) to 1.1 (3x3), 5: dense rows of large batches
template <int MODE, typename ET>
static int launch_pipe_rule(const GemmArgs& a, long long cap_rows, int nsamples, hipStream_t st) {
  // (each with its LDS request: cap_rows < 0, laud_init)
  auto t128x64 = [&](auto...) { return launch_pipe_t<MODE, ET, 128, 64, 2, 2, 1, 3>(a, cap_rows, nsamples, st); };
  auto t64x64 = [&](auto...) { return launch_pipe_t<MODE, ET, 64, 64, 2, 2, 1, 3>(a, cap_rows, nsamples, st); };
  constexpr bool CS = (MODE >= M_CS1 && MODE <= M_CS3), F32 = sizeof(ET) == 4;
  if constexpr (MODE == M_G2) {  // (a column tile is the 64 channels of whole groups)
    if constexpr (F32) return t64x64();
    else return t128x64();
  } else {
    constexpr bool TAPS = (MODE == M_CONV2 || MODE == M_SD2 || MODE == M_U2), DENSE = (MODE == M_SD1 || MODE == M_SD3 || MODE == M_CONV3);
    auto t64x128 = [&](auto...) { return launch_pipe_t<MODE, ET, 64, 128, 2, 2, 1, 3>(a, cap_rows, nsamples, st); };
    auto t64x128k = [&](auto...) { return launch_pipe_t<MODE, ET, 64, 128, 2, 2, 2, 6>(a, cap_rows, nsamples, st); };
    auto t128x128 = [&](auto...) { return launch_pipe_t<MODE, ET, 128, 128, 2, 4, 1, 4>(a, cap_rows, nsamples, st); };
    auto t256x128 = [&](auto...) { return launch_pipe_t<MODE, ET, 256, 128, 4, 2, 1, 3>(a, cap_rows, nsamples, st); };
    auto t128x256 = [&](auto...) { return launch_pipe_t<MODE, ET, 128, 256, 2, 4, 1, 3>(a, cap_rows, nsamples, st); };
    const long long rows = cap_rows * (MODE == M_CONV1 || CS ? nsamples : 1);
    const int kt = (TAPS || MODE == M_CS2 ? 9 : 1) * ((a.K + 8 * elem<ET>::per16 - 1) / (8 * elem<ET>::per16));
    auto tiles = [&](long long m, int bm, int bn) { return ((m + bm - 1) / bm) * ((a.Ncols + bn - 1) / bn); };
    const bool init = cap_rows < 0;
    int rc = LAUD_OK;
    auto all = [&rc](auto... t) { ((rc = rc == LAUD_OK ? t() : rc), ...); return rc; };
    if constexpr (F32) {
      // float32 is bound by its MFMAs (a sixteenth of the bf16 rate): the tile that wastes the fewest.  Dense and last 1x1s on 64 x 128, of
      // which a compute unit holds two or more at any K: 32 images, 64 x 128 / 128 x 128, last 1x1 in place at 0.86 of stage 1 46.5 / 53.4 us,
      // of stage 2 37.8 / 42.5 (out of place 40.3 / 45.9), of 256 -> 1024 channels on 18 x 18 51.2 / 63.8; shortcut and first 1x1 of stage 2's
      // first block 131 / 155.
      if constexpr (DENSE) return init ? all(t64x64, t64x128) : a.Ncols < 128 ? t64x64() : t64x128();
      if (init) return all(t64x64, t64x128, t128x128);
      return a.Ncols < 128 ? t64x64() : rows < 8192 ? t64x128() : t128x128();
    } else if constexpr (CS) {
      // Of one or two tiles a sample, all of them in one round of the chip: the six-slice ring.  First 1x1 and 3x3 of stage 4, 64 samples
      // of 7 x 7: 26.1 + 33.8 us with 64 x 128 and three slices, 15.9 + 23.1 here; the whole block 68.8 -> 54.2, one sample 43.1 ->
      // 38.4, 19 of 9 x 9 64.9 -> 51.1.  Past one round two workgroups a compute unit are the better: 96 samples 76.9 -> 83.8, 64 of 9 x 9
      // 83.7 -> 94.7; eight slices (512 channels on 8 x 8) 20.8 -> 21.1.
      if constexpr (MODE != M_CS3) {
        if (init) rc = t64x128k();
        else if (cap_rows <= 128 && kt >= 16 && tiles(cap_rows, 64, 128) * nsamples <= 256) return t64x128k();
      }
      if (init) return all(t64x128, t128x64);
      return cap_rows <= 64 ? t64x128() : t128x64();  // (cap_rows: rows of one sample)
    } else if constexpr (TAPS) {
      // Of listed rows half the capacity is taken to exist.  Stage 4, 128 images (listed, 3136 rows, 72 slices), 64 x 128 / 128 x
      // 128: 26 / 38 us; stage 2 (50176 rows, 18 slices) 36 / 26 us.  (256 x 128 there: 23, but 22 where 0.15 of the rows exist
      // and 128 x 128 takes 13.)  Dense rows, stage 2 in front of a stride: 64 x 128 / 128 x 128 / 256 x 128 61 / 52 / 48 us.
      if (init) return MODE == M_SD2 ? all(t128x64, t64x128k, t128x128, t256x128) : all(t128x64, t64x128k, t128x128);
      if (a.Ncols <= 64) return t128x64();
      const long long m = MODE == M_SD2 ? rows : rows / 2;
      auto cost = [&](int bm, double slice, double ends) { return (double)((tiles(m, bm, 128) + 255) / 256) * (kt * slice + ends); };
      const double c64 = cost(64, 0.285, 4.5), c128 = cost(128, 0.48, 4.5);
      if (c64 <= c128) return t64x128k();
      if constexpr (MODE == M_SD2)
        if (cost(256, 1.1, 5.) < c128) return t256x128();
      return t128x128();
    } else if constexpr (DENSE) {
      // Dense 1x1, 128 x 64 / 128 x 128 / 128 x 256: 100352 rows, 256 -> 512 channels 67 / 66 / 57 us; 6272 rows, 1024 -> 2048
      // 48 / 43 / 36 us, 512 -> 2048 29 / 29 / 25 us; short reductions are bound by memory, where two workgroups hide each other's ends:
      // 100352 rows, 64 -> 64 channels 22 / 38 / 51 us.
      if constexpr (MODE != M_SD1)
        if (init) rc = t128x128();
      if (init) return all(t128x64, t64x128k, t128x256);
      if (a.Ncols <= 64) return t128x64();
      const long long m = MODE == M_CONV3 ? rows / 2 : rows;
      // (a tile's LDS leaves a compute unit no room for a workgroup that copies: stage 4 out of place, 16 images, 0.15 / 0.86 34.2 / 38.3 us
      // with these, 34.9 / 36.3 with 128 x 64)
      if (kt >= 8 && tiles(rows, 64, 128) + a.cp.nblocks <= 256) return t64x128k();
      if (tiles(m, 128, 256) >= 192 && (MODE == M_SD1 ? a.Ncols >= 256 : kt >= 8 && a.Ncols >= 1024)) return t128x256();
      if constexpr (MODE != M_SD1)
        if (kt > 5 && tiles(m, 128, 128) >= 192) return t128x128();
      return t128x64();
    } else if constexpr (MODE == M_CONV1 || MODE == M_DENSE1) {
      // (blocks of stage 4, layer skipping, 48 / 64 images at 0.15: 46.4 / 47.2 us with 128 x 128, 42.7 / 44.2 with 64 x 128)
      // 6272 rows, 2048 -> 512 channels: 128 x 64 / 128 x 128 39 / 23 us; 100352 rows, 512 -> 128: 24 / 24 us, 401408 rows, 256 -> 64: 35 / 48
      if constexpr (MODE == M_CONV1) {
        if (init) rc = t64x128k();
        else if (kt >= 8 && a.Ncols > 64 && tiles(rows, 64, 128) <= 256) return t64x128k();
      }
      if (init) return all(t128x64, t128x128);
      return kt >= 16 && a.Ncols >= 256 ? t128x128() : t128x64();
    } else {  // the unfused schedule
      return t128x64();
    }
  }
}

template <int MODE>
static int launch_pipe_mode(int dtype, const GemmArgs& a, long long cap_rows, int nsamples, hipStream_t st) {
  return dtype == LAUD_BF16 ? launch_pipe_rule<MODE, bf16_t>(a, cap_rows, nsamples, st) : launch_pipe_rule<MODE, float>(a, cap_rows, nsamples, st);
}

}  // namespace laud
