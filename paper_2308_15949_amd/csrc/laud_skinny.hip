// The convolutions of a block when there are few rows (small batches, single images): same modes and arguments as the
// tiled kernel of laud_pipe.h, built for latency instead of throughput.
//
// With a few hundred rows a 64- or 128-row tile leaves most of the chip idle while each workgroup walks its whole reduction
// alone, slice after slice: what bounds such a launch is that serial chain (a 3x3 over 512 channels on one 7 x 7 image:
// 13 x 4 tiles, 72 slices each, 29 us).  Here a workgroup takes a small output tile (16*TM rows x 16*TN columns) and its
// NW waves SPLIT THE REDUCTION: wave w multiplies slices w, w+NW, ... (a slice: 128 bytes of every row of both operands) with
// the loads of D slices in flight in registers and no barrier in the loop; the NW partial tiles meet in LDS once, are added
// in wave order (fixed order: reproducible), and go through affine / residual / activation / rounding.
//   A lane loads 16 bytes so that eight consecutive lanes take one row's 128 bytes (a wave instruction: 8 rows), and the
// slice goes through a piece of LDS private to its wave into MFMA order.  Loading MFMA fragments straight from row-major
// memory puts consecutive lanes into different rows, and the CU then takes 16 bytes per cycle instead of 45 to 64 (measured
// 38 against 105 GB/s per CU).
// The MFMA computes the transposed tile (weights first), so a lane holds 4 x 4 consecutive channels of one row.
#include "laud_common.h"
#include "laud_gemm.h"

#include <atomic>
#include <type_traits>

namespace laud {

typedef __attribute__((ext_vector_type(4))) float f32x4;

// (LDS only: the weight loads stay in flight across this barrier)
__device__ __forceinline__ void lds_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#endif
}

// One 16-byte fragment pair: 16x16x32 bf16, or four k-steps of the 16x16x4 fp32 MFMA (lane group l/16 holds k-slots
// 4q .. 4q+3 of the 16-wide K group for both operands, so their pairing is consistent).
template <typename ET>
__device__ __forceinline__ void mma4(f32x4& acc, const uint4& a, const uint4& b) {
  if constexpr (sizeof(ET) == 2) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
  } else {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
  }
}

// A launch of this kind lives for a few microseconds, of which the instructions ahead of the first load are a good part
// (sixteen waves of a workgroup share four SIMDs), so divisions by run-time values are multiplications with reciprocals made
// on the host (fdiv; launch_skinny admits row numbers below 2^20).
struct SkinnyArgs {
  GemmArgs g;
  int cap_rows;               // rows (dense) or their upper bound (count on the device)
  int kch, KT;                // slices per tap, slices
  unsigned kmul;              // ceil(2^32 / kch), 0 for kch = 1
  int deal;                   // tiles to XCDs: 1 by row tile, 2 by column tile (a multiple of eight of them), 0 as they come
  float inv_ss, inv_s, inv_pps, inv_wp, inv_howo, inv_wo, inv_rt, inv_ct;
  PoolList pool;              // CONV2P
};

// CONV2P: with few patches every workgroup of the 3x3 decides all of them from the masker's projection -- one trip of loads, a ballot --
// instead of waiting for a launch that does (1.35 us and the gap behind it) and then for its count and list, two trips.  The first
// workgroup leaves mask, list and count for the last 1x1 and the caller.  Up to kPoolListMax patches, up to four a thread, of 1, 2 x 2 or 4 x 4 pixels.
// Summation order and decision as in laud_mask.hip.  (Blocks with their masker, before / here: one image of stage 1 / 2 / 3 / 4 18.1 / 15.2 / 15.6 /
// 19.5 -> 16.5 / 14.6 / 14.4 / 18.0 us, 16 images of stage 3 35.9 -> 34.5.  Decided ahead of the early exit, so that workgroups past the active
// rows load no weights: behind it four images of stage 4 took 25.7 instead of 23.8.)
template <int U>
struct PoolDecision {
  float v[U][16];
  int kept[U];
  __device__ __forceinline__ const float* base(const SkinnyArgs& ka, int q, int& n) const {
    const GemmArgs& a = ka.g;
    const int Wp = fdiv(a.W, ka.inv_s), pps = fdiv(a.H, ka.inv_s) * Wp;
    n = fdiv(q, ka.inv_pps);
    const int r = q - n * pps, py = fdiv(r, ka.inv_wp), px = r - py * Wp;
    return ka.pool.proj + ((size_t)n * a.H + py * a.S) * a.W + px * a.S;
  }
  template <int NT>
  __device__ __forceinline__ void load(const SkinnyArgs& ka, int tid) {
    const GemmArgs& a = ka.g;
    const float* b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u * NT >= ka.pool.n) break;  // (uniform, here and below)
      int n;
      b[u] = base(ka, min(tid + u * NT, ka.pool.n - 1), n);
      kept[u] = ka.pool.keep ? (int)ka.pool.keep[n] : 1;
    }
    const auto rows = [&](auto S) __attribute__((always_inline)) {  // (a map's width is a multiple of S: rows of a patch are aligned to their size)
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (u * NT < ka.pool.n)
#pragma unroll
          for (int y = 0; y < S; ++y) __builtin_memcpy(&v[u][S * y], __builtin_assume_aligned(b[u] + y * a.W, 4 * S), 4 * S);
    };
    if (a.S == 1) rows(std::integral_constant<int, 1>{});
    else if (a.S == 2) rows(std::integral_constant<int, 2>{});
    else rows(std::integral_constant<int, 4>{});
  }
  __device__ __forceinline__ float logit(const SkinnyArgs& ka, int u) const {
    const int S = ka.g.S;
    float acc = v[u][0];
    if (S > 1) {
#pragma unroll
      for (int k = 1; k < 4; ++k) acc += v[u][k];
    }
    if (S == 4) {
#pragma unroll
      for (int k = 4; k < 16; ++k) acc += v[u][k];
    }
    return acc / (float)(S * S) + ka.pool.bias;
  }
  // List and number of the active patches; s_cnt: counts of the waves, for every u.  `first`: the workgroup that leaves the results.
  template <int NT>
  __device__ __forceinline__ int list(const SkinnyArgs& ka, int tid, bool first, int* s_list, int* s_cnt) const {
    constexpr int NW = NT / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    float lg[U];
    bool on[U];
    unsigned long long bal[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u * NT >= ka.pool.n) break;
      lg[u] = logit(ka, u);
      on[u] = tid + u * NT < ka.pool.n && lg[u] > 0.f && kept[u] != 0;  // (not for NaN)
      bal[u] = __ballot(on[u]);
      if ((tid & (kWave - 1)) == 0) s_cnt[u * NW + wave] = __popcll(bal[u]);
    }
    lds_barrier();
    int pos[U], total = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u * NT >= ka.pool.n) break;
      pos[u] = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        if (w == wave) pos[u] = total + ballot_prefix(bal[u]);
        total += s_cnt[u * NW + w];
      }
      if (on[u]) s_list[pos[u]] = tid + u * NT;
    }
    lds_barrier();
    if (first) {
      const int Wp = fdiv(ka.g.W, ka.inv_s), pps = fdiv(ka.g.H, ka.inv_s) * Wp;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = tid + u * NT;
        if (q >= ka.pool.n) continue;
        ka.pool.mask[q] = on[u] ? 1 : 0;
        if (ka.pool.logits) ka.pool.logits[q] = lg[u];
        if (on[u]) const_cast<int32_t*>(ka.g.list)[pos[u]] = q;
        const int n = fdiv(q, ka.inv_pps);
        if (ka.pool.sample_offsets && q == n * pps) ka.pool.sample_offsets[n] = pos[u];
      }
      if (tid == 0) {
        *const_cast<int32_t*>(ka.g.count) = total;
        if (ka.pool.sample_offsets) ka.pool.sample_offsets[fdiv(ka.pool.n, ka.inv_pps)] = total;
      }
    }
    return total;
  }
};

template <int TM, int TN, int NW>
__host__ __device__ constexpr int skinny_lds() {
  constexpr int part = NW * 16 * TM * (16 * TN + 4) * 4, slices = NW * (16 * TM + 16 * TN) * 128;
  return part > slices ? part : slices;
}

// Workgroup L of a launch.
template <int MODE, typename ET, int TM, int TN, int NW, int D>
__device__ __forceinline__ void skinny_tile(const SkinnyArgs& ka, const int L) {
  const GemmArgs& a = ka.g;
  constexpr int BM = 16 * TM, BN = 16 * TN, NT = 64 * NW;
  constexpr int EPC = elem<ET>::per16, ES = (int)sizeof(ET), BKE = 8 * EPC;
  constexpr bool POOL = MODE == M_CONV2P, TAPS = (MODE == M_CONV2 || POOL || MODE == M_SD2 || MODE == M_G2);
  constexpr bool RES = (MODE == M_CONV3 || MODE == M_SD3);
  constexpr bool LISTED = (MODE == M_CONV2 || POOL || MODE == M_CONV3 || MODE == M_G2);
  constexpr int PSTR = BN + 4;  // floats per row of a partial tile
  extern __shared__ __align__(16) unsigned char smem[];
  // partial tiles [NW][BM][PSTR]; during the loop the same bytes are the waves' private slices [NW][(BM + BN) * 128 bytes]
  float* const part = reinterpret_cast<float*>(smem);
  float* const s_wm = reinterpret_cast<float*>(smem + skinny_lds<TM, TN, NW>());  // DENSE1: masker weights [K]
  __shared__ unsigned s_voff[BM], s_bad[BM];
  __shared__ int s_row[BM];
  __shared__ unsigned char s_inact[MODE == M_SD1 ? BM : 1];
  __shared__ float s_proj[MODE == M_DENSE1 ? NW * BM : 1];
  constexpr int PU = POOL ? kPoolListMax / NT : 1;  // patches a thread decides
  __shared__ int s_list[POOL ? kPoolListMax : 1], s_cnt[POOL ? kPoolListMax / kWave : 1];

  const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, lq = lane >> 4, l8 = lane >> 3, l7 = lane & 7;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if constexpr (MODE == M_CONV3) {
    if (a.cp.nblocks && L >= a.cp.first) {
      copy_inactive_part<NT>(a.cp, L - a.cp.first, a.cp.nblocks, smem);
      return;
    }
  }
  // which tile (consecutive workgroups go round-robin over the XCDs): the larger operand is read by one XCD only -- row tiles
  // dealt to the XCDs as in the tiled kernel, so that the next launch finds its rows in the same L2, or column tiles
  int rt, ct;
  {
    if (ka.deal == 1) {
      const int s = L >> 3, r8 = fdiv(s, ka.inv_ct);
      rt = r8 * 8 + (L & 7);
      ct = s - r8 * a.col_tiles;
      if (rt >= a.row_tiles) return;
    } else if (ka.deal == 2) {
      const int s = L >> 3, c8 = fdiv(s, ka.inv_rt);
      ct = c8 * 8 + (L & 7);
      rt = s - c8 * a.row_tiles;
    } else {
      ct = fdiv(L, ka.inv_rt);
      rt = L - ct * a.row_tiles;
    }
  }
  const int row0 = rt * BM, col0 = ct * BN;
  const int SS = a.S * a.S;
  int M;
  if constexpr (POOL) {
    PoolDecision<PU> decision;
    decision.template load<NT>(ka, tid);
    M = decision.template list<NT>(ka, tid, L == 0, s_list, s_cnt) * SS;
  } else {
    M = LISTED ? *a.count * SS : ka.cap_rows;
  }
  if (row0 >= M) return;

  constexpr unsigned kOob = 0x80000000u;
  const long long ashift = TAPS ? (long long)(a.W + 1) * a.lda * ES : 0;
  const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(reinterpret_cast<const char*>(a.A)) - ashift, 0, (int)kOob, 0x00020000);
  const __amdgpu_buffer_rsrc_t wrsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.Wt), 0, (int)kOob, 0x00020000);

  // ---- the row this thread looks up for the workgroup (first BM threads); its list entry is requested first -------------
  const int rrow = row0 + min(tid, BM - 1);
  int entry = 0;
  if constexpr (POOL) entry = s_list[list_entry(rrow, M, ka.inv_ss)];
  else if constexpr (LISTED) entry = a.list[list_entry(rrow, M, ka.inv_ss)];

  // ---- the weights of the first D slices: they depend on nothing but the tile ------------------------------------------
  // Every load is unconditional; a chunk that must read as zero (past K, past the wave's last slice, outside the image) gets
  // the top bit of its offset set, which lies outside the descriptor.  The bit is put together from sign bits: written as
  // conditions, the compiler branches around the loads and drains the counter where the paths meet.
  const int keff = MODE == M_G2 ? min(BN, a.K - col0) : a.K;  // group convolution: the tile's own input channels
  const int KT = ka.KT;
  unsigned voffA[2 * TM], abad[2 * TM], voffW[2 * TN];  // abad: bit t set = tap t reads as zero (bit 0 outside the tap modes)
  int wrel[2 * TN];
#pragma unroll
  for (int j = 0; j < 2 * TN; ++j) {
    const int c = min(col0 + 8 * j + l8, a.Ncols - 1);  // a column past the end re-reads the last one; its result is dropped
    voffW[j] = (unsigned)((c * a.ldw + (MODE == M_G2 ? 0 : l7 * EPC)) * ES);
    wrel[j] = 0;
    if constexpr (MODE == M_G2) wrel[j] = col0 + l7 * EPC - (c & ~(a.gw - 1));  // (group widths are powers of two)
  }
  u32x4 ra[D][2 * TM], rb[D][2 * TN];
  int kcs[D];
  auto tap_of = [&](int s) __attribute__((always_inline)) -> int {
    if constexpr (!TAPS) return 0;
    return ka.kmul ? (int)__umulhi((unsigned)s, ka.kmul) : s;
  };
  auto load_w = [&](int d, int i) __attribute__((always_inline)) {
    const int s = wave + i * NW, tap = tap_of(s), kc = s - tap * ka.kch;
    const int soff = (tap * (MODE == M_G2 ? a.gw : a.K) + (MODE == M_G2 ? 0 : kc * BKE)) * ES;
    const int bad = (KT - 1 - s) | (keff - 1 - kc * BKE - l7 * EPC);
#pragma unroll
    for (int j = 0; j < 2 * TN; ++j) {
      unsigned v = voffW[j] | ((unsigned)bad & kOob);
      if constexpr (MODE == M_G2) {
        const int rel = wrel[j] + kc * BKE;
        v = (voffW[j] + (unsigned)(rel * ES)) | ((unsigned)(bad | rel | (a.gw - 1 - rel)) & kOob);
      }
      rb[d][j] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, v, soff, 0);
    }
  };
  auto load_a = [&](int d, int i) __attribute__((always_inline)) {
    const int s = wave + i * NW, tap = tap_of(s), kc = s - tap * ka.kch;
    const int ky = (tap * 11) >> 5, kx = tap - ky * 3;  // (tap / 3 for the nine taps)
    const int soff = ((TAPS ? (ky * a.W + kx) * a.lda : 0) + kc * BKE) * ES;
    const int bad = (KT - 1 - s) | (keff - 1 - kc * BKE - l7 * EPC);
    kcs[d] = kc;
#pragma unroll
    for (int t = 0; t < 2 * TM; ++t)
      ra[d][t] = __builtin_amdgcn_raw_buffer_load_b128(
          arsrc, voffA[t] | ((unsigned)(bad | (int)(abad[t] << (31 - tap))) & kOob), soff, 0);
  };
  const int rounds = (KT + NW - 1) / NW;  // slices of the wave with the most
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < rounds) load_w(d, d);

  // ---- rows ----------------------------------------------------------------------------------------------------------
  const int sy = a.stride > 1 ? a.stride : 1;
  const int oH = a.stride > 1 ? a.Ho : a.H, oW = a.stride > 1 ? a.Wo : a.W;
  auto patch_pixel = [&](int rho, int q, int& n, int& yo, int& xo) __attribute__((always_inline)) {
    const int Wp = fdiv(oW, ka.inv_s), pps = fdiv(oH, ka.inv_s) * Wp;
    const int j = rho - fdiv(rho, ka.inv_ss) * SS;
    n = fdiv(q, ka.inv_pps);
    const int r2 = q - n * pps, py = fdiv(r2, ka.inv_wp), px = r2 - py * Wp, jy = fdiv(j, ka.inv_s);
    yo = py * a.S + jy;
    xo = px * a.S + j - jy * a.S;
  };
  if (tid < BM) {
    int pix = rrow, y = 0, x = 0, o = rrow;
    if constexpr (LISTED) {
      int n, yo, xo;
      patch_pixel(rrow, entry, n, yo, xo);
      if constexpr (MODE == M_CONV3) {
        o = (n * oH + yo) * oW + xo;
      } else {
        y = yo * sy; x = xo * sy;
        pix = (n * a.H + y) * a.W + x;
      }
    } else if constexpr (MODE == M_SD1 || MODE == M_SD2) {
      const int n = fdiv(rrow, ka.inv_howo), r2 = rrow - n * (a.Ho * a.Wo), yo = fdiv(r2, ka.inv_wo);
      y = yo * a.stride;
      x = (r2 - yo * a.Wo) * a.stride;
      pix = (n * a.H + y) * a.W + x;
    }
    unsigned mk = ~0u;
    if constexpr (TAPS)
      mk = ((y > 0 ? 0x7u : 0u) | 0x38u | (y < a.H - 1 ? 0x1c0u : 0u)) & ((x > 0 ? 0x49u : 0u) | 0x92u | (x < a.W - 1 ? 0x124u : 0u));
    const bool live = rrow < M;
    s_voff[tid] = ((unsigned)pix * (unsigned)a.lda + (unsigned)(MODE == M_G2 ? col0 : 0)) * (unsigned)ES;
    s_bad[tid] = live ? ~mk : ~0u;
    s_row[tid] = live ? o : -1;
    if constexpr (MODE == M_SD1) {
      // shortcut of a dynamic first block: the activation is applied here only where the branch will not be added
      bool inact = true;
      if (a.list != nullptr && live) {
        const int Hp = oH / a.S, Wp = oW / a.S;
        const int n = fdiv(rrow, ka.inv_howo), r2 = rrow - n * (a.Ho * a.Wo), yo = fdiv(r2, ka.inv_wo);
        const int q = (n * Hp + yo / a.S) * Wp + (r2 - yo * a.Wo) / a.S;
        const int cnt = *a.count;
        const int pos = lower_bound_dev(a.list, cnt, q);
        inact = !(pos < cnt && a.list[pos] == q);
      }
      s_inact[tid] = inact ? 1 : 0;
    }
  }
  const bool do_proj = MODE == M_DENSE1 && ct == 0 && a.wmask != nullptr;
  if (do_proj)
    for (int k = tid; k < a.K; k += NT) s_wm[k] = a.wmask[k];
  lds_barrier();
#pragma unroll
  for (int t = 0; t < 2 * TM; ++t) {
    voffA[t] = s_voff[8 * t + l8] + (unsigned)(l7 * 16);
    abad[t] = s_bad[8 * t + l8];
  }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < rounds) load_a(d, d);

  // ---- while those are on their way: affine and residual of this thread's share -------------------------------------
  constexpr int UPR = BN / 4;                        // units of four channels per row
  constexpr int UN = (BM * UPR + NT - 1) / NT;       // units per thread
  struct alignas(4 * ES) R4 { ET v[4]; };
  float4 sc[UN], sh[UN];
  R4 res[UN];
#pragma unroll
  for (int q = 0; q < UN; ++q) {
    // units past the tile and columns past the end read valid addresses; their results are dropped
    const int u = min(tid + q * NT, BM * UPR - 1), r = u / UPR, col = min(col0 + (u - r * UPR) * 4, a.Ncols - 4);
    __builtin_memcpy(&sc[q], a.scale + col, 16);
    __builtin_memcpy(&sh[q], a.shift + col, 16);
    if constexpr (RES) res[q] = *reinterpret_cast<const R4*>((const ET*)a.Res + (size_t)max(s_row[r], 0) * a.ldo + col);
  }

  f32x4 acc[TM][TN];
  float psum[TM];
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    psum[t] = 0.f;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[t][j][e] = 0.f;
  }
  // this wave's slice in LDS: row r keeps chunk c at position c ^ (r & 7) (rows of A, then rows of the weights)
  unsigned char* const mine = smem + wave * (BM + BN) * 128;
  const unsigned wpos = (unsigned)(l8 * 128 + ((l7 ^ l8) << 4));
  auto multiply = [&](int d) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 2 * TM; ++t) *reinterpret_cast<u32x4*>(mine + t * 1024 + wpos) = ra[d][t];
#pragma unroll
    for (int j = 0; j < 2 * TN; ++j) *reinterpret_cast<u32x4*>(mine + BM * 128 + j * 1024 + wpos) = rb[d][j];
#pragma unroll
    for (int kg = 0; kg < 2; ++kg) {
      const unsigned rpos = (unsigned)(l15 * 128 + (((4 * kg + lq) ^ (l15 & 7)) << 4));
      uint4 av[TM], bv[TN];
#pragma unroll
      for (int t = 0; t < TM; ++t) av[t] = *reinterpret_cast<const uint4*>(mine + t * 2048 + rpos);
#pragma unroll
      for (int j = 0; j < TN; ++j) bv[j] = *reinterpret_cast<const uint4*>(mine + BM * 128 + j * 2048 + rpos);
#pragma unroll
      for (int t = 0; t < TM; ++t) {
#pragma unroll
        for (int j = 0; j < TN; ++j) mma4<ET>(acc[t][j], bv[j], av[t]);
        if constexpr (MODE == M_DENSE1) {
          if (do_proj) {
            const int k = min(kcs[d] * BKE + (4 * kg + lq) * EPC, a.K - EPC);  // (past K the activation reads as zero)
            ET xe[EPC];
            __builtin_memcpy(xe, &av[t], 16);
#pragma unroll
            for (int e = 0; e < EPC; ++e) psum[t] += elem<ET>::load(&xe[e]) * s_wm[k + e];
          }
        }
      }
    }
  };
  int i0 = 0;
  for (; i0 + D < rounds; i0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      multiply(d);
      load_w(d, i0 + d + D);
      load_a(d, i0 + d + D);
    }
  }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (i0 + d < rounds) multiply(d);

  // ---- the partial tiles meet (in the bytes of the slices: every wave is done with its own, and only with its own) ------
  __syncthreads();
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int j = 0; j < TN; ++j)
      *reinterpret_cast<float4*>(part + (wave * BM + 16 * t + l15) * PSTR + 16 * j + 4 * lq) =
          make_float4(acc[t][j][0], acc[t][j][1], acc[t][j][2], acc[t][j][3]);
  if constexpr (MODE == M_DENSE1) {
    if (do_proj) {
#pragma unroll
      for (int t = 0; t < TM; ++t) {
        float p = psum[t];
        p += __shfl_xor(p, 16, kWave);
        p += __shfl_xor(p, 32, kWave);
        if (lq == 0) s_proj[wave * BM + 16 * t + l15] = p;
      }
    }
  }
  __syncthreads();
  if constexpr (MODE == M_DENSE1) {
    if (do_proj && tid < BM && row0 + tid < M) {
      float p = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) p += s_proj[w * BM + tid];
      a.proj[row0 + tid] = p;
    }
  }
#pragma unroll
  for (int q = 0; q < UN; ++q) {
    const int u = tid + q * NT, r = u / UPR, c4 = (u - r * UPR) * 4, col = col0 + c4;
    if (u >= BM * UPR || col >= a.Ncols) continue;
    const int orow = s_row[r];
    if (orow < 0) continue;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float4 p = *reinterpret_cast<const float4*>(part + (w * BM + r) * PSTR + c4);
      v[0] += p.x; v[1] += p.y; v[2] += p.z; v[3] += p.w;
    }
    const float scv[4] = {sc[q].x, sc[q].y, sc[q].z, sc[q].w}, shv[4] = {sh[q].x, sh[q].y, sh[q].z, sh[q].w};
    R4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = v[e] * scv[e] + shv[e];
      if constexpr (RES) {
        v[e] += elem<ET>::load(&res[q].v[e]);
        if (a.relu) v[e] = fmaxf(v[e], 0.f);
      } else if constexpr (MODE == M_SD1) {
        if (a.relu && s_inact[r]) v[e] = fmaxf(v[e], 0.f);
      } else {
        v[e] = fmaxf(v[e], 0.f);
      }
      elem<ET>::store(&o.v[e], v[e]);
    }
    *reinterpret_cast<R4*>((ET*)a.Out + (size_t)orow * a.ldo + col) = o;
  }
}

template <int MODE, typename ET, int TM, int TN, int NW, int D>
__global__ __launch_bounds__(64 * NW) void k_skinny(const SkinnyArgs ka) {
  prefetch_args<sizeof(SkinnyArgs)>();
  skinny_tile<MODE, ET, TM, TN, NW, D>(ka, blockIdx.x);
}

// Two dense 1x1s that read the same input and do not wait for each other -- the shortcut of a first block and its first 1x1 -- as
// one launch: workgroups from `split` on take the second.  (One image, first block of stage 1 / 2 / 3 / 4 at ratio 0.15: 19.8 /
// 17.8 / 17.1 / 23.5 -> 16.9 / 15.3 / 14.8 / 17.0 us.)  The second's tiles are dealt to the XCDs from `split` on: where that is not a
// multiple of eight, the 3x3 behind finds h1 in another XCD's L2 than it would behind a launch of its own.
struct SkinnyPair { SkinnyArgs p[2]; int split; };
template <typename ET, int TM, int TN, int NW, int D>
__global__ __launch_bounds__(64 * NW) void k_skinny_pair(const SkinnyPair ka) {
  prefetch_args<sizeof(SkinnyPair)>();
  const int second = (int)blockIdx.x >= ka.split;
  skinny_tile<M_SD1, ET, TM, TN, NW, D>(ka.p[second], (int)blockIdx.x - (second ? ka.split : 0));
}

// ---- host side ------------------------------------------------------------------------------------------------------
// More than 64 KB of dynamic LDS has to be requested once per kernel and device (idempotent; see gemm_request_lds).
template <int MODE, typename ET, int TM, int TN, int NW, int D>
static int skinny_request_lds() {
  static std::atomic<unsigned> done{0};  // one bit per device ordinal (ordinals >= 32 repeat the request)
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return LAUD_ERR_HIP;
  const unsigned bit = dev >= 0 && dev < 32 ? 1u << dev : 0u;
  if (bit && (done.load(std::memory_order_acquire) & bit)) return LAUD_OK;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_skinny<MODE, ET, TM, TN, NW, D>),
                          hipFuncAttributeMaxDynamicSharedMemorySize,
                          skinny_lds<TM, TN, NW>() + (MODE == M_DENSE1 ? 4096 * 4 : 0)) != hipSuccess)
    return LAUD_ERR_HIP;
  done.fetch_or(bit, std::memory_order_release);
  return LAUD_OK;
}

// The arguments of a launch and its workgroups (without those that copy).
template <int MODE, typename ET, int TM, int TN>
static unsigned skinny_args(GemmArgs a, long long cap_rows, SkinnyArgs& k) {
  constexpr bool TAPS = (MODE == M_CONV2 || MODE == M_CONV2P || MODE == M_SD2 || MODE == M_G2);
  constexpr int BKE = 8 * elem<ET>::per16;
  a.row_tiles = (int)((cap_rows + 16 * TM - 1) / (16 * TM));
  a.col_tiles = (a.Ncols + 16 * TN - 1) / (16 * TN);
  k = SkinnyArgs{};
  k.g = a;
  k.cap_rows = (int)cap_rows;
  k.kch = ((MODE == M_G2 ? 16 * TN : a.K) + BKE - 1) / BKE;
  k.KT = (TAPS ? 9 : 1) * k.kch;
  k.kmul = k.kch > 1 ? (unsigned)((0x100000000ull + k.kch - 1) / k.kch) : 0u;
  const int oH = a.stride > 1 ? a.Ho : a.H, oW = a.stride > 1 ? a.Wo : a.W;
  k.inv_s = 1.f / a.S; k.inv_ss = 1.f / (a.S * a.S);
  k.inv_wp = 1.f / (oW / a.S); k.inv_pps = 1.f / ((oH / a.S) * (oW / a.S));
  k.inv_howo = a.Ho > 0 ? 1.f / (a.Ho * a.Wo) : 0.f; k.inv_wo = a.Wo > 0 ? 1.f / a.Wo : 0.f;
  k.inv_rt = 1.f / a.row_tiles; k.inv_ct = 1.f / a.col_tiles;
  const bool by_row = cap_rows > (long long)a.Ncols * (TAPS ? 9 : 1) && a.row_tiles >= 64;
  k.deal = by_row ? 1 : (a.col_tiles & 7) == 0 ? 2 : 0;
  return (unsigned)((by_row ? (a.row_tiles + 7) / 8 * 8 : a.row_tiles) * a.col_tiles);
}

// cap_rows < 0: only make the request (laud_init)
template <int MODE, typename ET, int TM, int TN, int NW, int D>
static int launch_skinny_t(const GemmArgs& a, long long cap_rows, hipStream_t st, const PoolList* pool = nullptr) {
  const int rc = skinny_request_lds<MODE, ET, TM, TN, NW, D>();
  if (rc != LAUD_OK || cap_rows < 0) return rc;
  SkinnyArgs k;
  unsigned grid = skinny_args<MODE, ET, TM, TN>(a, cap_rows, k);
  const int lds = skinny_lds<TM, TN, NW>() + (MODE == M_DENSE1 && a.wmask ? a.K * 4 : 0);
  if constexpr (MODE == M_CONV2P) k.pool = *pool;
  if constexpr (MODE == M_CONV3) {
    k.g.cp.first = (int)grid;
    grid += (unsigned)a.cp.nblocks;
  }
  hipLaunchKernelGGL((k_skinny<MODE, ET, TM, TN, NW, D>), dim3(grid), dim3(64 * NW), lds, st, k);
  return check_launch();
}

template <typename ET, int TM, int TN, int NW, int D>
static int launch_pair_t(const GemmArgs& a, long long rows_a, const GemmArgs& b, long long rows_b, hipStream_t st) {
  constexpr int lds = skinny_lds<TM, TN, NW>();
  static std::atomic<unsigned> done{0};  // (as in skinny_request_lds)
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return LAUD_ERR_HIP;
  const unsigned bit = dev >= 0 && dev < 32 ? 1u << dev : 0u;
  if (!bit || !(done.load(std::memory_order_acquire) & bit)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_skinny_pair<ET, TM, TN, NW, D>), hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
      return LAUD_ERR_HIP;
    done.fetch_or(bit, std::memory_order_release);
  }
  if (rows_a < 0) return LAUD_OK;  // only the request (laud_init)
  SkinnyPair k;
  k.split = (int)skinny_args<M_SD1, ET, TM, TN>(a, rows_a, k.p[0]);
  const unsigned grid = (unsigned)k.split + skinny_args<M_SD1, ET, TM, TN>(b, rows_b, k.p[1]);
  hipLaunchKernelGGL((k_skinny_pair<ET, TM, TN, NW, D>), dim3(grid), dim3(64 * NW), lds, st, k);
  return check_launch();
}

template <int MODE, typename ET>
static int launch_skinny_e(const GemmArgs& a, long long cap_rows, hipStream_t st, const PoolList* pool) {
  constexpr int BKE = 8 * elem<ET>::per16;
  constexpr bool TAPS = (MODE == M_CONV2 || MODE == M_CONV2P || MODE == M_SD2 || MODE == M_G2);
  if constexpr (MODE == M_G2) {
    // 64-channel column tiles: they hold whole groups.  bf16: nine slices on three waves, all of a wave's under way at once, so
    // that a compute unit holds two workgroups (on eight waves their LDS let it hold one, and a second round took 10.6 us).  float32: eighteen slices, MFMAs as long as loads: eight waves.
    if constexpr (sizeof(ET) == 2) return launch_skinny_t<MODE, ET, 1, 4, 3, 3>(a, cap_rows, st, pool);
    else return launch_skinny_t<MODE, ET, 1, 4, 8, 2>(a, cap_rows, st, pool);
  } else {
    if (cap_rows < 0) {
      int rc = launch_skinny_t<MODE, ET, 1, 1, 8, 8>(a, -1, st);
      if (rc == LAUD_OK) rc = launch_skinny_t<MODE, ET, 1, 1, 4, 4>(a, -1, st);
      if (rc == LAUD_OK) rc = launch_skinny_t<MODE, ET, 2, 2, 8, 4>(a, -1, st);
      if (rc == LAUD_OK) rc = launch_skinny_t<MODE, ET, 2, 2, 4, 4>(a, -1, st);
      if (rc == LAUD_OK) rc = launch_skinny_t<MODE, ET, 2, 4, 4, 3>(a, -1, st);
      if (rc == LAUD_OK) rc = launch_skinny_t<MODE, ET, 4, 4, 4, 2>(a, -1, st);
      return rc;
    }
    // the largest tile that still gives most compute units a workgroup (float32: one and a half; its MFMAs, sixteen times
    // slower, are then what a workgroup's time is made of); eight waves where a wave of four would walk many slices
    const int kt = (TAPS ? 9 : 1) * ((a.K + BKE - 1) / BKE);
    auto tiles = [&](int tm, int tn) { return ((cap_rows + 16 * tm - 1) / (16 * tm)) * ((a.Ncols + 16 * tn - 1) / (16 * tn)); };
    constexpr int fill = sizeof(ET) == 2 ? 192 : 384;
    if (tiles(4, 4) >= fill) return launch_skinny_t<MODE, ET, 4, 4, 4, 2>(a, cap_rows, st, pool);
    if (tiles(2, 4) >= fill) return launch_skinny_t<MODE, ET, 2, 4, 4, 3>(a, cap_rows, st, pool);
    const bool small = tiles(2, 2) < 192;
    if (kt > 8) return small ? launch_skinny_t<MODE, ET, 1, 1, 8, 8>(a, cap_rows, st, pool) : launch_skinny_t<MODE, ET, 2, 2, 8, 4>(a, cap_rows, st, pool);
    return small ? launch_skinny_t<MODE, ET, 1, 1, 4, 4>(a, cap_rows, st, pool) : launch_skinny_t<MODE, ET, 2, 2, 4, 4>(a, cap_rows, st, pool);
  }
}

int launch_skinny(int mode, int dtype, const GemmArgs& a, long long cap_rows, hipStream_t st, const PoolList* pool) {
  switch (mode) {
#define LAUD_SKINNY_MODE(M) case M: return dtype == LAUD_BF16 ? launch_skinny_e<M, bf16_t>(a, cap_rows, st, pool) : launch_skinny_e<M, float>(a, cap_rows, st, pool)
    LAUD_SKINNY_MODE(M_CONV2);
    LAUD_SKINNY_MODE(M_CONV2P);
    LAUD_SKINNY_MODE(M_CONV3);
    LAUD_SKINNY_MODE(M_DENSE1);
    LAUD_SKINNY_MODE(M_SD1);
    LAUD_SKINNY_MODE(M_SD2);
    LAUD_SKINNY_MODE(M_SD3);
    LAUD_SKINNY_MODE(M_G2);
#undef LAUD_SKINNY_MODE
    default: return LAUD_ERR_UNSUPPORTED;
  }
}

template <typename ET>
static int launch_pair_e(const GemmArgs& a, long long rows_a, const GemmArgs& b, long long rows_b, hipStream_t st) {
  if (rows_a < 0) {
    int rc = launch_pair_t<ET, 1, 1, 8, 8>(a, -1, b, -1, st);
    if (rc == LAUD_OK) rc = launch_pair_t<ET, 1, 1, 4, 4>(a, -1, b, -1, st);
    if (rc == LAUD_OK) rc = launch_pair_t<ET, 2, 2, 8, 4>(a, -1, b, -1, st);
    if (rc == LAUD_OK) rc = launch_pair_t<ET, 2, 2, 4, 4>(a, -1, b, -1, st);
    if (rc == LAUD_OK) rc = launch_pair_t<ET, 2, 4, 4, 3>(a, -1, b, -1, st);
    if (rc == LAUD_OK) rc = launch_pair_t<ET, 4, 4, 4, 2>(a, -1, b, -1, st);
    return rc;
  }
  // the tile rule of launch_skinny_e for the two together (the same reduction length)
  const int kt = (a.K + 8 * elem<ET>::per16 - 1) / (8 * elem<ET>::per16);
  auto tiles = [&](int tm, int tn) {
    auto of = [&](const GemmArgs& g, long long m) { return ((m + 16 * tm - 1) / (16 * tm)) * ((g.Ncols + 16 * tn - 1) / (16 * tn)); };
    return of(a, rows_a) + of(b, rows_b);
  };
  constexpr int fill = sizeof(ET) == 2 ? 192 : 384;
  if (tiles(4, 4) >= fill) return launch_pair_t<ET, 4, 4, 4, 2>(a, rows_a, b, rows_b, st);
  if (tiles(2, 4) >= fill) return launch_pair_t<ET, 2, 4, 4, 3>(a, rows_a, b, rows_b, st);
  const bool small = tiles(2, 2) < 192;
  if (kt > 8) return small ? launch_pair_t<ET, 1, 1, 8, 8>(a, rows_a, b, rows_b, st) : launch_pair_t<ET, 2, 2, 8, 4>(a, rows_a, b, rows_b, st);
  return small ? launch_pair_t<ET, 1, 1, 4, 4>(a, rows_a, b, rows_b, st) : launch_pair_t<ET, 2, 2, 4, 4>(a, rows_a, b, rows_b, st);
}
int launch_skinny_pair(int dtype, const GemmArgs& a, long long rows_a, const GemmArgs& b, long long rows_b, hipStream_t st) {
  return dtype == LAUD_BF16 ? launch_pair_e<bf16_t>(a, rows_a, b, rows_b, st) : launch_pair_e<float>(a, rows_a, b, rows_b, st);
}

// The line is counted in 64 x 64 output tiles: past 256 of them this kernel's own 64 x 64 tiles are a second round.  Blocks of bf16
// at ratios 0.15 / 0.5 / 0.86, us, with this kernel | with the one that takes the launch past the line (k_pipe, k_group):
//   3x3, 72 slices (stage 4)   160 tiles 39.8 / 41.1 / 48.5 | 46.6 / 46.9 / 47.7     288 tiles 42.7 / 44.2 / 45.2 | 42.4 / 44.5 / 45.4
//                              320 tiles 42.3 / 44.6 / 69.0 | 42.4 / 45.1 / 51.1
//   3x3, 18 slices (stage 2)   172 tiles 17.7 / 18.9 / 23.5 | 19.2 / 20.3 / 22.4     294 tiles 20.3 / 22.5 / 25.4 | 19.6 / 21.7 / 24.2
//   3x3, nine slices (stage 1)  98 tiles 13.7 / 14.6 / 15.2 | 14.9 / 15.5 / 16.1     196 tiles 17.4 / 18.6 / 21.0 | 16.6 / 17.5 / 19.8
//   last 1x1, 512 -> 2048      192 tiles 24.2 / 30.6 / 37.3 | 25.0 / 31.5 / 38.0     224 tiles 23.7 / 24.8 / 25.4 | 24.1 / 25.5 / 26.4
//   last 1x1, 128 -> 512       104 tiles 12.0 / 12.8 / 15.5 | 11.8 / 12.7 / 15.4     200 tiles 14.9 / 15.6 / 16.5 | 13.6 / 14.4 / 15.0
//   first 1x1 (ratio 0.5)      2048 -> 512, 192 tiles 45.4 | 43.1     512 -> 128, 124 tiles 17.2 | 17.9, 246 tiles 22.8 | 21.9
//   group 3x3 (RegNetY-800MF)   49 tiles 11.5 / 11.6 / 11.5 | 10.9 / 11.0 / 11.0     125 tiles 14.5 / 16.6 / 18.0 | 14.1 / 15.2 / 16.2
// The numbers below are where the sides met before k_pipe and k_group, which are up to 2 us a block faster ahead of them: the sides meet
// at 288 tiles with 72 slices, at about 170 with fewer, at 100 to 150 for the 1x1s of up to eight slices; the group 3x3 has no such
// point down to 49 tiles.  In float32 the tiled kernel is bound by its MFMAs on few workgroups much longer (3x3 of stage 3 at 0.15 /
// 0.86: 408 tiles 103 / 169 | 134 / 155, 516 tiles 140 / 210 | 232 / 256).
bool skinny_wanted(int mode, int dtype, const GemmArgs& a, long long cap_rows) {
  const bool taps = mode == M_CONV2 || mode == M_SD2 || mode == M_G2, res = mode == M_CONV3 || mode == M_SD3;
  const int bke = dtype == LAUD_BF16 ? 64 : 32;
  const int kt = (taps ? 9 : 1) * (((mode == M_G2 ? 64 : a.K) + bke - 1) / bke);
  const long long t = ((cap_rows + 63) / 64) * ((a.Ncols + 63) / 64);
  int most = taps ? (kt > 9 ? 288 : 224) : (kt > 8 || res ? 208 : 256);
  if (dtype == LAUD_F32 && kt > 8) most = 512;
  if (mode == M_G2) most = 128;
  return cap_rows < (1 << 20) && t <= most;
}

// ... and for two 1x1s in one launch: together they have to fit the chip in one round too.  (RegNetY-800MF, first block of stage 3 at
// four images, 245 + 65 tiles: 27.8 us in two launches, 28.5 in one; ResNet stage 4 at four images, 104 + 128: 27.5 and 23.3.)
bool skinny_pair_wanted(int dtype, const GemmArgs& a, long long rows_a, const GemmArgs& b, long long rows_b) {
  auto tiles = [](const GemmArgs& g, long long m) { return ((m + 63) / 64) * ((g.Ncols + 63) / 64); };
  return skinny_wanted(M_SD1, dtype, a, rows_a) && skinny_wanted(M_SD1, dtype, b, rows_b) && tiles(a, rows_a) + tiles(b, rows_b) <= 256;
}

int skinny_init_device() {
  const GemmArgs none{};
  for (int mode : {M_CONV2, M_CONV2P, M_CONV3, M_DENSE1, M_SD1, M_SD2, M_SD3, M_G2})
    for (int dtype : {LAUD_BF16, LAUD_F32})
      if (launch_skinny(mode, dtype, none, -1, nullptr) != LAUD_OK) return LAUD_ERR_HIP;
  for (int dtype : {LAUD_BF16, LAUD_F32})
    if (launch_skinny_pair(dtype, none, -1, none, -1, nullptr) != LAUD_OK) return LAUD_ERR_HIP;
  return LAUD_OK;
}

}  // namespace laud
