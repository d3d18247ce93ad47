// The group 3x3 of the RegNetY blocks (mode G2) for many rows, bf16, on gfx950 MFMA.
//
// A tile of 64 output channels reads the 64 input channels of its own groups, and a wave's 32 channels, with groups of up to 32, only
// their own 32: a reduction of 9 x 32.  As a general tile the product is a chain of nine short slices with a barrier each.  Here a
// workgroup keeps its 64 channels' weights in registers, in MFMA order, and walks over tiles of 64 rows: all nine taps' rows are
// requested at once (72 KB of LDS, so that two workgroups share a compute unit and hide each other's waits), waited for once and
// multiplied without a barrier.  (Loaded per tile, the weights cost more than the rows: in MFMA order a lane's 16 bytes lie in a
// cache line of their own.)  RegNetY-800MF blocks of 128 images at ratio 0.5, as a general tile / here: stage 1 93.7 / 85.0 us, stage 2 80.0 /
// 73.6, stage 3 61.3 / 56.6.  An XCD walks over one contiguous eighth of the rows, where its taps find their neighbours in its L2.
#include "laud_common.h"
#include "laud_gemm.h"
#include "laud_tile_util.h"

#include <algorithm>
#include <atomic>

namespace laud {

namespace group {
constexpr int kBM = 64, kBN = 64, kThreads = 256;
constexpr unsigned kOob = 0x80000000u;
constexpr int kTap = kBM * 128;                 // a tap's rows: 64 channels each
constexpr int kTab = 9 * kTap;                  // scale, shift [64] floats; offset, unreadable taps [64]
constexpr int kLds = kTab + 2 * kBN * 4 + 2 * kBM * 4;
constexpr int kPerXcd = 64;                     // workgroups of an XCD: two for each of its 32 compute units
static_assert(kGroupMaxC <= kPerXcd * kBN, "every column tile has a workgroup");
}  // namespace group

struct GroupArgs {
  GemmArgs g;
  FastDiv ct, s, ss, pps, wp;
};

// KW: K steps of 16 channels a wave takes per tap: 2 (groups of up to 32 channels: the wave's own 32), 4 (groups of 64)
template <int KW>
__global__ __launch_bounds__(group::kThreads) void k_group(const GroupArgs ka) {
  using namespace group;
  prefetch_args<sizeof(GroupArgs)>();
  const GemmArgs& a = ka.g;
  extern __shared__ __align__(16) unsigned char smem[];
  float* const s_scale = reinterpret_cast<float*>(smem + kTab);
  float* const s_shift = s_scale + kBN;
  unsigned* const s_voff = reinterpret_cast<unsigned*>(s_shift + kBN);
  unsigned* const s_bad = s_voff + kBM;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  const int l31 = lane & 31, lhi = lane >> 5, l8 = lane >> 3, l7 = lane & 7;
  // workgroup b: column tile of its XCD's b >> 3, rows from the XCD's eighth on
  const int slot = blockIdx.x >> 3, xcd = blockIdx.x & 7, walker = fast_div(slot, ka.ct), step = fast_div(kPerXcd, ka.ct);
  const int col0 = (slot - walker * a.col_tiles) * kBN;
  const int SS = a.S * a.S, M = *a.count * SS, ntiles = (M + kBM - 1) / kBM, per = (ntiles + 7) >> 3;
  const int last = min((xcd + 1) * per, ntiles);
  int tile = xcd * per + walker;
  if (walker >= step || tile >= last) return;
  int entry = tid < kBM ? a.list[fast_div(min(tile * kBM + tid, M - 1), ka.ss)] : 0;  // (rows past the last one repeat its entry)

  // ---- weights: lane = output channel, 8 of the window's input channels; what lies outside the channel's group reads as zero -----
  const int C = a.Ncols, gw = a.gw;
  u32x4 w[9][KW];
  {
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.Wt), 0, C * 9 * gw * 2, 0x00020000);
    const int c = col0 + 32 * wn + l31;
#pragma unroll
    for (int kk = 0; kk < KW; ++kk) {
      const int rel = col0 + (KW == 2 ? 32 * wn : 0) + 16 * kk + 8 * lhi - (c & ~(gw - 1));  // (group widths are powers of two)
      const unsigned v = (unsigned)(c * 9 * gw + rel) * 2u | ((unsigned)(rel | (gw - 1 - rel) | (C - 1 - c)) & kOob);
#pragma unroll
      for (int t = 0; t < 9; ++t) w[t][kk] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, v, t * gw * 2, 0);
    }
  }
  if (tid >= kBM && tid < kBM + 2 * kBN) {
    const int i = tid - kBM, col = col0 + (i & (kBN - 1));
    (i < kBN ? s_scale : s_shift)[i & (kBN - 1)] = col < C ? (i < kBN ? a.scale : a.shift)[col] : 0.f;
  }
  // instruction i of wave w loads rows 8 (w + 4 i) .. +7 of a tap; chunk c of row r lies at c ^ (r & 7) ^ ((r >> 3) & 1).  The
  // taps reach one row and one pixel back: the descriptor starts that far before h1.
  const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(reinterpret_cast<const char*>(a.A)) - (long long)(a.W + 1) * a.lda * 2, 0, (int)kOob, 0x00020000);
  const int chunk = l7 ^ l8 ^ (wave & 1);
  const unsigned outside = col0 + 8 * chunk < C ? 0u : kOob;  // (channels past the last one: the row's next pixel)
  const unsigned swz = (unsigned)(32 * wm + l31) * 128u + (((unsigned)lhi ^ (unsigned)(l31 & 7) ^ ((unsigned)(l31 >> 3) & 1u)) << 4);
  for (; tile < last; tile += step) {
    // ---- rows: one thread looks a row up for the workgroup ------------------------------------------------------------------------
    const int row0 = tile * kBM;
    if (tid < kBM) {
      const int rho = min(row0 + tid, M - 1), j = rho - fast_div(rho, ka.ss) * SS;
      const int sy = a.stride > 1 ? a.stride : 1, Wp = fast_div(a.stride > 1 ? a.Wo : a.W, ka.s), pps = fast_div(a.stride > 1 ? a.Ho : a.H, ka.s) * Wp;
      const int n = fast_div(entry, ka.pps), r2 = entry - n * pps, py = fast_div(r2, ka.wp), px = r2 - py * Wp, jy = fast_div(j, ka.s);
      const int y = (py * a.S + jy) * sy, x = (px * a.S + j - jy * a.S) * sy;  // centre of the 3x3 on the input grid
      const unsigned mk = ((y > 0 ? 0x7u : 0u) | 0x38u | (y < a.H - 1 ? 0x1c0u : 0u)) & ((x > 0 ? 0x49u : 0u) | 0x92u | (x < a.W - 1 ? 0x124u : 0u));
      s_voff[tid] = ((unsigned)((n * a.H + y) * a.W + x) * (unsigned)a.lda + (unsigned)col0) * 2u;
      s_bad[tid] = ~mk;
      if (tile + step < last) entry = a.list[fast_div(min(row0 + step * kBM + tid, M - 1), ka.ss)];
    }
    lds_wait();
    wg_barrier();  // the rows; and everyone is done with the tile before
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = 8 * (wave + 4 * i) + l8;
      const unsigned voff = (s_voff[r] + (unsigned)chunk * 16u) | outside, bad = s_bad[r];
#pragma unroll
      for (int t = 0; t < 9; ++t)
        dma16(arsrc, voff | ((bad << (31 - t)) & kOob), (unsigned)((t / 3 * a.W + t % 3) * a.lda * 2), (unsigned)(t * kTap + (wave + 4 * i) * 1024));
    }
    f32x16 acc[2];
    acc[0] = acc[1] = f32x16{};
    vm_wait<0>();
    wg_barrier();
    if (col0 + 32 * wn >= C) continue;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int kk = 0; kk < KW; ++kk) {
        const unsigned kg = (KW == 2 ? 2 * wn : 0) + kk;
        const uint4 f = *reinterpret_cast<const uint4*>(smem + t * kTap + (swz ^ (kg << 5)));
        acc[(t * KW + kk) & 1] = mma_bf16(w[t][kk], f, acc[(t * KW + kk) & 1]);
      }
    float v[16];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 sc = *reinterpret_cast<const float4*>(s_scale + 32 * wn + 8 * g + 4 * lhi);
      const float4 sh = *reinterpret_cast<const float4*>(s_shift + 32 * wn + 8 * g + 4 * lhi);
      const float scv[4] = {sc.x, sc.y, sc.z, sc.w}, shv[4] = {sh.x, sh.y, sh.z, sh.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * g + e] = fmaxf((acc[0][4 * g + e] + acc[1][4 * g + e]) * scv[e] + shv[e], 0.f);
    }
    to_consecutive_channels(v);  // 0-3, 8-11, 4-7, 12-15: channels 16 lhi + 0 .. 15
    const int orow = row0 + 32 * wm + l31, col = col0 + 32 * wn + 16 * lhi;
    if (orow < M) {
      __bf16* const op = reinterpret_cast<__bf16*>(a.Out) + (size_t)orow * a.ldo + col;
      if (col < C) *reinterpret_cast<uint4*>(op) = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[8], v[9]), pack_bf16(v[10], v[11]));
      if (col + 8 < C) *reinterpret_cast<uint4*>(op + 8) = make_uint4(pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]), pack_bf16(v[12], v[13]), pack_bf16(v[14], v[15]));
    }
  }
}

// ---- host side ------------------------------------------------------------------------------------------------------
int group_init_device() {
  static std::atomic<unsigned> done{0};  // one bit per device ordinal (ordinals >= 32 repeat the request)
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return LAUD_ERR_HIP;
  const unsigned bit = dev >= 0 && dev < 32 ? 1u << dev : 0u;
  if (bit && (done.load(std::memory_order_acquire) & bit)) return LAUD_OK;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_group<2>), hipFuncAttributeMaxDynamicSharedMemorySize, group::kLds) != hipSuccess ||
      hipFuncSetAttribute(reinterpret_cast<const void*>(&k_group<4>), hipFuncAttributeMaxDynamicSharedMemorySize, group::kLds) != hipSuccess)
    return LAUD_ERR_HIP;
  done.fetch_or(bit, std::memory_order_release);
  return LAUD_OK;
}

int launch_group(const GemmArgs& args, long long cap_rows, hipStream_t st) {
  if (group_init_device() != LAUD_OK) return LAUD_ERR_HIP;
  GroupArgs k{};
  k.g = args;
  GemmArgs& a = k.g;
  a.row_tiles = (int)((cap_rows + group::kBM - 1) / group::kBM);
  a.col_tiles = (a.Ncols + group::kBN - 1) / group::kBN;
  const int oH = a.stride > 1 ? a.Ho : a.H, oW = a.stride > 1 ? a.Wo : a.W;
  k.ct = make_fast_div(a.col_tiles); k.s = make_fast_div(a.S); k.ss = make_fast_div(a.S * a.S);
  k.pps = make_fast_div((oH / a.S) * (oW / a.S)); k.wp = make_fast_div(oW / a.S);
  const dim3 grid((unsigned)(8 * std::min<long long>(group::kPerXcd, (long long)((a.row_tiles + 7) / 8) * a.col_tiles)));
  if (a.gw <= 32) hipLaunchKernelGGL((k_group<2>), grid, dim3(group::kThreads), group::kLds, st, k);
  else hipLaunchKernelGGL((k_group<4>), grid, dim3(group::kThreads), group::kLds, st, k);
  return check_launch();
}

}  // namespace laud
