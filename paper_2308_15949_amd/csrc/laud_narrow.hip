// 3x3 -> last 1x1 -> residual add (or projection shortcut) in ONE kernel for the 64-wide bf16 blocks (c_mid = 64, c_out = 256:
// the blocks of ResNet stage 1), gfx950.
//
// These blocks are bound by memory traffic (dense 136 FLOP per byte), and as separate launches h2, and in a first block the
// shortcut, make a round trip through it: at 128 images 42 + 55 us for the two convolutions of a dynamic block at ratio 0.5,
// 72 + 121 + 100 us for those of a static first block with its shortcut.  All weights of such a block fit a compute unit, so
// here a workgroup keeps them there for its whole life and walks over its tiles:
//
//   * one workgroup = 128 rows (active pixels of the index list, or all output pixels) x all channels, 8 waves.  In the
//     3x3 wave (wn, wm) owns mid channels 32 wn .. +31 of rows 32 wm .. +31, its weights (9 taps x 64 channels) in
//     registers as far as these go (seven taps, four with a shortcut), the rest in LDS; in the last 1x1 wave w owns output channels 32 w .. +31 of all rows.
//   * a tap's rows of h1 (64 channels = one 128-byte slice) come with LDS-direct loads into a ring of four slices, swizzled
//     as in the fused kernel of the 256-wide blocks; one barrier per tap.  h2 goes through LDS once.  The rows of a
//     projection shortcut (64 input channels) are one more slice.
//   * the next tile's list entries are requested during the 3x3, its first three slices during the last 1x1; the residual
//     is requested ahead of the fourth tap and used after the ninth.
//   * tiles are dealt so that an XCD works on one contiguous eighth of the rows: its taps find their neighbours in its L2.
//
// With a shortcut: blocks in front of a stride and maps too small for the rectangles of laud_first.hip (128 images of 112 x 112 to 56 x 56 122
// us, 8192 maps of 7 x 7 91 us, the first 1x1 ahead of it not counted).
// Vector-memory waits: see laud_tail.hip; the loads younger than the slice waited for are counted at each wait.
#include "laud_common.h"
#include "laud_tile_util.h"

#include <atomic>

namespace laud {

namespace narrow {
constexpr int kMid = 64, kOut = 256, kBM = 128, kThreads = 512;
constexpr int kStage = kBM * 128, kRing = 4, kAhead = kRing - 1;  // slices requested ahead of the one in use
constexpr int kH2 = kRing * kStage, kX = kH2 + kStage, kTab = kX + kStage;
constexpr int kTabFloats = 2 * kMid + 4 * kOut;         // s2 t2 | s3 t3 | s_sc t_sc
constexpr int kRows = kTab + kTabFloats * 4;            // output rows of two tiles
// taps whose weights stay in registers; the others' lie in LDS in MFMA order
template <bool SC> constexpr int reg_taps() { return SC ? 4 : 7; }
constexpr int kW2 = kRows + 2 * kBM * 4;                // [tap - reg_taps][wn][kg][lane] 16 bytes
template <bool SC> constexpr int lds_bytes() { return kW2 + (9 - reg_taps<SC>()) * 8192; }
constexpr unsigned kOob = 0x80000000u;
static_assert(lds_bytes<false>() <= 160 * 1024 && lds_bytes<true>() <= 160 * 1024, "LDS");
static_assert(kMid * 9 * kMid * 2 <= kTab, "w2 passes through the ring, h2 and shortcut regions on its way into registers");
}  // namespace narrow

// vm_wait with a count that is a constant once the loop around it is unrolled
__device__ __forceinline__ void vm_wait_n(int n) {
  switch (n) {
    case 0: vm_wait<0>(); break;
    case 2: vm_wait<2>(); break;
    case 4: vm_wait<4>(); break;
    case 6: vm_wait<6>(); break;
    case 8: vm_wait<8>(); break;
    case 10: vm_wait<10>(); break;
    case 12: vm_wait<12>(); break;
    case 14: vm_wait<14>(); break;
    case 16: vm_wait<16>(); break;
    case 18: vm_wait<18>(); break;
    default: vm_wait<0>(); break;
  }
}

template <bool SC>
__global__ __launch_bounds__(narrow::kThreads) void k_narrow(const NarrowArgs a) {
  using namespace narrow;
  prefetch_args<sizeof(NarrowArgs)>();
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, lhi = lane >> 5, l8 = lane >> 3, l7 = lane & 7;
  const int wn = wave & 1, wm = wave >> 1;
  if (!SC && a.cp.nblocks && (int)blockIdx.x >= a.cp.first) {
    copy_inactive_part<kThreads>(a.cp, blockIdx.x - a.cp.first, a.cp.nblocks, smem);
    return;
  }
  const int SS = a.S * a.S;
  const int M = SC ? a.m_rows : *a.count * SS;
  const int ntiles = (M + kBM - 1) / kBM;
  // workgroup b walks tiles first, first + stride, ... of its XCD's eighth
  const int wgs = SC || !a.cp.nblocks ? (int)gridDim.x : a.cp.first;
  const int per = (ntiles + 7) >> 3, xcd = blockIdx.x & 7;
  const int last = min((xcd + 1) * per, ntiles), step = wgs >> 3;
  int tile = xcd * per + (int)(blockIdx.x >> 3);
  if (tile >= last) return;

  float* const s_s2 = reinterpret_cast<float*>(smem + kTab);
  float* const s_t2 = s_s2 + kMid;
  float* const s_s3 = s_t2 + kMid;
  float* const s_t3 = s_s3 + kOut;
  float* const s_ss = s_t3 + kOut;
  float* const s_ts = s_ss + kOut;
  int* const s_orow = reinterpret_cast<int*>(smem + kRows);

  // ---- weights into registers, through LDS (whole lines from memory; MFMA order from row-major memory would put consecutive
  // lanes into different rows) ---------------------------------------------------------------------------------------
  const __amdgpu_buffer_rsrc_t w2rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.w2), 0, kMid * 9 * kMid * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t w3rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.w3), 0, kOut * kMid * 2, 0x00020000);
  constexpr int kW2KB = kMid * 9 * kMid * 2 / 1024, kW3KB = kOut * kMid * 2 / 1024;
  for (int i = wave; i < kW2KB; i += 8) dma16(w2rs, lane * 16u, (unsigned)i * 1024u, (unsigned)i * 1024u);
  for (int i = tid; i < kMid; i += kThreads) { s_s2[i] = a.s2[i]; s_t2[i] = a.t2[i]; }
  for (int i = tid; i < kOut; i += kThreads) {
    s_s3[i] = a.s3[i];
    s_t3[i] = a.t3[i];
    if constexpr (SC) { s_ss[i] = a.ssc[i]; s_ts[i] = a.tsc[i]; }
  }
  vm_wait<0>();
  lds_wait();
  wg_barrier();
  constexpr int RT = reg_taps<SC>();
  u32x4 w2r[RT][4], w3r[4], wsr[4];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int kg = 0; kg < 4; ++kg) {
      if (t < RT || wm == 0) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(smem + (32 * wn + l31) * (9 * kMid * 2) + t * 128 + kg * 32 + lhi * 16);
        if (t < RT) w2r[t < RT ? t : 0][kg] = v;
        else *reinterpret_cast<u32x4*>(smem + kW2 + (t - RT) * 8192 + ((wn * 4 + kg) * 64 + lane) * 16) = v;
      }
    }
  lds_wait();
  wg_barrier();
  for (int i = wave; i < kW3KB; i += 8) dma16(w3rs, lane * 16u, (unsigned)i * 1024u, (unsigned)i * 1024u);
  if constexpr (SC) {
    const __amdgpu_buffer_rsrc_t wsrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.wsc), 0, kOut * kMid * 2, 0x00020000);
    for (int i = wave; i < kW3KB; i += 8) dma16(wsrs, lane * 16u, (unsigned)i * 1024u, (unsigned)(kW3KB + i) * 1024u);
  }
  vm_wait<0>();
  wg_barrier();
#pragma unroll
  for (int kg = 0; kg < 4; ++kg) {
    w3r[kg] = *reinterpret_cast<const u32x4*>(smem + (32 * wave + l31) * 128 + kg * 32 + lhi * 16);
    if constexpr (SC) wsr[kg] = *reinterpret_cast<const u32x4*>(smem + kW3KB * 1024 + (32 * wave + l31) * 128 + kg * 32 + lhi * 16);
  }
  lds_wait();
  wg_barrier();

  // ---- rows: instruction i of wave w loads rows 64 i + 8 w .. +7 of a slice; row r keeps chunk c at c ^ (r & 7) ^ ((r >> 3) & 1)
  const int sy = a.stride;
  const int Hp = a.Ho / a.S, Wp = a.Wo / a.S;
  unsigned voffA[2], amask[2];
  int entry[2] = {0, 0};
  auto request_entries = [&](int t) __attribute__((always_inline)) {
    if constexpr (!SC) {
#pragma unroll
      for (int i = 0; i < 2; ++i) entry[i] = a.list[list_entry(t * kBM + 64 * i + 8 * wave + l8, M, a.inv_ss)];
    }
  };
  auto describe = [&](int t, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = 64 * i + 8 * wave + l8, rho = t * kBM + r;
      int n, yo, xo;
      if constexpr (SC) {
        n = fdiv(rho, a.inv_howo);
        const int r2 = rho - n * (a.Ho * a.Wo);
        yo = fdiv(r2, a.inv_wo);
        xo = r2 - yo * a.Wo;
      } else {
        const int q = entry[i], j = rho - fdiv(rho, a.inv_ss) * SS;
        n = fdiv(q, a.inv_pps);
        const int r2 = q - n * (Hp * Wp), py = fdiv(r2, a.inv_wp), px = r2 - py * Wp, jy = fdiv(j, a.inv_s);
        yo = py * a.S + jy;
        xo = px * a.S + j - jy * a.S;
      }
      const int y = yo * sy, x = xo * sy;  // centre of the 3x3 on the input grid
      const bool live = t < last && rho < M;  // (tiles from `last` on belong to another XCD's workgroups)
      voffA[i] = (unsigned)((n * a.H + y) * a.W + x) * 128u + (((unsigned)l7 ^ (unsigned)l8 ^ (wave & 1u)) << 4);
      const unsigned mk = ((y > 0 ? 0x7u : 0u) | 0x38u | (y < a.H - 1 ? 0x1c0u : 0u)) &
                          ((x > 0 ? 0x49u : 0u) | 0x92u | (x < a.W - 1 ? 0x124u : 0u));
      amask[i] = live ? mk : 0u;
      if (l7 == 0) s_orow[buf * kBM + r] = live ? (n * a.Ho + yo) * a.Wo + xo : -1;
    }
  };
  const __amdgpu_buffer_rsrc_t h1rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(reinterpret_cast<const char*>(a.h1)) - (long long)(a.W + 1) * 128, 0, (int)kOob, 0x00020000);
  const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(SC ? a.x : a.h1), 0, (int)kOob, 0x00020000);
  constexpr int NS = SC ? 10 : 9;  // slices of a tile; slice 9: the shortcut's input rows
  auto issue_A = [&](int s) __attribute__((always_inline)) {
    const unsigned soff = s < 9 ? (unsigned)((s / 3) * a.W + s % 3) * 128u : 0u;
    const unsigned base = (s < 9 ? (unsigned)(s % kRing) * kStage : (unsigned)kX) + wave * 1024u;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const unsigned v = ((amask[i] >> (s < 9 ? s : 4)) & 1u) ? voffA[i] : kOob;  // (the centre tap is inside for every live row)
      dma16(s < 9 ? h1rs : xrs, v, soff, base + i * 8192u);
    }
  };
  // fragment address of K step kg inside 32 rows of a slice: swz ^ (kg << 5)
  const unsigned swz = (unsigned)l31 * 128u + (((unsigned)lhi ^ (unsigned)(l31 & 7) ^ ((unsigned)(l31 >> 3) & 1u)) << 4);
  const float floor_ = act_floor(SC || a.relu);
  const __bf16* const resp = reinterpret_cast<const __bf16*>(a.res);
  __bf16* const outp = reinterpret_cast<__bf16*>(a.out);

  request_entries(tile);
  describe(tile, 0);
#pragma unroll
  for (int s = 0; s < kAhead; ++s) issue_A(s);
  int buf = 0;
  lds_wait();
  wg_barrier();  // the output rows of the first tile
  for (; tile < last; tile += step, buf ^= 1) {
    // the residual rows of this tile and the list entries of the next one
    uint4 res[4][2];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if constexpr (!SC) {
        const __bf16* rp = resp + (size_t)max(s_orow[buf * kBM + 32 * t + l31], 0) * kOut + wave * 32 + lhi * 16;
        res[t][0] = *reinterpret_cast<const uint4*>(rp);
        res[t][1] = *reinterpret_cast<const uint4*>(rp + 8);
      }
    }
    request_entries(tile + step);
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    // ---- the 3x3 -------------------------------------------------------------------------------------------------
    constexpr int kR = SC ? 0 : 10;  // residual and list loads, between slices kAhead - 1 and kAhead
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      // loads younger than slice s: the slices behind it that have been requested, and the residual where it is
      vm_wait_n(2 * ((s + kAhead - 1 < NS - 1 ? s + kAhead - 1 : NS - 1) - s) + (s < kAhead ? kR : 0));
      lds_wait();    // (this wave's reads of slice s - 1: its MFMAs, and their wait, may stand behind the barrier)
      wg_barrier();  // everyone's part of slice s is there, and everyone is done with slice s - 1
      if (s + kAhead < NS) issue_A(s + kAhead);
      if (s < 9) {
        const unsigned char* pa = smem + (unsigned)(s % kRing) * kStage + wm * 4096u;
        uint4 fa[4];
#pragma unroll
        for (int kg = 0; kg < 4; ++kg) fa[kg] = *reinterpret_cast<const uint4*>(pa + (swz ^ (kg << 5)));
#pragma unroll
        for (int kg = 0; kg < 4; ++kg) {
          const u32x4 w = s < RT ? w2r[s < RT ? s : 0][kg]
                                 : *reinterpret_cast<const u32x4*>(smem + kW2 + (s - RT) * 8192 + ((wn * 4 + kg) * 64 + lane) * 16);
          acc = mma_bf16(w, fa[kg], acc);
        }
      }
    }
    // ---- h2 = relu(s2 * acc + t2) -> LDS; the next tile's rows ------------------------------------------------------
    {
      float v[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 sc = *reinterpret_cast<const float4*>(s_s2 + 32 * wn + 8 * g + 4 * lhi);
        const float4 sh = *reinterpret_cast<const float4*>(s_t2 + 32 * wn + 8 * g + 4 * lhi);
        v[4 * g + 0] = fmaxf(acc[4 * g + 0] * sc.x + sh.x, 0.f);
        v[4 * g + 1] = fmaxf(acc[4 * g + 1] * sc.y + sh.y, 0.f);
        v[4 * g + 2] = fmaxf(acc[4 * g + 2] * sc.z + sh.z, 0.f);
        v[4 * g + 3] = fmaxf(acc[4 * g + 3] * sc.w + sh.w, 0.f);
      }
      to_consecutive_channels(v);
      const unsigned r = 32u * wm + l31, f = (r & 7u) ^ ((r >> 3) & 1u), ch = wn * 4u + lhi * 2u;
      unsigned char* row = smem + kH2 + r * 128u;
      *reinterpret_cast<uint4*>(row + ((ch ^ f) << 4)) =
          make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[8], v[9]), pack_bf16(v[10], v[11]));
      *reinterpret_cast<uint4*>(row + (((ch + 1u) ^ f) << 4)) =
          make_uint4(pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]), pack_bf16(v[12], v[13]), pack_bf16(v[14], v[15]));
    }
    describe(tile + step, buf ^ 1);  // (past this workgroup's last tile: no live rows, nothing is fetched)
    lds_wait();
    wg_barrier();  // h2 complete; everyone is done with the slices
#pragma unroll
    for (int s = 0; s < kAhead; ++s) issue_A(s);
    // ---- the last 1x1 (and the shortcut), one 32-row block at a time; the affine of this wave's channels is read
    // once per tile (per block it took as much LDS time as the fragments) -------------------------------
    float4 sc[4], sh[4], s4[4], t4[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int c = 32 * wave + 8 * g + 4 * lhi;
      sc[g] = *reinterpret_cast<const float4*>(s_s3 + c);
      sh[g] = *reinterpret_cast<const float4*>(s_t3 + c);
      if constexpr (SC) {
        s4[g] = *reinterpret_cast<const float4*>(s_ss + c);
        t4[g] = *reinterpret_cast<const float4*>(s_ts + c);
      }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x16 o, os;
#pragma unroll
      for (int e = 0; e < 16; ++e) { o[e] = 0.f; os[e] = 0.f; }
#pragma unroll
      for (int k2 = 0; k2 < 4; k2 += 2) {
        uint4 fh[2], fx[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          fh[k] = *reinterpret_cast<const uint4*>(smem + kH2 + t * 4096 + (swz ^ ((k2 + k) << 5)));
          if constexpr (SC) fx[k] = *reinterpret_cast<const uint4*>(smem + kX + t * 4096 + (swz ^ ((k2 + k) << 5)));
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          o = mma_bf16(w3r[k2 + k], fh[k], o);
          if constexpr (SC) os = mma_bf16(wsr[k2 + k], fx[k], os);
        }
      }
      float v[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        v[4 * g + 0] = o[4 * g + 0] * sc[g].x + sh[g].x;
        v[4 * g + 1] = o[4 * g + 1] * sc[g].y + sh[g].y;
        v[4 * g + 2] = o[4 * g + 2] * sc[g].z + sh[g].z;
        v[4 * g + 3] = o[4 * g + 3] * sc[g].w + sh[g].w;
        if constexpr (SC) {
          v[4 * g + 0] += os[4 * g + 0] * s4[g].x + t4[g].x;
          v[4 * g + 1] += os[4 * g + 1] * s4[g].y + t4[g].y;
          v[4 * g + 2] += os[4 * g + 2] * s4[g].z + t4[g].z;
          v[4 * g + 3] += os[4 * g + 3] * s4[g].w + t4[g].w;
        }
      }
      to_consecutive_channels(v);  // 0-3, 8-11, 4-7, 12-15: channels 32 wave + 16 lhi + 0 .. 15
      const float y[16] = {v[0], v[1], v[2], v[3], v[8], v[9], v[10], v[11], v[4], v[5], v[6], v[7], v[12], v[13], v[14], v[15]};
      unsigned pk[8];
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        float lo = y[2 * d], hi = y[2 * d + 1];
        if constexpr (!SC) {
          const uint4 rr = res[t][d / 4];
          const unsigned u = d % 4 == 0 ? rr.x : d % 4 == 1 ? rr.y : d % 4 == 2 ? rr.z : rr.w;
          lo += __uint_as_float(u << 16);
          hi += __uint_as_float(u & 0xffff0000u);
        }
        pk[d] = pack_bf16(fmaxf(lo, floor_), fmaxf(hi, floor_));
      }
      const int orow = s_orow[buf * kBM + 32 * t + l31];
      if (orow >= 0) {
        __bf16* op = outp + (size_t)orow * kOut + wave * 32 + lhi * 16;
        *reinterpret_cast<uint4*>(op) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        *reinterpret_cast<uint4*>(op + 8) = make_uint4(pk[4], pk[5], pk[6], pk[7]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  vm_wait<0>();  // (the slices requested for the tile that does not exist)
}

// ---- host side ------------------------------------------------------------------------------------------------------
bool narrow_supported(int dtype, int c_mid, int c_out, long long rows) {
  // (reciprocal divisions: rows and patches below 2^21; below 14336 rows the small tiles of laud_skinny.hip take the launch)
  return dtype == LAUD_BF16 && c_mid == narrow::kMid && c_out == narrow::kOut && rows > 14336 && rows < (1 << 21);
}

static int g_narrow_cus[32];
int narrow_init_device() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 32) return LAUD_ERR_HIP;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return LAUD_ERR_HIP;
  g_narrow_cus[dev] = cus / 8 * 8;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_narrow<false>), hipFuncAttributeMaxDynamicSharedMemorySize,
                          narrow::lds_bytes<false>()) != hipSuccess)
    return LAUD_ERR_HIP;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_narrow<true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             narrow::lds_bytes<true>()) == hipSuccess ? LAUD_OK : LAUD_ERR_HIP;
}

int launch_narrow(const NarrowArgs& args, hipStream_t st) {
  static std::atomic<unsigned> done{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 32) return LAUD_ERR_HIP;
  const unsigned bit = 1u << dev;
  if (!(done.load(std::memory_order_acquire) & bit)) {
    if (narrow_init_device() != LAUD_OK) return LAUD_ERR_HIP;
    done.fetch_or(bit, std::memory_order_release);
  }
  NarrowArgs a = args;
  const int tiles = (a.m_rows + narrow::kBM - 1) / narrow::kBM;
  unsigned grid = (unsigned)(tiles < g_narrow_cus[dev] ? (tiles + 7) / 8 * 8 : g_narrow_cus[dev]);
  a.inv_s = 1.f / a.S; a.inv_ss = 1.f / (a.S * a.S);
  a.inv_wp = 1.f / (a.Wo / a.S); a.inv_pps = 1.f / ((a.Ho / a.S) * (a.Wo / a.S));
  a.inv_howo = 1.f / (a.Ho * a.Wo); a.inv_wo = 1.f / a.Wo;
  a.cp.first = (int)grid;
  StageScope scope(LAUD_STAGE_CONV2, st);
  if (a.x) {
    hipLaunchKernelGGL((k_narrow<true>), dim3(grid), dim3(narrow::kThreads), narrow::lds_bytes<true>(), st, a);
  } else {
    grid += (unsigned)a.cp.nblocks;
    hipLaunchKernelGGL((k_narrow<false>), dim3(grid), dim3(narrow::kThreads), narrow::lds_bytes<false>(), st, a);
  }
  return check_launch();
}

}  // namespace laud
