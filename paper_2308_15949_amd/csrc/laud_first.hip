// The static first block of a stage with 64 input and mid channels, 256 output channels and no stride (ResNet stage 1), bf16, in ONE
// kernel: first 1x1 -> 3x3 -> last 1x1 + projection shortcut, gfx950.
//
// What bounds it is memory at large batches: the input once, the output (four times as many channels) once, 61 us for 128 images of 56 x 56
// at the rate of a copy (272 MB of traffic measured, 257 of them input and output).  h1 and h2 stay on the compute unit; with a first 1x1 in a launch of its own, h1 went out and came back nine-fold,
// tap by tap.  First 1x1 and k_narrow / here: 128 images 126 to 133 / 92 to 106 us (one machine and another), 32 images 44.9 / 33.8, 8
// images 19.7 / 15.6, 50 images of 72 x 72 74.3 / 61.8.  One and four images, three and four launches / here: 16.8 / 13.4 and 24.4 / 14.1.
//
//   * one workgroup = a rectangle of up to 128 output pixels at a time; it keeps all weights for its whole life (the 3x3's and the last
//     1x1s' in registers) and walks over rectangles.  Four waves (one per SIMD) make h1 and h2 of one rectangle, the other four the output of
//     the rectangle before: either's chain of loads, MFMAs and roundings hides behind the other's, and a wave holds the weights of its
//     part only.  (All eight waves going through the three convolutions together: 120 us where this takes 101, 38.7 where 33.8.)
//   * the rectangle's input pixels with their halo (up to 192) come with LDS-direct loads a rectangle ahead; h1 is made from them once for
//     all taps (a quarter to a half more rows than outputs), with zeros where the 3x3's padding is.
//   * first four waves: wave (wn, half) makes mid channels 32 wn .. +31, of h1 for 32-pixel blocks half, half + 2, half + 4, of h2 for blocks
//     2 half and 2 half + 1.  Others: output channels 64 w .. +63 of all pixels.  Rows of input and h2 lie in LDS as 128 bytes with chunk c
//     at c ^ (r & 7) ^ ((r >> 3) & 1).  What a lane needs to know of its pixels is worked out once and kept (divisions a rectangle cost 13 us
//     of 108).
//   * two barriers a rectangle: h1 complete; h2 and the next input complete.  The others meet the first one behind five of their eight
//     blocks (behind three or four, the makers' part takes the longer: 3 and 1 us more).
#include "laud_common.h"
#include "laud_tile_util.h"

#include <atomic>

namespace laud {

namespace first {
constexpr int kMid = 64, kOut = 256, kThreads = 512, kRows = 128, kHalo = 192;
constexpr int kXBytes = kHalo * 128, kXBufs = 3;             // input: in the first waves' hands, in the others', under way
// A pixel of h1 takes 144 bytes (nine 16-byte units: a tap is a distance that is the same for every pixel) and a rectangle's row 14 units
// more: 32 output pixels in a row of rectangles' rows jump by two inputs from one row to the next.  (Conflicts are 29 % of the kernel's LDS
// cycles all the same, SQ_LDS_BANK_CONFLICT; an LDS instruction is under way in 4 % of a wave's time.)
constexpr int kH1Pix = 144, kH1Pad = 224, kMaxTh = 18;
constexpr int kH1 = kXBufs * kXBytes, kH2 = kH1 + kHalo * kH1Pix + (kMaxTh + 2) * kH1Pad;  // h2: being made, being used
constexpr int kTab = kH2 + 2 * kRows * 128;                  // s1 t1 s2 t2 [64] | s3, s_sc, t3 + t_sc [256]
constexpr int kW1 = kTab + (4 * kMid + 3 * kOut) * 4;        // w1: [wn][kg][lane] 16 bytes
constexpr int kLds = kW1 + 8192;
constexpr unsigned kOob = 0x80000000u;
static_assert(kMid * 9 * kMid * 2 <= kTab && kLds <= 160 * 1024, "weights pass through the rows' regions on their way into registers");
}  // namespace first

struct FirstAt { int n, y, x; };  // sample and first output pixel of a rectangle
__device__ __forceinline__ FirstAt first_at(const FirstArgs& a, int t) {
  const int n = fast_div(t, a.d_pern), r = t - n * a.pern, y = fast_div(r, a.d_ntx);
  return {n, y * a.th, (r - y * a.ntx) * a.tw};
}
// address of this lane's chunk of K step 0 of row r (step kg: ^ kg << 5)
__device__ __forceinline__ unsigned first_row(int r, int lhi) {
  return (unsigned)r * 128u + (((unsigned)lhi ^ (unsigned)(r & 7) ^ ((unsigned)(r >> 3) & 1u)) << 4);
}

// h1 and h2 of this workgroup's rectangles (waves 0 .. 3)
__device__ __forceinline__ void first_make(const FirstArgs& a, const int tile0, const int step, const int count, const u32x4 (&w2r)[9][4]) {
  using namespace first;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int l31 = lane & 31, lhi = lane >> 5, wn = wave & 1, half = wave >> 1;
  const float* const s_s1 = reinterpret_cast<const float*>(smem + kTab);
  const float* const s_t1 = s_s1 + kMid;
  const float* const s_s2 = s_t1 + kMid;
  const float* const s_t2 = s_s2 + kMid;
  const int RW = a.tw + 2, npx = (a.th + 2) * RW, nout = a.th * a.tw;
  const int pitch = RW * kH1Pix + kH1Pad;
  const unsigned char* tap0[2];  // this lane's chunk of K step 0, tap 0
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int o = 32 * (2 * half + b) + l31, y = fast_div(o, a.d_tw), x = o - y * a.tw;
    tap0[b] = smem + kH1 + (o < nout ? y * pitch + x * kH1Pix : 0) + lhi * 16;
  }
  const unsigned ch = wn * 4u + lhi * 2u;  // the two chunks of mid channels 32 wn .. +31 that this lane stores, at c0 and c1 of a row
  auto put_row = [&](unsigned char* c0, unsigned char* c1, float (&v)[16], unsigned keep) __attribute__((always_inline)) {
    to_consecutive_channels(v);
    *reinterpret_cast<uint4*>(c0) =
        make_uint4(pack_bf16(v[0], v[1]) & keep, pack_bf16(v[2], v[3]) & keep, pack_bf16(v[8], v[9]) & keep, pack_bf16(v[10], v[11]) & keep);
    *reinterpret_cast<uint4*>(c1) =
        make_uint4(pack_bf16(v[4], v[5]) & keep, pack_bf16(v[6], v[7]) & keep, pack_bf16(v[12], v[13]) & keep, pack_bf16(v[14], v[15]) & keep);
  };
  int at1[kHalo / 64];  // pixel half + 2 j of h1 this lane makes a row of: y << 16 | x in the rectangle with its halo, -1 past its end
#pragma unroll
  for (int j = 0; j < kHalo / 64; ++j) {
    const int r = 32 * (half + 2 * j) + l31, y = fast_div(r, a.d_rw);
    at1[j] = r < npx ? y << 16 | (r - y * RW) : -1;
  }
  wg_barrier();  // the first input
  int buf = 0, tile = tile0;
  for (int i = 0; i < count; ++i, tile += step) {
    const unsigned xb = buf * kXBytes;
    buf = buf == kXBufs - 1 ? 0 : buf + 1;
    // ---- h1 = relu(s1 * acc + t1), zero outside the image -----------------------------------------------------------------
    const FirstAt p = first_at(a, tile);
#pragma unroll
    for (int j = 0; j < kHalo / 64; ++j) {
      if (32 * (half + 2 * j) >= npx) break;
      f32x16 acc = f32x16{};
      const unsigned pa = xb + first_row(32 * (half + 2 * j) + l31, lhi);
      uint4 fa[4];
#pragma unroll
      for (int kg = 0; kg < 4; ++kg) fa[kg] = *reinterpret_cast<const uint4*>(smem + (pa ^ (kg << 5)));
#pragma unroll
      for (int kg = 0; kg < 4; ++kg) acc = mma_bf16(*reinterpret_cast<const u32x4*>(smem + kW1 + ((wn * 4 + kg) * 64 + lane) * 16), fa[kg], acc);
      const int ry = at1[j] >> 16, rx = at1[j] & 0xffff, y = p.y - 1 + ry, x = p.x - 1 + rx;
      const bool in = (unsigned)y < (unsigned)a.H && (unsigned)x < (unsigned)a.W;
      float v[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 sc = *reinterpret_cast<const float4*>(s_s1 + 32 * wn + 8 * g + 4 * lhi);
        const float4 sh = *reinterpret_cast<const float4*>(s_t1 + 32 * wn + 8 * g + 4 * lhi);
        v[4 * g + 0] = fmaxf(acc[4 * g + 0] * sc.x + sh.x, 0.f);
        v[4 * g + 1] = fmaxf(acc[4 * g + 1] * sc.y + sh.y, 0.f);
        v[4 * g + 2] = fmaxf(acc[4 * g + 2] * sc.z + sh.z, 0.f);
        v[4 * g + 3] = fmaxf(acc[4 * g + 3] * sc.w + sh.w, 0.f);
      }
      unsigned char* const px = smem + kH1 + ry * pitch + rx * kH1Pix + ch * 16;
      if (at1[j] >= 0) put_row(px, px + 16, v, in ? ~0u : 0u);
      __builtin_amdgcn_sched_barrier(0);
    }
    lds_wait();
    wg_barrier();  // h1 complete
    // ---- h2 = relu(s2 * acc + t2): two K steps of a tap at a time, read one ahead of their MFMAs ---------------------------------
    {
      f32x16 acc[2] = {f32x16{}, f32x16{}};
      uint4 fa[2][2][2];
      auto read2 = [&](int q) __attribute__((always_inline)) {  // K steps 2 (q & 1), + 1 of tap q >> 1
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int k = 0; k < 2; ++k)
            fa[q & 1][b][k] = *reinterpret_cast<const uint4*>(tap0[b] + (q / 6 * pitch + q / 2 % 3 * kH1Pix) + (2 * (q & 1) + k) * 32);
      };
      read2(0);
#pragma unroll
      for (int q = 0; q < 18; ++q) {
        if (q + 1 < 18) read2(q + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int b = 0; b < 2; ++b) acc[b] = mma_bf16(w2r[q >> 1][2 * (q & 1) + k], fa[q & 1][b][k], acc[b]);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float v[16];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 sc = *reinterpret_cast<const float4*>(s_s2 + 32 * wn + 8 * g + 4 * lhi);
          const float4 sh = *reinterpret_cast<const float4*>(s_t2 + 32 * wn + 8 * g + 4 * lhi);
          v[4 * g + 0] = fmaxf(acc[b][4 * g + 0] * sc.x + sh.x, 0.f);
          v[4 * g + 1] = fmaxf(acc[b][4 * g + 1] * sc.y + sh.y, 0.f);
          v[4 * g + 2] = fmaxf(acc[b][4 * g + 2] * sc.z + sh.z, 0.f);
          v[4 * g + 3] = fmaxf(acc[b][4 * g + 3] * sc.w + sh.w, 0.f);
        }
        const unsigned r = 32 * (2 * half + b) + l31, f = (r & 7) ^ (r >> 3 & 1);
        unsigned char* const row = smem + kH2 + (i & 1) * (kRows * 128) + r * 128;
        put_row(row + ((ch ^ f) << 4), row + (((ch + 1) ^ f) << 4), v, ~0u);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    lds_wait();
    wg_barrier();  // h2 and the next input complete
  }
  wg_barrier();
  wg_barrier();  // (the others' last rectangle)
}

// The last 1x1 and the shortcut of the rectangle before (waves 4 .. 7)
__device__ __forceinline__ void first_finish(const FirstArgs& a, const int tile0, const int step, const int count, const u32x4 (&w3r)[2][4],
                                             const u32x4 (&wsr)[2][4]) {
  using namespace first;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, w4 = __builtin_amdgcn_readfirstlane(((int)threadIdx.x >> 6) - 4);
  const int l31 = lane & 31, lhi = lane >> 5, l8 = lane >> 3, l7 = lane & 7;
  const float* const s_s3 = reinterpret_cast<const float*>(smem + kTab) + 4 * kMid;
  const float* const s_ss = s_s3 + kOut;
  const float* const s_t = s_ss + kOut;
  const int RW = a.tw + 2, npx = (a.th + 2) * RW, nout = a.th * a.tw;
  unsigned ctr[4];
  int oy[4];  // the output pixel of block t: y << 16 | x in the rectangle; -1 past its end
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int o = 32 * t + l31, y = fast_div(o, a.d_tw), x = o - y * a.tw;
    oy[t] = o < nout ? y << 16 | x : -1;
    ctr[t] = first_row(o < nout ? (y + 1) * RW + x + 1 : 0, lhi);
  }
  const unsigned own = first_row(l31, lhi);
  const __amdgpu_buffer_rsrc_t ors = __builtin_amdgcn_make_buffer_rsrc(a.out, 0, (int)kOob, 0x00020000);
  const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.x), 0, (int)kOob, 0x00020000);
  const unsigned chunk = ((unsigned)l7 ^ (unsigned)l8 ^ (w4 & 1u)) << 4;
  // the pixels this lane requests, from the first output pixel: y << 16 | x & 0xffff; past the end 16384 rows up, outside maps that are not
  // taller and any pixel of those that are (nobody uses what comes to these rows)
  int ld[kHalo / 32];
#pragma unroll
  for (int i = 0; i < kHalo / 32; ++i) {
    const int r = 8 * (w4 + 4 * i) + l8, y = fast_div(r, a.d_rw);
    ld[i] = r < npx ? (y - 1) << 16 | ((r - y * RW - 1) & 0xffff) : -0x40000000;
  }
  auto request = [&](int t, int buf) __attribute__((always_inline)) {  // rows 8 (w4 + 4 i) .. +7 with instruction i
    const FirstAt p = first_at(a, t);
#pragma unroll
    for (int i = 0; i < kHalo / 32; ++i) {
      const int y = p.y + (ld[i] >> 16), x = p.x + (short)ld[i];
      const bool in = (unsigned)y < (unsigned)a.H && (unsigned)x < (unsigned)a.W;
      dma16(xrs, in ? (unsigned)((p.n * a.H + y) * a.W + x) * 128u + chunk : kOob, 0, (unsigned)(buf * kXBytes + (w4 + 4 * i) * 1024));
    }
  };
  request(tile0, 0);
  vm_wait<0>();
  wg_barrier();  // the first input
  if (count > 1) request(tile0 + step, 1);
  wg_barrier();
  vm_wait<0>();
  wg_barrier();  // h1 and h2 of the first rectangle, input of the second
  int buf = 0, tile = tile0;
  for (int i = 0; i < count; ++i, tile += step) {
    const unsigned xb = buf * kXBytes, hb = kH2 + (i & 1) * (kRows * 128);
    buf = buf == kXBufs - 1 ? 0 : buf + 1;
    const FirstAt p = first_at(a, tile);
    // the input after the next goes where the one before this was (past the last: the last one again, so that the count below holds)
    request(i + 2 < count ? tile + 2 * step : tile, buf == kXBufs - 1 ? 0 : buf + 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      float4 sc[4], s4[4], sh[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int c = 64 * w4 + 32 * j + 8 * g + 4 * lhi;
        sc[g] = *reinterpret_cast<const float4*>(s_s3 + c);
        s4[g] = *reinterpret_cast<const float4*>(s_ss + c);
        sh[g] = *reinterpret_cast<const float4*>(s_t + c);
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (j == 1 && t == 1) wg_barrier();  // (h1 of the next rectangle)
        f32x16 o = f32x16{}, os = f32x16{};
#pragma unroll
        for (int kg = 0; kg < 4; ++kg) {
          const uint4 fh = *reinterpret_cast<const uint4*>(smem + hb + t * 4096 + (own ^ (kg << 5)));
          const uint4 fx = *reinterpret_cast<const uint4*>(smem + xb + (ctr[t] ^ (kg << 5)));
          o = mma_bf16(w3r[j][kg], fh, o);
          os = mma_bf16(wsr[j][kg], fx, os);
        }
        float v[16];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          v[4 * g + 0] = fmaxf(o[4 * g + 0] * sc[g].x + (os[4 * g + 0] * s4[g].x + sh[g].x), 0.f);
          v[4 * g + 1] = fmaxf(o[4 * g + 1] * sc[g].y + (os[4 * g + 1] * s4[g].y + sh[g].y), 0.f);
          v[4 * g + 2] = fmaxf(o[4 * g + 2] * sc[g].z + (os[4 * g + 2] * s4[g].z + sh[g].z), 0.f);
          v[4 * g + 3] = fmaxf(o[4 * g + 3] * sc[g].w + (os[4 * g + 3] * s4[g].w + sh[g].w), 0.f);
        }
        to_consecutive_channels(v);  // 0-3, 8-11, 4-7, 12-15: channels 64 w4 + 32 j + 16 lhi + 0 .. 15
        const int y = p.y + (oy[t] >> 16), x = p.x + (oy[t] & 0xffff);
        const unsigned at = oy[t] >= 0 && y < a.H && x < a.W ? (unsigned)((p.n * a.H + y) * a.W + x) * (kOut * 2u) + w4 * 128u + lhi * 32u : kOob;
        const u32x4 lo = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[8], v[9]), pack_bf16(v[10], v[11])};
        const u32x4 hi = {pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]), pack_bf16(v[12], v[13]), pack_bf16(v[14], v[15])};
        // (always sixteen stores a rectangle, which the wait below counts on: pixels that do not exist lie outside the descriptor)
        // (no scalar offset: behind a 16-byte buffer store that has one the compiler leaves no wait state before a vector
        // instruction writes the store's data registers again, and the store then takes what was written)
        __builtin_amdgcn_raw_buffer_store_b128(lo, ors, at + j * 64, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(hi, ors, at + j * 64 + 16, 0, 0);
        __builtin_amdgcn_sched_barrier(0);  // one block at a time (registers)
      }
    }
    vm_wait<16>();  // the input requested above: behind it are this rectangle's sixteen stores
    wg_barrier();  // done with this rectangle's h2 and input; the next one's are complete
  }
  vm_wait<0>();  // (the input nobody waited for)
}

__global__ __launch_bounds__(first::kThreads) void k_first(const FirstArgs a) {
  using namespace first;
  prefetch_args<sizeof(FirstArgs)>();
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, lhi = lane >> 5;
  // workgroup b walks rectangles of its XCD's eighth
  const int per = (a.ntiles + 7) >> 3, xcd = blockIdx.x & 7;
  const int last = min((xcd + 1) * per, a.ntiles), step = (int)gridDim.x >> 3;
  const int tile = xcd * per + (int)(blockIdx.x >> 3);
  if (tile >= last) return;
  const int count = (last - tile + step - 1) / step;

  // ---- weights into registers, through LDS (whole lines from memory) ------------------------------------------------
  auto stage = [&](const void* w, int kb, int at) __attribute__((always_inline)) {  // kb KB of w to LDS byte `at`
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(w), 0, kb * 1024, 0x00020000);
    for (int i = wave; i < kb; i += kThreads / 64) dma16(rs, lane * 16u, (unsigned)i * 1024u, (unsigned)(at + i * 1024));
  };
  constexpr int kW2KB = kMid * 9 * kMid * 2 / 1024, kW3KB = kOut * kMid * 2 / 1024, kW1KB = kMid * kMid * 2 / 1024;
  float* const s_tab = reinterpret_cast<float*>(smem + kTab);
  static_assert((kW2KB + kW1KB) * 1024 <= kTab, "w2 and w1 pass through together");
  stage(a.w2, kW2KB, 0);
  stage(a.w1, kW1KB, kW2KB * 1024);
  for (int i = tid; i < kMid; i += kThreads) {
    s_tab[i] = a.s1[i]; s_tab[kMid + i] = a.t1[i]; s_tab[2 * kMid + i] = a.s2[i]; s_tab[3 * kMid + i] = a.t2[i];
  }
  for (int i = tid; i < kOut; i += kThreads) {
    s_tab[4 * kMid + i] = a.s3[i]; s_tab[4 * kMid + kOut + i] = a.ssc[i]; s_tab[4 * kMid + 2 * kOut + i] = a.t3[i] + a.tsc[i];
  }
  vm_wait<0>();
  lds_wait();
  wg_barrier();
  if (wave < 4) {
    const int wn = wave & 1;
    u32x4 w2r[9][4];
#pragma unroll
    for (int kg = 0; kg < 4; ++kg) {
      const unsigned at = kg * 32 + lhi * 16;
#pragma unroll
      for (int t = 0; t < 9; ++t) w2r[t][kg] = *reinterpret_cast<const u32x4*>(smem + (32 * wn + l31) * (9 * kMid * 2) + t * 128 + at);
      if (wave < 2)
        *reinterpret_cast<u32x4*>(smem + kW1 + ((wn * 4 + kg) * 64 + lane) * 16) =
            *reinterpret_cast<const u32x4*>(smem + kW2KB * 1024 + (32 * wn + l31) * 128 + at);
    }
    lds_wait();
    wg_barrier();
    stage(a.w3, kW3KB, 0);
    stage(a.wsc, kW3KB, kW3KB * 1024);
    vm_wait<0>();
    wg_barrier();
    wg_barrier();
    first_make(a, tile, step, count, w2r);
  } else {
    lds_wait();
    wg_barrier();
    stage(a.w3, kW3KB, 0);
    stage(a.wsc, kW3KB, kW3KB * 1024);
    vm_wait<0>();
    wg_barrier();
    u32x4 w3r[2][4], wsr[2][4];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int kg = 0; kg < 4; ++kg) {
        const unsigned at = (64 * (wave - 4) + 32 * j + l31) * 128 + kg * 32 + lhi * 16;
        w3r[j][kg] = *reinterpret_cast<const u32x4*>(smem + at);
        wsr[j][kg] = *reinterpret_cast<const u32x4*>(smem + kW3KB * 1024 + at);
      }
    lds_wait();
    wg_barrier();
    first_finish(a, tile, step, count, w3r, wsr);
  }
}

// ---- host side ------------------------------------------------------------------------------------------------------
static int g_first_cus[32];
int first_init_device() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 32) return LAUD_ERR_HIP;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return LAUD_ERR_HIP;
  g_first_cus[dev] = cus / 8 * 8;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_first), hipFuncAttributeMaxDynamicSharedMemorySize, first::kLds) == hipSuccess
             ? LAUD_OK : LAUD_ERR_HIP;
}

// workgroups that fill the current device once; 0: no device, or one that cannot be set up
static int first_workgroups() {
  static std::atomic<unsigned> done{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 32) return 0;
  const unsigned bit = 1u << dev;
  if (!(done.load(std::memory_order_acquire) & bit)) {
    if (first_init_device() != LAUD_OK) return 0;
    done.fetch_or(bit, std::memory_order_release);
  }
  return g_first_cus[dev];
}

bool first_plan(int dtype, int c_in, int c_mid, int c_out, int stride, FirstArgs* args) {
  FirstArgs& a = *args;
  const long long rows = (long long)a.N * a.H * a.W;
  // (outputs below 1 GiB.  A workgroup has its weights to fetch, whatever the map: up to a few hundred pixels three launches of small tiles
  // are as fast.  24 x 24 / 40 x 40 / 56 x 56 pixels: 11.7 / 15.0 / 16.8 us, here 12.6 / 13.0 / 13.4.)
  if (stride != 1 || dtype != LAUD_BF16 || c_in != first::kMid || c_mid != first::kMid || c_out != first::kOut || rows <= 1024 ||
      rows >= (1 << 21))
    return false;
  const int wgs = first_workgroups();
  if (wgs <= 0) return false;
  // the rectangle: fewest of them for a map, then the smallest halo
  long long best = 1LL << 60;
  for (int tw = 1; tw <= a.W && tw <= first::kRows; ++tw) {
    int th = first::kRows / tw < a.H ? first::kRows / tw : a.H;
    while (th > 1 && ((th + 2) * (tw + 2) > first::kHalo || th > first::kMaxTh)) --th;
    if ((th + 2) * (tw + 2) > first::kHalo) continue;
    const int nty = (a.H + th - 1) / th, ntx = (a.W + tw - 1) / tw;
    th = (a.H + nty - 1) / nty;
    const long long cost = (long long)nty * ntx * 1024 + (th + 2) * (tw + 2);
    if (cost < best) { best = cost; a.th = th; a.tw = tw; a.ntx = ntx; a.pern = nty * ntx; }
  }
  a.ntiles = a.N * a.pern;
  // A rectangle costs about the same however full it is (about 5 us a round of them, 12 the first), and none spans two samples: what counts is
  // the rounds against those of the other routes, whose tiles are full whatever the map.
  //   small tiles (up to 14336 rows): 1200 / 2700 / 4600 rows of 2 x 2 / 3 x 3 / 3 x 3 (2 rounds here) 13.3 / 18.3 / 18.8 us there, 16.4 / 16.5 /
  //   16.8 here; 12272 / 12288 rows of 4 x 4 (3) 22.8 / 22.7, 23.0 / 22.1; 14000 of 7 x 7 / 5 x 5 / 4 x 4 (2 / 3 / 4) 24.3 / 23.7 / 24.0, 17.9 /
  //   21.7 / 26.0.
  //   k_narrow's rounds of 128 rows a workgroup take 8 us with the first 1x1 ahead of them: 30000 rows (1 of its rounds) of 8 x 8 / 7 x 7 (2 /
  //   3 here) 20.1 / 19.9, 19.3 / 23.5; 100000 (4) of 12 x 12 / 8 x 8 / 4 x 4 (6 / 7 / 25) 42.5 / 42.1 / 42, 39.1 / 43.1 / 116; 400000 (13)
  //   of 9 x 9 / 12 x 12 / 4 x 4 (20 / 22 / 98) 108 / 112 / 110, 108 / 118 / 428.
  const long long rounds = (a.ntiles + wgs - 1) / wgs;
  if (!narrow_supported(dtype, c_mid, c_out, rows)) return rounds == 1 || (rounds - 2) * 9728 + 2560 <= rows;
  const long long full = (rows + (long long)first::kRows * wgs - 1) / ((long long)first::kRows * wgs);
  return 5 * rounds <= 8 * full + 2;
}

int launch_first(const FirstArgs& args, hipStream_t st) {
  const int wgs = first_workgroups();
  if (wgs <= 0) return LAUD_ERR_HIP;
  FirstArgs a = args;
  a.d_rw = make_fast_div(a.tw + 2); a.d_tw = make_fast_div(a.tw); a.d_pern = make_fast_div(a.pern); a.d_ntx = make_fast_div(a.ntx);
  const unsigned grid = (unsigned)(a.ntiles < wgs ? (a.ntiles + 7) / 8 * 8 : wgs);
  StageScope scope(LAUD_STAGE_CONV2, st);
  hipLaunchKernelGGL(k_first, dim3(grid), dim3(first::kThreads), first::kLds, st, a);
  return check_launch();
}

}  // namespace laud
