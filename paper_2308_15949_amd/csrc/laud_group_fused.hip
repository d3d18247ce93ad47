// First 1x1 and group 3x3 of the RegNetY blocks in one launch, bf16, on gfx950 MFMA: h1 stays in LDS.
//
// On narrow maps the two launches are bound by h1, which goes out and comes back nine taps wide, and by their starts and ends.  Here a
// workgroup takes a tile of up to 64 output pixels -- whole patches, or rows of one larger patch -- and 64 channels (whole groups: the
// 3x3 reads the same 64 channels of h1), makes h1 on the tile's input pixels with their halo and takes the 3x3 from there.  The halo is
// made once per tile: 81 pixels for 16 outputs of a 4 x 4 patch at stride two (64 without a halo), 36 without stride, 16 for 4
// of a 2 x 2 patch, which the 1x1's short reductions allow.  The pixel lists (k_need) are not needed either.
// First blocks of RegNetY-800MF, 128 images (pixel lists, first 1x1, 3x3 before): stage 1 18 + 75 + 66 -> 64 us, stage 2 7 + 40 + 33 -> 53,
// stage 3 5 + 38 + 17 -> 45; identity block of stage 2, whole samples, 15 + 17 -> 33 (not taken there).
//   Rows of x and of w1 come by LDS-direct loads in slices of 64 channels (32 at a time, half lines of the L2, took 10 % longer from three
// slices on) through a ring of two slots, without stride of three smaller ones.  h1 lies over the second slot, so that the first slices
// of the next tile are under way while the 3x3 runs.  The 3x3 has two taps in an MFMA of 16 channels (groups are no wider), its weights in
// registers for the workgroup's life, 40 instead of the 72 of k_group's one tap with 32; what a lane reads of h1 for each tap is the
// same in every tile.  What bounds it: the vector ALU's share of h1 (scale, maximum, rounding: 60 instructions per 32 x 32 block) and a
// slice's trip (1.1 us with two workgroups a compute unit).
#include "laud_common.h"
#include "laud_gemm.h"
#include "laud_tile_util.h"

#include <algorithm>
#include <atomic>

namespace laud {

typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace gfuse {
constexpr int kBN = 64, kThreads = 256, kPerXcd = 64;  // workgroups of an XCD: two for each of its 32 compute units
constexpr unsigned kOob = 0x80000000u;
// A tile: up to 32 Q outputs from up to CAP pixels of h1, slices of 64 channels of x and w1 through a ring of SLOTS slots.  Stride two
// takes <1>, as its outputs need up to nine pixels each; without stride <2>.
template <int Q>
struct Tile {
  static constexpr int kOut = 32 * Q, kCap = Q == 1 ? 192 : 144, kSlots = Q == 1 ? 2 : 3, kBlocks = 3;  // blocks of 32 pixels a wave makes
  static constexpr int kWAt = kCap * 128, kSlot = kWAt + kBN * 128;   // w1's slice lies behind the rows
  static constexpr int kH1 = kSlot, kTurn = kH1 + kCap * 128;         // h1 and the turned results lie over the second slot
  static constexpr int kTab = kSlots * kSlot;                         // offsets of the rows of two tiles
  static constexpr int kZero = kTab + 2 * kCap * 4;                   // 64 zero bytes; scale, shift of the 3x3
  static constexpr int kLds = kZero + 64 + 2 * kBN * 4;
  static_assert(kTurn + 4 * 1024 * Q <= 2 * kSlot && kZero % 64 == 0 && 2 * kLds <= 160 * 1024, "LDS of two workgroups");
  static_assert(2 * kBlocks * 32 * 128 <= kSlot && 2 * kBlocks * 32 >= kCap, "MFMAs read whole blocks of rows");
};
}  // namespace gfuse

struct GroupFusedArgs {
  GemmArgs g;                      // the 3x3, with A = x, lda = K = c_in
  const void* w1; const float* s1; const float* t1;
  int rows, strips, patches;       // output rows of a patch a tile takes, tiles a patch, patches a tile
  int hw, nh;                      // width of the halo, pixels of a tile's patch with its halo
  FastDiv ct, hwd, nhd, s, unit, pps, wp, st;
};

template <int Q>
__global__ __launch_bounds__(gfuse::kThreads, 2) void k_group_fused(const GroupFusedArgs ka) {
  using namespace gfuse;
  using T = Tile<Q>;
  constexpr int CAP = T::kCap, SLOTS = T::kSlots, NB = T::kBlocks, NI = (CAP / 8 + 3) / 4;
  static_assert(CAP <= kThreads, "a thread looks up one pixel");
  prefetch_args<sizeof(GroupFusedArgs)>();
  const GemmArgs& a = ka.g;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned* const s_voff = reinterpret_cast<unsigned*>(smem + T::kTab);  // [2][CAP]
  float* const s_aff = reinterpret_cast<float*>(smem + T::kZero + 64);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  const int l31 = lane & 31, lhi = lane >> 5, l15 = lane & 15, l4 = lane >> 4;
  // workgroup b: column tile of its XCD's b >> 3, tiles from the XCD's eighth on
  const int slot = blockIdx.x >> 3, xcd = blockIdx.x & 7, walker = fast_div(slot, ka.ct), step = fast_div(kPerXcd, ka.ct);
  const int col0 = (slot - walker * a.col_tiles) * kBN;
  const int cnt = *a.count, ntiles = ka.strips > 1 ? cnt * ka.strips : (cnt + ka.patches - 1) / ka.patches, per = (ntiles + 7) >> 3;
  const int last = min((xcd + 1) * per, ntiles);
  int tile = xcd * per + walker;
  if (walker >= step || tile >= last) return;
  const int C = a.Ncols, K = a.K, nsl = (K + 63) >> 6, sy = a.stride > 1 ? a.stride : 1;

  // ---- the pixel of h1 this thread looks up: patch of the tile, row and column in it; its list entry a tile ahead --------------------
  const int pp = fast_div(tid, ka.nhd), pw = tid - pp * ka.nh, pr = fast_div(pw, ka.hwd), pc = pw - pr * ka.hw;
  int entry;
  const auto fetch = [&](int t) __attribute__((always_inline)) {
    entry = a.list[min(ka.strips > 1 ? fast_div(t, ka.st) : t * ka.patches + pp, cnt - 1)];
  };
  fetch(tile);
  // offsets of a tile's rows in x; a pixel outside the image, or past the list, lies outside the descriptor
  const auto look_up = [&](int t, unsigned* dst) __attribute__((always_inline)) {
    const int Wp = fast_div(sy > 1 ? a.Wo : a.W, ka.s), pps = fast_div(sy > 1 ? a.Ho : a.H, ka.s) * Wp;
    const int strip = ka.strips > 1 ? t - fast_div(t, ka.st) * ka.strips : 0;
    const int n = fast_div(entry, ka.pps), e = entry - n * pps, py = fast_div(e, ka.wp), px = e - py * Wp;
    const int y = (py * a.S + strip * ka.rows) * sy - 1 + pr, x = px * a.S * sy - 1 + pc;
    const bool ok = pp < ka.patches && (ka.strips > 1 || t * ka.patches + pp < cnt) && (unsigned)y < (unsigned)a.H && (unsigned)x < (unsigned)a.W;
    if (tid < CAP) dst[tid] = ok ? (unsigned)((n * a.H + y) * a.W + x) * (unsigned)(K * 2) : kOob;
  };

  // ---- the 3x3's weights, two taps an MFMA: lane = output channel l15 of 16, 8 input channels of the same 16, tap 2 j + (l4 >> 1);
  // what lies outside the channel's group is zero -----------------------------------------------------------------------------------
  u32x4 w[5][2];
  {
    const int gw = a.gw;
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.Wt), 0, C * 9 * gw * 2, 0x00020000);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = col0 + 32 * wn + 16 * h + l15;
      const int rel = col0 + 32 * wn + 16 * h + 8 * (l4 & 1) - (c & ~(gw - 1));  // (group widths are powers of two)
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        const int t = 2 * j + (l4 >> 1);
        w[j][h] = __builtin_amdgcn_raw_buffer_load_b128(
            wrsrc, (unsigned)((c * 9 + t) * gw + rel) * 2u | ((unsigned)(rel | (gw - 1 - rel) | (C - 1 - c) | (8 - t)) & kOob), 0, 0);
      }
    }
  }
  if (tid < 2 * kBN) {
    const int col = col0 + (tid & (kBN - 1));
    s_aff[tid] = col < C ? (tid < kBN ? a.scale : a.shift)[col] : 0.f;
  } else if (tid < 2 * kBN + 16) {
    *reinterpret_cast<float*>(smem + T::kZero + (tid - 2 * kBN) * 4) = 0.f;
  }
  // ---- LDS-direct loads: instruction j fills rows 8 j .. +7 of a slot, eight lanes a row; chunk c of row r lies at c ^ (r & 7) ^ ((r >> 3) & 1)
  const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.A), 0, (int)kOob, 0x00020000);
  const __amdgpu_buffer_rsrc_t w1rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(ka.w1), 0, C * K * 2, 0x00020000);
  const int chunk = (lane & 7) ^ (lane >> 3) ^ (wave & 1), njx = (ka.patches * ka.nh + 7) >> 3, mine = (njx - wave + 3) >> 2;  // of the rows' instructions
  const int wrow = col0 + 8 * wave + (lane >> 3);
  const unsigned w1off = (unsigned)(wrow * K + 8 * chunk) * 2u, w1far = wrow + 32 < C ? 0u : kOob, w1near = wrow < C ? 0u : kOob;
  unsigned voff[NI];
  const auto offsets = [&](const unsigned* tab) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NI; ++i) voff[i] = tab[min(8 * (wave + 4 * i) + (lane >> 3), CAP - 1)] + 16u * chunk;
  };
  const auto issue = [&](int s, unsigned slot_at, bool weights) __attribute__((always_inline)) {
    const unsigned base = __builtin_amdgcn_readfirstlane(slot_at + (unsigned)wave * 1024u);
    const unsigned tail = (unsigned)(K - 1 - 64 * s - 8 * chunk) & kOob;  // channels past the last one: zero on both sides
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (i < mine) dma16(xrsrc, voff[i] | tail, (unsigned)s * 128u, base + (unsigned)i * 4096u);
    if (weights) {
      dma16(w1rsrc, w1off | tail | w1near, (unsigned)s * 128u, base + T::kWAt);
      dma16(w1rsrc, (w1off + (unsigned)K * 64u) | tail | w1far, (unsigned)s * 128u, base + T::kWAt + 4096u);
    }
  };
  // at most one slice's loads of this wave under way (fewer, where list entries or results came later)
  const auto wait_one = [&]() __attribute__((always_inline)) {
    switch (mine) {
      case 0: vm_wait<2>(); break;
      case 1: vm_wait<3>(); break;
      case 2: vm_wait<4>(); break;
      case 3: vm_wait<5>(); break;
      case 4: vm_wait<6>(); break;
      default: vm_wait<7>(); break;
    }
  };
  // slice s lies in the slot with this address: in turn the first, the third, the second, which is h1's between its tiles
  const auto next_slot = [&](unsigned at) __attribute__((always_inline)) { return SLOTS == 2 ? T::kSlot - at : at == 0 ? 2u * T::kSlot : at - T::kSlot; };
  const unsigned frag = (unsigned)l31 * 128u + (((unsigned)lhi ^ ((unsigned)l31 & 7u) ^ ((unsigned)(l31 >> 3) & 1u)) << 4);
  // row r of h1 lies at r ^ ((r >> 1) & 1), its 16-byte chunk c at c ^ ((r >> 1 ^ r >> 4) & 7): no bank conflicts for sixteen rows in a
  // row, nor for every second one
  const auto h1_at = [&](int r, int c) __attribute__((always_inline)) {
    return (unsigned)T::kH1 + (unsigned)(r ^ (r >> 1 & 1)) * 128u + (unsigned)((c ^ (r >> 1 ^ r >> 4)) & 7) * 16u;
  };
  unsigned tap[Q][5];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int i = 16 * (Q * wm + q) + l15, p0 = fast_div(i, ka.unit), un = ka.rows * a.S, p = p0 < ka.patches ? p0 : 0, o = p0 < ka.patches ? i - p0 * un : 0;
    const int oy = fast_div(o, ka.s), b = p * ka.nh + oy * sy * ka.hw + (o - oy * a.S) * sy;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      const int t = 2 * j + (l4 >> 1);
      tap[q][j] = t < 9 ? h1_at(b + t / 3 * ka.hw + t % 3, 4 * wn + (l4 & 1)) : (unsigned)T::kZero;  // (there is no tenth tap)
    }
  }
  // where a lane's four channels 8 g + 4 lhi of row 32 wm + l31 go: ^ g << 4; those of the i-th block 64 i rows on: ^ 64 where i is odd
  const unsigned put = h1_at(32 * wm + l31, 4 * wn) + 8 * lhi;
  const int put_odd = (put & 64) ? -64 : 64;
  float sc1[16], sh1[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int col = min(col0 + 32 * wn + 8 * (e / 4) + 4 * lhi + e % 4, C - 1);
    sc1[e] = ka.s1[col];
    sh1[e] = ka.t1[col];
  }
  int par = 0;
  look_up(tile, s_voff);
  fetch(tile + step);
  lds_wait();
  wg_barrier();
  offsets(s_voff);
  issue(0, 0, true);
  if (SLOTS > 2 && nsl > 1) issue(1, next_slot(0), true);
  for (; tile < last; tile += step, par ^= 1) {
    const bool more = tile + step < last;
    // ---- first 1x1 -----------------------------------------------------------------------------------------------------------------
    f32x16 acc[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) acc[i] = f32x16{};
    unsigned at = 0, ahead = T::kSlot;  // slots of slice s, of slice s + SLOTS - 1
    for (int s = 0; s < nsl; ++s) {
      if (SLOTS > 2 && s + 1 < nsl) wait_one(); else vm_wait<0>();
      lds_wait();
      wg_barrier();  // slice s is there, everyone is done with the one before, or with h1
      if (s + SLOTS - 1 < nsl) issue(s + SLOTS - 1, ahead, true);
      if (s == 0) {
        if (more) look_up(tile + step, s_voff + (par ^ 1) * CAP);
        fetch(tile + 2 * step);
      }
      const int left = K - 64 * s;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        if (16 * ks < left) {  // (all four without a branch need 50 registers more, and are slower)
          const unsigned f = at + (frag ^ (ks << 5));
          const u32x4 wf = *reinterpret_cast<const u32x4*>(smem + f + T::kWAt + wn * 4096);
#pragma unroll
          for (int i = 0; i < NB; ++i)
            acc[i] = mma_bf16(wf, *reinterpret_cast<const uint4*>(smem + f + wm * 4096 + i * 8192), acc[i]);
        }
      ahead = at;
      at = next_slot(at);
    }
    // (The compiler, which does not see the LDS-direct loads, waits for the entry here and not behind some of them.)
    asm volatile("" : "+v"(entry));
    lds_wait();
    wg_barrier();  // everyone is done with the ring
    if (more) {
      offsets(s_voff + (par ^ 1) * CAP);
      issue(0, 0, nsl > 1);  // (a single slice of w1 stays)
      if (SLOTS > 2 && nsl > 1) issue(1, next_slot(0), true);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int r = 32 * (2 * i + wm) + l31;
      const bool in = 64 * i + 63 < CAP || r < CAP, ok = s_voff[par * CAP + (in ? r : 0)] < kOob;  // the padding is zero
      const unsigned at = put + (((i & 1) ? put_odd : 0u) + i * 8192);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaxf(acc[i][4 * g + e] * sc1[4 * g + e] + sh1[4 * g + e], 0.f);
        const u32x2 two = {ok ? pack_bf16(v[0], v[1]) : 0u, ok ? pack_bf16(v[2], v[3]) : 0u};
        if (in) *reinterpret_cast<u32x2*>(smem + (at ^ (g << 4))) = two;
      }
    }
    lds_wait();
    wg_barrier();  // h1
    // ---- group 3x3 -----------------------------------------------------------------------------------------------------------------
    f32x4 o[Q][2];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int h = 0; h < 2; ++h) o[q][h] = f32x4{};
#pragma unroll
    for (int j = 0; j < 5; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const u32x4 f = *reinterpret_cast<const u32x4*>(smem + (tap[q][j] ^ (h << 5)));
          o[q][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[j][h]), __builtin_bit_cast(bf16x8, f), o[q][h], 0, 0, 0);
        }
    // a lane holds channels 16 h + 4 l4 .. +3 of pixel 16 q + l15
    unsigned char* const turn = smem + T::kTurn + wave * (1024 * Q);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4 sc = *reinterpret_cast<const f32x4*>(s_aff + 32 * wn + 16 * h + 4 * l4);
      const f32x4 sh = *reinterpret_cast<const f32x4*>(s_aff + kBN + 32 * wn + 16 * h + 4 * l4);
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaxf(o[q][h][e] * sc[e] + sh[e], 0.f);
        const u32x2 two = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        *reinterpret_cast<u32x2*>(turn + row_put((l4 & 1) * 32 + 16 * q + l15, 2 * h + (l4 >> 1))) = two;
      }
    }
    // compact rows of the tile: patches in the list's order, rows of a patch one after the other
    const int SS = a.S * a.S, te = ka.strips > 1 ? fast_div(tile, ka.st) : tile * ka.patches, first = ka.strips > 1 ? (tile - te * ka.strips) * ka.rows : 0;
    const int nrows = ka.strips > 1 ? min(ka.rows, a.S - first) * a.S : min(ka.patches, cnt - te) * SS;
    const long long row0 = (long long)te * SS + first * a.S;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const u32x4 r = *reinterpret_cast<const u32x4*>(turn + row_get(lane, q));
      const int i = 16 * (Q * wm + q) + (lane >> 2), col = col0 + 32 * wn + 8 * (lane & 3);
      if (i < nrows && col < C) *reinterpret_cast<u32x4*>(reinterpret_cast<__bf16*>(a.Out) + (size_t)(row0 + i) * a.ldo + col) = r;
    }
  }
}

// ---- host side ------------------------------------------------------------------------------------------------------
int group_fused_init_device() {
  static std::atomic<unsigned> done{0};  // one bit per device ordinal (ordinals >= 32 repeat the request)
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return LAUD_ERR_HIP;
  const unsigned bit = dev >= 0 && dev < 32 ? 1u << dev : 0u;
  if (bit && (done.load(std::memory_order_acquire) & bit)) return LAUD_OK;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_group_fused<1>), hipFuncAttributeMaxDynamicSharedMemorySize, gfuse::Tile<1>::kLds) != hipSuccess ||
      hipFuncSetAttribute(reinterpret_cast<const void*>(&k_group_fused<2>), hipFuncAttributeMaxDynamicSharedMemorySize, gfuse::Tile<2>::kLds) != hipSuccess)
    return LAUD_ERR_HIP;
  done.fetch_or(bit, std::memory_order_release);
  return LAUD_OK;
}

namespace {
// How a patch of S x S outputs is cut into tiles of up to `out` outputs whose pixels with halo are up to `cap`; false: not at all.
bool cut(int S, int stride, GroupFusedArgs* k) {
  const int out = stride > 1 ? gfuse::Tile<1>::kOut : gfuse::Tile<2>::kOut, cap = stride > 1 ? gfuse::Tile<1>::kCap : gfuse::Tile<2>::kCap;
  const int hw = (S - 1) * stride + 3;
  if (S > out || 3 * hw > cap) return false;
  int rows = std::min(S, out / S);
  while (((rows - 1) * stride + 3) * hw > cap) --rows;
  k->strips = (S + rows - 1) / rows;
  k->rows = rows = (S + k->strips - 1) / k->strips;
  k->hw = hw;
  k->nh = ((rows - 1) * stride + 3) * hw;
  k->patches = k->strips > 1 ? 1 : std::min(out / (S * S), cap / k->nh);
  return true;
}
}  // namespace

// Against first 1x1 and 3x3 in launches of their own, whole blocks of the RegNetY-400MF / -800MF stages at ratios 0.2 / 0.5 / 0.9.
// Stride two, where the first 1x1 makes four pixels of h1 for each output that the 3x3 leaves: 128 images of stage 1 (32 -> 64)
// 95.5 / 155 / 241 -> 64.8 / 96.7 / 136 us, stage 2 (64 -> 144) 74.9 / 103 / 136 -> 61.0 / 83.7 / 118, stage 3 (144 -> 320) 62.7 / 82.1 /
// 103 -> 49.8 / 71.5 / 92.2, one image of stage 1 23.2 / 28.1 / 33.4 -> 21.0 / 25.8 / 30.6.  A reduction of more than 96 channels on one
// image (196 outputs) is faster split over the waves of the small tiles' workgroups (stage 3 22.5 / 23.1, stage 4 31.9 / 34.5), and one of
// more than 256 pays for its halo once there is more than a round of tiles (stage 4, 128 images, S = 1: 71 / 88 / 112 -> 63 / 85 / 119).
// Without stride the halo is all overhead: a tile costs its slices whatever it yields, so that the more there are, the more outputs it
// has to have.  128 images at 0.5, of S = 2 / 4 / 7 (36, 64, 49 outputs a tile): 64 channels 111 / 96 / 90 -> 104 / 79 / 78, 144
// channels 91 / 83 / 81 -> 93 / 75 / 77, 320 channels (S = 2 / 7) 58 / 53 -> 65 / 54.  Whole samples have no pixel lists to save: 144 channels
// of 28 x 28 70.8 -> 72.2, 104 channels 49.9 -> 48.4.  In one round of tiles the launch saved outweighs any halo (stage 3 of 8 images,
// S = 2, 208 / 320 channels 29.0 / 31.9 -> 26.4 / 30.0); 196 rows of 320 channels are even, of 784 33.6 -> 38.7.
bool group_fused_wanted(int dtype, int c_in, int c_mid, int group_width, int S, int stride, bool whole, long long cap_rows) {
  GroupFusedArgs k{};
  if (dtype != LAUD_BF16 || group_width > 16 || c_mid > kGroupMaxC || !cut(S, stride, &k)) return false;
  const long long patches = cap_rows / (S * S), tiles = k.strips > 1 ? patches * k.strips : (patches + k.patches - 1) / k.patches;
  const bool one_round = tiles * ((c_mid + gfuse::kBN - 1) / gfuse::kBN) <= 8 * gfuse::kPerXcd;
  if (stride > 1) return c_in <= 96 || (cap_rows > 256 && (c_in <= 256 || (c_in <= 384 && one_round)));
  const int outputs = k.strips > 1 ? S * S / k.strips : k.patches * S * S;
  return outputs >= 32 + 6 * ((c_in + 63) / 64) + (whole ? 8 : 0) || (one_round && (c_in <= 256 || (c_in <= 384 && cap_rows > 1024)));
}

int launch_group_fused(const GemmArgs& args, const void* w1, const float* s1, const float* t1, long long cap_rows, hipStream_t st) {
  if (group_fused_init_device() != LAUD_OK) return LAUD_ERR_HIP;
  GroupFusedArgs k{};
  k.g = args;
  GemmArgs& a = k.g;
  const int stride = a.stride > 1 ? a.stride : 1;
  if (!cut(a.S, stride, &k)) return LAUD_ERR_UNSUPPORTED;
  k.w1 = w1; k.s1 = s1; k.t1 = t1;
  const int oH = stride > 1 ? a.Ho : a.H, oW = stride > 1 ? a.Wo : a.W;
  const long long patches = cap_rows / (a.S * a.S), tiles = k.strips > 1 ? patches * k.strips : (patches + k.patches - 1) / k.patches;
  a.row_tiles = (int)tiles;
  a.col_tiles = (a.Ncols + gfuse::kBN - 1) / gfuse::kBN;
  k.ct = make_fast_div(a.col_tiles); k.hwd = make_fast_div(k.hw); k.nhd = make_fast_div(k.nh); k.s = make_fast_div(a.S);
  k.unit = make_fast_div(k.rows * a.S); k.st = make_fast_div(k.strips);
  k.pps = make_fast_div((oH / a.S) * (oW / a.S)); k.wp = make_fast_div(oW / a.S);
  const dim3 grid((unsigned)(8 * std::min<long long>(gfuse::kPerXcd, (tiles + 7) / 8 * a.col_tiles)));
  if (stride > 1) hipLaunchKernelGGL((k_group_fused<1>), grid, dim3(gfuse::kThreads), gfuse::Tile<1>::kLds, st, k);
  else hipLaunchKernelGGL((k_group_fused<2>), grid, dim3(gfuse::kThreads), gfuse::Tile<2>::kLds, st, k);
  return check_launch();
}

}  // namespace laud
