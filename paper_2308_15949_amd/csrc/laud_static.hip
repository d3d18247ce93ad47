// Static stem of the ResNet body (the whole-body workload): 7x7 stride-2 conv on the 3-channel image with
// folded-BN affine and ReLU, then 3x3 stride-2 max pooling.  Outside the dynamic hot path (it runs once
// per image and is not masked): the usual shape (bf16, 64 channels) is one kernel straight from the image to the
// pooled map, other shapes go through an im2col kernel and the dense MFMA GEMMs (launch_dense_affine), and a plain
// kernel pools.
#include "laud_common.h"
#include "laud_tile_util.h"

#include <algorithm>
#include <atomic>

namespace laud {

constexpr int kStemK = 7 * 7 * 3;  // reduction length of the stem conv ...

constexpr int kStemKp = 152;       // ... padded to a multiple of 8 (16-byte chunks of the GEMM)

// im2col of the 7x7 stride-2 pad-3 windows: row = output pixel, column k = (ky*7 + kx)*3 + c, zero
// outside the image and in the padding columns.  One thread per (row, 8 consecutive columns).
template <typename ET>
__global__ __launch_bounds__(256) void k_stem_im2col(const ET* __restrict__ x, int N, int Hin, int Win, int Ho, int Wo,
                                                     ET* __restrict__ cols) {
  constexpr int CH = kStemKp / 8;
  const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
  if (id >= (long long)N * Ho * Wo * CH) return;
  const int ch = (int)(id % CH);
  const long long pix = id / CH;
  const int n = (int)(pix / (Ho * Wo)), r = (int)(pix - (long long)n * Ho * Wo);
  const int yo = r / Wo, xo = r - yo * Wo;
  ET v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k = ch * 8 + e;
    const int tap = k / 3, c = k - tap * 3;
    const int yy = yo * 2 - 3 + tap / 7, xx = xo * 2 - 3 + tap % 7;
    const bool ok = k < kStemK && yy >= 0 && yy < Hin && xx >= 0 && xx < Win;
    v[e] = ok ? x[(((size_t)n * Hin + yy) * Win + xx) * 3 + c] : (ET)0;
  }
  // 8 elements = one 16-byte store (bf16) or two (float32)
  uint4 raw[sizeof(v) / 16];
  __builtin_memcpy(raw, v, sizeof(v));
  uint4* dst = reinterpret_cast<uint4*>(cols + (size_t)pix * kStemKp + ch * 8);
#pragma unroll
  for (int q = 0; q < (int)(sizeof(v) / 16); ++q) dst[q] = raw[q];
}

typedef __attribute__((ext_vector_type(16))) float stem_f32x16;

// ---- the usual stem (bf16, 64 output channels) in one kernel: 7x7 stride-2 conv, affine, ReLU, 3x3 stride-2 max pooling ----
// As two kernels the conv's output (four times the image, eight times the result) makes a round trip through memory: 190 + 60
// us at 128 images of 224 x 224.  Here it stays in LDS.
//   * A workgroup takes strips of 7 pooled rows (16 conv rows, one of them to spare) and walks along x in steps of 16 conv
//     columns = 8 pooled columns; the step's conv columns and the last one of the step before lie in LDS, so the pooling windows
//     that reach one column back find it there.
//   * Image rows, products and pooling of a step are phases between barriers, each bound by something else; two workgroups a
//     compute unit fill each other's (62.5 KB of LDS, 128 registers a lane).  A wave brings whole image rows, a dword a lane, so what a
//     row and a dword stand for is scalar or the same for all rows.  With 101 KB of LDS, one workgroup a compute unit, 32 conv columns
//     and dwords dealt out over the threads (a division, bounds and masks for each) and copies of 240 bytes (reads in conflict): 128 / 256 images of
//     224 x 224 85.2 / 162 us, here 62.4 / 118; two such workgroups without the rest 80.2 / 151; 8 / 32 images 14.5 / 27.0 -> 14.4 / 26.0.
//   * Implicit GEMM per step: 256 rows (conv pixels) x 64 channels.  A window row is 21 consecutive values of the image
//     (7 pixels x 3 channels), padded to 24 = three 16-byte fragments: K = 7 x 24 (+ 8) = 176 in eleven 32x32x16 steps.  A
//     fragment starts 12 * column bytes into the image row, so each image row is kept in LDS four times, shifted by 0, 12,
//     24 and 36 bytes: column x reads copy x % 4, where its fragments are 16-byte aligned.  The 48 bytes of a window in its copy
//     are no other window's, so the padding is stored as zeros (the pixel beside the window, met by zero weights, would
//     make a NaN of an infinity).
//   * 8 waves: wave (wm, wn) computes rows 64 wm .. +63, channels 32 wn .. +31, weights in 44 registers per lane for the
//     workgroup's whole life.  The next step's image rows are on their way in registers meanwhile.
//   * ReLU leaves bf16 values whose bit patterns order like 16-bit integers: pooling is a packed integer maximum, and
//     positions outside the conv's output count as zeros.
constexpr int kSpRows = 7, kSpCols = 8;               // pooled rows of a strip, pooled columns of a step
constexpr int kSpIn = 37;                             // image rows of a strip: 2 * 15 + 7
constexpr int kSpCopyDw = 48;                         // dwords of a copy: four windows
constexpr int kSpCopy = 4 * kSpCopyDw, kSpRowB = 4 * kSpCopy;  // bytes of a copy (192: the fragments of 16 conv columns meet 16 bank groups), of a row
constexpr int kSpZero = kSpIn * kSpRowB;              // 16 bytes of zeros
constexpr int kSpConv = (kSpZero + 16 + 255) / 256 * 256;
constexpr int kSpSlots = 17;                          // conv columns in LDS: 0 .. 14 of the step, the last one of this and the previous step
constexpr int kSpAff = kSpConv + 16 * kSpSlots * 128; // conv values [16 rows][17 columns][64 channels]
constexpr int kSpLds = kSpAff + 2 * 64 * 4;           // scale and shift
// Place of conv column c of a step (-1: the last one of the step before).  Columns two apart, which a pooling read takes together, lie in
// different halves of the 256 bytes LDS serves at once; 16-byte chunk ch of a column is at ch ^ sp_swizzle(c): the sixteen columns of a
// block's store are spread over all of them.
__device__ __forceinline__ unsigned sp_slot(int c, int step) {
  return c < 0 ? 15u + ((unsigned)(step - 1) & 1u) : c == 15 ? 15u + ((unsigned)step & 1u) : (unsigned)((c & 12) | ((c & 1) << 1) | ((c >> 1) & 1));
}
__device__ __forceinline__ unsigned sp_swizzle(int c) { return ((unsigned)c & 1u) | (((unsigned)c >> 1) & 6u); }
constexpr int kSpThreads = 512, kSpLoads = (kSpIn + 7) / 8;  // image rows a wave brings, a dword of each per lane
__global__ __launch_bounds__(kSpThreads, 4) void k_stem_pool_bf16(const bf16_t* __restrict__ x, int N, int Hin, int Win, int Hc, int Wc,
                                                               int Hp, int Wp, int strips, int chunks, int chunk_steps,
                                                               const bf16_t* __restrict__ w7, const float* __restrict__ s,
                                                               const float* __restrict__ t, bf16_t* __restrict__ out) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, lhi = lane >> 5, wm = wave >> 1, wn = wave & 1;
  if (tid < 4) reinterpret_cast<unsigned*>(smem + kSpZero)[tid] = 0u;
  // weights into registers, through LDS: K step st of this lane is window row f / 3, values 8 (f % 3) .. +7, f = 2 st + lhi
  {
    unsigned* d = reinterpret_cast<unsigned*>(smem);
    for (int i = tid; i < 64 * kStemK / 2; i += kSpThreads) d[i] = reinterpret_cast<const unsigned*>(w7)[i];
  }
  __syncthreads();
  u32x4 wr[11];
#pragma unroll
  for (int st = 0; st < 11; ++st) {
    const int f = 2 * st + lhi, ky = f / 3, j = f - ky * 3;
    const bf16_t* src = reinterpret_cast<const bf16_t*>(smem) + (32 * wn + l31) * kStemK + ky * 21 + 8 * j;
    unsigned e[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) e[k] = ky < 7 && 8 * j + k < 21 ? (unsigned)src[k] : 0u;
    wr[st] = u32x4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
  }
  if (tid < 128) reinterpret_cast<float*>(smem + kSpAff)[tid] = tid < 64 ? s[tid] : t[tid - 64];
  // fragment addresses of this lane's first 32-row block (two conv rows; the second lies two rows on), without the K step's part: of lane
  // half 1 the next fragment, which is 16 bytes on or opens the next window row
  const unsigned abase = (unsigned)(2 * (wm * 4 + (l31 >> 4)) * kSpRowB + (l31 & 3) * kSpCopy + ((l31 & 15) >> 2) * 48);
  const unsigned same_row = abase + lhi * 16, next_row = abase + lhi * (kSpRowB - 32);
  // which bits of this lane's dword lie inside the window it belongs to in copy q (dwords 10 and 11 of a window's twelve: its last value
  // and the padding)
  unsigned inside[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) inside[q] = lane % 12 == (10 + 3 * q) % 12 ? 0xffffu : lane % 12 == (11 + 3 * q) % 12 ? 0u : ~0u;
  const int units = N * strips * chunks, nsteps = (Wp + kSpCols - 1) / kSpCols;
  for (int u = blockIdx.x; u < units; u += gridDim.x) {
    const int c = u % chunks, ns = u / chunks, n = ns / strips, p0 = (ns - n * strips) * kSpRows;
    const int first = c * chunk_steps, stop = min(first + chunk_steps, nsteps);
    const int iy0 = 4 * p0 - 5, cy0 = 2 * p0 - 1;  // first image row, first conv row
    const int s0 = first > 0 ? first - 1 : 0;      // the step before supplies the conv column to the left
    unsigned pre[kSpLoads];
    // A lane brings dword `lane` of rows wave + 8 i of a step: values e, e + 1 of the row's 3 Win, outside the image zero.  The load reads the
    // nearest two values there are; what they stand for is worked out when they are stored, a step later.
    auto request = [&](int step) __attribute__((always_inline)) {
      const int e = min(max((32 * step - 3) * 3 + 2 * lane, 0), 3 * Win - 2);
#pragma unroll
      for (int i = 0; i < kSpLoads; ++i) {
        const int iy = min(max(iy0 + wave + 8 * i, 0), Hin - 1);
        __builtin_memcpy(&pre[i], x + ((size_t)n * Hin + iy) * Win * 3 + e, 4);
      }
    };
    auto store_rows = [&](int step) __attribute__((always_inline)) {
      const int e = (32 * step - 3) * 3 + 2 * lane;
      const int shl = e < 0 ? 16 : 0, shr = e > 3 * Win - 2 ? 16 : 0;
      const unsigned live = e < -1 || e > 3 * Win - 1 ? 0u : ~0u;
      unsigned v[kSpLoads];
#pragma unroll
      for (int i = 0; i < kSpLoads; ++i) {
        const int iy = iy0 + wave + 8 * i;
        v[i] = ((pre[i] << shl) >> shr) & (iy >= 0 && iy < Hin ? live : 0u);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (lane >= 3 * q && lane < 3 * q + kSpCopyDw) {
#pragma unroll
          for (int i = 0; i < kSpLoads; ++i)
            if (wave + 8 * i < kSpIn)
              *reinterpret_cast<unsigned*>(smem + (wave + 8 * i) * kSpRowB + lane * 4 + q * (kSpCopy - 12)) = v[i] & inside[q];
        }
    };
    request(s0);
    __syncthreads();  // the weights, or the previous unit's last reads
    for (int step = s0; step < stop; ++step) {
      store_rows(step);
      __syncthreads();
      if (step + 1 < stop) request(step + 1);
      stem_f32x16 acc[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
      uint4 fa[2][2];  // fragments of the two blocks, read one K step ahead of their products
      auto fragments = [&](int st) __attribute__((always_inline)) {
        // lane half h: fragment f = 2 st + h; the last one (f = 21) has zero weights and reads zeros
        const int f = 2 * st;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const unsigned o = (unsigned)((f / 3 + 4 * i) * kSpRowB + f % 3 * 16);
          const unsigned at = st == 10 ? (lhi ? (unsigned)kSpZero : abase + o) : (f % 3 == 2 ? next_row : same_row) + o;
          fa[st & 1][i] = *reinterpret_cast<const uint4*>(smem + at);
        }
      };
      fragments(0);
#pragma unroll
      for (int st = 0; st < 11; ++st) {
        if (st < 10) fragments(st + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i] = mma_bf16(wr[st], fa[st & 1][i], acc[i]);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int rr = wm * 64 + i * 32 + l31, r = rr >> 4, C = rr & 15, X = 16 * step + C, Y = cy0 + r;
        const bool live = Y >= 0 && Y < Hc && X < Wc;
        float v[16];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 sc = *reinterpret_cast<const float4*>(smem + kSpAff + (32 * wn + 8 * g + 4 * lhi) * 4);
          const float4 sh = *reinterpret_cast<const float4*>(smem + kSpAff + 256 + (32 * wn + 8 * g + 4 * lhi) * 4);
          v[4 * g + 0] = fmaxf(acc[i][4 * g + 0] * sc.x + sh.x, 0.f);
          v[4 * g + 1] = fmaxf(acc[i][4 * g + 1] * sc.y + sh.y, 0.f);
          v[4 * g + 2] = fmaxf(acc[i][4 * g + 2] * sc.z + sh.z, 0.f);
          v[4 * g + 3] = fmaxf(acc[i][4 * g + 3] * sc.w + sh.w, 0.f);
        }
        to_consecutive_channels(v);
        uint4 c0 = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[8], v[9]), pack_bf16(v[10], v[11]));
        uint4 c1 = make_uint4(pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]), pack_bf16(v[12], v[13]), pack_bf16(v[14], v[15]));
        if (!live) c0 = c1 = make_uint4(0, 0, 0, 0);
        unsigned char* const at = smem + kSpConv + ((unsigned)r * kSpSlots + sp_slot(C, step)) * 128u;
        const unsigned ch = (wn * 4u + lhi * 2u) ^ sp_swizzle(C);
        *reinterpret_cast<uint4*>(at + (ch << 4)) = c0;
        *reinterpret_cast<uint4*>(at + ((ch ^ 1u) << 4)) = c1;
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
      if (step >= first && tid < kSpRows * kSpCols * 8) {
        const unsigned ch = tid & 7u;
        const int q = (tid >> 3) & (kSpCols - 1), p = tid >> 6, P = p0 + p, X = step * kSpCols + q;
        typedef __attribute__((ext_vector_type(8))) short s16x8;
        s16x8 m = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int dx = -1; dx < 2; ++dx) {
          const int c = 2 * q + dx;
          if (c < 0 && step == 0) continue;
          const unsigned at = kSpConv + (2 * p * kSpSlots + sp_slot(c, step)) * 128 + ((ch ^ sp_swizzle(c & 15)) << 4);
#pragma unroll
          for (int dy = 0; dy < 3; ++dy)
            m = __builtin_elementwise_max(m, *reinterpret_cast<const s16x8*>(smem + at + dy * kSpSlots * 128));
        }
        if (P < Hp && X < Wp) *reinterpret_cast<s16x8*>(out + (((size_t)n * Hp + P) * Wp + X) * 64 + ch * 8) = m;
      }
    }
    __syncthreads();
  }
}

// Weights [c_out][7][7][3] -> [c_out][kStemKp] with zero padding columns.
template <typename ET>
__global__ void k_stem_pack_weights(const ET* __restrict__ w7, int c_out, ET* __restrict__ wp) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= c_out * kStemKp) return;
  const int o = i / kStemKp, k = i - o * kStemKp;
  wp[i] = k < kStemK ? w7[o * kStemK + k] : (ET)0;
}

// One thread per (output pixel, 8 channels).
template <typename ET>
__global__ __launch_bounds__(256) void k_maxpool3x3s2(const ET* __restrict__ in, int N, int H, int W, int C, int Ho,
                                                      int Wo, ET* __restrict__ out) {
  const int groups = C / 8;
  const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
  if (id >= (long long)N * Ho * Wo * groups) return;
  const int g = (int)(id % groups);
  const long long pix = id / groups;
  const int n = (int)(pix / (Ho * Wo)), r = (int)(pix - (long long)n * Ho * Wo);
  const int yo = r / Wo, xo = r - yo * Wo;
  float m[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) m[e] = -INFINITY;
  for (int ky = 0; ky < 3; ++ky) {
    const int yy = yo * 2 - 1 + ky;
    if (yy < 0 || yy >= H) continue;
    for (int kx = 0; kx < 3; ++kx) {
      const int xx = xo * 2 - 1 + kx;
      if (xx < 0 || xx >= W) continue;
      const ET* p = in + (((size_t)n * H + yy) * W + xx) * C + g * 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) m[e] = fmaxf(m[e], elem<ET>::load(p + e));
    }
  }
  ET* po = out + (size_t)pix * C + g * 8;
#pragma unroll
  for (int e = 0; e < 8; ++e) elem<ET>::store(po + e, m[e]);
}

// Stem of the RegNet backbones: 3x3 stride-2 pad-1 conv from the 3-channel image, affine, ReLU.  One thread per
// output pixel: the 27 inputs of its window are read once into registers, then the output channels are produced
// eight at a time from the 27 x c_out float32 weights in LDS (all lanes read the same weight: a broadcast).
// Takes what the matrix-core kernel below does not.
template <typename ET>
__global__ __launch_bounds__(256) void k_stem3x3(const ET* __restrict__ in, int N, int H, int W, int Ho, int Wo,
                                                 const ET* __restrict__ w, const float* __restrict__ s,
                                                 const float* __restrict__ t, int C, ET* __restrict__ out) {
  extern __shared__ float s_w3[];  // [27][C] weights (tap-major, output channel fastest), then scale [C], shift [C]
  for (int i = threadIdx.x; i < 27 * C; i += 256) {
    const int o = i % C, k = i / C;
    s_w3[i] = elem<ET>::load(w + (size_t)o * 27 + k);
  }
  float* s_sc = s_w3 + 27 * C;
  float* s_sh = s_sc + C;
  for (int i = threadIdx.x; i < C; i += 256) { s_sc[i] = s[i]; s_sh[i] = t[i]; }
  __syncthreads();
  const long long pix = (long long)blockIdx.x * 256 + threadIdx.x;
  if (pix >= (long long)N * Ho * Wo) return;
  const int n = (int)(pix / (Ho * Wo)), r = (int)(pix - (long long)n * Ho * Wo);
  const int yo = r / Wo, xo = r - yo * Wo;
  float v[27];
#pragma unroll
  for (int ky = 0; ky < 3; ++ky) {
    const int yy = yo * 2 - 1 + ky;
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
      const int xx = xo * 2 - 1 + kx;
      const bool ok = yy >= 0 && yy < H && xx >= 0 && xx < W;
      const ET* p = in + (((size_t)n * H + (ok ? yy : 0)) * W + (ok ? xx : 0)) * 3;
#pragma unroll
      for (int c = 0; c < 3; ++c) v[(ky * 3 + kx) * 3 + c] = ok ? elem<ET>::load(p + c) : 0.f;
    }
  }
  ET* po = out + (size_t)pix * C;
  for (int g = 0; g < C; g += 8) {
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
    for (int k = 0; k < 27; ++k) {
      const float* wk = s_w3 + k * C + g;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += v[k] * wk[e];
    }
    ET o8[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) elem<ET>::store(&o8[e], fmaxf(acc[e] * s_sc[g + e] + s_sh[g + e], 0.f));
    if constexpr (sizeof(ET) == 2) {
      uint4 q;
      __builtin_memcpy(&q, o8, 16);
      *reinterpret_cast<uint4*>(po + g) = q;
    } else {
      uint4 q0, q1;
      __builtin_memcpy(&q0, o8, 16);
      __builtin_memcpy(&q1, o8 + 4, 16);
      reinterpret_cast<uint4*>(po + g)[0] = q0;
      reinterpret_cast<uint4*>(po + g)[1] = q1;
    }
  }
}

// The same on the matrix cores, for bf16 images of even width and c_out a multiple of 32.  One wave makes 32 output pixels of
// one row x 32 channels: a window row is nine consecutive values of the image; with the value ahead of them (zeroed here: it
// may be anything) they start at a 4-byte boundary, ten values = five dwords.  K = 32: four fragments of eight, the first eight
// values of each of the three window rows and the last pairs of all three together.  Fragments are loaded from the image as
// they are (neighbouring windows overlap in the cache); rows outside the image lie outside the descriptor and read as zero.
// The vector-ALU kernel reads 27 x c_out weights from LDS per wave of 64 pixels, which is what bounds it: about 105 us at 128
// images of 224 x 224 and 32 channels; this one takes 42 (142 MB read and written: 3.4 TB/s of a copy's 4.3).
constexpr int kS3Waves = 4, kS3Blocks = 2048;  // eight workgroups per compute unit, each wave walking over its tiles
__global__ __launch_bounds__(64 * kS3Waves) void k_stem3x3_mfma(const bf16_t* __restrict__ in, unsigned in_bytes, int rows, int H, int W,
                                                                int Ho, int Wo, int xtiles, const bf16_t* __restrict__ w,
                                                                const float* __restrict__ s, const float* __restrict__ t, int C,
                                                                bf16_t* __restrict__ out) {
  const int lane = threadIdx.x & 63, l31 = lane & 31, lhi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int c0 = 32 * blockIdx.y;
  constexpr unsigned kOob = 0x80000000u;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(in), 0, (int)in_bytes, 0x00020000);
  // weights of channel c0 + l31: fragment lhi, then fragment 2 + lhi
  u32x4 wr[2];
  {
    const bf16_t* wc = w + (size_t)(c0 + l31) * 27;
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const int f = 2 * st + lhi;
      unsigned e[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int i = f < 3 ? f * 9 + k - 1 : (k >> 1) * 9 + 7 + (k & 1);
        const bool none = f < 3 ? k == 0 : k > 5;
        e[k] = none ? 0u : (unsigned)wc[none ? 0 : i];
      }
      wr[st] = u32x4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
    }
  }
  float4 sc[4], sh[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    __builtin_memcpy(&sc[g], s + c0 + 8 * g + 4 * lhi, 16);
    __builtin_memcpy(&sh[g], t + c0 + 8 * g + 4 * lhi, 16);
  }
  const int units = rows * xtiles;
  for (int u = blockIdx.x * kS3Waves + wave; u < units; u += gridDim.x * kS3Waves) {
    const int R = u / xtiles, x0 = (u - R * xtiles) * 32, n = R / Ho, yo = R - n * Ho;
    const int xo = min(x0 + l31, Wo - 1), yc = 2 * yo;  // (pixels past the row's end repeat the last one; not stored)
    const unsigned rowb = (unsigned)W * 6u, mid = (unsigned)(n * H + yc) * rowb;
    const unsigned top = yc > 0 ? mid - rowb : kOob, bot = yc + 1 < H ? mid + rowb : kOob;
    // (the leftmost window starts outside the image: its load starts at the row and is moved up below)
    const unsigned lead = 12u * xo - (xo > 0 ? 8u : 0u), tail = lhi ? 12u * xo + 8u : kOob;
    u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(rs, (lhi ? mid : top) + lead, 0, 0);
    u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(rs, (lhi ? kOob : bot) + lead, 0, 0);
    const unsigned d0 = __builtin_amdgcn_raw_buffer_load_b32(rs, (top + tail) | (tail & kOob) | (top & kOob), 0, 0);
    const unsigned d1 = __builtin_amdgcn_raw_buffer_load_b32(rs, mid + tail, 0, 0);
    const unsigned d2 = __builtin_amdgcn_raw_buffer_load_b32(rs, (bot + tail) | (tail & kOob) | (bot & kOob), 0, 0);
    auto window = [&](const u32x4& v) __attribute__((always_inline)) {
      return xo > 0 ? make_uint4(v.x & 0xffff0000u, v.y, v.z, v.w) : make_uint4(0u, 0u, v.x, v.y);
    };
    const uint4 fa = window(a), wb = window(b);
    const uint4 fb = make_uint4(lhi ? d0 : wb.x, lhi ? d1 : wb.y, lhi ? d2 : wb.z, lhi ? 0u : wb.w);
    stem_f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    acc = mma_bf16(wr[0], fa, acc);
    acc = mma_bf16(wr[1], fb, acc);
    float v[16];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      v[4 * g + 0] = fmaxf(acc[4 * g + 0] * sc[g].x + sh[g].x, 0.f);
      v[4 * g + 1] = fmaxf(acc[4 * g + 1] * sc[g].y + sh[g].y, 0.f);
      v[4 * g + 2] = fmaxf(acc[4 * g + 2] * sc[g].z + sh[g].z, 0.f);
      v[4 * g + 3] = fmaxf(acc[4 * g + 3] * sc[g].w + sh[g].w, 0.f);
    }
    to_consecutive_channels(v);
    if (x0 + l31 < Wo) {
      uint4* po = reinterpret_cast<uint4*>(out + ((size_t)R * Wo + xo) * C + c0 + 16 * lhi);
      po[0] = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[8], v[9]), pack_bf16(v[10], v[11]));
      po[1] = make_uint4(pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]), pack_bf16(v[12], v[13]), pack_bf16(v[14], v[15]));
    }
  }
}

}  // namespace laud

using namespace laud;

extern "C" int laud_stem3x3(const void* x, int N, int Hin, int Win, int dtype, const void* w3, const float* s,
                            const float* t, int c_out, void* out, void* stream) {
  if (!x || !w3 || !s || !t || !out || N <= 0 || Hin <= 0 || Win <= 0 || c_out <= 0) return LAUD_ERR_INVALID_ARG;
  if (dtype != LAUD_F32 && dtype != LAUD_BF16) return LAUD_ERR_INVALID_ARG;
  if (c_out % 8 || c_out > 256) return LAUD_ERR_UNSUPPORTED;
  const int Ho = (Hin - 1) / 2 + 1, Wo = (Win - 1) / 2 + 1;
  const long long work = (long long)N * Ho * Wo;
  if ((work + 255) / 256 > 0x7fffffffLL) return LAUD_ERR_UNSUPPORTED;
  hipStream_t st = (hipStream_t)stream;
  clear_stale_error();
  const long long in_bytes = (long long)N * Hin * Win * 6;
  if (dtype == LAUD_BF16 && c_out % 32 == 0 && Win % 2 == 0 && Win >= 4 && in_bytes < 0x7fffffffLL && (reinterpret_cast<uintptr_t>(x) & 3u) == 0) {
    const int xtiles = (Wo + 31) / 32;
    const long long units = (long long)N * Ho * xtiles;
    const long long wgs = std::min<long long>((units + kS3Waves - 1) / kS3Waves, kS3Blocks);
    hipLaunchKernelGGL(k_stem3x3_mfma, dim3((unsigned)wgs, (unsigned)(c_out / 32)), dim3(64 * kS3Waves), 0, st, (const bf16_t*)x,
                       (unsigned)in_bytes, N * Ho, Hin, Win, Ho, Wo, xtiles, (const bf16_t*)w3, s, t, c_out, (bf16_t*)out);
    return check_launch();
  }
  const unsigned blocks = (unsigned)((work + 255) / 256);
  const size_t lds = (size_t)29 * c_out * sizeof(float);
  if (dtype == LAUD_BF16)
    hipLaunchKernelGGL((k_stem3x3<bf16_t>), dim3(blocks), dim3(256), lds, st, (const bf16_t*)x, N, Hin, Win, Ho, Wo,
                       (const bf16_t*)w3, s, t, c_out, (bf16_t*)out);
  else
    hipLaunchKernelGGL((k_stem3x3<float>), dim3(blocks), dim3(256), lds, st, (const float*)x, N, Hin, Win, Ho, Wo,
                       (const float*)w3, s, t, c_out, (float*)out);
  return check_launch();
}

namespace laud {
// Requests the stem kernel's LDS once per device; the device's compute units.
int stem_init_device(int* cus_out) {
  static std::atomic<int> cus_of[32];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 32) return LAUD_ERR_HIP;
  int cus = cus_of[dev].load(std::memory_order_acquire);
  if (cus == 0) {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return LAUD_ERR_HIP;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_stem_pool_bf16), hipFuncAttributeMaxDynamicSharedMemorySize, kSpLds) !=
        hipSuccess)
      return LAUD_ERR_HIP;
    cus_of[dev].store(cus, std::memory_order_release);
  }
  if (cus_out) *cus_out = cus;
  return LAUD_OK;
}
}  // namespace laud

namespace {
struct StemWs { size_t cols, wp, conv, bytes; };
StemWs stem_ws_layout(int N, int Hin, int Win, int c_out, int dtype) {
  const size_t eb = elem_bytes(dtype), rows = (size_t)N * ((Hin - 1) / 2 + 1) * ((Win - 1) / 2 + 1);
  StemWs w;
  size_t o = 0;
  w.cols = o; o += align_up(rows * kStemKp * eb, 256);
  w.wp = o;   o += align_up((size_t)c_out * kStemKp * eb, 256);
  w.conv = o; o += align_up(rows * c_out * eb, 256);
  w.bytes = o;
  return w;
}
}  // namespace

extern "C" size_t laud_stem_workspace(int N, int Hin, int Win, int c_out, int dtype) {
  if (N <= 0 || Hin <= 0 || Win <= 0 || c_out <= 0 || (dtype != LAUD_F32 && dtype != LAUD_BF16)) return 0;
  return stem_ws_layout(N, Hin, Win, c_out, dtype).bytes;
}

extern "C" int laud_stem(const void* x, int N, int Hin, int Win, int dtype, const void* w7, const float* s,
                         const float* t, int c_out, void* out, void* ws, size_t ws_bytes, void* stream) {
  if (!x || !w7 || !s || !t || !out || N <= 0 || Hin <= 0 || Win <= 0 || c_out <= 0) return LAUD_ERR_INVALID_ARG;
  if (dtype != LAUD_F32 && dtype != LAUD_BF16) return LAUD_ERR_INVALID_ARG;
  if (c_out % 8) return LAUD_ERR_UNSUPPORTED;
  if (!ws || ws_bytes < laud_stem_workspace(N, Hin, Win, c_out, dtype)) return LAUD_ERR_WORKSPACE;
  const int Hc = (Hin - 1) / 2 + 1, Wc = (Win - 1) / 2 + 1;  // 7x7, stride 2, pad 3
  const int Hp = (Hc - 1) / 2 + 1, Wp = (Wc - 1) / 2 + 1;    // 3x3, stride 2, pad 1
  const long long rows = (long long)N * Hc * Wc;
  if (rows > 0x7fffffffLL / 2) return LAUD_ERR_UNSUPPORTED;
  hipStream_t st = (hipStream_t)stream;
  clear_stale_error();
  const StemWs L = stem_ws_layout(N, Hin, Win, c_out, dtype);
  char* wsb = (char*)ws;
  void *cols = wsb + L.cols, *wp = wsb + L.wp, *conv = wsb + L.conv;
  if (dtype == LAUD_BF16 && c_out == 64 && (reinterpret_cast<uintptr_t>(w7) & 3u) == 0) {
    int cus;
    if (stem_init_device(&cus) != LAUD_OK) return LAUD_ERR_HIP;
    // with fewer strips than compute units a strip is cut along x (each cut repeats one step)
    const int strips = (Hp + kSpRows - 1) / kSpRows, nsteps = (Wp + kSpCols - 1) / kSpCols;
    const long long ns = (long long)N * strips;
    const int chunks = (int)std::min<long long>(nsteps, std::max<long long>(1, cus / ns));
    const int chunk_steps = (nsteps + chunks - 1) / chunks;
    hipLaunchKernelGGL(k_stem_pool_bf16, dim3((unsigned)std::min<long long>(ns * chunks, 2 * cus)), dim3(kSpThreads), kSpLds, st,
                       (const bf16_t*)x, N, Hin, Win, Hc, Wc, Hp, Wp, strips, chunks, chunk_steps, (const bf16_t*)w7, s, t,
                       (bf16_t*)out);
    return check_launch();
  }
  const unsigned iblocks = (unsigned)((rows * (kStemKp / 8) + 255) / 256);
  const unsigned wblocks = (unsigned)((c_out * kStemKp + 255) / 256);
  const unsigned pblocks = (unsigned)(((long long)N * Hp * Wp * (c_out / 8) + 255) / 256);
  if (dtype == LAUD_BF16) {
    hipLaunchKernelGGL((k_stem_im2col<bf16_t>), dim3(iblocks), dim3(256), 0, st, (const bf16_t*)x, N, Hin, Win, Hc, Wc,
                       (bf16_t*)cols);
    hipLaunchKernelGGL((k_stem_pack_weights<bf16_t>), dim3(wblocks), dim3(256), 0, st, (const bf16_t*)w7, c_out,
                       (bf16_t*)wp);
  } else {
    hipLaunchKernelGGL((k_stem_im2col<float>), dim3(iblocks), dim3(256), 0, st, (const float*)x, N, Hin, Win, Hc, Wc,
                       (float*)cols);
    hipLaunchKernelGGL((k_stem_pack_weights<float>), dim3(wblocks), dim3(256), 0, st, (const float*)w7, c_out,
                       (float*)wp);
  }
  if (check_launch() != LAUD_OK) return LAUD_ERR_HIP;
  int rc = launch_dense_affine(dtype, cols, wp, s, t, conv, rows, kStemKp, c_out, 1, st);
  if (rc != LAUD_OK) return rc;
  if (dtype == LAUD_BF16)
    hipLaunchKernelGGL((k_maxpool3x3s2<bf16_t>), dim3(pblocks), dim3(256), 0, st, (const bf16_t*)conv, N, Hc, Wc, c_out,
                       Hp, Wp, (bf16_t*)out);
  else
    hipLaunchKernelGGL((k_maxpool3x3s2<float>), dim3(pblocks), dim3(256), 0, st, (const float*)conv, N, Hc, Wc, c_out, Hp,
                       Wp, (float*)out);
  return check_launch();
}
