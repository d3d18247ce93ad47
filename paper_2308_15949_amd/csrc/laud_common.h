// Shared host/device helpers of the gfx950 dynamic-bottleneck library (internal header).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "laud.h"

namespace laud {

constexpr int kWave = 64;  // CDNA wavefront width

// ---- workspace carving: every sub-buffer starts on a 256-byte boundary ------------------
__host__ __device__ inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ---- element types -----------------------------------------------------------------------
// bf16 is stored as its 16-bit pattern; arithmetic is always float32.
typedef uint16_t bf16_t;

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// Round-to-nearest-even, quiet NaN preserved.
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)0x7fc0;
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

template <typename ET> struct elem;
template <> struct elem<float> {
  static constexpr int per16 = 4;  // elements per 16-byte chunk
  __device__ static __forceinline__ float load(const float* p) { return *p; }
  __device__ static __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct elem<bf16_t> {
  static constexpr int per16 = 8;
  __device__ static __forceinline__ float load(const bf16_t* p) { return bf16_to_f32(*p); }
  __device__ static __forceinline__ void store(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

// ---- wave-level primitives ---------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

// Brings a kernel's whole argument block into the scalar cache with one round trip: one word of every 64-byte line is
// requested before anything else.  The compiler loads arguments where they are first used, one line and one trip to memory
// after the other, which a launch of a few microseconds notices.
template <int BYTES>
__device__ __forceinline__ void prefetch_args() {
  const __attribute__((address_space(4))) unsigned* p =
      (const __attribute__((address_space(4))) unsigned*)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr int kLines = (BYTES + 63) / 64;
  unsigned v[kLines];
#pragma unroll
  for (int i = 0; i < kLines; ++i) v[i] = p[i * 16];
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
  for (int i = 0; i < kLines; ++i) asm volatile("" ::"s"(v[i]));
#endif
}

// Number of set bits of a 64-bit ballot below the calling lane.
__device__ __forceinline__ int ballot_prefix(unsigned long long b) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
}

// Exclusive scan of one count per wave across the (at most 64) waves of a block: every wave leaves
// its count in wsum[wave], one barrier, then each wave scans the counts with wave shuffles (no thread
// walks the list alone).  Returns the sum of the counts of the waves before this one; *total gets the
// block's sum.  wsum must not be reused by the next call before another barrier: alternate two arrays.
__device__ __forceinline__ int scan_wave_counts(int count, int nwaves, int* wsum, int* total) {
  const int lane = lane_id(), wave = (int)threadIdx.x / kWave;
  if (lane == 0) wsum[wave] = count;
  __syncthreads();
  const int v = lane < nwaves ? wsum[lane] : 0;
  int incl = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int t = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += t;
  }
  *total = __shfl(incl, kWave - 1, kWave);
  return __shfl(incl - v, wave, kWave);
}

// lower_bound over a sorted list by a whole wave: 64 probes per round instead of one, so a list of n entries
// takes ceil(log64 n) dependent round trips.  Every lane of the wave must call it; all get the result.
__device__ __forceinline__ int wave_lower_bound(const int32_t* v, int n, int key) {
  const int lane = lane_id();
  int lo = 0, hi = n;  // the answer lies in [lo, hi]
  while (hi > lo) {
    const int step = (hi - lo + kWave - 1) / kWave;
    const int pos = lo + lane * step;
    const bool below = pos < hi && v[pos] < key;  // true for a prefix of the lanes (sorted list)
    const int c = __popcll(__ballot(below));
    if (c == 0) {
      hi = lo;
    } else {
      const int nhi = min(lo + c * step, hi);
      lo = lo + (c - 1) * step + 1;
      hi = nhi;
    }
  }
  return lo;
}

// The same for two keys at once (their round trips overlap).
__device__ __forceinline__ void wave_lower_bound2(const int32_t* v, int n, int key0, int key1, int& r0, int& r1) {
  const int lane = lane_id();
  int lo[2] = {0, 0}, hi[2] = {n, n};
  const int key[2] = {key0, key1};
  while (hi[0] > lo[0] || hi[1] > lo[1]) {
    int step[2], val[2];
    bool in[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      step[i] = (hi[i] - lo[i] + kWave - 1) / kWave;
      const int pos = lo[i] + lane * step[i];
      in[i] = pos < hi[i];
      val[i] = v[in[i] ? pos : 0];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (hi[i] <= lo[i]) continue;
      const int c = __popcll(__ballot(in[i] && val[i] < key[i]));
      if (c == 0) {
        hi[i] = lo[i];
      } else {
        const int nhi = min(lo[i] + c * step[i], hi[i]);
        lo[i] = lo[i] + (c - 1) * step[i] + 1;
        hi[i] = nhi;
      }
    }
  }
  r0 = lo[0];
  r1 = lo[1];
}

// n / d by the reciprocal 1 / d, exact for n below 2^21: (n + 1/2) / d is at least 1 / 2d away from an integer, the product's
// error is below (n + 1) / d * 2^-23.
__host__ __device__ __forceinline__ int fdiv(int n, float inv) { return (int)(((float)n + 0.5f) * inv); }

// n / d for 0 <= n < 2^31 as a multiplication and a shift, exact: mul = ceil(2^(31+l) / d) with 2^l >= d exceeds 2^(31+l) / d by
// less than 1, which over n < 2^31 adds less than 1 / d to the quotient.
struct FastDiv { uint32_t mul, shift; };
inline FastDiv make_fast_div(int d) {
  uint32_t l = 0;
  while ((1ull << l) < (unsigned long long)d) ++l;
  return {(uint32_t)(((1ull << (31 + l)) + d - 1) / d), l};
}
__device__ __forceinline__ int fast_div(int n, FastDiv f) { return (int)(__umulhi((unsigned)n << 1, f.mul) >> f.shift); }

// Whether the 3x3 window (at spatial stride 1 or 2) of any active output pixel covers input pixel (y, x); pm: mask of the patches
// [rows][Wp] of the sample.  Output rows ceil((y-1)/stride) .. floor((y+1)/stride), clipped, lie in at most three rows of
// patches: nine look-ups that do not wait for each other.
__device__ __forceinline__ bool window_active(const unsigned char* pm, int y, int x, int stride, int Ho, int Wo, int Wp, FastDiv d_s) {
  const int y0 = max(stride > 1 ? y >> 1 : y - 1, 0), y2 = min(stride > 1 ? (y + 1) >> 1 : y + 1, Ho - 1), y1 = min(y0 + 1, y2);
  const int x0 = max(stride > 1 ? x >> 1 : x - 1, 0), x2 = min(stride > 1 ? (x + 1) >> 1 : x + 1, Wo - 1), x1 = min(x0 + 1, x2);
  const int r[3] = {fast_div(y0, d_s) * Wp, fast_div(y1, d_s) * Wp, fast_div(y2, d_s) * Wp};
  const int c[3] = {fast_div(x0, d_s), fast_div(x1, d_s), fast_div(x2, d_s)};
  unsigned any = 0;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) any |= pm[r[i] + c[j]];
  return any != 0;
}

// Entry of an index list that row `rho` of a launch over `rows` >= 1 rows (entries * S * S) belongs to.  Rows past the last one
// repeat its entry: a caller's list may end, and its memory with it, at the last of its *count entries.
__host__ __device__ __forceinline__ int list_entry(int rho, int rows, float inv_ss) {
  return fdiv(rho < rows ? rho : rows - 1, inv_ss);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

__device__ __forceinline__ int wave_sum_int(int v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// ---- host-side launch checking -----------------------------------------------------------
// hipGetLastError() reports (and clears) the last error of ANY earlier HIP call of the thread,
// the caller's included; each entry point clears that state once, after validation and before
// its first launch, so that check_launch() sees only the library's own launches.
inline void clear_stale_error() { (void)hipGetLastError(); }
inline int check_launch() { return hipGetLastError() == hipSuccess ? LAUD_OK : LAUD_ERR_HIP; }

inline bool valid_fmap(const laud_fmap& f) {
  return f.N > 0 && f.H > 0 && f.W > 0 && f.C > 0 && (f.dtype == LAUD_F32 || f.dtype == LAUD_BF16);
}
inline size_t elem_bytes(int dtype) { return dtype == LAUD_BF16 ? 2 : 4; }

// Compaction works on blocks of this many mask bytes.
constexpr int kCompactBlock = 4096;
inline size_t compact_ws_bytes(long long n) {
  long long nb = (n + kCompactBlock - 1) / kCompactBlock;
  return align_up((size_t)(nb > 0 ? nb : 1) * sizeof(int32_t), 256);
}

// Launches the ordered compaction of `n` mask bytes on `stream` (see laud_mask.hip).
int launch_compact(const uint8_t* mask, int n, int32_t* idx, int32_t* count, int32_t* sample_offsets,
                   int per_sample, int32_t* block_counts, hipStream_t stream);

// Pools a per-pixel masker projection over S x S patches, thresholds, and launches the ordered
// compaction (one launch for small patch counts); see laud_mask.hip.
int launch_pool_compact(const float* proj, int N, int H, int W, int S, float bias, const uint8_t* keep, uint8_t* mask,
                        float* logits, int32_t* idx, int32_t* count, int32_t* sample_offsets, int32_t* block_counts,
                        hipStream_t stream);

// Dense GEMM + per-column affine (+ ReLU) on the MFMA kernels of laud_pipe.h and laud_skinny.hip:
// Out[r][c] = act(scale[c] * sum_k A[r][k] * Wt[c][k] + shift[c]), A [rows][K], Wt [ncols][K], all of `dtype`.
int launch_dense_affine(int dtype, const void* A, const void* Wt, const float* scale, const float* shift, void* Out,
                        long long rows, int K, int ncols, int relu, hipStream_t stream);

// The SE module on the compact rows h2 [rows][C] of the active patches (pps patches per sample, SS pixels per
// patch, at most cap_rows rows); see laud_se.hip.  `scratch` holds N*(2*C + se_width) floats.
constexpr int kSeMaxC = 4096, kSeMaxHidden = 1024;  // widest layer / SE hidden layer the kernels keep in LDS
int launch_se(int dtype, int N, int pps, int SS, int C, const laud_group_se* e, void* h2, const int32_t* idx,
              const int32_t* count, float* scratch, long long cap_rows, hipStream_t stream);

// Out-of-place calls: pixels of inactive patches keep their value, so they are copied from x to out, bit for bit.  The copy
// rides in extra workgroups of the block's last launch (nblocks of them, from workgroup id `first` on): it has nothing to
// wait for but the index list, and the compute units that launch leaves idle carry it.  (As a launch of its own it took 4 us
// on one image and 14 us on 128 images of the stage-3 map.)
struct InactiveCopy {
  const uint4* x;
  uint4* out;
  const int32_t* idx;    // ascending active patch ids
  const int32_t* count;
  int npatch, Hp, Wp;    // patches, patch grid
  int S, W, H;           // patch size, map size
  int cpp;               // 16-byte chunks per pixel
  int first, nblocks;
};
constexpr int kCopyPatches = 1024;  // most patches one workgroup takes at a time
InactiveCopy inactive_copy(const void* x, void* out, const laud_fmap& fx, int S, const int32_t* idx, const int32_t* count);

// Share `part` of `nparts` of the copy, counted in pixel rows of patches (a patch may be a whole map); flags: kCopyPatches bytes
// of LDS.
template <int NT>
__device__ __forceinline__ void copy_inactive_part(const InactiveCopy& c, int part, int nparts, unsigned char* flags) {
  // (a vector type of the compiler's own: an array of the uint4 struct went to scratch memory, 80 bytes a lane that every
  // wave of the launch was given, tiles included)
  typedef __attribute__((ext_vector_type(4))) unsigned chunk;
  const chunk* const x = reinterpret_cast<const chunk*>(c.x);
  chunk* const out = reinterpret_cast<chunk*>(c.out);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int cnt = *c.count;
  const int rows = c.npatch * c.S, per = (rows + nparts - 1) / nparts;
  const int r0 = part * per, r1 = min(r0 + per, rows);  // (parts behind the last row: nothing)
  if (r0 >= r1) return;
  const int p0 = r0 / c.S, p1 = (r1 + c.S - 1) / c.S;
  const int rowc = c.S * c.cpp;  // chunks in one pixel row of a patch
  for (int q0 = p0; q0 < p1; q0 += kCopyPatches) {
    const int n = min(kCopyPatches, p1 - q0);
    for (int i = tid; i < n; i += NT) flags[i] = 0;
    const int lo = wave_lower_bound(c.idx, cnt, q0);
    __syncthreads();
    for (int i = tid; i < n && lo + i < cnt; i += NT) {  // at most n entries of the sorted list fall into the range
      const int q = c.idx[lo + i] - q0;
      if (q < n) flags[q] = 1;
    }
    __syncthreads();
    for (int r = max(r0, q0 * c.S) + wave; r < min(r1, (q0 + n) * c.S); r += NT / kWave) {  // one wave per pixel row of a patch
      const int q = r / c.S;
      if (flags[q - q0]) continue;
      const int s = q / (c.Hp * c.Wp), g = q - s * (c.Hp * c.Wp), py = g / c.Wp, px = g - py * c.Wp;
      const size_t off = (((size_t)s * c.H + py * c.S + (r - q * c.S)) * c.W + px * c.S) * c.cpp;
      int i = lane;
      for (; i + 3 * kWave < rowc; i += 4 * kWave) {
        chunk v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = x[off + i + u * kWave];
#pragma unroll
        for (int u = 0; u < 4; ++u) out[off + i + u * kWave] = v[u];
      }
      for (; i < rowc; i += kWave) out[off + i] = x[off + i];
    }
    __syncthreads();
  }
}

// conv2 -> conv3 -> residual add in one kernel (laud_tail.hip), for the shapes tail_supported() names.
struct TailArgs {
  const void* h1;        // [pixels of the input grid][MID] bf16, conv1's output at pixel positions
  const void* wpacked;   // w2 and w3 in MFMA fragment order (launch_tail_pack), tail_packed_bytes() bytes
  const float* s2; const float* t2;  // [MID]
  const float* s3; const float* t3;  // [cout]
  const void* res;       // residual [output pixels][cout] (x, or the shortcut already in `out`)
  void* out;             // [output pixels][cout]; may alias res
  const int32_t* count;  // device: number of active patches
  const int32_t* list;   // device: ascending active patch ids
  int H, W;              // input grid of h1
  int S;                 // patch size on the output grid
  int stride, Ho, Wo;    // spatial stride of the 3x3 and the output grid (stride 1: Ho = H, Wo = W)
  int cout;
  int relu;
  int pb;                // tile height in blocks of 32 pixels (1..3); 0 = chosen on the device from the count
  // channel skipping (Fig. 2(c)) on whole samples (S = H: a "patch" is a sample, `list` the samples in processing
  // order): sbits[i] = kept channel groups (bit g) of the i-th sample of the list, cs_group = channels per group (a
  // multiple of 64).  Input slices of groups no row of a tile keeps are skipped in the 3x3, and h2 is zeroed in the
  // groups a row drops.  Null: no channel mask.
  const uint8_t* sbits;
  int cs_group;
  InactiveCopy cp;       // nblocks 0: in place
  int wg_target;         // workgroups that fill the device once (its compute units; set by launch_tail)
  FastDiv d_s, d_ss, d_wp, d_pps;  // S, S * S, patches of a row and of a sample (set by launch_tail)
};

bool tail_supported(int dtype, int c_mid, int c_out);
int tail_init_device();
size_t tail_packed_bytes(int c_mid, int c_out);
// re-orders w2 [c_mid][3][3][c_mid] and w3 [c_out][c_mid] into the order the fused kernel streams them
int launch_tail_pack(const void* w2, const void* w3, int c_out, void* packed, hipStream_t stream);
// cap_rows: pixels of the output map, the upper bound of the active ones (grid size); the count itself stays on the device
int launch_tail(const TailArgs& a, long long cap_rows, hipStream_t stream);

// conv1 on every pixel (+ masker projection) with register-resident weights (laud_head.hip), for head_supported() shapes.
struct HeadArgs {
  const void* x;         // [m_rows][K] bf16
  const void* wpacked;   // w1 in MFMA fragment order (launch_head_pack), head_packed_bytes() bytes
  const float* s1; const float* t1;  // [256]
  void* h1;              // [m_rows][256] bf16
  int m_rows, K;
  const float* wmask;    // masker weights [K] or null
  float* proj;           // [m_rows] per-pixel projection (with wmask)
  // sparse form (the gather fused into the first 1x1): rows are pixel ids taken from per-group lists; list == null: dense
  const int32_t* list;   // [ngroups][group_rows] ascending pixel ids of the dilated active set
  const int32_t* counts; // [ngroups] device: valid entries per group
  int group_rows;        // capacity of one group's list
  // ... or the active patches themselves: every workgroup works out its group's list, m_rows groups of gs samples (N in all), at
  // most kHeadGroup pixels each; patches of S x S on the output grid Ho x Wo, spatial stride `stride`, input grid H x W
  const int32_t* idx; const int32_t* count;
  int N, gs, S, stride, Ho, Wo, H, W;
  FastDiv d_hw, d_w, d_s;  // set by launch_head
  // rows = the pixels of listed samples (layer gate ahead of a spatially static first 1x1): slist [scap] ascending kept
  // sample ids, *scount of them valid (device), hw pixels per sample; m_rows = scap * hw is the capacity.  Null: all rows.
  // scap 0: a list that ends with its last valid entry (m_rows: N * hw).
  const int32_t* slist;
  const int32_t* scount;
  int scap;
  // channel skipping: rbits[n] = kept channel groups (bit g) of sample n, hw = pixels per sample, cs_group = channels per
  // group (a multiple of 32); h1 is written as zero in the groups a row's sample drops.  Null: no channel mask.
  const uint8_t* rbits;
  int hw, cs_group;
  int pb;                // tile height in blocks of 32 pixels (2 or 4); 0 = chosen by launch_head (dense rows) or on the device (lists)
  int wg_target;         // workgroups that fill the device once (its compute units; set by launch_head)
};
constexpr int kHeadGroup = 4096;
bool head_supported(int dtype, int c_in, int c_mid);
int head_init_device();
size_t head_packed_bytes(int c_in);
int launch_head_pack(const void* w1, int c_in, void* packed, hipStream_t stream);
int launch_head(const HeadArgs& a, hipStream_t stream);

// 3x3 -> last 1x1 -> residual add / projection shortcut of the 64-wide bf16 blocks in one kernel (laud_narrow.hip), for
// narrow_supported() shapes and row counts.
struct NarrowArgs {
  const void* h1;        // [input pixels][64]
  const void* w2; const void* w3;  // [64][3][3][64], [256][64]
  const float* s2; const float* t2; const float* s3; const float* t3;
  const void* res;       // residual [output pixels][256]; may alias out
  void* out;
  const int32_t* count;  // active patches (device) and their ascending ids; null with a shortcut (every output pixel)
  const int32_t* list;
  int m_rows;            // rows, or their upper bound where the count is on the device
  int H, W, S, stride, Ho, Wo, relu;
  // projection shortcut instead of a residual (static first block): x [input pixels][64] read at the 3x3's centre
  const void* x; const void* wsc; const float* ssc; const float* tsc;
  InactiveCopy cp;
  float inv_s, inv_ss, inv_wp, inv_pps, inv_howo, inv_wo;  // set by launch_narrow
};
bool narrow_supported(int dtype, int c_mid, int c_out, long long rows);
int narrow_init_device();
int launch_narrow(const NarrowArgs& a, hipStream_t stream);

// The static first block of ResNet stage 1 (64 -> 64 -> 256, no stride, bf16) in one kernel (laud_first.hip), for
// the shapes and maps that first_plan() takes.
struct FirstArgs {
  const void* x; void* out;        // [N][H][W][64], [N][H][W][256]
  const void* w1; const void* w2; const void* w3; const void* wsc;  // [64][64], [64][3][3][64], [256][64], [256][64]
  const float* s1; const float* t1; const float* s2; const float* t2; const float* s3; const float* t3;
  const float* ssc; const float* tsc;
  int N, H, W;
  int th, tw, ntx, pern, ntiles;   // rectangles of th x tw outputs, ntx a row of them, pern a sample (set by first_plan)
  FastDiv d_rw, d_tw, d_pern, d_ntx;  // set by launch_first
};
bool first_plan(int dtype, int c_in, int c_mid, int c_out, int stride, FirstArgs* a);  // N, H, W given
int first_init_device();
int launch_first(const FirstArgs& a, hipStream_t stream);

int stem_init_device(int* cus_out);

// Stage timing (see laud_stage_timing_enable): RAII bracket around the launches of one stage.
extern bool g_stage_timing_on;
void stage_mark(int stage, hipStream_t stream, bool begin);
struct StageScope {
  int stage;
  hipStream_t stream;
  StageScope(int s, hipStream_t st) : stage(s), stream(st) {
    if (g_stage_timing_on) stage_mark(stage, stream, true);
  }
  ~StageScope() {
    if (g_stage_timing_on) stage_mark(stage, stream, false);
  }
};

}  // namespace laud
