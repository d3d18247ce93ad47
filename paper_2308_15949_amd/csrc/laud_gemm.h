// What the implicit-GEMM kernels of the three convolutions share (laud_gemm.hip, laud_pipe.h, laud_skinny.hip, laud_group.hip): modes,
// arguments, and for the modes without lists where a row of the activation operand comes from and a row of the result goes to.
#pragma once

#include "laud_common.h"

namespace laud {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) u32x4* gptr16;  // 16-byte chunk in global memory

enum { M_CONV1 = 0, M_CONV2 = 1, M_CONV3 = 2, M_CS1 = 3, M_CS2 = 4, M_CS3 = 5, M_DENSE1 = 6, M_U1 = 7, M_U2 = 8, M_U3 = 9,
       M_SD1 = 10, M_SD2 = 11, M_SD3 = 12, M_G2 = 13,
       M_CONV2P = 14 };  // CONV2 that decides the patches itself (PoolList; laud_skinny.hip only)

struct GemmArgs {
  const void* A;         // activations the rows are gathered from
  const void* Wt;        // weights [Ncols][ldw]
  const float* scale;    // per-output-channel affine
  const float* shift;
  void* Out;
  const void* Res;       // residual (CONV3 / CS3); may alias Out
  const int32_t* count;  // device: number of units (pixels for CONV1, patches for CONV2/3)
  const int32_t* list;   // device: pixel ids (CONV1) or active patch ids (CONV2/3)
  const uint8_t* cmask;  // CS: [N][D]
  int K;                 // reduction length per tap (full width)
  int ldw;               // weight row stride, elements
  int Ncols;             // output channels (full width)
  int H, W, S;
  int lda;               // A row stride, elements
  int ldo;               // Out/Res row stride, elements
  int relu;
  int D, G;              // CS: groups per sample, channels per group
  int row_tiles, col_tiles;
  int group_rows, tiles_per_group;  // CONV1: pixel lists are kept per group of samples
  int hw;                // CONV1: pixels of a sample where `list` holds samples, whose pixels are all rows; 0: pixel lists
  int m_rows;            // DENSE1, SD1..3: number of rows (all output pixels), known on the host
  int stride, Ho, Wo;    // SD1, SD2: spatial stride and output size (H, W are the input size)
  int gw;                // G2: channels per group of the 3x3
  // Workgroups past the tiles (CONV1 / DENSE1 launches only) copy the block's w2 / w3 into the fused tail kernel's
  // streaming order while the first 1x1 runs; pk_out == null: none.
  const void* pk_w2; const void* pk_w3; void* pk_out; int pk_chunks; int pk_first_block;
  const float* wmask;    // DENSE1: masker weights [K] or null
  float* proj;           // DENSE1: per-pixel masker projection sum_c w[c]*x[pixel][c], [m_rows]
  InactiveCopy cp;       // CONV3: copy of the inactive patches in extra workgroups (nblocks 0: none)
};

// The masker's decision of a map's patches from the per-pixel projection, made by every workgroup of the 3x3 that runs on them.
constexpr int kPoolListMax = 1024;
struct PoolList {
  const float* proj; const uint8_t* keep;  // [N*H*W]; [N] or null
  uint8_t* mask; float* logits;            // [n]; logits or null
  int32_t* sample_offsets;                 // [N + 1] or null
  float bias;
  int n;                                   // patches, up to kPoolListMax
};

// Few rows: small tiles, the reduction split over the waves of a workgroup (laud_skinny.hip).  cap_rows: number of rows, or
// its upper bound where the count is on the device.
bool skinny_wanted(int mode, int dtype, const GemmArgs& a, long long cap_rows);
int launch_skinny(int mode, int dtype, const GemmArgs& a, long long cap_rows, hipStream_t stream, const PoolList* pool = nullptr);
int skinny_init_device();
// Two dense 1x1s (M_SD1) on the same input and reduction length in one launch.
bool skinny_pair_wanted(int dtype, const GemmArgs& a, long long rows_a, const GemmArgs& b, long long rows_b);
int launch_skinny_pair(int dtype, const GemmArgs& a, long long rows_a, const GemmArgs& b, long long rows_b, hipStream_t stream);

// The group 3x3 in bf16, many rows, up to kGroupMaxC channels (laud_group.hip).
constexpr int kGroupMaxC = 4096;
int launch_group(const GemmArgs& a, long long cap_rows, hipStream_t stream);
int group_init_device();
// First 1x1 and group 3x3 in one launch (laud_group_fused.hip; `whole`: a patch is a whole sample): `a` as for the 3x3 on the listed patches, but A = x, K = c_in.
bool group_fused_wanted(int dtype, int c_in, int c_mid, int group_width, int S, int stride, bool whole, long long cap_rows);
int launch_group_fused(const GemmArgs& a, const void* w1, const float* s1, const float* t1, long long cap_rows, hipStream_t stream);
int group_fused_init_device();

// Many rows (laud_pipe.h); nsamples: samples of channel skipping, groups of CONV1's pixel lists.
int launch_pipe_a(int mode, int dtype, const GemmArgs& a, long long cap_rows, int nsamples, hipStream_t stream);
int launch_pipe_b(int mode, int dtype, const GemmArgs& a, long long cap_rows, int nsamples, hipStream_t stream);
int launch_pipe_c(int mode, int dtype, const GemmArgs& a, long long cap_rows, int nsamples, hipStream_t stream);
inline int launch_pipe(int mode, int dtype, const GemmArgs& a, long long cap_rows, int nsamples, hipStream_t stream) {
  if (mode == M_CONV1 || mode == M_DENSE1 || mode == M_SD1) return launch_pipe_a(mode, dtype, a, cap_rows, nsamples, stream);
  if (mode == M_CONV2 || mode == M_SD2 || mode == M_G2) return launch_pipe_b(mode, dtype, a, cap_rows, nsamples, stream);
  return launch_pipe_c(mode, dtype, a, cap_rows, nsamples, stream);
}

// ---- one 16-byte fragment pair -> MFMA ------------------------------------------------------
template <typename ET>
__device__ __forceinline__ void mma16(f32x16& acc, const uint4& a, const uint4& b) {
  if constexpr (sizeof(ET) == 2) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc,
                                                  0, 0, 0);
  } else {
    // Four k-steps of the 32x32x2 fp32 MFMA; lane group l/32 holds k-slots {4h..4h+3} of this
    // 8-wide K group for A and B alike, so the pairing of A and B elements is consistent.
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
  }
}

// Row of the activation operand that row `rho` of a launch starts from, for the modes whose rows follow from their number alone
// (the listed and strided ones are looked up in the kernels); the row-of-taps modes also need the centre (y, x) of the 3x3.
template <int MODE>
__device__ __forceinline__ size_t source_row(const GemmArgs& a, int rho, int sample, int& y, int& x) {
  static_assert((MODE >= M_CS1 && MODE <= M_U3) || MODE == M_SD3, "rows of this mode are looked up in its kernel");
  y = 0; x = 0;
  if constexpr (MODE == M_DENSE1 || MODE == M_U1 || MODE == M_U3 || MODE == M_SD3) {
    return (size_t)rho;
  } else if constexpr (MODE == M_U2) {
    // row = (patch p, pixel j of the patch); its centre inside the gathered (S+2) x (S+2) tile
    const int E = a.S + 2, SS = a.S * a.S;
    const int p = rho / SS, j = rho - p * SS;
    return (size_t)p * E * E + (size_t)(j / a.S + 1) * E + (j % a.S + 1);
  } else {  // CS1, CS2, CS3
    if constexpr (MODE == M_CS2) {
      y = rho / a.W;
      x = rho - y * a.W;
    }
    return (size_t)sample * (a.H * a.W) + rho;
  }
}

// Row of the output (and residual) buffer that row `rho` of the result belongs to, for the same modes; U1: -2 - row for a position
// outside the image (stored as zeros).
template <int MODE>
__device__ __forceinline__ int output_row(const GemmArgs& a, int rho, int sample, int Hp, int Wp) {
  static_assert((MODE >= M_CS1 && MODE <= M_U3) || MODE == M_SD3, "rows of this mode are looked up in its kernel");
  if constexpr (MODE == M_DENSE1 || MODE == M_U2 || MODE == M_U3 || MODE == M_SD3) {
    return rho;
  } else if constexpr (MODE == M_U1) {
    const int E = a.S + 2;
    const int p = rho / (E * E), e = rho - p * (E * E);
    const int q = a.list[p];
    const int r2 = q % (Hp * Wp);
    const int yy = (r2 / Wp) * a.S - 1 + e / E, xx = (r2 % Wp) * a.S - 1 + e % E;
    return (yy >= 0 && yy < a.H && xx >= 0 && xx < a.W) ? rho : -2 - rho;
  } else {
    return sample * a.H * a.W + rho;
  }
}

// first position of a sorted list whose value is not below `key`
__device__ __forceinline__ int lower_bound_dev(const int32_t* v, int n, int key) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (v[mid] < key) lo = mid + 1; else hi = mid;
  }
  return lo;
}

}  // namespace laud
