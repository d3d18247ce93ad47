// Squeeze-and-excitation module of the group-convolution / SE blocks (the RegNetY backbones of Sec. 4), applied
// to the compact rows h2 of the active patches between the 3x3 and the last 1x1 of a dynamic block.
#include "laud_common.h"
#include "laud_tile_util.h"

#include <type_traits>
#include <algorithm>

namespace laud {

// The sample's active patches are a contiguous range of the ascending index list, so its h2 rows are contiguous too, and
// the whole module of a sample -- channel means, the two fully connected layers, rows multiplied by the gate in place --
// can be the work of one workgroup in one launch: nothing of it needs another sample.  As four dependent launches it takes
// 20 to 28 us per block at 32 to 128 images, mostly launch and memory latency; samples that are too much for one
// compute unit take those (se_one_launch).  The squeeze averages over the sample's computed pixels; a sample without
// active patches has no rows.  All sums have a fixed order.
constexpr int kSeThreads = 1024, kSeChunks = 128, kSeLanes = 16;

// dst[o] = f(w[o] . v + b[o]), o < n, for vectors of length len in LDS: sixteen lanes per output, 64 outputs at a time.  A
// thread's share of the weights is a sequence of items (pass over the outputs, 16-byte step along the row); the first kSePre
// of them are loaded before anything else the kernel does (they depend on nothing), the rest four at a time.  Loads return in
// order, so that the list and the rows wait for them: a pass or a step that there is not is not loaded, nor a lane past the last one.
// The biases are in LDS: from memory every pass waited for its own.
// (Positions are counted up instead of divided out: sixteen waves share four SIMDs, and a division per item and wave cost more
// than the loads.)
constexpr int kSePre = 8, kSeOutputs = kSeThreads / kSeLanes;
struct SeItems {
  int l, o0, n, q4, ks, passes;
  __amdgpu_buffer_rsrc_t w;
  int p, k;  // position of the next load
  __device__ __forceinline__ SeItems(const float* wt, int n_, int len)
      : l((int)threadIdx.x & (kSeLanes - 1)), o0((int)threadIdx.x / kSeLanes), n(n_), q4(len / 4), ks((len / 4 + kSeLanes - 1) / kSeLanes),
        passes((n_ + kSeOutputs - 1) / kSeOutputs),
        w(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(wt), 0, n_ * len * 4, 0x00020000)), p(0), k(0) {}
  __device__ __forceinline__ u32x4 next() {
    u32x4 r = {0, 0, 0, 0};
    if (p < passes) {
      const int o = p * kSeOutputs + o0, c = k * kSeLanes + l;
      r = __builtin_amdgcn_raw_buffer_load_b128(w, o < n && c < q4 ? (unsigned)(o * q4 + c) * 16u : 0x80000000u, 0, 0);
      if (++k == ks) { k = 0; ++p; }
    }
    return r;
  }
};
// Sum over a row of sixteen lanes, the lanes 8, 4, 2 and 1 apart (rotations: what they add has that period).
template <int N>
__device__ __forceinline__ float add_rotated(float v) {
  return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x120 + N, 0xf, 0xf, true));
}
// Four items with weights r; steps (p, k) on.
template <bool SIGMOID>
__device__ __forceinline__ void se_items(const SeItems& it, int& p, int& k, const u32x4* r, const float* v, const float* b, float& acc, float* dst) {
  float4 x[4];
  float bias[4];
  int pp = p, kk = k;
#pragma unroll
  for (int u = 0; u < 4; ++u) {  // (what lies in LDS is under way together)
    x[u] = reinterpret_cast<const float4*>(v)[min(kk * kSeLanes + it.l, it.q4 - 1)];
    bias[u] = b[min(pp * kSeOutputs + it.o0, it.n - 1)];
    if (++kk == it.ks) { kk = 0; ++pp; }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (p >= it.passes) return;
    if (k * kSeLanes + it.l < it.q4)
      acc += __uint_as_float(r[u].x) * x[u].x + __uint_as_float(r[u].y) * x[u].y + __uint_as_float(r[u].z) * x[u].z + __uint_as_float(r[u].w) * x[u].w;
    if (++k == it.ks) {  // the output is complete
      acc = add_rotated<1>(add_rotated<2>(add_rotated<4>(add_rotated<8>(acc))));
      const int o = p * kSeOutputs + it.o0;
      if (it.l == 0 && o < it.n) {
        const float s = acc + bias[u];
        dst[o] = SIGMOID ? 1.f / (1.f + __expf(-s)) : fmaxf(s, 0.f);
      }
      acc = 0.f;
      k = 0;
      ++p;
    }
  }
}
template <bool SIGMOID>
__device__ __forceinline__ void se_layer(SeItems& it, const u32x4 (&pre)[kSePre], const float* v, const float* b, float* dst) {
  float acc = 0.f;
  int p = 0, k = 0;
#pragma unroll
  for (int t = 0; t < kSePre; t += 4) se_items<SIGMOID>(it, p, k, pre + t, v, b, acc, dst);
  while (p < it.passes) {
    u32x4 r[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) r[u] = it.next();
    se_items<SIGMOID>(it, p, k, r, v, b, acc, dst);
  }
}
// rows of w whose length is no multiple of four (not 16-byte aligned)
template <bool SIGMOID>
__device__ __forceinline__ void se_layer_any(const float* __restrict__ w, const float* v, int n, int len,
                                             const float* b, float* dst) {
  const int l = threadIdx.x % kSeLanes, o0 = threadIdx.x / kSeLanes;
  for (int o1 = 0; o1 < n; o1 += kSeThreads / kSeLanes) {
    const int o = min(o1 + o0, n - 1);
    float acc = 0.f;
    for (int k = l; k < len; k += kSeLanes) acc += w[(size_t)o * len + k] * v[k];
#pragma unroll
    for (int d = kSeLanes / 2; d > 0; d >>= 1) acc += __shfl_xor(acc, d, kWave);
    if (l == 0 && o1 + o0 < n) {
      const float s = acc + b[o];
      dst[o] = SIGMOID ? 1.f / (1.f + __expf(-s)) : fmaxf(s, 0.f);
    }
  }
}

template <typename ET>
__device__ __forceinline__ uint4 se_scaled(const uint4& v, const float (&g)[elem<ET>::per16]) {
  if constexpr (sizeof(ET) == 4) {
    return make_uint4(__float_as_uint(__uint_as_float(v.x) * g[0]), __float_as_uint(__uint_as_float(v.y) * g[1]),
                      __float_as_uint(__uint_as_float(v.z) * g[2]), __float_as_uint(__uint_as_float(v.w) * g[3]));
  } else {
    auto two = [&](unsigned u, int i) __attribute__((always_inline)) {
      return pack_bf16(__uint_as_float(u << 16) * g[i], __uint_as_float(u & 0xffff0000u) * g[i + 1]);
    };
    return make_uint4(two(v.x, 0), two(v.y, 2), two(v.z, 4), two(v.w, 6));
  }
}
template <typename ET>
__device__ __forceinline__ void se_add(float (&acc)[elem<ET>::per16], const uint4& v) {
  const unsigned u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (sizeof(ET) == 4) {
      acc[i] += __uint_as_float(u[i]);
    } else {
      acc[2 * i] += __uint_as_float(u[i] << 16);
      acc[2 * i + 1] += __uint_as_float(u[i] & 0xffff0000u);
    }
  }
}

// Means over a sample's rows for the block of up to kSeChunks 16-byte channel chunks that starts at chunk cb: the threads are
// (chunk lane, row phase), every thread keeps eight row loads in flight, and the row phases are added in a fixed order.
template <typename ET>
__device__ __forceinline__ void se_means(const uint4* base, int rows, int cpr, int cb, float inv, float* s_part, float* dst) {
  constexpr int EPC = elem<ET>::per16;
  const int tid = threadIdx.x, nch = min(kSeChunks, cpr - cb);
  // chunk lanes: a power of two that divides the thread count
  const int cs = 32 - __builtin_clz(max(nch - 1, 1)), CP = 1 << cs, RP = kSeThreads >> cs, cl = tid & (CP - 1), rp = tid >> cs;
  float acc[EPC];
#pragma unroll
  for (int e = 0; e < EPC; ++e) acc[e] = 0.f;
  if (cl < nch) {
    const uint4* col = base + cb + cl;
    int r = rp;
    for (; r + 7 * RP < rows; r += 8 * RP) {
      uint4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = col[(size_t)(r + u * RP) * cpr];
#pragma unroll
      for (int u = 0; u < 8; ++u) se_add<ET>(acc, v[u]);
    }
    for (; r < rows; r += RP) {
      const uint4 v = col[(size_t)r * cpr];
      se_add<ET>(acc, v);
    }
  }
#pragma unroll
  for (int e = 0; e < EPC; ++e) s_part[(rp * CP + cl) * EPC + e] = acc[e];
  __syncthreads();
  // the row phases are halved until they are few enough for one thread per value: the same pairs every time
  int left = RP;
  for (; left * nch * EPC > 2 * kSeThreads && left > 1;) {
    left >>= 1;
    for (int k = tid; k < left * CP * EPC; k += kSeThreads) s_part[k] += s_part[left * CP * EPC + k];
    __syncthreads();
  }
  for (int k = tid; k < nch * EPC; k += kSeThreads) {
    float t = 0.f;
    for (int q = 0; q < left; ++q) t += s_part[q * CP * EPC + k];
    dst[cb * EPC + k] = t * inv;
  }
}

// One workgroup per sample.  A chain of dependent memory trips is most of its time, so there are as few as can be: the count; the
// whole index list (kWave to kSeList entries: every workgroup counts the entries of the samples ahead of its own, which a search
// takes three or four trips for); the rows, which stay in registers until they are rescaled.  (Samples of more rows are read twice.)
// Blocks of RegNetY-800MF stage 3 at ratio 0.5 (every sample's rows kept): 25.5 -> 22.9 us for one sample, 56.5 -> 54.1 us for 128; a
// block of more rows (stage 1, 128 samples) as before.  Lists of more than 8192 entries are searched: two trips of loads gained nothing.
constexpr int kSeKeep = 8, kSeList = 8 * kSeThreads;
template <typename ET>
__global__ __launch_bounds__(kSeThreads) void k_se(ET* __restrict__ h2, const int32_t* __restrict__ idx,
                                                   const int32_t* __restrict__ count, int pps, int SS, int C, int se_w,
                                                   const float* __restrict__ w1, const float* __restrict__ b1,
                                                   const float* __restrict__ w2, const float* __restrict__ b2) {
  constexpr int EPC = elem<ET>::per16, NW = kSeThreads / kWave;
  __shared__ __align__(16) float s_part[kSeThreads * EPC];  // [row phase][chunk lane][EPC]
  __shared__ __align__(16) float s_z[kSeMaxC];              // means, then gates
  __shared__ __align__(16) float s_h[kSeMaxHidden];
  __shared__ float s_sums[kSeThreads];
  __shared__ float s_b1[kSeMaxHidden], s_b2[kSeMaxC];
  __shared__ int s_below[2][NW];
  const int n = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  SeItems it1(w1, se_w, C), it2(w2, C, se_w);
  const float bias1 = tid < se_w ? b1[tid] : 0.f, bias2 = tid < C ? b2[tid] : 0.f;
  u32x4 pre1[kSePre], pre2[kSePre];
  const bool vec2 = (se_w & 3) == 0;  // (C is a multiple of eight)
#pragma unroll
  for (int t = 0; t < kSePre; ++t) {
    pre1[t] = it1.next();
    if (vec2) pre2[t] = it2.next();
  }
  const int cnt = *count;
  int lo, hi;
  if (cnt > kWave && cnt <= kSeList) {
    int below[2] = {0, 0};  // entries ahead of this sample's first, and of the next sample's
    const auto below_in = [&](auto U) {  // U entries per thread, all requested before the first is used
      int e[decltype(U)::value];
#pragma unroll
      for (int u = 0; u < decltype(U)::value; ++u) e[u] = idx[min(tid + u * kSeThreads, cnt - 1)];
#pragma unroll
      for (int u = 0; u < decltype(U)::value; ++u) {
        const bool in = tid + u * kSeThreads < cnt;
        below[0] += __popcll(__ballot(in && e[u] < n * pps));
        below[1] += __popcll(__ballot(in && e[u] < (n + 1) * pps));
      }
    };
    if (cnt <= kSeThreads) below_in(std::integral_constant<int, 1>{});
    else below_in(std::integral_constant<int, kSeList / kSeThreads>{});
    if (lane == 0) { s_below[0][wave] = below[0]; s_below[1][wave] = below[1]; }
    __syncthreads();
    lo = hi = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) { lo += s_below[0][w]; hi += s_below[1][w]; }
  } else {
    wave_lower_bound2(idx, cnt, n * pps, (n + 1) * pps, lo, hi);
  }
  const int rows = (hi - lo) * SS;
  if (rows == 0) return;
  s_b1[tid] = bias1;  // (read behind the means' barriers)
  s_b2[tid] = bias2;
  for (int i = tid + kSeThreads; i < C; i += kSeThreads) s_b2[i] = b2[i];
  const int cpr = C / EPC;  // 16-byte chunks per row
  uint4* const base = reinterpret_cast<uint4*>(h2 + (long long)lo * SS * C);
  const float inv = 1.f / (float)rows;
  // a thread's chunk column and first row, as many rows at a time as the threads make
  const float inv_cpr = 1.f / (float)cpr;
  const int RP = fdiv(kSeThreads, inv_cpr), rp = fdiv(tid, inv_cpr), cl = tid - rp * cpr;
  const bool keep = C <= kSeThreads && rows <= kSeKeep * RP;
  uint4 v[kSeKeep];
  if (keep) {
    uint4* const col = base + (size_t)rp * cpr + cl;
    const bool on = rp < RP;
#pragma unroll
    for (int u = 0; u < kSeKeep; ++u) {
      v[u] = make_uint4(0, 0, 0, 0);
      if (on && rp + u * RP < rows) v[u] = col[(size_t)u * RP * cpr];
    }
    float acc[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[e] = 0.f;
#pragma unroll
    for (int u = 0; u < kSeKeep; ++u) se_add<ET>(acc, v[u]);
    if (on) {
#pragma unroll
      for (int e = 0; e < EPC; ++e) s_part[rp * C + cl * EPC + e] = acc[e];
    }
    __syncthreads();
    // the row phases of a channel are added by G threads, then these
    const float inv_c = 1.f / (float)C;
    const int G = fdiv(kSeThreads, inv_c), g = fdiv(tid, inv_c), c = tid - g * C;
    if (g < G) {
      float t = 0.f;
#pragma unroll 4
      for (int q = g; q < RP; q += G) t += s_part[q * C + c];
      if (G > 1) s_sums[g * C + c] = t;
      else s_z[c] = t * inv;
    }
    if (G > 1) __syncthreads();
    if (G > 1 && tid < C) {
      float t = 0.f;
      for (int q = 0; q < G; ++q) t += s_sums[q * C + tid];
      s_z[tid] = t * inv;
    }
    __syncthreads();
  } else {
    for (int cb = 0; cb < cpr; cb += kSeChunks) {
      se_means<ET>(base, rows, cpr, cb, inv, s_part, s_z);
      __syncthreads();
    }
  }
  se_layer<false>(it1, pre1, s_z, s_b1, s_h);
  __syncthreads();
  if (vec2) se_layer<true>(it2, pre2, s_h, s_b2, s_z);
  else se_layer_any<true>(w2, s_h, C, se_w, s_b2, s_z);
  __syncthreads();
  // h2[row][:] *= gate, rounded to the storage type
  if (keep) {
    if (rp >= RP) return;
    float g[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) g[e] = s_z[cl * EPC + e];
    uint4* const col = base + (size_t)rp * cpr + cl;
#pragma unroll
    for (int u = 0; u < kSeKeep; ++u)
      if (rp + u * RP < rows) col[(size_t)u * RP * cpr] = se_scaled<ET>(v[u], g);
    return;
  }
  for (int cb = 0; cb < cpr; cb += kSeChunks) {
    const int nch = min(kSeChunks, cpr - cb);
    const int cs = 32 - __builtin_clz(max(nch - 1, 1)), CP = 1 << cs, RP2 = kSeThreads >> cs, cl2 = tid & (CP - 1), rp2 = tid >> cs;
    if (cl2 >= nch) continue;
    float g[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) g[e] = s_z[(cb + cl2) * EPC + e];
    uint4* col = base + cb + cl2;
    int r = rp2;
    for (; r + 3 * RP2 < rows; r += 4 * RP2) {
      uint4 x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = col[(size_t)(r + u * RP2) * cpr];
#pragma unroll
      for (int u = 0; u < 4; ++u) col[(size_t)(r + u * RP2) * cpr] = se_scaled<ET>(x[u], g);
    }
    for (; r < rows; r += RP2) col[(size_t)r * cpr] = se_scaled<ET>(col[(size_t)r * cpr], g);
  }
}

// ---- the same in four launches: means with one workgroup per sample and block of channels, the two layers batched over samples
// and tiled over outputs, the rescaling over all rows -------------------------------------------------------------------
// grid (ceil(chunks per row / kSeChunks), N): z[n][c] = mean over the sample's rows (zeros for a sample without rows)
template <typename ET>
__global__ __launch_bounds__(kSeThreads) void k_se_squeeze(const ET* __restrict__ h2, const int32_t* __restrict__ idx,
                                                           const int32_t* __restrict__ count, int pps, int SS, int C,
                                                           float* __restrict__ z) {
  constexpr int EPC = elem<ET>::per16;
  __shared__ __align__(16) float s_part[kSeThreads * EPC];
  const int n = blockIdx.y, cnt = *count;
  int lo, hi;
  wave_lower_bound2(idx, cnt, n * pps, (n + 1) * pps, lo, hi);
  const int rows = (hi - lo) * SS;
  se_means<ET>(reinterpret_cast<const uint4*>(h2 + (long long)lo * SS * C), rows, C / EPC, (int)blockIdx.x * kSeChunks,
               rows > 0 ? 1.f / (float)rows : 0.f, s_part, z + (size_t)n * C);
}

// The two small fully connected layers, batched over groups of kFcSamples samples so that a weight row read
// from L2 serves the whole group, and tiled over the outputs so that the grid fills the chip:
//   k_se_fc1: hid[n][k] = relu(w1[k] . z[n] + b1[k])
//   k_se_fc2: gate[n][c] = sigmoid(w2[c] . hid[n] + b2[c])
// One wave per four outputs at a time, lanes stride over the reduction with 16-byte loads, all loads of a
// step issued before their use.
constexpr int kFcSamples = 8, kFcThreads = 256, kFc1Tile = 16, kFc2Tile = 32;

// Sums 32 per-lane values over the 64 lanes of a wave with 32 shuffles instead of 32 x 6: each step exchanges
// one half of the remaining values with the partner lane and keeps the other half, so the number of values
// halves while the number of lanes summed doubles.  Returns, in lane l, the total of value
// 16*b5 + 8*b4 + 4*b3 + 2*b2 + b1 (b_i = bit i of l); lanes l and l^1 hold the same value.
template <int HALF>
__device__ __forceinline__ void wave_reduce_step(float (&v)[32], int lane) {  // xor distance 2*HALF
  const bool upper = (lane & (2 * HALF)) != 0;
#pragma unroll
  for (int i = 0; i < HALF; ++i) {
    const float keep = upper ? v[i + HALF] : v[i], send = upper ? v[i] : v[i + HALF];
    v[i] = keep + __shfl_xor(send, 2 * HALF, kWave);
  }
}
__device__ __forceinline__ float wave_reduce_32(float (&v)[32]) {
  const int lane = lane_id();
  wave_reduce_step<16>(v, lane);
  wave_reduce_step<8>(v, lane);
  wave_reduce_step<4>(v, lane);
  wave_reduce_step<2>(v, lane);
  wave_reduce_step<1>(v, lane);
  return v[0] + __shfl_xor(v[0], 1, kWave);
}

__global__ __launch_bounds__(kFcThreads) void k_se_fc1(const float* __restrict__ z, int N, int C, int se_w,
                                                       const float* __restrict__ w1, const float* __restrict__ b1,
                                                       float* __restrict__ hid) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n0 = blockIdx.y * kFcSamples, k0 = blockIdx.x * kFc1Tile + wave * 4;
  if (k0 >= se_w) return;  // whole wave; the kernel has no barrier
  float acc[4 * kFcSamples];  // [output u][sample g]
#pragma unroll
  for (int i = 0; i < 4 * kFcSamples; ++i) acc[i] = 0.f;
  const int c4n = C / 4;
  for (int c4 = lane; c4 < c4n; c4 += kWave) {
    float4 w[4], zz[kFcSamples];
#pragma unroll
    for (int u = 0; u < 4; ++u) w[u] = reinterpret_cast<const float4*>(w1 + (size_t)min(k0 + u, se_w - 1) * C)[c4];
#pragma unroll
    for (int g = 0; g < kFcSamples; ++g) zz[g] = reinterpret_cast<const float4*>(z + (size_t)min(n0 + g, N - 1) * C)[c4];
#pragma unroll
    for (int g = 0; g < kFcSamples; ++g)
#pragma unroll
      for (int u = 0; u < 4; ++u)
        acc[u * kFcSamples + g] += w[u].x * zz[g].x + w[u].y * zz[g].y + w[u].z * zz[g].z + w[u].w * zz[g].w;
  }
  // even lane l ends up with the sum of (output u, sample g), 8u + g = l / 2: the 32 results leave in one
  // store, and the bias loads of the lanes run side by side instead of one after the other
  const float mine = wave_reduce_32(acc);
  if ((lane & 1) == 0) {
    const int n = n0 + (lane >> 1) % kFcSamples, k = k0 + (lane >> 1) / kFcSamples;
    if (n < N && k < se_w) hid[(size_t)n * se_w + k] = fmaxf(mine + b1[k], 0.f);
  }
}

__global__ __launch_bounds__(kFcThreads) void k_se_fc2(const float* __restrict__ hid, int N, int C, int se_w,
                                                       const float* __restrict__ w2, const float* __restrict__ b2,
                                                       float* __restrict__ gate) {
  __shared__ __align__(16) float s_h[kFcSamples][kSeMaxHidden];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n0 = blockIdx.y * kFcSamples;
  for (int i = tid; i < kFcSamples * se_w; i += kFcThreads) {
    const int g = i / se_w, k = i - g * se_w;
    s_h[g][k] = hid[(size_t)min(n0 + g, N - 1) * se_w + k];
  }
  __syncthreads();
  const bool vec = (se_w % 4) == 0;  // every row of w2 16-byte aligned
  for (int pass = 0; pass < 2; ++pass) {
    const int c0 = blockIdx.x * kFc2Tile + wave * 8 + pass * 4;
    if (c0 >= C) break;
    float acc[4 * kFcSamples];  // [output u][sample g]
#pragma unroll
    for (int i = 0; i < 4 * kFcSamples; ++i) acc[i] = 0.f;
    if (vec) {
      for (int k4 = lane; k4 < se_w / 4; k4 += kWave) {
        float4 w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = reinterpret_cast<const float4*>(w2 + (size_t)min(c0 + u, C - 1) * se_w)[k4];
#pragma unroll
        for (int g = 0; g < kFcSamples; ++g) {
          const float4 h = reinterpret_cast<const float4*>(s_h[g])[k4];
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[u * kFcSamples + g] += w[u].x * h.x + w[u].y * h.y + w[u].z * h.z + w[u].w * h.w;
        }
      }
    } else {
      for (int k = lane; k < se_w; k += kWave) {
        float w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = w2[(size_t)min(c0 + u, C - 1) * se_w + k];
#pragma unroll
        for (int g = 0; g < kFcSamples; ++g) {
          const float h = s_h[g][k];
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[u * kFcSamples + g] += w[u] * h;
        }
      }
    }
    const float mine = wave_reduce_32(acc);  // even lane l: (output u, sample g), 8u + g = l / 2
    if ((lane & 1) == 0) {
      const int n = n0 + (lane >> 1) % kFcSamples, c = c0 + (lane >> 1) / kFcSamples;
      if (n < N && c < C) gate[(size_t)n * C + c] = 1.f / (1.f + __expf(-(mine + b2[c])));
    }
  }
}

// h2[row][:] *= gate[sample of the row][:], rounded to the storage type; grid-stride over 16-byte chunks.
template <typename ET>
__global__ __launch_bounds__(256) void k_se_scale(ET* __restrict__ h2, const int32_t* __restrict__ idx,
                                                  const int32_t* __restrict__ count, int pps, int SS, int C,
                                                  const float* __restrict__ gate) {
  constexpr int EPC = elem<ET>::per16;
  const int cpr = C / EPC;
  const long long total = (long long)*count * SS * cpr;
  uint4* base = reinterpret_cast<uint4*>(h2);
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long long)gridDim.x * 256) {
    const int row = (int)(i / cpr), c = (int)(i - (long long)row * cpr);
    const int n = idx[row / SS] / pps;
    uint4 v = base[i];
    const float4* g4 = reinterpret_cast<const float4*>(gate + (size_t)n * C + c * EPC);
    float g[EPC];
#pragma unroll
    for (int u = 0; u < EPC / 4; ++u) {
      const float4 q = g4[u];
      g[4 * u] = q.x; g[4 * u + 1] = q.y; g[4 * u + 2] = q.z; g[4 * u + 3] = q.w;
    }
    ET t[EPC];
    __builtin_memcpy(t, &v, 16);
#pragma unroll
    for (int e = 0; e < EPC; ++e) elem<ET>::store(&t[e], elem<ET>::load(&t[e]) * g[e]);
    __builtin_memcpy(&v, t, 16);
    base[i] = v;
  }
}

// One launch where a sample is little work for the one compute unit it then has: its rows, which pass three times, and the
// weights of the layers, which every sample reads.  Both ways measured over 48 to 2048 channels, 4 x 4 to 224 x 224 pixels, 1 to
// 256 samples and ratios 0.15 to 0.95 (bf16): with rows of up to 400 KB (800 KB from 16 samples on: the four launches then
// take longer as well) and weights of up to 256 KB one launch saves 1 to 16 us everywhere; at one sample and ratio 0.95 it
// costs 3 us at 450 KB of rows, 15 us at 1.2 MB and 40 us at 2.4 MB, and with 1.2 MB of weights (784 channels) 2 to 15 us at
// any number of rows up to 300 KB.
static bool se_one_launch(int dtype, int N, long long rows, int C, int se_w) {
  return rows * C * (long long)elem_bytes(dtype) <= (N < 16 ? 400 : 800) * 1024 && 2LL * C * se_w * 4 <= 256 * 1024;
}

// The SE module on the compact rows h2 of the active patches (pps patches per sample, SS pixels per patch, at most cap_rows
// rows).  `scratch` (float32: means [N][C], gates [N][C], hidden units [N][se_w]) must not be in use: the callers pass the h1
// region, which is dead once the 3x3 has run.
int launch_se(int dtype, int N, int pps, int SS, int C, const laud_group_se* e, void* h2, const int32_t* idx,
              const int32_t* count, float* scratch, long long cap_rows, hipStream_t st) {
  StageScope scope(LAUD_STAGE_SE, st);
  const int sw = e->se_width;
  if (se_one_launch(dtype, N, (long long)pps * SS, C, sw)) {
    if (dtype == LAUD_BF16)
      hipLaunchKernelGGL(k_se<bf16_t>, dim3(N), dim3(kSeThreads), 0, st, (bf16_t*)h2, idx, count, pps, SS, C, sw, e->w_se1,
                         e->b_se1, e->w_se2, e->b_se2);
    else
      hipLaunchKernelGGL(k_se<float>, dim3(N), dim3(kSeThreads), 0, st, (float*)h2, idx, count, pps, SS, C, sw, e->w_se1,
                         e->b_se1, e->w_se2, e->b_se2);
    return check_launch();
  }
  float* z = scratch;
  float* gate = z + (size_t)N * C;
  float* hid = gate + (size_t)N * C;
  const int cpr = (int)(C * elem_bytes(dtype) / 16);
  const dim3 sq((unsigned)((cpr + kSeChunks - 1) / kSeChunks), (unsigned)N);
  const unsigned ngrp = (unsigned)((N + kFcSamples - 1) / kFcSamples);
  const dim3 g1((unsigned)((sw + kFc1Tile - 1) / kFc1Tile), ngrp), g2((unsigned)((C + kFc2Tile - 1) / kFc2Tile), ngrp);
  const unsigned sblocks = (unsigned)std::min<long long>((cap_rows * cpr + 1023) / 1024, 8192);
  if (dtype == LAUD_BF16)
    hipLaunchKernelGGL(k_se_squeeze<bf16_t>, sq, dim3(kSeThreads), 0, st, (const bf16_t*)h2, idx, count, pps, SS, C, z);
  else
    hipLaunchKernelGGL(k_se_squeeze<float>, sq, dim3(kSeThreads), 0, st, (const float*)h2, idx, count, pps, SS, C, z);
  hipLaunchKernelGGL(k_se_fc1, g1, dim3(kFcThreads), 0, st, z, N, C, sw, e->w_se1, e->b_se1, hid);
  hipLaunchKernelGGL(k_se_fc2, g2, dim3(kFcThreads), 0, st, hid, N, C, sw, e->w_se2, e->b_se2, gate);
  if (dtype == LAUD_BF16)
    hipLaunchKernelGGL(k_se_scale<bf16_t>, dim3(sblocks), dim3(256), 0, st, (bf16_t*)h2, idx, count, pps, SS, C, gate);
  else
    hipLaunchKernelGGL(k_se_scale<float>, dim3(sblocks), dim3(256), 0, st, (float*)h2, idx, count, pps, SS, C, gate);
  return check_launch();
}

}  // namespace laud
