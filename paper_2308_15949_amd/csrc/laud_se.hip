// Squeeze-and-excitation module of the group-convolution / SE blocks (the RegNetY backbones of Sec. 4), applied
// to the compact rows h2 of the active patches between the 3x3 and the last 1x1 of a dynamic block.
#include "laud_common.h"
#include "laud_tile_util.h"

namespace laud {

// The sample's active patches are a contiguous range of the ascending index list, so its h2 rows are contiguous too, and
// the whole module of a sample -- channel means, the two fully connected layers, rows multiplied by the gate in place --
// is the work of one workgroup in one launch: nothing of it needs another sample.  (As four dependent launches it took
// 20 to 28 us per block at 32 to 128 images, mostly launch and memory latency; the weights are read once per sample from
// L2, at most 1.2 MB for the widest backbone.)  The squeeze averages over the sample's computed pixels; a sample without
// active patches has no rows.  All sums have a fixed order.
constexpr int kSeThreads = 1024, kSeChunks = 128, kSeLanes = 16;

// dst[o] = f(w[o] . v + b[o]), o < n, for vectors of length len in LDS: sixteen lanes per output, 64 outputs at a time.  A
// thread's share of the weights is a sequence of items (pass over the outputs, 16-byte step along the row); the first kSePre
// of them are loaded before anything else the kernel does (they depend on nothing), the rest four at a time.
// (Positions are counted up instead of divided out: sixteen waves share four SIMDs, and a division per item and wave cost more
// than the loads.)
constexpr int kSePre = 8, kSeOutputs = kSeThreads / kSeLanes;
struct SeItems {
  int l, o0, n, q4, ks, passes;
  const float4* w;
  int p, k;  // position of the next load
  __device__ __forceinline__ SeItems(const float* wt, int n_, int len)
      : l((int)threadIdx.x & (kSeLanes - 1)), o0((int)threadIdx.x / kSeLanes), n(n_), q4(len / 4), ks((len / 4 + kSeLanes - 1) / kSeLanes),
        passes((n_ + kSeOutputs - 1) / kSeOutputs), w(reinterpret_cast<const float4*>(wt)), p(0), k(0) {}
  __device__ __forceinline__ float4 next() {  // items past the end re-read a valid row; never used
    const float4 r = w[(size_t)min(p * kSeOutputs + o0, n - 1) * q4 + min(k * kSeLanes + l, q4 - 1)];
    if (++k == ks) { k = 0; ++p; }
    return r;
  }
};
// Item (p, k) with weights r; steps (p, k) on.
template <bool SIGMOID>
__device__ __forceinline__ void se_item(const SeItems& it, int& p, int& k, const float4& r, const float* v,
                                        const float* __restrict__ b, float& acc, float* dst) {
  const int c = k * kSeLanes + it.l;
  if (c < it.q4) {
    const float4 x = reinterpret_cast<const float4*>(v)[c];
    acc += r.x * x.x + r.y * x.y + r.z * x.z + r.w * x.w;
  }
  if (++k == it.ks) {  // the output is complete
#pragma unroll
    for (int d = kSeLanes / 2; d > 0; d >>= 1) acc += __shfl_xor(acc, d, kWave);
    const int o = p * kSeOutputs + it.o0;
    if (it.l == 0 && o < it.n) {
      const float s = acc + b[o];
      dst[o] = SIGMOID ? 1.f / (1.f + __expf(-s)) : fmaxf(s, 0.f);
    }
    acc = 0.f;
    k = 0;
    ++p;
  }
}
template <bool SIGMOID>
__device__ __forceinline__ void se_layer(SeItems& it, const float4 (&pre)[kSePre], const float* v, const float* __restrict__ b,
                                         float* dst) {
  float acc = 0.f;
  int p = 0, k = 0;
#pragma unroll
  for (int t = 0; t < kSePre; ++t)
    if (p < it.passes) se_item<SIGMOID>(it, p, k, pre[t], v, b, acc, dst);
  while (p < it.passes) {
    float4 r[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) r[u] = it.next();
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (p < it.passes) se_item<SIGMOID>(it, p, k, r[u], v, b, acc, dst);
  }
}
// rows of w whose length is no multiple of four (not 16-byte aligned)
template <bool SIGMOID>
__device__ __forceinline__ void se_layer_any(const float* __restrict__ w, const float* v, int n, int len,
                                             const float* __restrict__ b, float* dst) {
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

// One workgroup per sample.  For the means and the rescaling the threads are (chunk lane, row phase) over blocks of up to
// 128 16-byte channel chunks; every thread keeps eight row loads in flight; the row phases are added in a fixed order.
template <typename ET>
__global__ __launch_bounds__(kSeThreads) void k_se(ET* __restrict__ h2, const int32_t* __restrict__ idx,
                                                   const int32_t* __restrict__ count, int pps, int SS, int C, int se_w,
                                                   const float* __restrict__ w1, const float* __restrict__ b1,
                                                   const float* __restrict__ w2, const float* __restrict__ b2) {
  constexpr int EPC = elem<ET>::per16;
  __shared__ __align__(16) float s_part[kSeThreads * EPC];  // [row phase][chunk lane][EPC]
  __shared__ __align__(16) float s_z[kSeMaxC];              // means, then gates
  __shared__ __align__(16) float s_h[kSeMaxHidden];
  const int n = blockIdx.x, tid = threadIdx.x;
  SeItems it1(w1, se_w, C), it2(w2, C, se_w);
  float4 pre1[kSePre], pre2[kSePre];
  const bool vec2 = (se_w & 3) == 0;  // (C is a multiple of eight)
#pragma unroll
  for (int t = 0; t < kSePre; ++t) {
    pre1[t] = it1.next();
    if (vec2) pre2[t] = it2.next();
  }
  const int cnt = *count;
  int lo, hi;
  wave_lower_bound2(idx, cnt, n * pps, (n + 1) * pps, lo, hi);
  const int rows = (hi - lo) * SS;
  if (rows == 0) return;
  const int cpr = C / EPC;  // 16-byte chunks per row
  uint4* const base = reinterpret_cast<uint4*>(h2 + (long long)lo * SS * C);
  const float inv = 1.f / (float)rows;
  for (int cb = 0; cb < cpr; cb += kSeChunks) {
    const int nch = min(kSeChunks, cpr - cb);
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
      s_z[cb * EPC + k] = t * inv;
    }
    __syncthreads();
  }
  se_layer<false>(it1, pre1, s_z, b1, s_h);
  __syncthreads();
  if (vec2) se_layer<true>(it2, pre2, s_h, b2, s_z);
  else se_layer_any<true>(w2, s_h, C, se_w, b2, s_z);
  __syncthreads();
  // h2[row][:] *= gate, rounded to the storage type
  for (int cb = 0; cb < cpr; cb += kSeChunks) {
    const int nch = min(kSeChunks, cpr - cb);
    const int cs = 32 - __builtin_clz(max(nch - 1, 1)), CP = 1 << cs, RP = kSeThreads >> cs, cl = tid & (CP - 1), rp = tid >> cs;
    if (cl >= nch) continue;
    float g[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) g[e] = s_z[(cb + cl) * EPC + e];
    uint4* col = base + cb + cl;
    int r = rp;
    for (; r + 3 * RP < rows; r += 4 * RP) {
      uint4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = col[(size_t)(r + u * RP) * cpr];
#pragma unroll
      for (int u = 0; u < 4; ++u) col[(size_t)(r + u * RP) * cpr] = se_scaled<ET>(v[u], g);
    }
    for (; r < rows; r += RP) col[(size_t)r * cpr] = se_scaled<ET>(col[(size_t)r * cpr], g);
  }
}

// The SE module on the compact rows h2 of the active patches (pps patches per sample, SS pixels per patch).
int launch_se(int dtype, int N, int pps, int SS, int C, const laud_group_se* e, void* h2, const int32_t* idx,
              const int32_t* count, hipStream_t st) {
  StageScope scope(LAUD_STAGE_SE, st);
  if (dtype == LAUD_BF16)
    hipLaunchKernelGGL(k_se<bf16_t>, dim3(N), dim3(kSeThreads), 0, st, (bf16_t*)h2, idx, count, pps, SS, C, e->se_width,
                       e->w_se1, e->b_se1, e->w_se2, e->b_se2);
  else
    hipLaunchKernelGGL(k_se<float>, dim3(N), dim3(kSeThreads), 0, st, (float*)h2, idx, count, pps, SS, C, e->se_width,
                       e->w_se1, e->b_se1, e->w_se2, e->b_se2);
  return check_launch();
}

}  // namespace laud
