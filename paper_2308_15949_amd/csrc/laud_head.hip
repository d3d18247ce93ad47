// The first 1x1 of the block on EVERY pixel, with the one-channel spatial masker's per-pixel projection taken from the
// same reads of x (Sec. 3.4 "Operator fusion for spatial maskers"; App. B item 1), for gfx950: bf16, c_mid = 256,
// c_in a multiple of 256.  Same construction as the fused conv2 -> conv3 kernel (laud_tail.hip):
//
//   * one workgroup = 64 or 128 pixels x all 256 mid channels, 8 waves; wave w owns channels 32w .. 32w+31 and keeps
//     its weight fragments in registers, streamed from the packed copy of w1 (four K slices held / in flight);
//   * x reaches LDS with LDS-direct 16-byte loads into a four-stage ring of 128-byte K slices, swizzled on the
//     global side; one barrier per slice, in its middle; fragments are read one K step ahead of their MFMAs;
//   * the MFMAs compute the transposed tile, so a lane holds 4 x 4 consecutive channels of a pixel: h1 = relu(s1 * acc + t1)
//     goes through 4 KB of LDS a wave and leaves with four lanes on 64 bytes of a row;
//   * the masker projection sum_c w[c] * x[pixel][c] is formed on the vector ALU from the same LDS slices, every wave an equal share
//     of every slice, partial sums meet in LDS at the end.
//
// What bounds it (128 x 14 x 14 x 1024, 196 tiles of 128 rows): 16 slices of 1024 cycles of MFMAs, beside 768 of the vector-memory path, at 1.9 GHz.
// What is not a MFMA stands behind one each, in pieces that take no longer: the two waves of a SIMD issue in step, and what both do between
// their MFMAs the matrix pipe waits for.  In a row ahead of the MFMAs, with the projection of a K step on one wave and the rows' 16-byte stores
// 512 bytes apart, a slice took 1610 cycles, the stores 4200, the launch 21.8 us.  Now (stamps, one input over and over): 5518 cycles until the
// first rows are there, 16 x 1268, stores 2708, projection 1276: 15.6 us at 1.91 GHz, 0.6 between the workgroups, 2.6 of the launch around
// them.  With x cold in HBM a slice takes 1664 (3.3 TB/s) and the launch 24.7.
#include "laud_common.h"
#include "laud_tail_pack.h"
#include "laud_tile_util.h"

#include <atomic>

namespace laud {

namespace head {
constexpr int kMid = 256;
constexpr int kMaxPB = 4;                     // a workgroup takes PB = 2 or 4 blocks of 32 pixels
constexpr int kThreads = 512, kWaves = 8;
constexpr int kARing = 4;
constexpr int kWRing = 4;                     // weight slices in registers
constexpr unsigned kOob = 0x80000000u;
constexpr int kMaxK = 4096;
__host__ __device__ constexpr int a_stage(int pb) { return 32 * pb * 128; }  // one 128-byte K slice of every pixel row
// behind the activation ring: s1, t1 [256] floats, the tile's output rows [32*pb] (int), partial sums of the projection
// [8 / pb][32*pb], the waves' turning buffers (two pixel blocks of 32 rows x 64 bytes each), masker weights [K] floats
constexpr int kTurn = 2 * 32 * 64;
__host__ __device__ constexpr int tab_off(int pb) { return kARing * a_stage(pb); }
__host__ __device__ constexpr int orow_off(int pb) { return tab_off(pb) + 2 * kMid * 4; }
__host__ __device__ constexpr int part_off(int pb) { return orow_off(pb) + 32 * pb * 4; }
__host__ __device__ constexpr int turn_off(int pb) { return part_off(pb) + kWaves * 32 * 4; }
__host__ __device__ constexpr int wm_off(int pb) { return turn_off(pb) + kWaves * kTurn; }
__host__ __device__ constexpr int lds_bytes(int K, int pb) { return wm_off(pb) + K * 4; }
// where a workgroup makes its list (no projection then): behind everything a tile of either height writes ahead of its loop
constexpr int kListOff = turn_off(kMaxPB);
static_assert(wm_off(2) <= kListOff && kHeadGroup + kHeadGroup / kWave * 4 + 128 * 4 <= kWaves * kTurn, "the list's tables share their bytes");
// time of one tile of 64 / 128 pixels in the same unit (measured 14-17 and 21-26 us at K = 1024): a workgroup streams
// all of w1 whatever its height
constexpr int kCost2 = 2, kCost4 = 3;
}  // namespace head

// w1 [256][K] in MFMA fragment order: slice b (K chunk of 64), wave w, K step kg, lane l hold the 16 bytes
// W1[channel 32w + l%32][k = 64b + 16kg + 8*(l/32) .. +7].
__device__ __forceinline__ void head_pack_chunk(int idx, const uint4* __restrict__ w1, int K, uint4* __restrict__ out) {
  const int l = idx & 63, kg = (idx >> 6) & 3, w = (idx >> 8) & 7, b = idx >> 11;
  const int ch = 32 * w + (l & 31), k = 64 * b + kg * 16 + (l >> 5) * 8;
  out[idx] = w1[((size_t)ch * K + k) / 8];
}
__global__ __launch_bounds__(256) void k_pack_head_weights(const uint4* __restrict__ w1, int K, uint4* __restrict__ out) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx < (K / 64) * tail::kSliceChunks) head_pack_chunk(idx, w1, K, out);
}

// One tile of 32*PB rows: rows row0 .. of the dense map, or (listed) of a pixel list with M entries whose entries for
// this lane's rows (row0 + 64i + 8*wave + lane/8) the caller has already requested.
template <bool PROJ, int PB>
__device__ __forceinline__ void head_tile(const HeadArgs& a, const int row0, const int M, const bool listed,
                                          const int (&pixsp)[PB / 2]) {
  using namespace head;
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int kBM = 32 * PB, kAStage = a_stage(PB), kTabOff = tab_off(PB);
  constexpr int kAI = PB / 2;  // LDS-direct instructions per wave and activation slice (8 rows each)
  static_assert(PB % 2 == 0, "an activation instruction of all eight waves covers 64 rows");
  float* const s_s1 = reinterpret_cast<float*>(smem + kTabOff);
  float* const s_t1 = s_s1 + kMid;
  int* const s_orow = reinterpret_cast<int*>(smem + orow_off(PB));
  float* const s_part = reinterpret_cast<float*>(smem + part_off(PB));
  float* const s_wm = reinterpret_cast<float*>(smem + wm_off(PB));

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, lhi = lane >> 5, l8 = lane >> 3, l7 = lane & 7;
  const int K = a.K, NSL = K / 64;
  // Channel skipping (dense rows only): the mask multiplies the 3x3's input, so h1 is stored as zero in the groups a
  // row's sample drops.  Bit t: the row of pixel block t this lane stores keeps the group of this wave's 32 channels.
  unsigned hkeep = ~0u;
  if (a.rbits != nullptr && !listed) {
    hkeep = 0;
#pragma unroll
    for (int t = 0; t < PB; ++t) {
      const int n = min(row0 + 32 * t + l31, M - 1) / a.hw;
      hkeep |= (((unsigned)a.rbits[n] >> ((wave * 32) / a.cs_group)) & 1u) << t;
    }
  }

  // ---- per-channel tables: requested ahead of the streams, stored to LDS behind them -------------------------------
  static_assert(kThreads == 2 * kMid, "a thread takes one entry of s1 or t1");
  const float tab = tid < kMid ? a.s1[tid] : a.t1[tid - kMid];
  constexpr int kWm = PROJ ? kMaxK / kThreads : 1;
  float wm[kWm];
  if constexpr (PROJ) {
#pragma unroll
    for (int i = 0; i < kWm; ++i)
      if (i * kThreads < K) wm[i] = a.wmask[min(i * kThreads + tid, K - 1)];
  }

  // ---- weight stream: four slices in registers -------------------------------------------------------------------
  // (buffer loads: see laud_tail.hip)
  const __amdgpu_buffer_rsrc_t wrs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.wpacked), 0, NSL * (tail::kSliceChunks * 16), 0x00020000);
  const unsigned wlane = (unsigned)(wave * 4096 + lane * 16);
  u32x4 wr[kWRing][4];
  auto load_W = [&](int buf, int b, int kg) __attribute__((always_inline)) {
    const int bb = b < NSL ? b : NSL - 1;  // past the end: the last slice again (keeps the load count uniform)
    wr[buf][kg] = __builtin_amdgcn_raw_buffer_load_b128(wrs, wlane + kg * 1024, bb * (tail::kSliceChunks * 16), 0);
  };

  // ---- activation rows: instruction i of wave w loads rows 64i + 8w .. +7; row r keeps chunk c at position
  // c ^ (r&7) ^ ((r>>3)&1) ---------------------------------------------------------------------------------------
  unsigned voffA[kAI];
#pragma unroll
  for (int i = 0; i < kAI; ++i) {
    const int r = 64 * i + 8 * wave + l8;
    const int rho = row0 + r;
    const unsigned c = (unsigned)l7 ^ ((unsigned)(l8 & 7) ^ (wave & 1u));
    const int pixel = rho < M ? (listed ? pixsp[i] : rho) : -1;
    voffA[i] = pixel >= 0 ? (unsigned)pixel * (unsigned)(K * 2) + c * 16u : kOob;
    if (l7 == 0) s_orow[r] = pixel;
  }
  const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.x), 0, (int)kOob, 0x00020000);
  const unsigned ldsA = wave * 1024;
  auto issue_A = [&](int s) __attribute__((always_inline)) {
    const unsigned soff = (unsigned)s * 128u;
#pragma unroll
    for (int i = 0; i < kAI; ++i)
      dma16(xrs, s < NSL ? voffA[i] : kOob, soff, ldsA + (unsigned)(s & (kARing - 1)) * kAStage + i * 8192);
  };
  // slice by slice, so that the first multiplications wait for the first slice only
  static_assert(kARing == 4 && kWRing == 4, "the counts of the waits below");
#pragma unroll
  for (int s = 0; s < kWRing; ++s) {
    if (s < kARing - 1) issue_A(s);
#pragma unroll
    for (int kg = 0; kg < 4; ++kg) load_W(s, s, kg);
    __builtin_amdgcn_sched_barrier(0);
  }
  s_s1[tid] = tab;  // (s1, then t1)
  if constexpr (PROJ) {
#pragma unroll
    for (int i = 0; i < kWm; ++i)
      if (i * kThreads + tid < K) s_wm[i * kThreads + tid] = wm[i];
  }

  unsigned swz[4];
  {
    const unsigned f = (unsigned)(l31 & 7) ^ ((unsigned)(l31 >> 3) & 1u);
#pragma unroll
    for (int kg = 0; kg < 4; ++kg) swz[kg] = (unsigned)l31 * 128u + (((2u * kg + lhi) ^ f) << 4);
  }
  // of the two waves of a SIMD one goes first, the other's MFMAs fill what it leaves: in step both would wait and multiply at once
  if (wave < kWaves / 2) __builtin_amdgcn_s_setprio(1);
  f32x16 acc[PB];
#pragma unroll
  for (int t = 0; t < PB; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
  // The masker projection: wave w takes the pixel block w % PB in every kShare-th K step, the same work for every wave and slice
  // (a wave that took one step for all blocks kept the others waiting at the slice's barrier: 1610 cycles a slice, 1024 of them
  // MFMAs).  Four sums of a lane: as many products in a chain as the sums of sixteen lanes' steps had.
  constexpr int kShare = kWaves / PB;
  const int pblk = wave % PB, pshare = wave / PB;
  float psum[4] = {0.f, 0.f, 0.f, 0.f};
  uint4 pv = make_uint4(0, 0, 0, 0);
  float4 pw[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)};
  const unsigned swzp = (swz[0] ^ (unsigned)(pshare * 32)) + pblk * 4096;  // the chunk of K step pshare
  const float* const wmp = s_wm + pshare * 16 + lhi * 8;
  uint4 fa[2][PB];
  auto read_frag = [&](int buf, int s, int kg, int t) __attribute__((always_inline)) {
    fa[buf][t] = *reinterpret_cast<const uint4*>(smem + (unsigned)(s & (kARing - 1)) * kAStage + swz[kg] + t * 4096);
  };

  vm_wait<16 + 2 * kAI>();  // own part of the activations of slice 0 (behind them: W(0), A(1), W(1), A(2), W(2), W(3))
  lds_wait();
  wg_barrier();
#pragma unroll
  for (int t = 0; t < PB; ++t) read_frag(0, 0, 0, t);

  // Four slices = sixteen K steps with static register indices.  A weight register is refilled behind the step that
  // used it: a wave that issues its four loads of a slice in a row stands in the queue of the compute unit's vector-memory
  // path, which takes 64 bytes a cycle, and its MFMAs with it.  Vector-memory operations of a wave in program order, per
  // slice s: W(s+4) K steps 0, 1; A(s+3) x kAI [middle of s]; W(s+4) K steps 2, 3.  Needed at the barrier of slice s:
  // A(s+1), issued two slices earlier -- two steps of W, then W x 4 and A(s+2), then two steps of W are younger: 8 + kAI
  // loads; of the slices 0 and 1, whose A(s+1) lies ahead of the loop, 14 + kAI.  Loads past the last slice are issued all
  // the same so that the count holds to the end.
  for (int s0 = 0; s0 < NSL; s0 += 4) {
#pragma unroll
    for (int g = 0; g < 16; ++g) {
      const int s = s0 + g / 4, kg = g % 4;
      if (PROJ && g % kShare == 0) {
        pv = *reinterpret_cast<const uint4*>(smem + (unsigned)(s & (kARing - 1)) * kAStage + (swzp ^ (unsigned)(kg * 32)));
        pw[0] = *reinterpret_cast<const float4*>(wmp + s * 64 + kg * 16);
        pw[1] = *reinterpret_cast<const float4*>(wmp + s * 64 + kg * 16 + 4);
      }
#pragma unroll
      for (int t = 0; t < PB; ++t) {
        acc[t] = mma_bf16(wr[g / 4][kg], fa[g & 1][t], acc[t]);
        __builtin_amdgcn_sched_barrier(0);
        read_frag((g + 1) & 1, kg < 3 ? s : s + 1, (kg + 1) & 3, t);  // (behind the last slice: of a stage that nothing is done with)
        const int m = g % kShare * PB + t;  // eight MFMAs a chunk: two of its elements behind every second one
        if (PROJ && (m & 1)) {
          const int d = m / 2;
          const unsigned v = d == 0 ? pv.x : d == 1 ? pv.y : d == 2 ? pv.z : pv.w;
          const float4 w = pw[d / 2];
          psum[2 * (d & 1)] += __uint_as_float(v << 16) * (d & 1 ? w.z : w.x);
          psum[2 * (d & 1) + 1] += __uint_as_float(v & 0xffff0000u) * (d & 1 ? w.w : w.y);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      load_W(g / 4, s + kWRing, kg);
      __builtin_amdgcn_sched_barrier(0);
      if (kg == 1) {
        if (s < 2) vm_wait<14 + kAI>(); else vm_wait<8 + kAI>();
        wg_barrier();
        issue_A(s + kARing - 1);
      }
    }
  }

  // ---- h1 = relu(s1 * acc + t1); through LDS, so that four lanes store 64 bytes of a row (laud_tile_util.h: row_put, row_get) ------
  {
    const int cb = wave * 32;
    __bf16* const outp = reinterpret_cast<__bf16*>(a.h1);
    float4 sc[4], sh[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      sc[g] = *reinterpret_cast<const float4*>(s_s1 + cb + 8 * g + 4 * lhi);
      sh[g] = *reinterpret_cast<const float4*>(s_t1 + cb + 8 * g + 4 * lhi);
    }
#pragma unroll
    for (int t = 0; t < PB; ++t) {
      unsigned char* const turn = smem + turn_off(PB) + wave * kTurn + (t & 1) * 2048;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        u32x2 c = {pack_bf16(fmaxf(acc[t][4 * g] * sc[g].x + sh[g].x, 0.f), fmaxf(acc[t][4 * g + 1] * sc[g].y + sh[g].y, 0.f)),
                   pack_bf16(fmaxf(acc[t][4 * g + 2] * sc[g].z + sh[g].z, 0.f), fmaxf(acc[t][4 * g + 3] * sc[g].w + sh[g].w, 0.f))};
        if (!((hkeep >> t) & 1u)) c = u32x2{0, 0};  // channel skipping: the row's sample drops the group of this wave's channels
        *reinterpret_cast<u32x2*>(turn + row_put(lane, g)) = c;
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const u32x4 c = *reinterpret_cast<const u32x4*>(turn + row_get(lane, q));
        const int pixel = s_orow[32 * t + 16 * q + (lane >> 2)];
        if (pixel >= 0) *reinterpret_cast<u32x4*>(outp + (size_t)pixel * kMid + cb + (lane & 3) * 8) = c;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // ---- projection: the two K halves of a pixel sit in lanes l and l+32; then the shares of the block's waves --------
  if constexpr (PROJ) {
    const float half = (psum[0] + psum[1]) + (psum[2] + psum[3]);
    const float other = __shfl_xor(half, 32, kWave);
    if (lhi == 0) s_part[pshare * kBM + 32 * pblk + l31] = half + other;
    lds_wait();
    wg_barrier();
    if (tid < kBM && s_orow[tid] >= 0) {
      float p = 0.f;
#pragma unroll
      for (int w = 0; w < kShare; ++w) p += s_part[w * kBM + tid];
      a.proj[s_orow[tid]] = p;
    }
  }
}

// The tile height: dense rows are known on the host (a.pb set); for pixel lists the counts live on the device, and
// every workgroup takes the same decision from them -- the height with the smaller (rounds of workgroups over the
// compute units) x (time of one tile), as in the fused conv2 -> conv3 kernel.
template <bool PROJ>
__global__ __launch_bounds__(head::kThreads) void k_head(const HeadArgs a) {
  using namespace head;
  prefetch_args<sizeof(HeadArgs)>();
  int pb = a.pb;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, l8 = lane >> 3;
  if constexpr (!PROJ) {
    if (a.idx != nullptr) {
      // The dilated pixel list of the workgroup's group of samples, made here by every workgroup of the group for itself: a chain of
      // two memory round trips and three barriers (about 2 us), where a launch that writes the lists takes 7.  Workgroup id ->
      // (group, tile) as for lists below.  The height goes by the group's own count: groups need not agree.
      // (in bytes that a tile writes behind its loop only: a faster wave may be there while another still reads here)
      extern __shared__ __align__(16) unsigned char smem[];
      unsigned char* const s_pm = smem + kListOff;  // patch masks of the group's samples
      int* const s_cnt = reinterpret_cast<int*>(s_pm + kHeadGroup);
      int* const s_list = s_cnt + kHeadGroup / kWave;
      const unsigned touched = l2_touch(a.wpacked, a.K / 64 * tail::kSliceChunks * 16, kThreads);
      const int tid = threadIdx.x;
      const int g = blockIdx.x % a.m_rows, tile = blockIdx.x / a.m_rows;
      const int Wp = fast_div(a.Wo, a.d_s), pps = fast_div(a.Ho, a.d_s) * Wp, HW = a.H * a.W;
      const int n0 = g * a.gs, ns = min(a.gs, a.N - n0), q0 = n0 * pps, nq = ns * pps, npx = ns * HW;
      const int cnt = *a.count;
      for (int i = tid; i < (nq + 15) / 16; i += kThreads) reinterpret_cast<uint4*>(s_pm)[i] = make_uint4(0, 0, 0, 0);
      int lo = 0, hi = cnt;
      constexpr int kAtOnce = 16;  // entries of a thread requested before any is used: one round trip for lists of up to 8192
      if (cnt > kAtOnce * kThreads) wave_lower_bound2(a.idx, cnt, q0, q0 + nq, lo, hi);
      __syncthreads();
      for (int i0 = lo + tid; i0 < hi; i0 += kAtOnce * kThreads) {
        int e[kAtOnce];
#pragma unroll
        for (int u = 0; u < kAtOnce; ++u) e[u] = a.idx[min(i0 + u * kThreads, hi - 1)];
#pragma unroll
        for (int u = 0; u < kAtOnce; ++u)
          if (i0 + u * kThreads < hi && (unsigned)(e[u] - q0) < (unsigned)nq) s_pm[e[u] - q0] = 1;
      }
      __syncthreads();
      constexpr int kSteps = kHeadGroup / kThreads;
      unsigned need = 0;  // bit it: this thread's pixel it * kThreads + tid of the group is in the list
      int ahead[kSteps];  // ... and the list's pixels ahead of it in its wave's 64
#pragma unroll
      for (int it = 0; it < kSteps; ++it) {
        ahead[it] = 0;
        if (it * kThreads >= npx) continue;
        const int pp = it * kThreads + tid;
        bool in = false;
        if (pp < npx) {
          const int ln = fast_div(pp, a.d_hw), q = pp - ln * HW, y = fast_div(q, a.d_w), x = q - y * a.W;
          in = window_active(s_pm + ln * pps, y, x, a.stride, a.Ho, a.Wo, Wp, a.d_s);
        }
        const unsigned long long b = __ballot(in);
        if (lane == 0) s_cnt[it * (kThreads / kWave) + wv] = __popcll(b);
        ahead[it] = ballot_prefix(b);
        need |= (in ? 1u : 0u) << it;
      }
      __syncthreads();
      const int c = lane < (npx + kThreads - 1) / kThreads * (kThreads / kWave) ? s_cnt[lane] : 0;
      int incl = c;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int t = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += t;
      }
      const int M = __shfl(incl, kWave - 1, kWave);
      if (pb == 0) {
        const int t2 = (M + 63) / 64 * a.m_rows, t4 = (M + 127) / 128 * a.m_rows;
        const int c2 = ((t2 + a.wg_target - 1) / a.wg_target) * kCost2, c4 = ((t4 + a.wg_target - 1) / a.wg_target) * kCost4;
        pb = c2 <= c4 ? 2 : 4;
      }
      pb = __builtin_amdgcn_readfirstlane(pb);
      const int row0 = tile * 32 * pb;
      l2_touched(touched);
      if (row0 >= M) return;
#pragma unroll
      for (int it = 0; it < kSteps; ++it) {
        if (it * kThreads >= npx) continue;
        const int r = __shfl(incl - c, it * (kThreads / kWave) + wv, kWave) + ahead[it] - row0;
        if (((need >> it) & 1u) && (unsigned)r < 32u * pb) s_list[r] = n0 * HW + it * kThreads + tid;
      }
      __syncthreads();
      const int r8 = 8 * wv + l8;
      const int p2[1] = {s_list[r8]}, p4[2] = {s_list[r8], s_list[64 + r8]};  // (rows past the last one: not used)
      if (pb == 2) head_tile<false, 2>(a, row0, M, true, p2);
      else head_tile<false, 4>(a, row0, M, true, p4);
      return;
    }
  }
  if (a.slist != nullptr) {
    // Rows = the pixels of the kept samples, in list order: row -> (slot = row / hw, pixel of sample slist[slot]).  The
    // count lives on the device, so the height is decided here (as for pixel lists), and the sample ids of this lane's
    // rows are requested for both candidate heights together with the count.
    const int r8 = 8 * wv + l8;
    // A list without spare entries (scap 0) is read behind its count.
    int last = a.scap - 1;
    if (a.scap == 0) {
      last = __builtin_nontemporal_load(a.scount) - 1;  // (a load of its own: the other one is not to be waited for)
      if (last < 0) return;
    }
    auto pix_of = [&](int row) __attribute__((always_inline)) {
      const int slot = row / a.hw;
      return a.slist[min(slot, last)] * a.hw + (row - slot * a.hw);
    };
    const int p2[1] = {pix_of((int)blockIdx.x * 64 + r8)};
    const int p4[2] = {pix_of((int)blockIdx.x * 128 + r8), pix_of((int)blockIdx.x * 128 + 64 + r8)};
    const int M = *a.scount * a.hw;
    if (pb == 0) {
      const int t2 = (M + 63) >> 6, t4 = (M + 127) >> 7;
      const int c2 = ((t2 + a.wg_target - 1) / a.wg_target) * kCost2, c4 = ((t4 + a.wg_target - 1) / a.wg_target) * kCost4;
      pb = c2 <= c4 ? 2 : 4;
    }
    const int row0 = blockIdx.x * 32 * pb;
    if (row0 >= M) return;
    if (pb == 2) head_tile<PROJ, 2>(a, row0, M, true, p2);
    else head_tile<PROJ, 4>(a, row0, M, true, p4);
    return;
  }
  if (a.list == nullptr) {
    const int row0 = blockIdx.x * 32 * pb;
    if (row0 >= a.m_rows) return;
    const int none2[1] = {0}, none4[2] = {0, 0};
    if (pb == 2) head_tile<PROJ, 2>(a, row0, a.m_rows, false, none2);
    else head_tile<PROJ, 4>(a, row0, a.m_rows, false, none4);
    return;
  }
  if constexpr (!PROJ) {
    // Pixel lists per group of samples: a.m_rows groups of up to a.group_rows entries.  Workgroup id -> (group =
    // id % groups, tile = id / groups): consecutive ids (which go round-robin over the XCDs) cycle through the groups
    // at equal tile index, so the tiles that exist come first and evenly spread, the idle workgroups last.  Group
    // and tile do not depend on the counts, so the list entries of both candidate heights are requested together
    // with the counts: one memory round trip before the rows themselves.
    const int g = blockIdx.x % a.m_rows, tile = blockIdx.x / a.m_rows;
    const int32_t* const listp = a.list + (size_t)g * a.group_rows;
    const int cap = a.group_rows - 1;
    const int r8 = 8 * wv + l8;
    int p2[1], p4[2];
    p2[0] = listp[min(tile * 64 + r8, cap)];
    p4[0] = listp[min(tile * 128 + r8, cap)];
    p4[1] = listp[min(tile * 128 + 64 + r8, cap)];
    const int M = a.counts[g];
    if (pb == 0) {
      // the height with the smaller (rounds of workgroups over the compute units) x (time of one tile); the counts
      // are read one per lane and summed across the wave (every wave does the same)
      int t2 = 0, t4 = 0;
      for (int g0 = 0; g0 < a.m_rows; g0 += kWave) {
        const int c = g0 + lane < a.m_rows ? a.counts[g0 + lane] : 0;
        int v2 = (c + 63) >> 6, v4 = (c + 127) >> 7;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) { v2 += __shfl_xor(v2, d, kWave); v4 += __shfl_xor(v4, d, kWave); }
        t2 += v2;
        t4 += v4;
      }
      const int c2 = ((t2 + a.wg_target - 1) / a.wg_target) * kCost2, c4 = ((t4 + a.wg_target - 1) / a.wg_target) * kCost4;
      pb = c2 <= c4 ? 2 : 4;
    }
    const int row0 = tile * 32 * pb;
    if (row0 >= M) return;
    if (pb == 2) head_tile<false, 2>(a, row0, M, true, p2);
    else head_tile<false, 4>(a, row0, M, true, p4);
  }
}

// ---- host side -----------------------------------------------------------------------------------------------------
bool head_supported(int dtype, int c_in, int c_mid) {
  return dtype == LAUD_BF16 && c_mid == head::kMid && c_in % 256 == 0 && c_in <= head::kMaxK;
}
size_t head_packed_bytes(int c_in) { return align_up((size_t)(c_in / 64) * tail::kSliceChunks * 16, 256); }

static int g_head_cus[32];  // compute units of device d (written before the device's bit in launch_head's `done`)

int head_init_device() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 32) return LAUD_ERR_HIP;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return LAUD_ERR_HIP;
  g_head_cus[dev] = cus;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_head<true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                          head::lds_bytes(head::kMaxK, head::kMaxPB)) != hipSuccess)
    return LAUD_ERR_HIP;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_head<false>), hipFuncAttributeMaxDynamicSharedMemorySize,
                          head::lds_bytes(head::kMaxK, head::kMaxPB)) != hipSuccess)
    return LAUD_ERR_HIP;
  return LAUD_OK;
}

int launch_head_pack(const void* w1, int c_in, void* packed, hipStream_t st) {
  const int chunks = (c_in / 64) * tail::kSliceChunks;
  hipLaunchKernelGGL(k_pack_head_weights, dim3((chunks + 255) / 256), dim3(256), 0, st, (const uint4*)w1, c_in, (uint4*)packed);
  return check_launch();
}

int launch_head(const HeadArgs& args, hipStream_t st) {
  static std::atomic<unsigned> done{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 32) return LAUD_ERR_HIP;
  const unsigned bit = 1u << dev;
  if (!(done.load(std::memory_order_acquire) & bit)) {
    if (head_init_device() != LAUD_OK) return LAUD_ERR_HIP;
    done.fetch_or(bit, std::memory_order_release);
  }
  HeadArgs a = args;
  a.wg_target = g_head_cus[dev];
  unsigned grid;
  int lds_pb = head::kMaxPB;
  if (a.slist != nullptr) {
    // pixels of listed samples: capacity m_rows = scap * hw rows, the count is on the device
    if (a.pb != 2 && a.pb != 4) a.pb = 0;
    grid = (unsigned)((a.m_rows + (a.pb == 4 ? 127 : 63)) / (a.pb == 4 ? 128 : 64));
  } else if (a.list == nullptr && a.idx == nullptr) {
    // dense rows: the count is known here; the same rounds x tile-time cost the kernel uses for lists
    if (a.pb != 2 && a.pb != 4) {
      const long long t2 = (a.m_rows + 63) / 64, t4 = (a.m_rows + 127) / 128;
      const long long c2 = ((t2 + a.wg_target - 1) / a.wg_target) * head::kCost2;
      const long long c4 = ((t4 + a.wg_target - 1) / a.wg_target) * head::kCost4;
      a.pb = c2 <= c4 ? 2 : 4;
    }
    grid = (unsigned)((a.m_rows + 32 * a.pb - 1) / (32 * a.pb));
    lds_pb = a.pb;
  } else {
    // m_rows groups, each with up to group_rows entries: enough workgroups for the smaller tile height
    if (a.pb != 2 && a.pb != 4) a.pb = 0;
    if (a.idx) {
      a.group_rows = a.gs * a.H * a.W;
      a.d_hw = make_fast_div(a.H * a.W); a.d_w = make_fast_div(a.W); a.d_s = make_fast_div(a.S);
      // a workgroup without a tile has its group's list to make before it knows: of more than two rounds of them, half as many
      if ((long long)a.m_rows * ((a.group_rows + 63) / 64) > 2 * a.wg_target) a.pb = 4;
    }
    const int h = a.pb ? 32 * a.pb : 64;
    grid = (unsigned)a.m_rows * (unsigned)((a.group_rows + h - 1) / h);
  }
  StageScope scope(LAUD_STAGE_CONV1, st);
  if (a.wmask)
    hipLaunchKernelGGL((k_head<true>), dim3(grid), dim3(head::kThreads), head::lds_bytes(a.K, lds_pb), st, a);
  else
    hipLaunchKernelGGL((k_head<false>), dim3(grid), dim3(head::kThreads), head::lds_bytes(a.K, lds_pb), st, a);
  return check_launch();
}

}  // namespace laud
