// conv2 (3x3) -> conv3 (1x1) -> residual add of the dynamic bottleneck in ONE kernel for gfx950: the 3x3's
// output tile h2 never leaves the CU (Sec. 3.4 operator fusion; App. B items 2-3: gather inside the 3x3, scatter-add
// in the last 1x1).  bf16 operands, float32 accumulation; c_mid = 256, c_out a multiple of 256.
//
// One workgroup = 32, 64 or 96 active pixels (rows of the compact list: active patch x pixel in patch; the height is
// chosen on the device from the count, see k_tail) x all 256 mid channels, 8 waves (two per SIMD).  Wave w owns mid
// channels 32w .. 32w+31 of the 3x3 and, per 256-wide column tile of the last 1x1, output channels 32w .. 32w+31 of
// that tile, for all pixels of the tile: the weight rows a wave multiplies are the rows it loads itself, so weights
// need no barrier; only the activation slices (loaded cooperatively) do.
//
//   * Operands reach LDS with LDS-direct 16-byte buffer loads (no VGPR staging, no ds_write): a wave instruction
//     drops 64 x 16 bytes = 8 rows of a 128-byte K slice.  Bank conflicts are avoided by an XOR swizzle of the 16-byte
//     chunk position applied on the global side: chunk c of row r lies at position c ^ (r&7) ^ ((r>>3)&1).
//   * Rings: 4 activation stages (4 KB per 32 pixels each), 4 weight stages (32 KB each, in registers).  One barrier
//     per slice, placed in the middle of the slice's MFMAs; fragments of the next K step (also across slices) are
//     read before the current step's MFMAs are issued.
//   * The MFMAs compute the transposed tile (weights as the first operand): a lane then holds, for one pixel,
//     4 x 4 consecutive channels, and h2 goes to LDS in 8-byte pieces.  The result passes through 4 KB of LDS a wave on its way to
//     memory, so that four lanes together hold 64 bytes of a row (laud_tile_util.h: turn_put, turn_get).
//   * h2 (pixels x 256 bf16) sits behind the activation ring in LDS; the last 1x1 streams w3 through the
//     same weight ring (no barrier at all in that phase), reads the residual, adds, applies the
//     activation, rounds and stores.
//
// What bounds it: the compute unit's vector-memory path of 64 bytes a cycle, at the clock this load leaves.  A 64-pixel tile brings 40 KB a slice
// of the 3x3 and 32 KB of weights, 8 KB of residual and 8 KB of results a slice of the last 1x1: 640 and 768 cycles of the path (MFMAs 512).
// Stamps, 12544 pixels in place, inputs in turn, 1.71 GHz: 1818 cycles until the count is there, 6514 list -> rows (in whose shadow the
// tables and the first weights come), 36 x 675, 1284 for h2, 16 x 931 with the last epilogue: 28.5 us, 1.2 more between the first and the last
// workgroup, 4.7 of the launch around them.  The launch 33.5 -> 31.0 us with tables and weights out of the rows' way, the last 1x1's
// epilogue in pieces of one MFMA's time and results stored through a descriptor (maps past its 2 GiB: WIDE).
//
// Channel skipping (Fig. 2(c)) rides on the same kernel (template flag CS): the "patches" are whole samples in
// mask-pattern order, the 3x3 leaves out the 64-channel input slices whose group no row of the tile keeps, and h2 is
// stored as zero in the groups a row drops.
//
// Vector-memory counter discipline: the LDS-direct loads are issued from inline assembly, so the compiler does
// not know them.  Every wait for them is an explicit s_waitcnt vmcnt(n), n = number of LOADS this wave issued
// after the ones needed (loads return in order; stores in flight only make such a wait longer, never shorter).
#include "laud_common.h"
#include "laud_tail_pack.h"
#include "laud_tile_util.h"

#include <atomic>
#include <type_traits>

namespace laud {

namespace tail {
// A workgroup takes PB blocks of 32 pixels (PB = 1 .. 3, chosen per launch on the device from the number of active
// pixels, see k_tail); the LDS layout depends on it.
constexpr int kMaxPB = 3;
constexpr int kCopyExtra = 128;               // workgroups beyond the tiles' capacity where inactive patches have to be copied
constexpr int kARing = 4;
constexpr int kWRing = 3;                     // weight slices held / in flight in registers (4 without a channel mask)
constexpr unsigned kOob = 0x80000000u;        // offset outside every descriptor: reads as zero
__host__ __device__ constexpr int a_stage(int pb) { return 32 * pb * 128; }        // one 128-byte K slice of every pixel row
__host__ __device__ constexpr int h2_off(int pb) { return kARing * a_stage(pb); }  // h2 tile: 32*pb pixels x 512 bytes
__host__ __device__ constexpr int turn_off(int pb) { return h2_off(pb) + 32 * pb * kMid * 2; }  // kTurnBytes of every wave
__host__ __device__ constexpr int tab_off(int pb) { return turn_off(pb) + kWaves * kTurnBytes; }
// float tables in LDS behind the tiles: s2, t2 [256], then s3, t3 [cout], then the tile's output rows (int)
__host__ __device__ constexpr int lds_bytes(int pb, int cout) { return tab_off(pb) + (2 * kMid + 2 * cout) * 4 + 32 * pb * 4; }
}  // namespace tail

__global__ __launch_bounds__(256) void k_pack_tail_weights(const uint4* __restrict__ w2, const uint4* __restrict__ w3,
                                                           uint4* __restrict__ out, int nslices) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx < nslices * tail::kSliceChunks) tail_pack_chunk(idx, w2, w3, out);
}

#ifdef LAUD_TAIL_DBG
__device__ long long g_tail_dbg[1024 * 64];
#define TAIL_STAMP(i) do { if (tid == 0 && blockIdx.x < 1024) g_tail_dbg[blockIdx.x * 64 + (i)] = (long long)__builtin_readcyclecounter(); } while (0)
__device__ long long g_tail_fine[8 * 64];
// fine stamps: every wave of workgroup 0, slot i (0..63)
#define TAIL_FINE(i) do { if (blockIdx.x == 0 && lane == 0) g_tail_fine[wave * 64 + (i)] = (long long)__builtin_readcyclecounter(); } while (0)
#else
#define TAIL_STAMP(i) do { } while (0)
#define TAIL_FINE(i) do { } while (0)
#endif

// One tile: rows row0 .. row0 + 32*PB - 1 of the compact list of active pixels (M rows exist).
// NCT column tiles of 256 output channels (cout = 256 * NCT); CS: channel mask; WIDE: the output map has more than 2 GiB
template <int NCT, int PB, bool CS, bool WIDE>
__device__ __forceinline__ void tail_tile(const TailArgs& a, const int row0, const int M, const unsigned touched) {
  using namespace tail;
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int COUT = 256 * NCT;
  constexpr int kBM = 32 * PB;
  constexpr int kAStage = a_stage(PB), kAOff = 0, kH2Off = h2_off(PB), kTabOff = tab_off(PB), kTurnOff = turn_off(PB);
  constexpr int kNB = kSl2 + NCT * kKch;  // slices in the weight stream
  // LDS-direct instructions per wave and activation slice: an instruction of all eight waves covers 64 rows; with an
  // odd PB the last one is issued by waves 0-3 only
  constexpr int kAI = (PB + 1) / 2;
  // Two accumulator sets (the epilogue of a column tile behind the next tile's MFMAs) while the registers allow it:
  // three pixel blocks keep one set and run the epilogue after its tile
  constexpr bool DUAL = PB <= 2;
  float* const s_s2 = reinterpret_cast<float*>(smem + kTabOff);
  float* const s_t2 = s_s2 + kMid;
  float* const s_s3 = s_t2 + kMid;
  float* const s_t3 = s_s3 + COUT;
  int* const s_orow = reinterpret_cast<int*>(s_t3 + COUT);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, lhi = lane >> 5, l8 = lane >> 3, l7 = lane & 7;
  const bool lastA = !(PB & 1) || wave < 4;  // this wave takes part in the last activation instruction of a slice

  TAIL_STAMP(0);
  const int SS = a.S * a.S;
  int qsp[(PB + 1) / 2];
#pragma unroll
  for (int i = 0; i < (PB + 1) / 2; ++i) qsp[i] = a.list[fast_div(min(row0 + 64 * i + 8 * wave + l8, M - 1), a.d_ss)];  // (see list_entry)
  // ---- channel skipping: which input slices of the 3x3 this tile needs ---------------------------------------------
  // The tile's rows belong to the list entries (samples) row0/SS .. (row0+kBM-1)/SS; a K chunk (64 input channels) is
  // needed if any of them keeps the chunk's group.  n2 = slices of the 3x3 that are multiplied (9 taps x kept
  // chunks, tap-major); position i of that sequence is slice sid(i) of the packed stream, and the stream goes on
  // into the last 1x1 (all of it: h2 is zero where a row drops a group) behind position n2.
  int n2 = kSl2;
  unsigned kcpack = 0xe4u;  // kept K chunks, two bits each (0, 1, 2, 3)
  int nkc = kKch;
  if constexpr (CS) {
    const int e0 = row0 / SS, e1 = min(row0 + kBM - 1, M - 1) / SS;
    unsigned u = 0;
    for (int e = e0; e <= e1; ++e) u |= a.sbits[e];
    kcpack = 0; nkc = 0;
#pragma unroll
    for (int kc = 0; kc < kKch; ++kc)
      if ((u >> ((kc * 64) / a.cs_group)) & 1u) { kcpack |= (unsigned)kc << (2 * nkc); ++nkc; }
    n2 = 9 * nkc;
  }
  auto sid = [&](int i) __attribute__((always_inline)) -> int {  // packed-stream slice at position i
    if constexpr (!CS) return i;
    if (i >= n2) return kSl2 + (i - n2);
    const int tap = i / nkc, j = i - tap * nkc;
    return tap * kKch + (int)((kcpack >> (2 * j)) & 3u);
  };

  // ... and, per pixel block t of this lane's rows, whether the row keeps the group of this wave's 32 channels (bit t)
  unsigned hkeep = ~0u;
  if constexpr (CS) {
    hkeep = 0;
#pragma unroll
    for (int t = 0; t < PB; ++t) {
      const int e = min(row0 + 32 * t + l31, M - 1) / SS;
      hkeep |= (((unsigned)a.sbits[e] >> ((wave * 32) / a.cs_group)) & 1u) << t;
    }
  }

  // ---- per-channel affine tables: requested with the list entries, stored to LDS behind the first rows' requests -------------
  static_assert(kThreads == 2 * kMid, "a thread takes one entry of s2 or t2");
  float tab[1 + 4 * NCT / 2];
  tab[0] = tid < kMid ? a.s2[tid] : a.t2[tid - kMid];
#pragma unroll
  for (int i = 0; i < COUT / kThreads; ++i) {
    tab[1 + 2 * i] = a.s3[i * kThreads + tid];
    tab[2 + 2 * i] = a.t3[i * kThreads + tid];
  }

  // ---- weight stream: a ring of slices in registers (one in use, the others in flight) ------------------------------
  // (Buffer loads: a 64-bit address per lane takes vector instructions and register reads from the MFMAs.  One compute unit's
  // stream beside two MFMAs and two fragment reads a K step: 93 bytes a ns through such addresses, 119 through a descriptor; a
  // 64-pixel tile's slice 914 -> 784 cycles.)
  const __amdgpu_buffer_rsrc_t wrs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.wpacked), 0, kNB * kSliceChunks * 16, 0x00020000);
  const unsigned wlane = (unsigned)(wave * 4096 + lane * 16);
  auto fragment_W = [&](int b, int kg) __attribute__((always_inline)) -> u32x4 {  // K step kg of slice b
    return __builtin_amdgcn_raw_buffer_load_b128(wrs, wlane + kg * 1024, b * (kSliceChunks * 16), 0);
  };
  // Weight slices held / in flight in registers: four (every compute unit streams the same 1.7 MB at once, which keeps
  // the L2 at its bandwidth limit and its latency high: 37.3 against 38.3 us per launch with three); three with a
  // channel mask, whose slice sequences have 9, 18, 27 or 36 entries.
  constexpr int WR = CS ? kWRing : 4;
  static_assert(kSl2 % WR == 0, "the slice groups of the 3x3 must end where the last 1x1 starts");
  u32x4 wr[WR][4];
  auto load_W = [&](int buf, int i) __attribute__((always_inline)) {  // position i of the slice sequence
    const int b = sid(i);
#pragma unroll
    for (int kg = 0; kg < 4; ++kg) wr[buf][kg] = fragment_W(b, kg);
  };
  // (two slices ahead of the rows, which wait for the list, the others behind them: what the compute unit's path of 64 bytes a cycle
  // brings first is what the first multiplications need)
  constexpr int kFirstW = 2;
#pragma unroll
  for (int b = 0; b < kFirstW; ++b) load_W(b, b);

  // ---- activation rows: instruction i of wave w loads rows 64i + 8w .. +7, lane l the chunk position l%8 of row
  // 64i + 8w + l/8; row r keeps chunk c at position c ^ f(r), f(r) = (r&7) ^ ((r>>3)&1) (conflict-free fragment
  // reads; the swizzle is applied on the global side) -----------------------------------------------------------
  const int sy = a.stride;
  const int Wp = fast_div(a.Wo, a.d_s), pps = fast_div(a.Ho, a.d_s) * Wp;
  unsigned voffA[kAI], amask[kAI];
#pragma unroll
  for (int i = 0; i < kAI; ++i) {
    voffA[i] = 0; amask[i] = 0;
    const int r = 64 * i + 8 * wave + l8;
    const int rho = row0 + r;
    if (r >= kBM) continue;
    if (rho < M) {
      const int j = rho - fast_div(rho, a.d_ss) * SS, jy = fast_div(j, a.d_s);
      const int q = qsp[i];
      const int n = fast_div(q, a.d_pps), r2 = q - n * pps;
      const int py = fast_div(r2, a.d_wp), px = r2 - py * Wp;
      const int yo = py * a.S + jy, xo = px * a.S + j - jy * a.S;
      const int y = yo * sy, x = xo * sy;  // centre of the 3x3 on the input grid
      const unsigned pix = (unsigned)(n * a.H * a.W + y * a.W + x);
      const unsigned c = (unsigned)l7 ^ ((unsigned)(l8 & 7) ^ (wave & 1u));
      voffA[i] = pix * (kMid * 2u) + c * 16u;
      unsigned mk = 0;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int yy = y + t / 3 - 1, xx = x + t % 3 - 1;
        if (yy >= 0 && yy < a.H && xx >= 0 && xx < a.W) mk |= 1u << t;
      }
      amask[i] = mk;
      if (l7 == 0) s_orow[r] = n * (a.Ho * a.Wo) + yo * a.Wo + xo;
    } else if (l7 == 0) {
      s_orow[r] = -1;
    }
  }
  // taps reach one row and one pixel back: the descriptor starts that far before h1
  const long long ashift = (long long)(a.W + 1) * kMid * 2;
  const __amdgpu_buffer_rsrc_t h1rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(reinterpret_cast<const char*>(a.h1)) - ashift, 0, (int)kOob, 0x00020000);
  const unsigned ldsA = kAOff + wave * 1024;
  auto issue_A = [&](int s) __attribute__((always_inline)) {  // position s of the slice sequence -> ring stage s % 4
    const int b = s < n2 ? sid(s) : kSl2;
    const int tap = b / kKch, kc = b - tap * kKch;
    const int ky = tap / 3, kx = tap - ky * 3;
    const unsigned soff = (unsigned)((ky * a.W + kx) * kMid + kc * 64) * 2u;
#pragma unroll
    for (int i = 0; i < kAI; ++i) {
      if (i == kAI - 1 && !lastA) break;
      const unsigned v = (tap < 9 && ((amask[i] >> tap) & 1u)) ? voffA[i] : kOob;  // (positions past the 3x3: zeros)
      dma16(h1rs, v, soff, ldsA + (unsigned)(s & (kARing - 1)) * kAStage + i * 8192);
    }
  };
  issue_A(0);
  issue_A(1);
  issue_A(2);
#pragma unroll
  for (int b = kFirstW; b < WR; ++b) load_W(b, b);
  s_s2[tid] = tab[0];  // (s2, then t2)
#pragma unroll
  for (int i = 0; i < COUT / kThreads; ++i) {
    s_s3[i * kThreads + tid] = tab[1 + 2 * i];
    s_t3[i * kThreads + tid] = tab[2 + 2 * i];
  }

  // ---- fragment addresses: row lane%32 of a 32-row block, chunk 2*kg + lane/32, swizzled ------------------------
  unsigned swz[4];
  {
    const unsigned f = (unsigned)(l31 & 7) ^ ((unsigned)(l31 >> 3) & 1u);
#pragma unroll
    for (int kg = 0; kg < 4; ++kg) swz[kg] = (unsigned)l31 * 128u + (((2u * kg + lhi) ^ f) << 4);
  }

  f32x16 acc[PB];
#pragma unroll
  for (int t = 0; t < PB; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;

  uint4 fa[2][PB];  // activation fragments of the pixel blocks, read one K step ahead of their MFMAs
  auto read_frag2 = [&](int buf, int s, int kg, int t) __attribute__((always_inline)) {
    fa[buf][t] = *reinterpret_cast<const uint4*>(smem + kAOff + (unsigned)(s & (kARing - 1)) * kAStage + swz[kg] + t * 4096);
  };

  // ---- the 3x3 -----------------------------------------------------------------------------------------------
  vm_wait<4 * (WR - kFirstW)>();  // the first weights and this wave's part of activations 0-2 have landed
  l2_touched(touched);
  lds_wait();    // the tables written above
  wg_barrier();  // ... and everybody else's
  TAIL_STAMP(1);
#pragma unroll
  for (int t = 0; t < PB; ++t) read_frag2(0, 0, 0, t);

  // WR slices = 4 WR K steps with static register indices (weight buffer g/4, fragment buffer g%2).
  // One barrier per slice, in its middle: behind it everyone's activations of the next slice have landed and
  // everyone is done with the slice before this one, whose stage is refilled (three slices ahead).
  // A weight register is refilled behind the step that used it (a wave that issues the four loads of a slice in a row stands in
  // the queue of the compute unit's vector-memory path, and its MFMAs with it), a fragment read behind each MFMA.
  // Vector-memory operations of a wave in program order, per slice s: W(s+WR) K steps 0, 1; A(s+3) x kAI [middle of s]; W(s+WR)
  // K steps 2, 3.  Needed at the barrier of slice s: A(s+1), issued two slices earlier -- two steps of W, then W x 4 and A(s+2),
  // then two steps of W are younger: 8 + (this wave's activation instructions per slice) loads; of the first two slices all
  // have landed ahead of the loop.  Activation loads past the last slice are issued all the same (they read as zeros
  // into stages nobody reads any more) so that the count holds to the end.
  auto group2 = [&](int s0) __attribute__((always_inline)) {
    int refill = 0;
#pragma unroll
    for (int g = 0; g < 4 * WR; ++g) {
      const int s = s0 + g / 4, kg = g % 4;
      if (kg == 0) TAIL_STAMP(2 + s);
      if (kg == 0) refill = sid(s + WR);
#pragma unroll
      for (int t = 0; t < PB; ++t) {
        acc[t] = mma_bf16(wr[g / 4][kg], fa[g & 1][t], acc[t]);
        __builtin_amdgcn_sched_barrier(0);
        read_frag2((g + 1) & 1, kg < 3 ? s : s + 1, (kg + 1) & 3, t);  // (behind the last slice: of a stage that nothing is done with)
        __builtin_amdgcn_sched_barrier(0);
      }
      wr[g / 4][kg] = fragment_W(refill, kg);  // (the stream continues into the last 1x1)
      __builtin_amdgcn_sched_barrier(0);
      if (kg == 1) {
        if (lastA) vm_wait<8 + kAI>(); else vm_wait<8 + kAI - 1>();  // own part of the activations of slice s+1
        wg_barrier();        // everyone's; and everyone is done with slice s-1
        issue_A(s + 3);
      }
    }
  };
  for (int s = 0; s < n2; s += WR) group2(s);

  // ---- h2 = relu(s2 * acc + t2) -> LDS -------------------------------------------------------------------------
  TAIL_STAMP(38);
  {
    const int cb = wave * 32;
    float4 sc[4], sh[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      sc[g] = *reinterpret_cast<const float4*>(s_s2 + cb + 8 * g + 4 * lhi);
      sh[g] = *reinterpret_cast<const float4*>(s_t2 + cb + 8 * g + 4 * lhi);
    }
#pragma unroll
    for (int t = 0; t < PB; ++t) {
      // pixel row r, 512 bytes per row; 16-byte chunk c sits at position c ^ (r & 15); this lane's half of chunk 4 * wave + g
      const unsigned r = 32u * t + l31;
      unsigned char* row = smem + kH2Off + r * 512u + lhi * 8u;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        u32x2 c = {pack_bf16(fmaxf(acc[t][4 * g] * sc[g].x + sh[g].x, 0.f), fmaxf(acc[t][4 * g + 1] * sc[g].y + sh[g].y, 0.f)),
                   pack_bf16(fmaxf(acc[t][4 * g + 2] * sc[g].z + sh[g].z, 0.f), fmaxf(acc[t][4 * g + 3] * sc[g].w + sh[g].w, 0.f))};
        // the channel mask multiplies the 3x3's output: a row that drops this wave's group stores zeros
        if (CS && !((hkeep >> t) & 1u)) c = u32x2{0, 0};
        *reinterpret_cast<u32x2*>(row + (((wave * 4u + g) ^ (r & 15u)) << 4)) = c;
      }
      __builtin_amdgcn_sched_barrier(0);              // one pixel block at a time (register pressure)
    }
  }
  lds_wait();
  wg_barrier();  // h2 complete
  TAIL_STAMP(39);

  // ---- the last 1x1, column tile by column tile: no activation loads, no barriers ------------------------------
  // Two accumulator sets alternate between column tiles: while tile ct is multiplied into one, the other (tile
  // ct-1) goes through its epilogue -- affine, residual add, activation, rounding, store -- piece by piece: a quarter of a pixel
  // block is four pieces of about eight vector instructions, each behind one MFMA, which takes as long (in larger pieces both
  // waves of a SIMD multiplied first and then stood in line for the vector ALU: 1000 cycles a slice, 512 of them MFMAs).
  // Results go through the wave's part of the turning buffer; then lane l holds channels 8 * (l % 4) .. +7 of row 16 q + l / 4 of a
  // pixel block, q = 0, 1.  The row of the map is read from LDS where it is used (kept, its address costs the registers that the
  // accumulators need); a row that does not exist has an offset outside the descriptors: nothing is read or stored there.
  const unsigned ocol = (unsigned)(wave * 32 + (lane & 3) * 8) * 2u;
  const __amdgpu_buffer_rsrc_t resrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.res), 0, (int)kOob, 0x00020000);
  const __amdgpu_buffer_rsrc_t outrs = __builtin_amdgcn_make_buffer_rsrc(a.out, 0, (int)kOob, 0x00020000);
  unsigned char* const turn = smem + kTurnOff + wave * kTurnBytes;
  const unsigned hrow = kH2Off + (unsigned)l31 * 512u;  // h2 fragment rows: pixel block t at + t * 32 * 512
  const unsigned hx = (unsigned)(l31 & 15);
  auto read_frag3 = [&](int buf, int ks, int kg, int t) __attribute__((always_inline)) {
    const unsigned c = (unsigned)(ks * 8 + 2 * kg) + lhi;
    fa[buf][t] = *reinterpret_cast<const uint4*>(smem + hrow + t * (32 * 512) + ((c ^ hx) << 4));
  };
  const float floor_ = act_floor(a.relu);
  f32x16 acc2[DUAL ? PB : 1];  // the second accumulator set (odd column tiles)
  u32x4 res[PB][2];  // residual of the tile whose epilogue is pending
#pragma unroll
  for (int t = 0; t < PB; ++t) res[t][0] = res[t][1] = u32x4{0, 0, 0, 0};

  // Piece `part` of quarter u of pixel block t.  Quarters 0, 1: the affine of accumulator groups 2 u and 2 u + 1 of column tile `from`
  // into the turning buffer; 2, 3: residual, activation, rounding and store of 16 of its rows, then the request for the residual
  // that column tile `next` adds there.  (from, next outside the column tiles: none)
  float4 e0, e1;       // what a piece hands on to the next: scale and shift, or eight results
  unsigned eoff = 0;   // byte offset of the row's channels in column tile 0; WIDE: the row itself
  u32x4 epk = {0, 0, 0, 0};
  auto piece = [&](const f32x16& A, int from, int next, int t, int u, int part) __attribute__((always_inline)) {
    if (u < 2) {
      if (from < 0) return;
      const int g = 2 * u + part / 2, c = from * 256 + wave * 32 + 8 * g + 4 * lhi;
      if (!(part & 1)) {
        e0 = *reinterpret_cast<const float4*>(s_s3 + c);
        e1 = *reinterpret_cast<const float4*>(s_t3 + c);
      } else {
        *reinterpret_cast<float4*>(turn + turn_put(lane, g)) =
            make_float4(A[4 * g] * e0.x + e1.x, A[4 * g + 1] * e0.y + e1.y, A[4 * g + 2] * e0.z + e1.z, A[4 * g + 3] * e0.w + e1.w);
      }
      return;
    }
    const int q = u - 2;
    if (part == 0) {
      if (from >= 0) {
        e0 = *reinterpret_cast<const float4*>(turn + turn_get(lane, q, 0));
        e1 = *reinterpret_cast<const float4*>(turn + turn_get(lane, q, 1));
      }
      const int o = s_orow[32 * t + 16 * q + (lane >> 2)];
      eoff = WIDE ? (unsigned)o : o >= 0 ? (unsigned)o * (COUT * 2u) + ocol : kOob;
    } else if (part < 3) {
      if (from < 0) return;
      const float4 x = part == 1 ? e0 : e1;
      const unsigned r0 = res[t][q][2 * part - 2], r1 = res[t][q][2 * part - 1];
      epk[2 * part - 2] = pack_bf16(fmaxf(x.x + __uint_as_float(r0 << 16), floor_), fmaxf(x.y + __uint_as_float(r0 & 0xffff0000u), floor_));
      epk[2 * part - 1] = pack_bf16(fmaxf(x.z + __uint_as_float(r1 << 16), floor_), fmaxf(x.w + __uint_as_float(r1 & 0xffff0000u), floor_));
    } else if constexpr (WIDE) {
      const int o = (int)eoff;
      const size_t at = (size_t)max(o, 0) * (COUT * 2) + ocol;
      if (from >= 0 && o >= 0) *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(a.out) + at + from * 512) = epk;
      if (next >= 0) res[t][q] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(a.res) + at + next * 512);
    } else {
      // (no scalar offset: behind a 16-byte buffer store that has one the compiler leaves no wait state before it writes the store's
      // first data register again, and the store then stores what was written)
      if (from >= 0) __builtin_amdgcn_raw_buffer_store_b128(epk, outrs, eoff + from * 512, 0, 0);
      if (next >= 0) res[t][q] = __builtin_amdgcn_raw_buffer_load_b128(resrs, eoff, next * 512, 0);
    }
  };

#pragma unroll
  for (int t = 0; t < PB; ++t) read_frag3(0, 0, 0, t);
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) {
#pragma unroll
    for (int st = 0; st < 4 * kKch; ++st) {
      const int ks = st / 4, kg = st % 4;
      const int b = kSl2 + ct * kKch + ks;
      const int BUF = b % WR;
      if (kg == 0) TAIL_STAMP(40 + ct * kKch + ks);
      const int cur = st & 1, nxt = cur ^ 1;
#pragma unroll
      for (int t = 0; t < PB; ++t) {
        f32x16& A = DUAL && (ct & 1) ? acc2[t] : acc[t];
        if (st == 0) A = mma_bf16(wr[BUF][kg], fa[cur][t], f32x16{});  // (a column tile starts from zero)
        else A = mma_bf16(wr[BUF][kg], fa[cur][t], A);
        __builtin_amdgcn_sched_barrier(0);
        if (kg < 3) read_frag3(nxt, ks, kg + 1, t);
        else if (b + 1 < kNB) read_frag3(nxt, (ks + 1) % kKch, 0, t);
        // 16 * PB MFMAs a column tile, four for each of the 4 * PB quarters of the tile before it; a residual register is refilled
        // where it is used up, a whole tile ahead of its next use
        const int m = st * PB + t, pt = m / 16, u = m / 4 % 4;
        if constexpr (DUAL) piece(ct & 1 ? acc[pt] : acc2[pt], ct - 1, ct, pt, u, m % 4);
        else if (u >= 2) piece(acc[pt], -1, ct, pt, u, m % 4);
        __builtin_amdgcn_sched_barrier(0);
      }
      // the weight register just used is refilled for one ring length later
      if (b + WR < kNB) wr[BUF][kg] = fragment_W(b + WR, kg);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (!DUAL || ct == NCT - 1) {  // one accumulator set, and the last tile: the epilogue follows its tile
#pragma unroll
      for (int t = 0; t < PB; ++t) {
#pragma unroll
        for (int i = 0; i < 16; ++i) piece(DUAL && (ct & 1) ? acc2[t] : acc[t], ct, -1, t, i / 4, i % 4);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  TAIL_STAMP(56);
}

// The tile height is chosen on the device, where the number of active patches is known.  A workgroup streams all
// weights whatever its height, and one workgroup fits a compute unit, so the time of a launch is (rounds of
// workgroups over the compute units) x (time of one tile); tiles of 32 / 64 / 96 pixels take about 3 : 4 : 6 time
// units (measured; a small tile is bound by its weight stream, a large one by LDS fragment reads + MFMAs).  Every
// workgroup evaluates the same three candidates and takes the cheapest: a small active set spreads over the whole
// chip, a large one does not leave a nearly empty last round.
template <int NCT, bool CS, bool WIDE>
__global__ __launch_bounds__(tail::kThreads) void k_tail(const TailArgs a) {
  using namespace tail;
  prefetch_args<sizeof(TailArgs)>();
  // (a body's blocks bring cold weights: 43.3 -> 36.5 us per launch in a ResNet-101 body, batch 128, ratio 0.5)
  const unsigned touched = l2_touch(a.wpacked, (kSl2 + NCT * kKch) * kSliceChunks * 16, kThreads);
  const int SS = a.S * a.S, b32 = blockIdx.x * 32;
  const int M = *a.count * SS;
  const int t32 = (M + 31) >> 5;
  int pb = a.pb;
  if (pb < 1 || pb > kMaxPB) {
    constexpr int kCost[kMaxPB] = {3, 4, 6};
    int best = 0x7fffffff;
    pb = 1;
#pragma unroll
    for (int c = 1; c <= kMaxPB; ++c) {
      const int tiles = (t32 + c - 1) / c;
      const int cost = ((tiles + a.wg_target - 1) / a.wg_target) * kCost[c - 1];
      if (cost < best) { best = cost; pb = c; }
    }
  }
  const int row0 = b32 * pb;
  if (row0 >= M) {
    vm_wait<0>();
    l2_touched(touched);
    if (a.cp.nblocks) {
      // the first workgroups past the tiles copy the inactive patches: eight for each compute unit the last round of tiles
      // leaves idle (each has a chain of four round trips ahead of its share; two, four and sixteen measured 2 to 4 us slower)
      extern __shared__ __align__(16) unsigned char smem[];
      const int tiles = (t32 + pb - 1) / pb, idle = a.wg_target - tiles % a.wg_target;
      const int nparts = min((int)gridDim.x - tiles, max(8 * idle, kCopyExtra));
      if ((int)blockIdx.x - tiles < nparts) copy_inactive_part<kThreads>(a.cp, blockIdx.x - tiles, nparts, smem);
    }
    return;
  }
  switch (pb) {
    case 1: tail_tile<NCT, 1, CS, WIDE>(a, row0, M, touched); break;
    case 2: tail_tile<NCT, 2, CS, WIDE>(a, row0, M, touched); break;
    default: tail_tile<NCT, 3, CS, WIDE>(a, row0, M, touched); break;
  }
}

#ifdef LAUD_TAIL_DBG
}  // namespace laud
extern "C" int laud_tail_fine_read(long long* host) {
  return hipMemcpyFromSymbol(host, HIP_SYMBOL(laud::g_tail_fine), 8 * 64 * 8) == hipSuccess ? 0 : -1;
}
extern "C" int laud_tail_dbg_read(long long* host, int nblocks) {
  return hipMemcpyFromSymbol(host, HIP_SYMBOL(laud::g_tail_dbg), (size_t)nblocks * 64 * 8) == hipSuccess ? 0 : -1;
}
namespace laud {
#endif

// ---- host side ---------------------------------------------------------------------------------------------------
bool tail_supported(int dtype, int c_mid, int c_out) {
  return dtype == LAUD_BF16 && c_mid == tail::kMid && (c_out == 1024);
}
size_t tail_packed_bytes(int c_mid, int c_out) { (void)c_mid; return align_up(tail::packed_bytes(c_out), 256); }

static int g_tail_cus[32];  // compute units of device d (written before the device's bit in launch_tail's `done`)

int tail_init_device() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 32) return LAUD_ERR_HIP;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return LAUD_ERR_HIP;
  g_tail_cus[dev] = cus;
  const auto request = [](const void* kernel) {
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, tail::lds_bytes(tail::kMaxPB, 1024)) == hipSuccess;
  };
  return request(reinterpret_cast<const void*>(&k_tail<4, false, false>)) && request(reinterpret_cast<const void*>(&k_tail<4, false, true>)) &&
                 request(reinterpret_cast<const void*>(&k_tail<4, true, false>)) ? LAUD_OK : LAUD_ERR_HIP;
}

int launch_tail_pack(const void* w2, const void* w3, int c_out, void* packed, hipStream_t st) {
  const int nslices = tail::packed_slices(c_out);
  const int chunks = nslices * tail::kSliceChunks;
  hipLaunchKernelGGL(k_pack_tail_weights, dim3((chunks + 255) / 256), dim3(256), 0, st, (const uint4*)w2, (const uint4*)w3,
                     (uint4*)packed, nslices);
  return check_launch();
}

int launch_tail(const TailArgs& args, long long cap_rows, hipStream_t st) {
  static std::atomic<unsigned> done{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 32) return LAUD_ERR_HIP;
  const unsigned bit = 1u << dev;
  if (!(done.load(std::memory_order_acquire) & bit)) {
    if (tail_init_device() != LAUD_OK) return LAUD_ERR_HIP;
    done.fetch_or(bit, std::memory_order_release);
  }
  TailArgs a = args;
  a.wg_target = g_tail_cus[dev];
  a.d_s = make_fast_div(a.S); a.d_ss = make_fast_div(a.S * a.S); a.d_wp = make_fast_div(a.Wo / a.S);
  a.d_pps = make_fast_div((a.Ho / a.S) * (a.Wo / a.S));
  // one workgroup per 32 rows of the capacity: enough for the smallest tile height; workgroups past the last tile
  // of the height chosen on the device leave at once
  unsigned grid = (unsigned)((cap_rows + 31) / 32);
  if (a.cp.nblocks) grid += tail::kCopyExtra;
  StageScope scope(LAUD_STAGE_CONV2, st);
  // results past a descriptor's 2 GiB (first blocks: c_out = 1024 is more than what bounds x and h1) go through 64-bit addresses, as
  // does the residual (channel skipping: c_out = c_in, which is bounded)
  const bool wide = cap_rows * a.cout * 2 > (long long)tail::kOob;
  if (a.sbits && wide) return LAUD_ERR_UNSUPPORTED;
  const dim3 block(tail::kThreads);
  const int lds = tail::lds_bytes(tail::kMaxPB, 1024);
  if (a.sbits) hipLaunchKernelGGL((k_tail<4, true, false>), dim3(grid), block, lds, st, a);
  else if (wide) hipLaunchKernelGGL((k_tail<4, false, true>), dim3(grid), block, lds, st, a);
  else hipLaunchKernelGGL((k_tail<4, false, false>), dim3(grid), block, lds, st, a);
  return check_launch();
}

}  // namespace laud
