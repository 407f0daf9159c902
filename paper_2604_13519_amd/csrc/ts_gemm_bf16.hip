// Skinny-M projection of a bf16 model for gfx950:  out[r][n] = sum_k X[r][k] * W[n][k],  r < R <= 80 per pass.
//
// With at most a few dozen rows the projection is a weight stream: every weight byte is
// used once, so the kernel is organised around the HBM read of W and nothing else.
//  * Arithmetic: IEEE half x IEEE half -> fp32 (v_mfma_f32_16x16x32_f16).  The bf16 weights are
//    re-encoded as half at model load (exact: half has more significand bits; the load rejects
//    magnitudes beyond half's range) and an activation arrives as the sum of two halves, about
//    22 significant bits, with two MFMAs per weight fragment and row tile.
//  * W is pre-tiled at model load into MFMA operand order (see k_repack_tiles): a wave's
//    16-byte-per-lane global load is one contiguous 1 KiB tile that feeds the MFMA directly as
//    the B operand - no LDS, no shuffles for weights.
//  * Each wave owns NT tiles of 16 output features and walks its K range in chunks of KC;
//    the weights of the next PF chunks are in flight (register ring) while the current one
//    is multiplied.
//  * The activations X (R x K, tiny) are shared by the WAVES waves of a workgroup through a
//    double-buffered LDS chunk and read as A operands with 16-byte LDS loads.  With one row tile, and two
//    where K is not split, they mostly go straight into a deeper LDS ring (k_gemm_few_bf16, see launch_mt).
//  * K is split two ways.  Inside a workgroup, KW waves share the same output columns and take
//    alternate k-steps of every chunk; their accumulators are added through LDS in a fixed
//    order at the end.  Across workgroups, partial sums go to a fp32
//    [split][row][col] buffer that the next row-wise kernel adds up in a fixed order
//    (deterministic, no atomics).  The in-workgroup split costs no memory traffic, the
//    cross-workgroup one costs a write and a read of the partial sums, so the planner uses as
//    little of the second as still fills the chip.
//  * gate/up variant (SWIGLU): the weight tiles of gate and up alternate, so a wave that owns
//    two neighbouring tiles holds gate and up of the same 16 features; with no cross-workgroup
//    split the epilogue applies SiLU(gate) * up and stores the product as half directly.
//  * lm_head variant (ARGMAX): no split; the epilogue reduces each row's maximum over the
//    workgroup's columns and emits one (value, index) partial per row, so the full logits
//    never have to reach memory.
#include "ts_internal.h"
#include "ts_device_utils.h"
#include <algorithm>
#include <type_traits>

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

namespace {

struct GemmArgs {
  const f16_t* X;      // [2 planes][rows][act_ld(K)] IEEE half (x = hi + lo)
  size_t x_plane;      // elements between the hi and the lo plane
  const f16_t* Wt;     // tiled weights, IEEE half
  float* out;          // [split][R][N] partial sums (nullptr for ARGMAX)
  float* logits;       // [R][N] or nullptr (ARGMAX only)
  float* aval;         // [R][amax_parts]
  int32_t* aidx;
  f16_t* act_out;      // SWIGLU: [2 planes][rows][act_ld(N/2)] gated product, IEEE half hi + lo
  size_t act_plane;    // elements between its planes
  unsigned long long* sat;   // counts gated products beyond half's range
  int R, N, K;
  int kper;            // k elements per split
  int n_tiles;         // ceil(N / 16)
  int kt_count;        // K / 32
  size_t split_stride; // R * N
  int amax_parts;
  int zero_row;        // where the rows past the last come from (see x_off)
  int groups, splits;  // column groups x K splits workgroups
  int runs;            // their place on the XCDs
};

enum { MODE_PARTIAL = 0, MODE_ARGMAX = 1, MODE_SWIGLU = 2 };

// The finish of both kernels below: joins the k-waves, applies the mode's epilogue and stores.  acc[mt][t] holds rows
// 4 (lane / 16) .. +4 of row tile mt and column lane % 16 of tile t; red: room for the sums of all waves, free to use.
template <int MT, int NT, int CS, int KW, int MODE>
__device__ __forceinline__ void finish(const GemmArgs& a, const f32x4 (&acc)[MT][NT], const int (&nt_idx)[NT], float* red, int group, int split) {
  constexpr bool ARGMAX = MODE == MODE_ARGMAX;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l15 = lane & 15, g = lane >> 4;
  const int cs = wave / KW, kq = wave % KW;
  // ARGMAX: best (value, column) of every row over the columns of each column set
  __shared__ float rv[ARGMAX ? CS : 1][ARGMAX ? MT * 16 : 1];
  __shared__ int ri[ARGMAX ? CS : 1][ARGMAX ? MT * 16 : 1];
  // value of output (row tile mt, row r of the lane group, tile t) goes to memory
  auto emit = [&](int mt, int r, const float (&v)[NT]) {
    const int row = mt * 16 + g * 4 + r;
    if (ARGMAX) {
      float bv = -INFINITY;
      int bi = 0x7fffffff;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int col = nt_idx[t] * 16 + l15;
        if (nt_idx[t] < a.n_tiles && col < a.N) {
          if (a.logits != nullptr && row < a.R) a.logits[(size_t)row * a.N + col] = v[t];
          amax_take(bv, bi, v[t], col);
        }
      }
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {       // reduce over the 16 lanes that hold this row
        const float ov = __shfl_xor(bv, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        amax_take(bv, bi, ov, oi);
      }
      if (l15 == 0) { rv[cs][row] = bv; ri[cs][row] = bi; }
      return;
    }
    if (row >= a.R) return;
    if (MODE == MODE_SWIGLU) {
      const int f = (nt_idx[0] >> 1) * 16 + l15;           // tiles 2j / 2j+1 = gate / up of features 16j..
      if (nt_idx[NT - 1] < a.n_tiles) {
        const float gv = v[0], uv = v[NT - 1];
        st_act_planes(a.act_out + (size_t)row * act_ld(a.N / 2) + f, a.act_plane, gv / (1.0f + expf(-gv)) * uv, a.sat);
      }
    } else {
      float* o = a.out + (size_t)split * a.split_stride;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int col = nt_idx[t] * 16 + l15;
        if (nt_idx[t] < a.n_tiles && col < a.N) o[(size_t)row * a.N + col] = v[t];
      }
    }
  };
  if (KW == 1) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) v[t] = acc[mt][t][r];
        emit(mt, r, v);
      }
  } else {
    // add the KW accumulators of a column set through LDS, one row tile at a time, always in the order kq = 0, 1, ...
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) red[((wave * 4 + r) * NT + t) * 64 + lane] = acc[mt][t][r];
      __syncthreads();
      for (int r = kq; r < 4; r += KW) {                 // this wave finishes rows r of the tile
        float v[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          float sum = 0.f;
#pragma unroll
          for (int k = 0; k < KW; ++k) sum += red[(((cs * KW + k) * 4 + r) * NT + t) * 64 + lane];
          v[t] = sum;
        }
        emit(mt, r, v);
      }
      __syncthreads();
    }
  }
  if (ARGMAX) {
    __syncthreads();
    if (tid < MT * 16 && tid < a.R) {
      float bv = rv[0][tid];
      int bi = ri[0][tid];
      for (int c = 1; c < CS; ++c) amax_take(bv, bi, rv[c][tid], ri[c][tid]);
      a.aval[(size_t)tid * a.amax_parts + group] = bv;
      a.aidx[(size_t)tid * a.amax_parts + group] = bi;
    }
  }
}

template <int MT, int NT, int CS, int KW, int KC, int PF, int MODE>
__global__ __launch_bounds__(64 * CS * KW) void k_gemm_bf16(GemmArgs a) {
  constexpr int WAVES = CS * KW;            // CS column sets x KW k-step owners
  constexpr int KSTEPS = KC / 32;           // MFMA k-steps per chunk
  constexpr int KSW = KSTEPS / KW;          // ... of which this wave multiplies KSW
  static_assert(KSTEPS % KW == 0 && KSW >= 1, "k-steps of a chunk must divide among the k-waves");
  static_assert(MODE != MODE_SWIGLU || NT == 2, "gate and up tiles alternate");
  // LDS row stride in elements.  A 16-byte read is served in four groups of 16 lanes that are not consecutive (lanes
  // 0-3, 12-15, 20-27 make the first): with rows 16 (2 mod 4) bytes apart, as with 32 more than KC, their 16-byte
  // vectors fall into 16 different bank groups.  16 bytes more left a conflict in every read, half of the LDS cycles
  // (counters: gate/up 65 rows 11.8 -> 7.2 M cycles).
  constexpr int XS = KC + 16;
  constexpr int NTHR = 64 * WAVES;
  constexpr int NBUF = PF + 1;              // weight register ring
  constexpr int PL = TS_ACT_PLANES;         // an activation is the sum of a hi and a lo half
  constexpr int XVP = MT * 16 * KC / 8;     // 16-byte vectors per plane of an X chunk
  constexpr int XV = PL * XVP;
  constexpr int XPT = (XV + NTHR - 1) / NTHR;
  // activation chunks [buffer][plane][row][k]; the same memory later serves the k-wave reduction
  constexpr size_t XS_BYTES = sizeof(f16_t) * 2 * PL * MT * 16 * XS;
  constexpr size_t RED_BYTES = KW > 1 ? sizeof(float) * WAVES * 4 * NT * 64 : 0;
  __shared__ __attribute__((aligned(16))) char smem[XS_BYTES > RED_BYTES ? XS_BYTES : RED_BYTES];
  f16_t (*xs)[PL][MT * 16][XS] = reinterpret_cast<f16_t (*)[PL][MT * 16][XS]>(smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l15 = lane & 15, g = lane >> 4;
  const int cs = wave / KW, kq = wave % KW;
  // Place: workgroups are dealt to the 8 XCDs round robin by id.  With a.runs each XCD takes a contiguous run of
  // the (split, column group) pairs in split order, else the pairs go round robin as they come (use_runs).
  const int units = a.groups * a.splits;
  const int unit = a.runs ? (int)((blockIdx.x & 7) * ((units + 7) / 8) + (blockIdx.x >> 3)) : (int)blockIdx.x;
  if (unit >= units) return;
  const int group = unit % a.groups, split = unit / a.groups;
  const int kbase0 = split * a.kper;
  const int n_chunks = a.kper / KC;

  // Addresses are (uniform 64-bit base) + (32-bit per-lane byte offset that never changes).
  const int cs_u = __builtin_amdgcn_readfirstlane(cs), kq_u = __builtin_amdgcn_readfirstlane(kq);
  const char* wbase[NT];                    // start of this wave's k range in each owned tile row
  int nt_idx[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    nt_idx[t] = (group * CS + cs_u) * NT + t;
    const int c = nt_idx[t] < a.n_tiles ? nt_idx[t] : a.n_tiles - 1;   // idle waves re-read a valid tile
    wbase[t] = reinterpret_cast<const char*>(a.Wt) + ((size_t)c * a.kt_count + kbase0 / 32 + kq_u * KSW) * 1024;
  }
  const uint32_t w_lane = lane * 16;
  // The workspace only grows, and a plane of one that held a very large batch passes 4 GiB: the plane is in the
  // base (a wave's 64 vectors lie in one plane), the lane offset covers the rows of this pass.
  static_assert(XVP % 64 == 0, "a wave stages from one plane");
  constexpr int XPP = XVP % NTHR == 0 ? XVP / NTHR : 0;     // staging rounds per plane; 0: a round holds vectors of both
  const char* xbase = reinterpret_cast<const char*>(a.X) + (size_t)kbase0 * 2;
  const size_t plane_bytes = a.x_plane * 2;
  bool x_lo[XPT];                           // which plane (uniform in a wave)
  uint32_t x_off[XPT];                      // byte offset of each staged vector within its plane and chunk
#pragma unroll
  for (int p = 0; p < XPT; ++p) {
    const int v = XPP ? tid + (p < XPP ? p : p - XPP) * NTHR : min(tid + p * NTHR, XV - 1);      // surplus threads re-read the last vector
    const int rl = (v % XVP) / (KC / 8), cv = v % (KC / 8);
    // rows past the last come from one spare row, which is zero: their lines are fetched once, and zeros cost the
    // matrix pipes little power.  17 rows (32 before): head of 8192 columns 19.4 -> 16.3 us, gate/up 40.6 -> 39.7 us,
    // O 9.2 -> 8.8 us
    const int row = rl < a.R ? rl : a.zero_row;
    x_lo[p] = XPP ? p >= XPP : __builtin_amdgcn_readfirstlane(v / XVP) != 0;
    x_off[p] = ((uint32_t)row * (uint32_t)act_ld(a.K) + cv * 8) * 2;
  }

  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  f16x8 w[NBUF][NT][KSW];
  u32x4 xr[NBUF][XPT];   // activation chunks travel the same register ring as the weights

  auto load_w = [&](f16x8 (&dst)[NT][KSW], int chunk) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int j = 0; j < KSW; ++j)
        dst[t][j] = __builtin_nontemporal_load(
            reinterpret_cast<const f16x8*>(wbase[t] + (size_t)chunk * (KSTEPS * 1024) + w_lane + j * 1024));
  };
  auto load_x = [&](u32x4 (&dst)[XPT], int chunk) {
    const char* hi = xbase + (size_t)chunk * (KC * 2);
    const char* lo = hi + plane_bytes;
#pragma unroll
    for (int p = 0; p < XPT; ++p) dst[p] = *reinterpret_cast<const u32x4*>((x_lo[p] ? lo : hi) + x_off[p]);   // never predicated, see below
  };
  auto store_x = [&](const u32x4 (&src)[XPT], int buf) {
#pragma unroll
    for (int p = 0; p < XPT; ++p) {
      const int v = tid + p * NTHR;
      if (XV % NTHR == 0 || v < XV)
        *reinterpret_cast<u32x4*>(&xs[buf][v / XVP][(v % XVP) / (KC / 8)][(v % (KC / 8)) * 8]) = src[p];
    }
  };
  auto mma_chunk = [&](const f16x8 (&wc)[NT][KSW], int buf) {
#pragma unroll
    for (int ks = 0; ks < KSW; ++ks) {
#pragma unroll
      for (int pl = 0; pl < PL; ++pl) {
        f16x8 xa[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          xa[mt] = *reinterpret_cast<const f16x8*>(&xs[buf][pl][mt * 16 + l15][(kq * KSW + ks) * 32 + g * 8]);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[mt], wc[t][ks], acc[mt][t], 0, 0, 0);
      }
    }
  };

  // Vector-memory loads complete in issue order as far as the wait counter is concerned, and
  // the compiler's wait for a load counts every later load that MIGHT not have been issued as
  // not issued.  Three consequences shape this loop.  The activation chunk of step c + PF is
  // requested together with the weights of step c + PF and waits in registers as long as they
  // do: were it requested one step ahead, storing it to LDS would first wait for every weight
  // load issued before it, and the weights would never be more than one step ahead either.  The
  // small X loads go out BEFORE the weight loads of the same step.  And no load is ever
  // predicated - a prefetch under an `if` would turn every wait into a wait for everything;
  // where nothing is left to prefetch the step re-requests the last chunk instead (an L2 hit
  // that is never used).
  const int last = n_chunks - 1;
  auto step = [&](f16x8 (&wcur)[NT][KSW], f16x8 (&wpf)[NT][KSW], u32x4 (&xpf)[XPT], const u32x4 (&xnext)[XPT], int c) {
    load_x(xpf, min(c + PF, last));
    __builtin_amdgcn_sched_barrier(0);
    load_w(wpf, min(c + PF, last));
    __builtin_amdgcn_sched_barrier(0);
    mma_chunk(wcur, c & 1);
    store_x(xnext, (c + 1) & 1);            // chunk c + 1, requested PF - 1 steps ago
    __syncthreads();
  };

#pragma unroll
  for (int b = 0; b < PF; ++b) {
    load_x(xr[b], min(b, last));
    __builtin_amdgcn_sched_barrier(0);
    load_w(w[b], min(b, last));
    __builtin_amdgcn_sched_barrier(0);
  }
  store_x(xr[0], 0);
  __syncthreads();

  // NBUF chunks per trip so that ring slots are compile-time register names
  int c0 = 0;
  for (; c0 + NBUF <= n_chunks; c0 += NBUF) {
#pragma unroll
    for (int b = 0; b < NBUF; ++b) step(w[b], w[(b + PF) % NBUF], xr[(b + PF) % NBUF], xr[(b + 1) % NBUF], c0 + b);
  }
#pragma unroll
  for (int b = 0; b < NBUF - 1; ++b)
    if (c0 + b < n_chunks) step(w[b], w[(b + PF) % NBUF], xr[(b + PF) % NBUF], xr[(b + 1) % NBUF], c0 + b);

  finish<MT, NT, CS, KW, MODE>(a, acc, nt_idx, reinterpret_cast<float*>(smem), group, split);
}

// One row tile (up to 16 rows), and two where K is not split across workgroups: the same stream with the activations
// going straight into the LDS, RD chunks deep.  In the kernel above the weights are one or two chunks of 128 k ahead, and
// the ring cannot be deeper because the activations share its registers; here they are RD - 1 chunks of 64 ahead.
// A group is the activations and weights of one chunk; a step waits for its own group, meets the other waves (all
// have their pieces in LDS, and none still reads the slot of the chunk before), requests group c + RD - 1 into that
// slot and multiplies.  Loads in the loop are never predicated: past the end they re-request the last chunk.
// Measured (between events, kernel above : this one): 9 rows head of 128256 columns 183 : 172 us (6.1 TB/s); 1 row QKV
// 12.5 : 12.2, O 9.5 : 9.3, 32B-class O 18.8 : 18.1, QKV 20.8 : 20.2; calls 842 : 832 us (decode), 32B-class layers 415 : 410.
// 17 rows: gate/up 41.6 : 41.0, head of 8192 18.4 : 17.9, but the short ranges of QKV 13.6 : 14.0 and O 10.9 : 11.3.  From three row
// tiles on the kernel above is the better one (38 rows down 25.3 : 28.7, 65 rows 28.8 : 32.3, O 14.1 : 15.1 us), with chunks
// of 128 k and three or four slots too (26.9, 30.6, 15.0; at 1 row 21.6 : 22.2 for down).  Nor is the step of the many-row
// kernel, which reads ahead and requests between products, any faster there (gemm_bf16_plan).
template <int MT, int NT, int CS, int KW, int KC, int RD, int MODE>
__global__ __launch_bounds__(64 * CS * KW) void k_gemm_few_bf16(GemmArgs a) {
  constexpr int WAVES = CS * KW;            // CS column sets x KW k-step owners
  constexpr int KSTEPS = KC / 32;           // MFMA k-steps per chunk
  constexpr int KSW = KSTEPS / KW;          // ... of which this wave multiplies KSW
  static_assert(KSTEPS % KW == 0 && KSW >= 1, "k-steps of a chunk must divide among the k-waves");
  static_assert(MODE != MODE_SWIGLU || NT == 2, "gate and up tiles alternate");
  constexpr int PL = TS_ACT_PLANES;         // an activation is the sum of a hi and a lo half
  constexpr int UPR = KC / 8;               // 16-byte vectors per row of a chunk
  constexpr int PPP = MT * 16 * UPR / 64;   // 1 KiB pieces per plane of a chunk: one direct-to-LDS load of a wave each
  constexpr int XN = (PL * PPP + WAVES - 1) / WAVES;      // pieces a wave stages; the surplus repeats the chunk's last one
  constexpr size_t XBYTES = (size_t)PL * PPP * 1024;
  constexpr int GN = XN + NT * KSW;         // loads of a group
  // one array per ring slot: the compiler then knows which loads a read of LDS has to wait for
  static_assert(RD * XBYTES <= 160 * 1024, "the activation chunks fit the LDS");
  __shared__ float red[KW > 1 ? WAVES * 4 * NT * 64 : 1];
  __shared__ __attribute__((aligned(1024))) char xs0[XBYTES], xs1[XBYTES], xs2[RD > 2 ? XBYTES : 16], xs3[RD > 3 ? XBYTES : 16], xs4[RD > 4 ? XBYTES : 16], xs5[RD > 5 ? XBYTES : 16];
  auto slot = [&](auto i_c) -> char* {
    constexpr int I = decltype(i_c)::value;
    if constexpr (I == 0) return xs0;
    else if constexpr (I == 1) return xs1;
    else if constexpr (I == 2) return xs2;
    else if constexpr (I == 3) return xs3;
    else if constexpr (I == 4) return xs4;
    else return xs5;
  };

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l15 = lane & 15, g = lane >> 4;
  const int cs = wave / KW, kq = wave % KW;
  // Place: workgroups are dealt to the 8 XCDs round robin by id.  With a.runs each XCD takes a contiguous run of
  // the (split, column group) pairs in split order, else the pairs go round robin as they come (use_runs).
  const int units = a.groups * a.splits;
  const int unit = a.runs ? (int)((blockIdx.x & 7) * ((units + 7) / 8) + (blockIdx.x >> 3)) : (int)blockIdx.x;
  if (unit >= units) return;
  const int group = unit % a.groups, split = unit / a.groups;
  const int kbase0 = split * a.kper;
  const int n_chunks = a.kper / KC;

  // Addresses are (uniform 64-bit base) + (32-bit per-lane byte offset that never changes).
  const int cs_u = __builtin_amdgcn_readfirstlane(cs), kq_u = __builtin_amdgcn_readfirstlane(kq), wave_u = __builtin_amdgcn_readfirstlane(wave);
  const char* wbase[NT];                    // start of this wave's k range in each owned tile row
  int nt_idx[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    nt_idx[t] = (group * CS + cs_u) * NT + t;
    const int c = nt_idx[t] < a.n_tiles ? nt_idx[t] : a.n_tiles - 1;   // idle waves re-read a valid tile
    wbase[t] = reinterpret_cast<const char*>(a.Wt) + ((size_t)c * a.kt_count + kbase0 / 32 + kq_u * KSW) * 1024;
  }
  const uint32_t w_lane = lane * 16;
  // a row's vectors stand permuted, so that the reads meet no bank twice (see XS above)
  auto swz = [](int row) { return KC == 128 ? row & 15 : row >> 1 & 7; };
  // The workspace only grows, and a plane of one that held a very large batch passes 4 GiB: the plane is in the
  // base, the lane offset covers the rows of this pass.
  const char* xbase = reinterpret_cast<const char*>(a.X) + (size_t)kbase0 * 2;
  const size_t plane_bytes = a.x_plane * 2;
  int piece[XN];
  uint32_t x_off[XN];
#pragma unroll
  for (int p = 0; p < XN; ++p) {
    piece[p] = min(p * WAVES + wave_u, PL * PPP - 1);
    const int rl = piece[p] % PPP * (64 / UPR) + lane / UPR;
    // rows past the last come from one spare row, which is zero: their lines are fetched once, and zeros cost the
    // matrix pipes little power.  17 rows (32 before): head of 8192 columns 19.4 -> 16.3 us, gate/up 40.6 -> 39.7 us,
    // O 9.2 -> 8.8 us
    const int row = rl < a.R ? rl : a.zero_row;
    x_off[p] = ((uint32_t)row * (uint32_t)act_ld(a.K) + ((lane % UPR) ^ swz(rl)) * 8) * 2;
  }

  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  f16x8 w[RD][NT][KSW];
  const int last_chunk = n_chunks - 1;
  auto request = [&](auto i_c, int chunk) __attribute__((always_inline)) {
    constexpr int I = decltype(i_c)::value;
    const int ch = min(chunk, last_chunk);
    const char* xc = xbase + (size_t)ch * (KC * 2);
#pragma unroll
    for (int p = 0; p < XN; ++p) {
      uint32_t o = x_off[p];
      asm("" : "+v"(o));
      __builtin_amdgcn_global_load_lds((const TS_GLOBAL void*)(xc + (piece[p] >= PPP ? plane_bytes : 0) + o),
                                       (TS_LDS void*)(slot(i_c) + piece[p] * 1024), 16, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    uint32_t wl = w_lane;
    asm("" : "+v"(wl));
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int j = 0; j < KSW; ++j)
        w[I][t][j] = __builtin_nontemporal_load(reinterpret_cast<const f16x8*>(wbase[t] + (size_t)ch * (KSTEPS * 1024) + wl + j * 1024));
    __builtin_amdgcn_sched_barrier(0);
  };
  uint32_t x_read[KSW];
#pragma unroll
  for (int j = 0; j < KSW; ++j) x_read[j] = l15 * (KC * 2) + (((kq * KSW + j) * 4 + g) ^ swz(l15)) * 16;
  // T < 0: a step of the loop.  T >= 0: step T of the rest, behind which no chunk is left to request.
  auto step = [&](auto i_c, auto t_c, int c) __attribute__((always_inline)) {
    constexpr int I = decltype(i_c)::value, T = decltype(t_c)::value;
    constexpr int LEFT = RD - 2 - (T < 0 ? 0 : T);           // later groups that may stay in flight
    wait_loads<(LEFT > 0 ? LEFT : 0) * GN>();
    if (T < 0) request(std::integral_constant<int, (I + RD - 1) % RD>{}, c + RD - 1);
#pragma unroll
    for (int ks = 0; ks < KSW; ++ks)
#pragma unroll
      for (int pl = 0; pl < PL; ++pl) {
        f16x8 xa[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          xa[mt] = *reinterpret_cast<const f16x8*>(slot(i_c) + pl * (PPP * 1024) + mt * (16 * KC * 2) + x_read[ks]);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[mt], w[I][t][ks], acc[mt][t], 0, 0, 0);
      }
  };
  auto ring = [&](auto n, auto&& f) __attribute__((always_inline)) {       // f(slot, number) for the first n slots
    constexpr int N = decltype(n)::value;
    if constexpr (N > 0) f(std::integral_constant<int, 0>{});
    if constexpr (N > 1) f(std::integral_constant<int, 1>{});
    if constexpr (N > 2) f(std::integral_constant<int, 2>{});
    if constexpr (N > 3) f(std::integral_constant<int, 3>{});
    if constexpr (N > 4) f(std::integral_constant<int, 4>{});
    if constexpr (N > 5) f(std::integral_constant<int, 5>{});
  };
  using Loop = std::integral_constant<int, -1>;
  using Rest = std::integral_constant<int, RD - 1>;
  ring(Rest{}, [&](auto i_c) __attribute__((always_inline)) { request(i_c, decltype(i_c)::value); });
  int c0 = 0;
  for (; c0 + RD <= n_chunks; c0 += RD)
    ring(std::integral_constant<int, RD>{}, [&](auto i_c) __attribute__((always_inline)) { step(i_c, Loop{}, c0 + decltype(i_c)::value); });
  ring(Rest{}, [&](auto i_c) __attribute__((always_inline)) {
    constexpr int I = decltype(i_c)::value;
    if (c0 + I < n_chunks) step(i_c, i_c, c0 + I);
    else                                                 // a request past the end
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < KSW; ++j) keep_loaded(w[I][t][j]);
  });
  // nothing may still be on its way into the LDS when it is used otherwise or given back
  wait_loads<0>();

  finish<MT, NT, CS, KW, MODE>(a, acc, nt_idx, red, group, split);
}

// One row tile, and two where K is not split: k_gemm_few_bf16, with chunks of 64 k and six slots, or, with four k-waves (one
// k-step of a chunk each), of 128 and four.  The four k-waves of a small model's gate/up are the exception, on short ranges (4 to
// 16 chunks) the ring does not pay for its longer prologue.  Us between events, k_gemm_bf16 : k_gemm_few_bf16 -
// gate/up of 1, 16 and 26 rows, K 512 x 3072 columns 6.1 : 6.1, 6.2 : 6.2, 7.0 : 7.1, K 1024 x 5632 6.7 : 7.1, 7.3 : 7.6, 8.7 : 8.7,
// K 2048 x 11264 12.9 : 13.1, 14.8 : 15.1, 18.1 : 18.0; arg-max, K 512 x 2048 6.5 : 6.5, 6.9 : 6.8, 8.2 : 7.8, K 1024 x 8192
// 8.5 : 8.4, 8.9 : 8.7, 10.4 : 9.9.
template <int NT, int CS, int KW, int KC, int PF, int MODE>
void launch_mt(int mt, dim3 grid, hipStream_t s, const GemmArgs& a) {
  const dim3 block(64 * CS * KW);
  constexpr bool FEW = KW <= 2 || MODE == MODE_ARGMAX;
  constexpr int FKC = KW > 2 ? 128 : 64, FRD = KW > 2 ? 4 : 6;
  switch (mt) {
    case 1:
      if constexpr (FEW) hipLaunchKernelGGL((k_gemm_few_bf16<1, NT, CS, KW, FKC, FRD, MODE>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((k_gemm_bf16<1, NT, CS, KW, KC, PF, MODE>), grid, block, 0, s, a);
      break;
    case 2:
      if constexpr (FEW && MODE != MODE_PARTIAL) hipLaunchKernelGGL((k_gemm_few_bf16<2, NT, CS, KW, FKC, FRD, MODE>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((k_gemm_bf16<2, NT, CS, KW, KC, PF, MODE>), grid, block, 0, s, a);
      break;
    case 3: hipLaunchKernelGGL((k_gemm_bf16<3, NT, CS, KW, KC, PF, MODE>), grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL((k_gemm_bf16<4, NT, CS, KW, KC, PF, MODE>), grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL((k_gemm_bf16<5, NT, CS, KW, KC, PF, MODE>), grid, block, 0, s, a); break;
  }
}

// The compiled tile shapes.  shape id -> (NT, CS, KW): tiles per wave, column sets and
// k-waves per workgroup.  In k_gemm_bf16 all use chunks of 128 k (the LDS holds two buffers of the activation chunk in
// both planes, 90 KiB for 80 rows); the k-wave shapes hold fewer weight registers per chunk and prefetch two to
// four chunks ahead instead of one.  launch_mt has the chunks and the ring of k_gemm_few_bf16.  A plan's K split is a whole
// number of 128 k (kShapeKC) for either.
constexpr int kNumShapes = 7;
const int kShapeNT[kNumShapes] = {1, 2, 1, 2, 2, 1, 2};
const int kShapeCS[kNumShapes] = {4, 4, 8, 8, 4, 2, 1};
const int kShapeKW[kNumShapes] = {1, 1, 1, 1, 2, 4, 4};
const int kShapeKC[kNumShapes] = {128, 128, 128, 128, 128, 128, 128};

template <int MODE>
void launch_shape(int shape, int mt, dim3 grid, hipStream_t s, const GemmArgs& a) {
  switch (shape) {
    case 0: if (MODE != MODE_SWIGLU) launch_mt<1, 4, 1, 128, 1, MODE == MODE_SWIGLU ? MODE_PARTIAL : MODE>(mt, grid, s, a); break;
    case 1: launch_mt<2, 4, 1, 128, 1, MODE>(mt, grid, s, a); break;
    case 2: if (MODE != MODE_SWIGLU) launch_mt<1, 8, 1, 128, 1, MODE == MODE_SWIGLU ? MODE_PARTIAL : MODE>(mt, grid, s, a); break;
    case 3: launch_mt<2, 8, 1, 128, 1, MODE>(mt, grid, s, a); break;
    case 4: launch_mt<2, 4, 2, 128, 2, MODE>(mt, grid, s, a); break;
    case 5: if (MODE == MODE_ARGMAX) launch_mt<1, 2, 4, 128, 4, MODE_ARGMAX>(mt, grid, s, a); break;
    case 6: if (MODE == MODE_SWIGLU) launch_mt<2, 1, 4, 128, 3, MODE_SWIGLU>(mt, grid, s, a); break;
    default: break;
  }
}

bool shape_supports(int shape, int mode) {
  // 32 columns a workgroup, for small projections that cannot split K across workgroups: gate/up of a 512-wide
  // model (3072 columns, 26 rows) 7.4 us on 24 workgroups of 128 columns, 5.2 us on 96
  if (shape >= 5) return mode == (shape == 5 ? MODE_ARGMAX : MODE_SWIGLU);
  if (mode == MODE_SWIGLU) return kShapeNT[shape] == 2;
  return true;
}

// plan.shape values from here on name a many-row configuration: kRowsShape0 + 4 * row tiles + cfg
constexpr int kRowsShape0 = 100;
constexpr size_t kRowsPartCap = (size_t)64 << 20;   // partial-sum elements a plan may use before a workspace exists

// Place of the workgroups on the XCDs.  In runs an XCD reads neighbouring weight tiles, and only the activations of
// one or two K splits pass through its L2 instead of all of them.  That pays (8B shape, round robin : runs, us between
// events): 1 row gate/up 44.4 : 40.0, QKV 14.3 : 12.7, O 11.9 : 9.8, down 22.1 : 21.5; 17 rows 45.3 : 41.7, 14.8 : 13.8,
// 12.0 : 11.0, 23.6 : 22.9; 65 rows O 15.2 : 14.3, down 29.8 : 29.1, gate/up the same.  Except where five row tiles meet a
// shape with one k-wave (one chunk in flight) and an XCD's run is a part of one K range of eight chunks or more,
// presumably because its workgroups then ask its L2 for the same activation lines at the same time, 40 KB a chunk each.  65 rows, from
// a trace: QKV (48 groups x 4 splits) 17.6 : 18.5, head of 128256 columns (501 groups) 204 : 211; half the K range
// (2048) 15.7 : 14.7, four row tiles 16.0 : 16.2 and 193 : 192, and two k-waves (head of 151936 columns) 324 : 316.
// The SwiGLU shapes stay in runs (51200 columns, one k-wave 101.4 : 100.2).
bool use_runs(int shape, int mode, int R, int chunks_per_split, int groups, int splits) {
  return !(R > 64 && mode != MODE_SWIGLU && kShapeKW[shape] == 1 && chunks_per_split >= 8 && (groups * splits + 7) / 8 < groups);
}

}  // namespace

int gemm_bf16_cols_per_group(int shape) { return kShapeNT[shape] * kShapeCS[shape] * 16; }
int gemm_bf16_chunk(int shape) { return shape >= kRowsShape0 ? gemm_rows_chunk((shape - kRowsShape0) % 4) : kShapeKC[shape]; }

// Tile shape and cross-workgroup K splits, from a byte count per CU:
//   rounds x (weight bytes one workgroup streams + 72 KB)     rounds = ceil(workgroups / CUs); start and finish
//                                                             of a round cost what 72 KB of streaming do (3 us)
// + write and read of the fp32 partial sums, shared by all CUs and 15 % dearer (only if splits > 1), at least 5 KB a split:
//   with few rows the kernel that adds them up pays for their number, not their bytes.  Rows of under 1024 columns
//   (512-wide models) pay that in proportion: K 1536 to 512 columns, 38 rows, 6 splits 7.3 us, 12 splits 6.4 us
// + 0.3 of the activation bytes (both planes) a workgroup stages from L2 per round.
// Measured on MI355X, a second round of workgroups costs a full round (the tail does not
// overlap), which the round count models.  mode: 0 partial sums, 1 arg-max (no split),
// 2 SwiGLU epilogue (no split).
// The constants come from a sweep of every (shape, splits) pair of the 8B projections, each with the change
// of the kernel behind it, between events.  One row, before the two fixed costs and with them: QKV 16 splits
// in three rounds 14.8 us, 4 splits in one 12.1 us; O 16 splits 14.9 us, 4 splits 8.3 us; down 21.9 and 20.2 us.
// 17 rows: QKV 17.5 and 14.1 us, down 22.9 and 22.0 us.  65 rows: unchanged plans.
// On the 32B-class shape, which set none of them (one request, events): 1 row QKV 19.7 -> 20.9 us (1280 workgroups
// that overlap on their CUs beat 200 there, which the round count does not see), O 20.1 -> 18.6 us, each norm behind
// a split 7.9 -> 7.0 us; 65 rows O 33.0 -> 27.5 us, head of 151936 columns 363 -> 316 us, the rest alike.  Two layers and a
// head of 8192 columns, 1 / 9 / 17 / 38 / 65 rows: 445 -> 418, 453 -> 427, 501 -> 450, 546 -> 509, 659 -> 603 us a call.
GemmPlan gemm_bf16_plan(const ts_model* m, int R, int N, int K, int mode) {
  // Batches: the many-row kernel.  Up to 80 rows the kernels of this file are the faster ones.  8B shape, us between events,
  // these : the many-row kernel by its best plan - 38, 65 and 80 rows QKV 15.1 : 20.3, 18.8 : 21.0, 19.5 : 21.2, O 12.0 : 14.8,
  // 14.2 : 15.8, 15.0 : 16.2, gate/up 43.8 : 50.7, 50.0 : 53.4, 52.2 : 53.4, down 23.9 : 28.4, 27.3 : 30.0, 29.7 : 30.5, head of
  // 8192 columns 24 : 45, 32 : 48, 34 : 48 - except for the head of 128256 columns from 64 rows on: 49 rows 186 : 188, 64 193 : 189,
  // 65 211 : 192, 80 213 : 193.
  if (R > TS_MROWS_PER_BLOCK) {
    int mt, cfg, splits;
    const size_t max_part = m->part_elems ? m->part_elems : kRowsPartCap;
    gemm_rows_plan(m, R, N, K, mode, max_part, &mt, &cfg, &splits);
    return GemmPlan{kRowsShape0 + mt * 4 + cfg, splits};
  }
  GemmPlan best{mode == MODE_SWIGLU ? 1 : 0, 1};
  double best_cost = 1e300;
  const int rows = ((R + 15) / 16) * 16;
  for (int shape = 0; shape < kNumShapes; ++shape) {
    if (!shape_supports(shape, mode)) continue;
    const int kc = kShapeKC[shape];
    if (K % kc) continue;
    const int chunks = K / kc;
    const int cols = gemm_bf16_cols_per_group(shape);
    const int groups = (N + cols - 1) / cols;
    for (int s = 1; s <= chunks && s <= 16; ++s) {
      if (chunks % s) continue;
      if (mode != MODE_PARTIAL && s > 1) break;
      const long wgs = (long)groups * s;
      const long rounds = (wgs + m->n_cu - 1) / m->n_cu;
      const double kper = (double)K / s;
      double cost = rounds * cols * kper * 2.0;
      // one row tile (the kernel with the deep ring): activations weigh little, splits more than their bytes, and neither
      // one tile per wave nor the number of waves matters.  One row, before and with its own constants: QKV 12.3 -> 11.8 us,
      // down 21.5 -> 20.9; 32B-class O 18.0 -> 16.6, down 42.5 -> 40.2 (9 rows 12.8 -> 12.6, 22.0 -> 21.2, 19.2 -> 18.7, 43.0 -> 41.2)
      // Gate/up and the arg-max keep the constants of the other rows.  Gate/up (28672 columns) and a head of 8192 get the best
      // shape with them at 1 - 32 rows; the one plan of a head is made for 80 rows (amax_parts is sized by it), and
      // for 128256 columns that is 6 - 9 % from the best one at 1 - 16 rows (153 : 166, 157 : 166, 158 : 165 us at 1, 9, 16 rows).
      const bool one = rows <= 16 && mode == MODE_PARTIAL;
      if (s > 1) cost += std::max(2.3 * s * R * (double)N * 4.0 / m->n_cu, (one && N >= 1024 ? 8.0 : 5.0) * std::min(N, 1024) * s);
      cost += (one ? 0.1 : 0.3) * rounds * rows * kper * 2.0 * TS_ACT_PLANES;
      // Measured (8B shape): over a long K range the k-wave shape wins by its deeper prefetch (gate/up, 32
      // chunks, 65 rows: 55.5 us against 57.7 us for the 4-wave shape of the same columns; down, 14 chunks, 1 to
      // 17 rows 21.7 - 22.9 against 22.2 - 23.8 us, from 38 rows on no more); over the short ranges of the split
      // projections its longer prologue and the cross-wave reduction are not amortised (O, 4 chunks, 65 rows:
      // 16.1 against 14.4 us; QKV, 8 chunks: 22.4 against 20.4 us).
      const bool long_k = kper / kc >= 16 || (kper / kc >= 12 && rows <= 32);
      if (!one && (long_k ? kShapeCS[shape] * kShapeKW[shape] < 6 : kShapeKW[shape] > 1)) cost *= 1.05;
      if (!one && kShapeNT[shape] < 2) cost *= 1.05;                     // one tile per wave reads twice the LDS per weight byte
      cost += rounds * 73728.0;
      if (cost < best_cost) { best_cost = cost; best.shape = shape; best.splits = s; }
    }
  }
  return best;
}

void launch_gemm_bf16(ts_model* m, const f16_t* X, const f16_t* Wt, float* out, int R, int N, int K, GemmPlan plan,
                      int mode, float* logits, f16_t* act_out) {
  if (plan.shape >= kRowsShape0) {
    const int code = plan.shape - kRowsShape0;
    launch_gemm_rows_bf16(m, X, Wt, out, R, N, K, code / 4, code % 4, plan.splits, mode, act_out, logits);
    return;
  }
  GemmArgs a;
  a.X = X; a.Wt = Wt; a.out = out; a.logits = logits;
  a.x_plane = (size_t)(m->ws_rows + TS_MROWS_PER_BLOCK) * act_ld(K);
  a.act_plane = (size_t)(m->ws_rows + TS_MROWS_PER_BLOCK) * act_ld(N / 2);
  a.aval = m->amax_val; a.aidx = m->amax_idx;
  a.act_out = act_out;
  a.sat = m->sat_count;
  a.R = R; a.N = N; a.K = K;
  // the first spare row, which nothing writes; the last real row where 32 bits do not reach the spare ones (those
  // outputs are not used, a row of zeros is only the cheaper one)
  a.zero_row = ((size_t)m->ws_rows + 1) * act_ld(K) * 2 < ((size_t)1 << 32) ? m->ws_rows : R - 1;
  const int splits = mode == MODE_PARTIAL ? plan.splits : 1;
  a.kper = K / splits;
  a.n_tiles = (N + 15) / 16;
  a.kt_count = K / 32;
  a.split_stride = (size_t)R * N;
  a.amax_parts = m->amax_parts;
  if (mode == MODE_ARGMAX) m->amax_used = (N + gemm_bf16_cols_per_group(plan.shape) - 1) / gemm_bf16_cols_per_group(plan.shape);
  const int cols = gemm_bf16_cols_per_group(plan.shape);
  const int groups = (N + cols - 1) / cols;
  const int mt = (R + 15) / 16;
  a.groups = groups; a.splits = splits;
  a.runs = use_runs(plan.shape, mode, R, a.kper / kShapeKC[plan.shape], groups, splits);
  dim3 grid((groups * splits + 7) / 8 * 8);
  if (mode == MODE_ARGMAX) launch_shape<MODE_ARGMAX>(plan.shape, mt, grid, m->stream, a);
  else if (mode == MODE_SWIGLU) launch_shape<MODE_SWIGLU>(plan.shape, mt, grid, m->stream, a);
  else launch_shape<MODE_PARTIAL>(plan.shape, mt, grid, m->stream, a);
}
