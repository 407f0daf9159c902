// Many-row projection of a bf16 model for gfx950:  out[r][n] = sum_k X[r][k] * W[n][k]  for R > 80 rows
// (batched verification: the rows of all requests of a pass share one weight stream).
//
// With hundreds of rows the projection is no longer a weight stream but a matrix-core problem:
// every weight fragment is multiplied with R / 16 activation fragments.  The kernel keeps the
// arithmetic (IEEE half x half -> fp32) and the data path of the skinny kernel - weights
// pre-tiled in MFMA operand order and loaded straight from global memory into registers,
// activations shared through LDS chunks - and changes the tile a wave owns:
//  * 4 tiles of 16 output features per wave (the skinny kernel has 2).  One 1 KiB activation
//    fragment read from LDS then feeds 4 MFMAs, 64 matrix-pipe cycles against 8 LDS-pipe
//    cycles; with 8 waves the LDS pipe is half as busy as the four matrix pipes.
//  * 4 to 8 row tiles (up to 128 rows) per workgroup.  The rows of a pass are cut into equal
//    row blocks; the row blocks of one weight slab get consecutive places on the same XCD, so that
//    the slab comes from HBM once and from that XCD's L2 for the other blocks.
//  * 8 waves as CS column sets x KW k-waves (8x1: 512 columns, 4x2: 256, 2x4: 128) plus K
//    splits across workgroups; the planner takes the combination with the least modelled time.
//    The k-waves of a column set add their accumulators through LDS,
//    one row tile at a time, in the order kq = 0, 1, ...; K splits write fp32 partial sums
//    [split][row][col] for the next row-wise kernel (deterministic, no atomics).
//  * Activations go from memory into the LDS directly (no registers on the way), two to four chunks
//    deep, requested together with the weights of the same chunk and waited for by count; the first
//    LDS read of a chunk is issued before the barrier that ends the one before, and the requests go
//    out between the first products of a chunk, so that the matrix pipes do not stand still at a chunk's
//    edge.  Through registers (one chunk ahead with k-waves, two without) against this, us:
//    132 rows gate/up 108 -> 78, down 57 -> 44; 2048 rows gate/up 765 -> 710 (1.27 -> 1.36 PFLOP/s, both planes
//    counted), down 345 -> 327, QKV 173 -> 159; 528 rows gate/up 224 -> 193.  What is left: the matrix pipes are
//    busy 76 % of the cycles (528 rows gate/up, counters) of a clock that the power holds down: random operands that stay in
//    registers sustain 1.88 PFLOP/s here, zeros 2.37.
//  * gate/up variant (SWIGLU): gate and up tiles alternate, a wave holds two (gate, up) pairs
//    and the epilogue stores SiLU(gate) * up as half.
//  * lm_head variant (ARGMAX, no K split): the epilogue reduces each row's maximum over the workgroup's
//    columns and emits one (value, index) partial per row and column group.  A small head takes the shapes of
//    256 or 128 columns like any other projection (8192 columns, 528 rows 119 -> 70 us, 260 rows x 5120 146 -> 59 us).
#include "ts_internal.h"
#include "ts_device_utils.h"
#include <algorithm>
#include <type_traits>

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

struct RowsArgs {
  const f16_t* X;      // [2 planes][x_rows][act_ld(K)] IEEE half (x = hi + lo)
  size_t x_plane;      // elements between the planes
  size_t act_plane;    // SWIGLU: elements between the planes of act_out
  unsigned long long* sat;   // counts gated products beyond half's range
  int x_rows;          // rows allocated (reads are clamped to them)
  const f16_t* Wt;     // tiled weights, IEEE half
  float* out;          // [split][R][N] partial sums
  f16_t* act_out;      // SWIGLU: [2 planes][x_rows][act_ld(N/2)] IEEE half
  float* logits;       // ARGMAX: [R][N] or nullptr
  float* aval;         // ARGMAX: [R][amax_stride] partial maxima, one per column group
  int32_t* aidx;
  int amax_stride;
  int R, N, K;
  int kper;            // k elements per split
  int n_tiles;         // ceil(N / 16)
  int kt_count;        // K / 32
  size_t split_stride; // R * N
  int n_groups;        // column groups
  int n_units;         // column groups x K splits: one weight slab each
  int n_rblocks;       // row blocks
};

enum { MODE_PARTIAL = 0, MODE_ARGMAX = 1, MODE_SWIGLU = 2 };
constexpr int NT = 4;        // tiles of 16 output features per wave
constexpr int WAVES = 8;

// Ring slots: the activations of a chunk take MT * KW * 2 KiB of LDS each, its weights 16 registers.  The 4-row-tile
// kernels with one or two k-waves run two workgroups per CU and have half the registers and LDS.
constexpr int ring_depth(int MT, int KW) { return KW <= 2 ? (MT <= 4 ? 3 : 4) : MT <= 4 ? 4 : MT <= 6 ? 3 : 2; }

template <int MT, int CS, int KW, int MODE>
__global__ __launch_bounds__(64 * WAVES, MT <= 4 && KW <= 2 ? 4 : 2) void k_gemm_rows_bf16(RowsArgs a) {
  static_assert(CS * KW == WAVES, "8 waves");
  constexpr int KC = KW * 32;             // k elements per staged chunk: one k-step per wave
  constexpr int PL = TS_ACT_PLANES;       // an activation is the sum of a hi and a lo half
  constexpr int UPR = KC / 8;             // 16-byte vectors per row of a chunk
  constexpr int PPP = MT * 16 * UPR / 64; // 1 KiB pieces per plane of a chunk: one direct-to-LDS load of a wave each
  constexpr int XN = (PL * PPP + WAVES - 1) / WAVES;      // pieces a wave stages; the surplus repeats its last one
  constexpr size_t XBYTES = (size_t)PL * PPP * 1024;
  constexpr int RD = ring_depth(MT, KW);
  constexpr bool AHEAD = RD >= 4;
  constexpr int FD = 1, RQ = 2;           // fragments read ahead; the fragment behind whose products the requests go out
  static_assert(RD * XBYTES <= 160 * 1024, "the activation chunks fit the LDS");
  // One array per ring slot: the compiler then knows which loads a read of LDS has to wait for (all of them, if the
  // slots were parts of one array).  The first two later serve the k-wave reduction and the arg-max.
  __shared__ __attribute__((aligned(1024))) char xs0[XBYTES], xs1[XBYTES], xs2[RD > 2 ? XBYTES : 16], xs3[RD > 3 ? XBYTES : 16];
  auto slot = [&](auto i_c) -> char* {
    constexpr int I = decltype(i_c)::value;
    if constexpr (I == 0) return xs0;
    else if constexpr (I == 1) return xs1;
    else if constexpr (I == 2) return xs2;
    else return xs3;
  };

  // place: XCD = blockIdx.x % 8; each takes an equal, contiguous run of the (weight slab, row block)
  // pairs, so that the row blocks of a slab follow each other on one XCD (two at a run's ends).  Whole
  // slabs dealt round robin loaded the XCDs unevenly (12 slabs: 2 on four of them, 1 on the others), and
  // the planner paid for it with K splits: 2048 rows x 6144 columns 180.4 us and four partial sums to
  // re-read (20.4 instead of 36.2 us in k_rope_kv now), 178.4 us and one (170 us with 32-bit lane offsets, below).
  const int wgs = a.n_units * a.n_rblocks;
  const int place = (blockIdx.x & 7) * ((wgs + 7) / 8) + (blockIdx.x >> 3);
  if (place >= wgs) return;
  const int rb = place % a.n_rblocks, unit = place / a.n_rblocks;
  const int group = unit % a.n_groups, split = unit / a.n_groups;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l15 = lane & 15, g = lane >> 4;
  const int cs = wave / KW, kq = wave % KW;
  const int row0 = rb * (MT * 16);
  const int kbase0 = split * a.kper;
  const int n_chunks = a.kper / KC;

  const int cs_u = __builtin_amdgcn_readfirstlane(cs), kq_u = __builtin_amdgcn_readfirstlane(kq);
  const char* wbase[NT];
  int nt_idx[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    nt_idx[t] = (group * CS + cs_u) * NT + t;
    const int c = nt_idx[t] < a.n_tiles ? nt_idx[t] : a.n_tiles - 1;   // idle waves re-read a valid tile
    wbase[t] = reinterpret_cast<const char*>(a.Wt) + ((size_t)c * a.kt_count + kbase0 / 32 + kq_u) * 1024;
  }
  const uint32_t w_lane = lane * 16;
  // Staging: lane l of a piece brings the vector that belongs at l x 16 bytes of it.  A row's vectors stand permuted
  // (swz), so that the 16-byte reads below meet no bank twice: each is served in groups of 16 lanes that hold rows 0-3
  // and 12-15 of one lane group and rows 4-11 of the next.
  auto swz = [](int row) { return KC == 128 ? row & 15 : KC == 64 ? row >> 1 & 7 : (row >> 2 & 1) * 3; };
  // Rows past the last hold what an earlier pass left, or zeros: their outputs are not stored.  (The kernels of few rows
  // read one spare row of zeros in their place, which costs the matrix pipes less power; not tried here.)
  // Plane and row block are in the base: both can be past 4 GiB in the workspace of a very large batch; the lane
  // offset covers the 64 to 128 rows of a block
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const char* xbase = reinterpret_cast<const char*>(a.X) + ((size_t)row0 * act_ld(a.K) + kbase0) * 2;
  const size_t plane_bytes = a.x_plane * 2;
  int piece[XN];
  uint32_t x_off[XN];
#pragma unroll
  for (int p = 0; p < XN; ++p) {
    piece[p] = p * WAVES + wave_u;
    if (piece[p] >= PL * PPP) piece[p] -= WAVES;
    const int rl = piece[p] % PPP * (64 / UPR) + lane / UPR;
    x_off[p] = ((uint32_t)min(rl, a.x_rows - 1 - row0) * (uint32_t)act_ld(a.K) + ((lane % UPR) ^ swz(rl)) * 8) * 2;
  }

  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Pipeline.  Group c = activations and weights of chunk c, requested RD - 1 steps ahead.  A step waits until its
  // group - with four slots the next one too, so that its first fragment can be read early - has arrived, meets the
  // other waves (all have their pieces in LDS, and none still reads the slot of the chunk before), and between its
  // products requests group c + RD - 1 into that slot.  Loads in the loop are never predicated (the counts rely on
  // it): past the end they re-request the last chunk.
  // Measured: fragments 1, 2, 3 ahead 528 rows gate/up 193, 208, 208 us; requests after the third fragment against
  // right after the barrier 330 rows gate/up 132 : 134 us; the next group waited for with three slots too: 193 -> 285 us.
  // The empty asm statements keep the lane offsets 32 bits wide up to the load, which then adds them to the
  // uniform base itself; left alone the compiler hoists 64-bit lane addresses, a register pair per load, out of
  // the loop, and the largest tiles spill around them.
  f16x8 w[RD][NT];
  const int last_chunk = n_chunks - 1;
  auto request = [&](auto i_c, int chunk) {
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
    for (int t = 0; t < NT; ++t) w[I][t] = *reinterpret_cast<const f16x8*>(wbase[t] + (size_t)ch * (KW * 1024) + wl);
    __builtin_amdgcn_sched_barrier(0);
  };
  const uint32_t x_read = l15 * (KC * 2) + ((kq * 4 + g) ^ swz(l15)) * 16;
  auto frag = [&](auto i_c, int f) {        // fragment f of a slot: row tile f / PL, plane f % PL
    return *reinterpret_cast<const f16x8*>(slot(i_c) + f % PL * (PPP * 1024) + f / PL * (16 * KC * 2) + x_read);
  };
  f16x8 xa[FD + 1];
  // T < 0: a step of the loop.  T >= 0: step T of the rest, behind which no chunk is left to request: the groups in
  // flight get fewer, and no request may be made for nothing (its weights, which nothing uses, would be left out by the
  // compiler, and the counts would be wrong).
  auto step = [&](auto i_c, auto t_c, int c) {
    constexpr int I = decltype(i_c)::value, T = decltype(t_c)::value;
    constexpr int NF = MT * PL, LEFT = RD - 2 - AHEAD - (T < 0 ? 0 : T);     // later groups that may stay in flight
    wait_loads<(LEFT > 0 ? LEFT : 0) * (XN + NT)>();
    if constexpr (!AHEAD) {
#pragma unroll
      for (int f = 0; f < FD; ++f) xa[f] = frag(i_c, f);
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      if (f + FD < NF) xa[(f + FD) % (FD + 1)] = frag(i_c, f + FD);
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[f / PL][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[f % (FD + 1)], w[I][t], acc[f / PL][t], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (T < 0 && f == RQ) request(std::integral_constant<int, (I + RD - 1) % RD>{}, c + RD - 1);
    }
    if constexpr (AHEAD) {
#pragma unroll
      for (int f = 0; f < FD; ++f) xa[f] = frag(std::integral_constant<int, (I + 1) % RD>{}, f);
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2 % RD>;
  using I3 = std::integral_constant<int, 3 % RD>;
  using Loop = std::integral_constant<int, -1>;
  request(I0{}, 0);
  if constexpr (RD > 2) request(I1{}, 1);
  if constexpr (RD > 3) request(I2{}, 2);
  if constexpr (AHEAD) {
    wait_loads<(RD - 2) * (XN + NT)>();
#pragma unroll
    for (int f = 0; f < FD; ++f) xa[f] = frag(I0{}, f);
  }
  int c0 = 0;
  for (; c0 + RD <= n_chunks; c0 += RD) {
    step(I0{}, Loop{}, c0);
    step(I1{}, Loop{}, c0 + 1);
    if constexpr (RD > 2) step(I2{}, Loop{}, c0 + 2);
    if constexpr (RD > 3) step(I3{}, Loop{}, c0 + 3);
  }
  // the rest; a slot that it does not reach holds a request past the end
  auto rest = [&](auto i_c) {
    constexpr int I = decltype(i_c)::value;
    if (c0 + I < n_chunks) step(i_c, i_c, c0 + I);
    else
#pragma unroll
      for (int t = 0; t < NT; ++t) keep_loaded(w[I][t]);
  };
  rest(I0{});
  if constexpr (RD > 2) rest(I1{});
  if constexpr (RD > 3) rest(I2{});
  // nothing may still be on its way into the LDS when it is used otherwise or given back
  wait_loads<0>();

  // ARGMAX: best (value, column) of every row over the 64 columns of each column set
  __shared__ float rv[MODE == MODE_ARGMAX ? CS : 1][MODE == MODE_ARGMAX ? MT * 16 : 1];
  __shared__ int ri[MODE == MODE_ARGMAX ? CS : 1][MODE == MODE_ARGMAX ? MT * 16 : 1];
  // value of output (row tile mt, row r of the lane group, tile t) goes to memory
  auto emit = [&](int mt, int r, const float (&v)[NT]) {
    const int row = row0 + mt * 16 + g * 4 + r;
    if (MODE == MODE_ARGMAX) {                // in-lane over the 4 tiles, then over the 16 lanes of the row
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
      for (int o = 8; o > 0; o >>= 1) {
        const float ov = __shfl_xor(bv, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        amax_take(bv, bi, ov, oi);
      }
      if (l15 == 0) { rv[cs][row - row0] = bv; ri[cs][row - row0] = bi; }
      return;
    }
    if (row >= a.R) return;
    if (MODE == MODE_SWIGLU) {
#pragma unroll
      for (int t = 0; t < NT; t += 2) {       // tiles 2j / 2j+1 = gate / up of features 16j..
        if (nt_idx[t + 1] < a.n_tiles) {
          const int f = (nt_idx[t] >> 1) * 16 + l15;
          const float gv = v[t], uv = v[t + 1];
          st_act_planes(a.act_out + (size_t)row * act_ld(a.N / 2) + f, a.act_plane, gv / (1.0f + expf(-gv)) * uv, a.sat);
        }
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
    // one row tile at a time through LDS (the activation slots are free now; the first four waves use one, the others
    // the next, and a column set's k-waves are all in one half): every wave stores its 16 values per lane, then k-wave kq finishes the rows
    // r = kq, kq + KW, .. of the tile, adding in the order kq = 0, 1, ...
    static_assert(KW == 1 || XBYTES >= sizeof(float) * 16 * NT * 64, "the sums of four waves fit a slot");
    float* red = reinterpret_cast<float*>(wave < 4 ? xs0 : xs1);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) red[(((wave & 3) * 4 + r) * NT + t) * 64 + lane] = acc[mt][t][r];
      __syncthreads();
      for (int r = kq; r < 4; r += KW) {
        float v[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          float sum = 0.f;
#pragma unroll
          for (int k = 0; k < KW; ++k) sum += red[((((cs * KW + k) & 3) * 4 + r) * NT + t) * 64 + lane];
          v[t] = sum;
        }
        emit(mt, r, v);
      }
      __syncthreads();
    }
  }
  if (MODE == MODE_ARGMAX) {
    __syncthreads();
    if (tid < MT * 16 && row0 + tid < a.R) {
      float bv = rv[0][tid];
      int bi = ri[0][tid];
      for (int c = 1; c < CS; ++c) amax_take(bv, bi, rv[c][tid], ri[c][tid]);
      a.aval[(size_t)(row0 + tid) * a.amax_stride + group] = bv;
      a.aidx[(size_t)(row0 + tid) * a.amax_stride + group] = bi;
    }
  }
}

// compiled (CS, KW) pairs; a chunk is one k-step per k-wave
constexpr int kNumCfg = 3;
constexpr int kMinMT = 4, kMaxMT = 8;   // compiled row tiles per workgroup
const int kCfgCS[kNumCfg] = {8, 4, 2};
const int kCfgKW[kNumCfg] = {1, 2, 4};
const int kCfgKC[kNumCfg] = {32, 64, 128};

template <int MT, int MODE>
void launch_cfg(int cfg, dim3 grid, hipStream_t s, const RowsArgs& a) {
  const dim3 block(64 * WAVES);
  switch (cfg) {
    case 0: hipLaunchKernelGGL((k_gemm_rows_bf16<MT, 8, 1, MODE>), grid, block, 0, s, a); break;
    case 1: hipLaunchKernelGGL((k_gemm_rows_bf16<MT, 4, 2, MODE>), grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL((k_gemm_rows_bf16<MT, 2, 4, MODE>), grid, block, 0, s, a); break;
  }
}

template <int MODE>
void launch_mt(int mt, int cfg, dim3 grid, hipStream_t s, const RowsArgs& a) {
  switch (mt) {
    case 4: launch_cfg<4, MODE>(cfg, grid, s, a); break;
    case 5: launch_cfg<5, MODE>(cfg, grid, s, a); break;
    case 6: launch_cfg<6, MODE>(cfg, grid, s, a); break;
    case 7: launch_cfg<7, MODE>(cfg, grid, s, a); break;
    default: launch_cfg<8, MODE>(cfg, grid, s, a); break;
  }
}

}  // namespace

int gemm_rows_chunk(int cfg) { return kCfgKC[cfg]; }

// Row tiles per workgroup (4..8: the rows are cut into equal blocks), configuration and K splits with the least
// modelled time.  max_part_elems bounds splits x R x N.  K is a multiple of 128 (check_config), so every chunk length fits.
//   workgroup = k-steps of a wave x (kStepTile x row tiles + kStep) + kFix + kFixTile x row tiles   (start, finish, joining k-waves)
//   launch    = rounds over the CUs x workgroup, less 8 % of the share of CUs that stay empty (clock), + 0.6 us per million partial sums
// where the 4-row-tile kernels with one or two k-waves need half the registers and LDS of a CU: two workgroups share
// one and take 1.75 times as long as one.  The constants (all in us) are fitted to a sweep of every (row tiles, configuration,
// splits) of the 8B and 32B-class projections at 18 and 8 row counts of 96 to 2048, each with the change of the
// kernels that read the sums: the chosen ones together take 0.5 % more than the best ones, at most 7 %
// (400 rows x 8192 columns of the head).  The model before, one efficiency per configuration: 3.9 %, at most 25 %.
void gemm_rows_plan(const ts_model* m, int R, int N, int K, int mode, size_t max_part_elems, int* mt_out, int* cfg_out,
                    int* splits_out) {
  static const double kStepTile[kNumCfg] = {0.125, 0.113, 0.160}, kStep[kNumCfg] = {0.200, 0.300, 0.400};
  static const double kPairStep[kNumCfg] = {0.768, 0.820, 0.0};          // four row tiles, two workgroups a CU
  static const double kFix[kNumCfg] = {11.0, 2.0, 4.0}, kFixTile[kNumCfg] = {0.0, 1.6, 0.7};
  const int tiles = (R + 15) / 16;
  double best = 1e300;
  for (int mt = kMinMT; mt <= kMaxMT; ++mt) {
    const int n_rblocks = (tiles + mt - 1) / mt;
    if (mt > kMinMT && n_rblocks == (tiles + mt - 2) / (mt - 1)) continue;   // same blocks, more idle rows
    for (int cfg = 0; cfg < kNumCfg; ++cfg) {
      const int chunks = K / kCfgKC[cfg];
      const int cols = kCfgCS[cfg] * NT * 16;
      const int groups = (N + cols - 1) / cols;
      if (mode == MODE_ARGMAX && groups > m->amax_parts) continue;       // room for the partial maxima of a row
      for (int s = 1; s <= chunks && s <= 8; ++s) {
        if (chunks % s) continue;
        if (mode != MODE_PARTIAL && s > 1) break;
        if (s > 1 && (size_t)s * R * N > max_part_elems) break;
        const long wgs = (long)groups * s * n_rblocks, rounds = (wgs + m->n_cu - 1) / m->n_cu;
        const bool pairs = mt <= 4 && cfg <= 1;
        const double steps = (double)(K / s / kCfgKC[cfg]);
        const double wg = steps * (pairs ? kPairStep[cfg] : kStepTile[cfg] * mt + kStep[cfg]) + kFix[cfg] + kFixTile[cfg] * mt;
        double cost = wg * (pairs ? rounds / 2 * 1.75 + rounds % 2 : rounds);
        cost *= 1.0 - 0.08 * (1.0 - (double)wgs / (double)(rounds * m->n_cu));
        if (s > 1) cost += 0.6e-6 * s * R * (double)N;
        if (cost < best) { best = cost; *mt_out = mt; *cfg_out = cfg; *splits_out = s; }
      }
    }
  }
}

void launch_gemm_rows_bf16(ts_model* m, const f16_t* X, const f16_t* Wt, float* out, int R, int N, int K, int mt, int cfg,
                           int splits, int mode, f16_t* act_out, float* logits) {
  RowsArgs a;
  a.x_rows = m->ws_rows + TS_MROWS_PER_BLOCK;
  a.X = X; a.Wt = Wt; a.out = out;
  a.x_plane = (size_t)a.x_rows * act_ld(K);
  a.act_plane = (size_t)a.x_rows * act_ld(N / 2);
  a.act_out = act_out;
  a.sat = m->sat_count;
  a.logits = logits; a.aval = m->amax_val; a.aidx = m->amax_idx; a.amax_stride = m->amax_parts;
  a.R = R; a.N = N; a.K = K;
  if (mode != MODE_PARTIAL) splits = 1;
  a.kper = K / splits;
  a.n_tiles = (N + 15) / 16;
  a.kt_count = K / 32;
  a.split_stride = (size_t)R * N;
  const int cols = kCfgCS[cfg] * NT * 16;
  a.n_groups = (N + cols - 1) / cols;
  a.n_units = a.n_groups * splits;
  a.n_rblocks = ((R + 15) / 16 + mt - 1) / mt;
  dim3 grid((unsigned)(a.n_units * a.n_rblocks + 7) / 8 * 8);
  if (mode == MODE_ARGMAX) m->amax_used = a.n_groups;       // partials the combine kernel has to look at
  if (mode == MODE_SWIGLU) launch_mt<MODE_SWIGLU>(mt, cfg, grid, m->stream, a);
  else if (mode == MODE_ARGMAX) launch_mt<MODE_ARGMAX>(mt, cfg, grid, m->stream, a);
  else launch_mt<MODE_PARTIAL>(mt, cfg, grid, m->stream, a);
}
