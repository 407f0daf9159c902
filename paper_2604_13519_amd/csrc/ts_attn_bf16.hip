// Tree-masked grouped-query attention of the draft rows over the paged KV cache (bf16, gfx950).
//
// Every row of a sequence attends to all committed positions [0, P), to the root row and
// to its own ancestors among the tree rows, whose K/V were just written to slots
// P .. P+M-1 (paper App. A.1: one forward pass with a tree-structured mask).  The mask is a
// 64-bit ancestor set per row plus "root is always visible"; it only matters for the key
// blocks that overlap [P, P+M).
//
// Work split: grid = (unit of key blocks, KV head x head group), see attn_bf16_units.  A workgroup streams
// its key range once in blocks of 64 keys (4 pages) through double-buffered LDS and serves
// up to 4 query heads of the same KV head, one wave per head, all M rows of that head per
// wave - so each K/V byte is read from HBM once per KV head.
//
// The two products run in IEEE half precision (v_mfma_f32_16x16x32_f16): the cache stays bf16
// and its entries are widened to half while they are staged into LDS (exact in half's normal
// range), Q arrives in half, and the probabilities are rounded to half - 11 significant bits
// instead of bf16's 8 where it matters most for the logits.
//
// MFMA formulation, chosen so that no operand needs a transpose or a cross-lane shuffle:
//   S^T[key][query] = K . Q^T     A = K tile from LDS (16 keys x 32 dims per step)
//                                 B = Q fragments, resident in registers
//   lane l then holds query (l % 16) and 4 keys of each 16-key tile, and the exponentials
//   of two 16-key tiles pack straight into the B operand of
//   O^T[dim][query] += V^T . P^T  A = V^T tile from LDS.  V pages are stored transposed in
//                                 the cache ([head_dim][16 tokens]) exactly for this.
// Soft-max is the running-max / rescale recurrence in fp32 on scores in log2 units, with a
// whole-number reference (the rounded-up maximum, followed lazily: see kRefSlack) so that every
// rescale is an exact power of two;
// probabilities 2^(s - ref) are rounded to half for the second product and the row sum
// accumulates those rounded values (an extra MFMA against an all-ones operand, fp32 exact).
// Partial (max, sum, O) per split (unit of its sequence) are combined by k_attn_merge.
#include <algorithm>
#include <type_traits>

#include "ts_internal.h"
#include "ts_device_utils.h"

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

namespace {

constexpr int KB = TS_ATTN_KB;   // keys per block

struct AttnArgs {
  const bf16_t* Qb;          // [rows][Hq*HD], IEEE half bit patterns
  const uint64_t* row_anc;   // [rows]
  const AttnUnit* units;
  uint16_t* part_o;          // per row [Hq][splits][HD], IEEE half: the split's output divided by its row sum
  float* part_ml;            // per row [Hq][splits][2]
  int layer, Hq, Hkv, n_units, n_cu;
  float scale;               // 1/sqrt(head_dim) * log2(e): scores are kept in log2 units
};

// 8 cache entries bf16 -> half (exact in half's normal range), done while staging into LDS
__device__ __forceinline__ u32x4 to_half8(u32x4 v) {
  return u32x4{bf16x2_to_f16x2(v.x), bf16x2_to_f16x2(v.y), bf16x2_to_f16x2(v.z), bf16x2_to_f16x2(v.w)};
}

// The running soft-max reference of a row follows its maximum lazily: it moves only when the
// rounded-up maximum exceeds it by more than this many powers of two.  Probabilities then reach
// 2^kRefSlack at most (half holds 2^15), every rescale stays an exact power of two, and the O
// rescale - 32 multiplies per row tile whenever any row of the wave moves its reference - runs a
// few times per row instead of at most half blocks of a long context.
// The probabilities are taken against the reference as it stands, and only their largest is looked
// at, in packed halves over all row tiles of a wave (4 instructions per tile and 32 keys; the maximum
// of the scores over a row's lanes, taken before the exponentials, was 20): one above 2^kRefSlack
// sends the wave through the path that moves references.  A row without a reference yet has kNoRef,
// which makes any visible score overflow to +inf and any masked one 0.
// Measured (with the two 32-key halves unrolled): 65 rows x 8 heads per KV head x 32768 keys x 4
// sequences 514 -> 416 us, 33 rows x 16 sequences 114 -> 106 us, 38 rows x 23011 keys 43.3 -> 40.0 us,
// 65 rows x 8192 keys 27.0 -> 25.3 us.
// What the kernel waits for, as it is now, by leaving parts out (us in a trace: all, without the K and V^T fragment reads
// out of LDS, without staging the next block, without the exponentials, without all three): the first of these 324, 241,
// 261, 283, 217; 33 rows x 16 sequences 94, 57, 68, 81, 46; 38 rows x 23011 keys 36, 23, 28, 34, 21; 65 rows x 8192 keys 23.8,
// 20.7, 22.0, 22.0, 18.2.  Two thirds (half with three tiles in one wave) are the matrix instructions and what
// surrounds them; of the rest the reads cost most, by the time products wait for them and not by the LDS's rate, which is
// 15 - 22 % busy (counters).
constexpr float kRefSlack = 8.f, kRefLimit = 256.f, kNoRef = -1e30f;

union Pack8 {
  f16x8 v;
  u32x2 h[2];
  uint32_t u[4];
};

// MT0 row tiles for the waves of the first row split, MT1 (0 = no second split) for the second
template <int HD, int MT0, int MT1, int HB>
__global__ __launch_bounds__(64 * HB * (MT1 > 0 ? 2 : 1), (HB * (MT1 > 0 ? 2 : 1) <= 4) ? 2 : 1) void k_attn_bf16(AttnArgs a) {
  constexpr int RS = MT1 > 0 ? 2 : 1;
  constexpr int KSQ = HD / 32;            // k-steps of the score product
  constexpr int DT = HD / 16;             // 16-dim tiles of the output
  constexpr int NTHR = 64 * HB * RS;
  constexpr int VPP = 2 * HD;             // 16-byte vectors per K page (and per V page)
  constexpr int VTS = 32;                 // LDS row stride of the V^T of a 32-key half block, in tokens
  constexpr int VPG = 2 * VPP;            // 16-byte vectors per page, K then V
  constexpr int JP = (VPG + NTHR - 1) / NTHR;   // staged vectors per thread and page
  constexpr int NV = 4 * JP;              // staged vectors per thread and key block
  // Both arrays are read without bank conflicts: a 16-byte read is served in groups of 16 lanes that hold rows 0-3 and
  // 12-15 of one lane group and rows 4-11 of the next, which suits rows 32 bytes apart (K) and 64-byte rows of which
  // the second half of every 8 has its four vectors reversed (V^T).  Rows 16 bytes apart left half of the LDS cycles
  // to conflicts (counters, 65 rows x 4 sequences: 80 -> 46 M cycles; time 397 -> 395 us).
  __shared__ __attribute__((aligned(16))) bf16_t ks_[2][KB][HD + 16];
  // V^T of a half block (2 pages = 32 keys): per head-dim row, the keys in the order the second
  // MFMA wants them - lane group g holds tokens 4g..4g+3 of the first page, then of the second -
  // so that a lane's operand is one 16-byte read, and a thread that stages 8 tokens of both pages writes two.
  __shared__ __attribute__((aligned(16))) bf16_t vs_[2][2][HD][VTS];

  auto v_col = [](int d, int grp) { return (grp ^ (d >> 2 & 1) * 3) * 8; };   // where lane group grp's 8 tokens of row d are
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l15 = lane & 15, g4 = lane >> 4;
  const int G = a.Hq / a.Hkv;
  const int subs = G / HB;
  // Workgroups are dealt to the 8 XCDs round-robin by linear id.  The `subs` workgroups that
  // share one (unit, KV head) read the same K/V, so they are given ids that
  // differ by 8: same XCD, same L2, dispatched back to back.
  const int bid = blockIdx.x;
  const int jj = bid >> 3;
  const int rest = (jj / subs) * 8 + (bid & 7);
  if (rest >= a.n_units * a.Hkv) return;
  const int g = rest % a.Hkv;
  const int h = g * G + (jj % subs) * HB + (wave % HB);
  const int tile0 = (wave / HB) * MT0;    // first 16-row tile of this wave
  const AttnUnit sd = a.units[rest / a.Hkv];
  const int P = sd.P, M = sd.M, T = P + M;
  const int b0 = sd.b0, b1 = sd.b1, split = sd.split;

  const size_t page_elems = (size_t)a.Hkv * 16 * HD;
  const TS_GLOBAL bf16_t* kl = (const TS_GLOBAL bf16_t*)sd.k_pool + (size_t)a.layer * sd.n_pages * page_elems + (size_t)g * 16 * HD;
  const TS_GLOBAL bf16_t* vl = (const TS_GLOBAL bf16_t*)sd.v_pool + (size_t)a.layer * sd.n_pages * page_elems + (size_t)g * 16 * HD;
  const TS_GLOBAL int32_t* ptab = (const TS_GLOBAL int32_t*)sd.page_table;

  // Staging of one key block (4 pages).  A thread always fetches the same vector of a page
  // (K vectors for the first VPP thread ids, V vectors after), so its source pointer is fixed
  // and a page only adds a wave-uniform offset: one scalar page-table load and no vector
  // address arithmetic per page.  Pages past the last key are clamped to the last one: their
  // keys are masked in the scores and their V entries (finite cache contents) meet zero
  // probabilities.
  const TS_GLOBAL bf16_t* my_src[JP];
#pragma unroll
  for (int j = 0; j < JP; ++j) {
    const int w = min(tid + j * NTHR, VPG - 1);
    my_src[j] = (w < VPP) ? (kl + (size_t)w * 8) : (vl + (size_t)(w - VPP) * 8);
  }
  // Page-table entries of a key block: one 16-byte load (the table is padded by four entries of
  // page 0), fetched a block ahead of the data loads that need it and moved to scalar registers
  // there.  Pages past the last key hold finite cache contents.
  typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
  auto load_pt = [&](int blk) { return *reinterpret_cast<const TS_GLOBAL i32x4*>(ptab + blk * 4); };
  u32x4 stage[NV];
  auto load_block = [&](const i32x4& pt) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const size_t pg = (size_t)__builtin_amdgcn_readfirstlane(pt[p]) * page_elems;
#pragma unroll
      for (int j = 0; j < JP; ++j)
        if (VPG % NTHR == 0 || tid + j * NTHR < VPG) stage[p * JP + j] = *reinterpret_cast<const TS_GLOBAL u32x4*>(my_src[j] + pg);
    }
  };
  // always inline: with one head per workgroup (64 threads, eight vectors a thread and page) the compiler left it
  // a function, which kept `stage` in scratch memory and moved every live register around its calls.  17 rows x
  // 8192 keys, 16 KV heads of one query head: 64 us, 115 us with the unrolled halves around the call, 25 us inline.
  auto store_block = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < 4; p += 2)
#pragma unroll
      for (int j = 0; j < JP; ++j) {
        const int w = tid + j * NTHR;
        if (VPG % NTHR != 0 && w >= VPG) continue;
        const u32x4 v0 = to_half8(stage[p * JP + j]), v1 = to_half8(stage[(p + 1) * JP + j]);
        if (w < VPP) {
          const int t = w / (HD / 8), dv = w % (HD / 8);
          *reinterpret_cast<u32x4*>(&ks_[buf][p * 16 + t][dv * 8]) = v0;
          *reinterpret_cast<u32x4*>(&ks_[buf][p * 16 + 16 + t][dv * 8]) = v1;
        } else {
          // 8 tokens of one head-dim row from either page of the half block: two lane groups' operands
          const int d = (w - VPP) >> 1, g0 = (w - VPP) & 1;
          *reinterpret_cast<u32x4*>(&vs_[buf][p >> 1][d][v_col(d, 2 * g0)]) = u32x4{v0.x, v0.y, v1.x, v1.y};
          *reinterpret_cast<u32x4*>(&vs_[buf][p >> 1][d][v_col(d, 2 * g0 + 1)]) = u32x4{v0.z, v0.w, v1.z, v1.w};
        }
      }
  };

  // The main loop, compiled once per tile count: the waves of the second row split usually own
  // fewer tiles (5 tiles = 3 + 2) and run a copy without the empty one.  Both copies execute
  // the same barriers.
  auto body = [&](auto mt_c) {
    constexpr int MT = decltype(mt_c)::value;
    // LDS operand fragments requested ahead of the MFMAs that consume them; 0 leaves the order to
    // the compiler (which requests a pair, waits, multiplies).  The explicit pipeline pays in the
    // 8-wave variants with two row splits (65 rows: -4 % with 4 query heads per KV head, -9 %
    // with 8) and with two tiles a wave (17 rows: 11.4 -> 10.7 us); three tiles in 4 waves have no
    // registers left for it (33 rows: 107 -> 144 us), measured.
    constexpr int FD = HB == 4 && (RS == 2 || MT0 == 2) ? 3 : 0;
    // The two 32-key halves of a block are unrolled, except where one wave holds three tiles of 128 dims: there
    // the copies cost registers that the kernel does not have.  One head per KV head (245 accumulation registers
    // instead of 256 and 24 spilled): 33 rows x 8192 keys 37.9 -> 29.3 us, 33 rows x 8 sequences 88.8 -> 65.0 us; four
    // heads (8 instead of 9 spilled, 36 B of scratch a lane; none before the probabilities took the standing
    // reference, and that was the slower kernel): 33 rows x 8 sequences of 8192 99 -> 98 us, before 102 us.
    // Unrolled against rolled elsewhere: 8 heads, 65 rows x 32768 keys 98.5 and 102 us; 64 dims, 48 rows 15.6 and
    // 16.1 us, ingestion 64.7 and 66.9 us (three or two waves per SIMD fit there instead of four or three: the
    // launches of one sequence place one workgroup per CU, and the batches are faster all the same: 65 rows x
    // 8 sequences 68.5 rolled, 67.2 us).
    constexpr int K2U = HD == 128 && RS == 1 && MT == 3 ? 1 : 2;
  // resident query fragments and ancestor masks of this wave's head
  f16x8 qf[MT][KSQ];
  uint64_t anc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int lrow = (tile0 + mt) * 16 + l15;
    const bf16_t* qp = a.Qb + (size_t)(sd.row0 + lrow) * a.Hq * HD + (size_t)h * HD + g4 * 8;
#pragma unroll
    for (int ks = 0; ks < KSQ; ++ks) qf[mt][ks] = *reinterpret_cast<const f16x8*>(qp + ks * 32);
    anc[mt] = lrow < M ? a.row_anc[sd.row0 + lrow] : 0ull;
  }

  f32x4 o[DT][MT], l_run[MT];              // l_run: the row sum, the same in all four elements
  float m_run[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    m_run[mt] = kNoRef;
    l_run[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  Pack8 ones;
#pragma unroll
  for (int i = 0; i < 4; ++i) ones.u[i] = 0x3c003c00u;   // half 1.0 x 8

  i32x4 pt_next = i32x4{0, 0, 0, 0};
  if (b0 < b1) {
    load_block(load_pt(b0));
    if (b0 + 1 < b1) pt_next = load_pt(b0 + 1);
    store_block(0);
  }
  // Every load issued so far (query fragments, ancestor masks, first block) is complete past
  // this point.  Without the explicit wait the compiler has to assume, at the loop head, that
  // the query loads may still be in flight, and guards the first MFMA of every pass with a
  // wait for ALL vector loads - which would include the next block's K/V just requested.
  __builtin_amdgcn_s_waitcnt(0x0F70);       // vmcnt(0)
  __syncthreads();

  // One of the two waves of a SIMD goes first wherever both could issue, so that they do not run their matrix and
  // their soft-max phases at the same time.  With eight waves a workgroup fills a CU, and waves w and w + 4 share a SIMD:
  // the first row split goes first (it has as many row tiles as the second or one more).  With up to four waves two
  // workgroups share a CU (the dispatcher puts one on every CU before any second one), and the later one goes first.
  // 33 rows x 16 sequences 89.0 -> 86.1 us, x 8 69.8 -> 69.0, 65 rows x 4 sequences x 32768 keys 299 -> 295.6 us; single
  // sequences the same.  Two query heads per KV head, 65 rows (four waves), by the row split as with eight : by the
  // workgroup: one sequence of 16384 keys 29.8 : 28.2, x 16 96.0 : 92.0 us.
  if (HB * RS == 8 ? wave < HB : ((uint32_t)bid / (uint32_t)a.n_cu & 1) != 0) __builtin_amdgcn_s_setprio(1);
  for (int blk = b0; blk < b1; ++blk) {
    const int cur = (blk - b0) & 1;
    const bool more = blk + 1 < b1;
    if (more) {
      load_block(pt_next);
      if (blk + 2 < b1) pt_next = load_pt(blk + 2);
    }

    // Two sub-blocks of 32 keys (2 pages) each: scores, mask, running soft-max, P.V.
    const int key0 = blk * KB;
    const bool masked = key0 + KB > P;
#pragma unroll K2U
    for (int k2 = 0; k2 < 2; ++k2) {
      // ---- S^T = K . Q^T -----------------------------------------------------------
      // With FD > 0 the K fragments come from LDS through a short software pipeline, FD of them
      // in flight ahead of the MFMAs that consume them; the scheduling barriers keep the stages
      // in this order.
      f32x4 s[2][MT];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) s[kt][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
      constexpr int NKF = 2 * KSQ;
      static_assert(FD <= NKF && FD <= DT, "pipeline deeper than the fragment count");
      auto k_frag = [&](int i) {
        return *reinterpret_cast<const f16x8*>(&ks_[cur][(2 * k2 + i / KSQ) * 16 + l15][(i % KSQ) * 32 + g4 * 8]);
      };
      auto v_frag = [&](int dt) { return *reinterpret_cast<const f16x8*>(&vs_[cur][k2][dt * 16 + l15][v_col(l15, g4)]); };
      f16x8 kf[NKF];
#pragma unroll
      for (int i = 0; i < FD; ++i) kf[i] = k_frag(i);
      if (FD > 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NKF; ++i) {
        if (FD == 0) kf[i] = k_frag(i);
        else if (i + FD < NKF) kf[i + FD] = k_frag(i + FD);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          s[i / KSQ][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[i], qf[mt][i % KSQ], s[i / KSQ][mt], 0, 0, 0);
        if (FD > 0) __builtin_amdgcn_sched_barrier(0);
      }
      // the first V^T fragments of the second product travel while the soft-max is computed
      f16x8 vf[DT];
#pragma unroll
      for (int dt = 0; dt < FD; ++dt) vf[dt] = v_frag(dt);
      if (FD > 0) __builtin_amdgcn_sched_barrier(0);

      // ---- mask (only blocks that reach past the committed context) ----------------------
      if (masked) {
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int key = key0 + (2 * k2 + kt) * 16 + g4 * 4 + r;
            const int srow = key - P;                      // tree row of this key (if >= 0)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
              bool vis = key < T;
              if (vis && srow > 0) vis = (anc[mt] >> (srow - 1)) & 1ull;
              if (!vis) s[kt][mt][r] = -INFINITY;
            }
          }
      }

      // ---- probabilities against the reference as it stands (see kRefSlack); a.scale =
      //      log2(e)/sqrt(hd) folds into the exponent
      Pack8 pb[MT];
      f16x2 top = {(_Float16)0.f, (_Float16)0.f};
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          pb[mt].u[i] = pack_f16x2(__builtin_amdgcn_exp2f(fmaf(s[i >> 1][mt][(i & 1) * 2], a.scale, -m_run[mt])),
                                   __builtin_amdgcn_exp2f(fmaf(s[i >> 1][mt][(i & 1) * 2 + 1], a.scale, -m_run[mt])));
          top = __builtin_elementwise_max(top, __builtin_bit_cast(f16x2, pb[mt].u[i]));
        }
      }
      // some score of the wave beyond the slack: move the references of those rows and start over
      if (__builtin_amdgcn_ballot_w64(fmaxf((float)top[0], (float)top[1]) > kRefLimit) != 0ull) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          float mx = -INFINITY;
#pragma unroll
          for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s[kt][mt][r]);
          const float m_ceil = ceilf(max_over_lane_groups(mx) * a.scale);
          const float m_new = (m_ceil > m_run[mt] + kRefSlack) ? m_ceil : m_run[mt];
          const float alpha = __builtin_amdgcn_exp2f(m_run[mt] - m_new);
          m_run[mt] = m_new;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) o[dt][mt] *= alpha;
          l_run[mt] *= alpha;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            pb[mt].u[i] = pack_f16x2(__builtin_amdgcn_exp2f(fmaf(s[i >> 1][mt][(i & 1) * 2], a.scale, -m_new)),
                                     __builtin_amdgcn_exp2f(fmaf(s[i >> 1][mt][(i & 1) * 2 + 1], a.scale, -m_new)));
        }
      }

      // ---- O^T += V^T . P^T ; row sums of the rounded probabilities from an all-ones operand ---
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        l_run[mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones.v, pb[mt].v, l_run[mt], 0, 0, 0);
      if (FD > 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        if (FD == 0) vf[dt] = v_frag(dt);
        else if (dt + FD < DT) vf[dt + FD] = v_frag(dt + FD);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          o[dt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf[dt], pb[mt].v, o[dt][mt], 0, 0, 0);
        if (FD > 0) __builtin_amdgcn_sched_barrier(0);
      }
    }

    if (more) store_block(cur ^ 1);
    __syncthreads();
  }

  // ---- partial results of this split ---------------------------------------------------
  // (reference, row sum) in fp32 and the split's own normalised output O / l in half: a convex
  // combination of V rows, so it can neither overflow nor lose more than half's 11 bits, the
  // precision the probabilities already have.  Half the bytes of fp32 partials, which is what
  // bounds this epilogue and the merge kernel.
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const float l = l_run[mt][0];  // already the sum over all keys (MFMA reduces over the lane groups)
    const int lrow = (tile0 + mt) * 16 + l15;
    if (lrow < M) {
      const size_t base = (size_t)(sd.part0 + lrow * sd.splits) * a.Hq + h * sd.splits + split;
      if (g4 == 0) {
        a.part_ml[base * 2 + 0] = m_run[mt] == kNoRef ? -INFINITY : m_run[mt];
        a.part_ml[base * 2 + 1] = l;
      }
      const float inv = l > 0.f ? 1.0f / l : 0.f;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        *reinterpret_cast<u32x2*>(a.part_o + base * HD + dt * 16 + g4 * 4) =
            u32x2{pack_f16x2(o[dt][mt][0] * inv, o[dt][mt][1] * inv), pack_f16x2(o[dt][mt][2] * inv, o[dt][mt][3] * inv)};
    }
  }
  };
  if (RS == 1 || wave / HB == 0) body(std::integral_constant<int, MT0>{});
  else body(std::integral_constant<int, (MT1 > 0 ? MT1 : MT0)>{});
}

// Combine the splits: out = sum_s w_s (O_s / l_s) / sum_s w_s with w_s = 2^(m_s - m*) l_s, stored as IEEE half.
// Two kernels, by the number of slots and splits:
//  * many (row, head) slots and up to kMergeFew splits (batches and context ingestion): a thread owns
//    8 dims of a slot and requests its splits eight at a time; no LDS.  One workgroup per slot is mostly
//    the cost of dispatching workgroups there: 65536 slots x 3 - 4 splits 66 -> 21.5 us, 16896 x 7 22.0 -> 12.0 us,
//    10656 x 10 14.7 -> 9.1 us.  Few slots want the other kernel, which spreads them over more CUs: 208 slots x
//    12 splits cost a pass of three layers 14 us more here.  The line, one workgroup per slot against a thread
//    per 8 dims: 4160 slots x 3 / 8 / 9 / 12 / 16 splits 8.6 : 6.6, 9.3 : 7.8, 8.8 : 8.5, 10.0 : 11.2, 9.2 : 11.8 us (past
//    eight splits a thread needs a second round of loads); with 9 - 16 splits 4224 slots 9.6 : 10.2, 5120 10.7 : 10.5,
//    5280 10.9 : 10.6, 6336 12.1 : 10.9, 8448 13.6 : 11.0 us; 2304 slots x 8 7.2 : 8.1 us.
//  * otherwise (one sequence over many workgroups: few slots, many splits): one workgroup per slot; its
//    256 threads form 256/(HD/4) groups, group j takes splits j, j+groups, ... so that every partial of
//    the slot is requested at once (the kernel is a single round of memory latency plus the
//    transfer); the groups' sums are then added through LDS in a fixed order.
constexpr int kMergeFew = 16;
bool merge_few(int slots, int splits) { return splits <= kMergeFew && slots >= (splits <= 8 ? 4096 : 5120); }

__global__ __launch_bounds__(256) void k_attn_merge_few(const uint16_t* __restrict__ part_o, const float* __restrict__ part_ml,
                                                        f16_t* __restrict__ Ab, size_t a_plane, int slots, int Hq, int HD, int all_splits,
                                                        const int2* __restrict__ row_part,
                                                        unsigned long long* __restrict__ sat) {
  const int tps = HD / 8;                  // threads per slot
  const int slot = blockIdx.x * (256 / tps) + threadIdx.x / tps, d8 = threadIdx.x % tps;
  if (slot >= slots) return;
  size_t base = (size_t)slot * all_splits;
  int splits = all_splits;
  if (row_part) {
    const int2 p = row_part[slot / Hq];
    base = (size_t)p.x * Hq + slot % Hq * p.y;
    splits = p.y;
  }
  const float2* ml = reinterpret_cast<const float2*>(part_ml) + base;
  const uint4* po = reinterpret_cast<const uint4*>(part_o) + base * tps + d8;
  float num[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, den = 0.f, mstar = -INFINITY;
  float2 w[kMergeFew];
#pragma unroll
  for (int s = 0; s < kMergeFew; ++s) w[s] = s < splits ? ml[s] : make_float2(-INFINITY, 0.f);
#pragma unroll
  for (int h = 0; h < kMergeFew; h += 8) {
    if (h >= splits) break;
    uint4 o[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) o[s] = h + s < splits ? po[(size_t)(h + s) * tps] : make_uint4(0u, 0u, 0u, 0u);
    if (h == 0) {
#pragma unroll
      for (int s = 0; s < kMergeFew; ++s) mstar = fmaxf(mstar, w[s].x);
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if (w[h + s].x == -INFINITY) continue;
      const float f = exp2f(w[h + s].x - mstar) * w[h + s].y;   // whole-number references: an exact power of two
      den += f;
      const uint32_t u[4] = {o[s].x, o[s].y, o[s].z, o[s].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f16x2 v = __builtin_bit_cast(f16x2, u[i]);
        num[2 * i] += f * (float)v[0];
        num[2 * i + 1] += f * (float)v[1];
      }
    }
  }
  // the attention output feeds the O projection as a hi and a lo half
  f16_t* dst = Ab + (size_t)(slot / Hq) * act_ld(Hq * HD) + slot % Hq * HD + d8 * 8;
  st_act_planes4(dst, a_plane, num[0] / den, num[1] / den, num[2] / den, num[3] / den, sat);
  st_act_planes4(dst + 4, a_plane, num[4] / den, num[5] / den, num[6] / den, num[7] / den, sat);
}

constexpr int kMergeMaxSplits = 512;

// Bound by its launch and one round of latency, so also by what stands before its loads: the division of the threads
// into groups is a constant, and a pass without differing split counts (every single request) has an instance that does
// not ask for them.  65 rows x 8192 keys, us in a trace of 32 layers: 6.08 before a row had a count of its own, 6.50 with
// it and one instance for both, 5.95 now.
template <int HD, bool RAGGED>
__global__ __launch_bounds__(256) void k_attn_merge(const uint16_t* __restrict__ part_o, const float* __restrict__ part_ml,
                                                    f16_t* __restrict__ Ab, size_t a_plane, int Hq, int all_splits,
                                                    const int2* __restrict__ row_part,
                                                    unsigned long long* __restrict__ sat) {
  __shared__ float s_m[kMergeMaxSplits], s_l[kMergeMaxSplits];
  __shared__ float4 r_num[256];
  __shared__ float r_den[256];
  const int tid = threadIdx.x;
  constexpr int tpp = HD / 4;              // threads per group: four dims of the head each
  constexpr int groups = 256 / tpp;
  const int grp = tid / tpp, d4 = tid % tpp;
  const int row = blockIdx.y, head = blockIdx.x;
  size_t base = ((size_t)row * Hq + head) * all_splits;
  int splits = all_splits;
  if (RAGGED) {
    const int2 p = row_part[row];
    base = (size_t)p.x * Hq + head * p.y;
    splits = p.y;
  }
  const float2* ml = reinterpret_cast<const float2*>(part_ml);
  const uint2* po = reinterpret_cast<const uint2*>(part_o);     // 4 halves
  for (int sp = tid; sp < splits; sp += 256) {
    const float2 v = ml[base + sp];
    s_m[sp] = v.x;
    s_l[sp] = v.y;
  }
  uint2 o4[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int sp = grp + u * groups;
    o4[u] = sp < splits ? po[(base + sp) * tpp + d4] : make_uint2(0u, 0u);
  }
  __syncthreads();
  float mstar = -INFINITY;
  for (int sp = 0; sp < splits; ++sp) mstar = fmaxf(mstar, s_m[sp]);
  float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
  float den = 0.f;
  for (int s0 = 0; s0 < splits; s0 += 4 * groups) {
    if (s0 > 0) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int sp = s0 + grp + u * groups;
        o4[u] = sp < splits ? po[(base + sp) * tpp + d4] : make_uint2(0u, 0u);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int sp = s0 + grp + u * groups;
      if (sp < splits && s_m[sp] != -INFINITY) {
        const float w = exp2f(s_m[sp] - mstar) * s_l[sp];   // whole-number references: an exact power of two
        den += w;
        const ts_f16x2 lo2 = __builtin_bit_cast(ts_f16x2, o4[u].x), hi2 = __builtin_bit_cast(ts_f16x2, o4[u].y);
        num.x += w * (float)lo2[0]; num.y += w * (float)lo2[1]; num.z += w * (float)hi2[0]; num.w += w * (float)hi2[1];
      }
    }
  }
  r_num[tid] = num;
  r_den[tid] = den;
  __syncthreads();
  if (grp != 0) return;
  for (int k = 1; k < groups; ++k) {
    const float4 t = r_num[k * tpp + d4];
    num.x += t.x; num.y += t.y; num.z += t.z; num.w += t.w;
    den += r_den[k * tpp + d4];
  }
  // the attention output feeds the O projection as a hi and a lo half
  st_act_planes4(Ab + row * act_ld(Hq * HD) + head * HD + d4 * 4, a_plane, num.x / den, num.y / den, num.z / den, num.w / den, sat);
}

// Rows are covered by RS waves per head, MT tiles of 16 rows each: (tiles -> RS x MT)
// 1 -> 1, 2 -> 2, 3 -> 3, 4 -> 2+2, 5 -> 3+2.  Two row-splits put two waves on every
// SIMD (256 registers each) and let one wave's soft-max arithmetic overlap the other's MFMAs.
template <int HD, int HB>
void launch_hb(int tiles, dim3 grid, hipStream_t s, const AttnArgs& a) {
  switch (tiles) {
    case 1: hipLaunchKernelGGL((k_attn_bf16<HD, 1, 0, HB>), grid, dim3(64 * HB), 0, s, a); break;
    case 2: hipLaunchKernelGGL((k_attn_bf16<HD, 2, 0, HB>), grid, dim3(64 * HB), 0, s, a); break;
    case 3: hipLaunchKernelGGL((k_attn_bf16<HD, 3, 0, HB>), grid, dim3(64 * HB), 0, s, a); break;
    case 4: hipLaunchKernelGGL((k_attn_bf16<HD, 2, 2, HB>), grid, dim3(128 * HB), 0, s, a); break;
    default: hipLaunchKernelGGL((k_attn_bf16<HD, 3, 2, HB>), grid, dim3(128 * HB), 0, s, a); break;
  }
}

template <int HD>
void launch_hd(int hb, int tiles, dim3 grid, hipStream_t s, const AttnArgs& a) {
  if (hb == 4) launch_hb<HD, 4>(tiles, grid, s, a);
  else if (hb == 2) launch_hb<HD, 2>(tiles, grid, s, a);
  else launch_hb<HD, 1>(tiles, grid, s, a);
}

// query heads of one KV head served by a workgroup (one wave each per row split)
int heads_per_block(int G) { return G >= 4 ? 4 : (G >= 2 ? 2 : 1); }

}  // namespace

// How the key blocks of a pass are dealt to workgroups.  A unit is a run of key blocks of one sequence; every
// KV head (times the head groups that share its K/V) makes one workgroup of each unit.
// One sequence: as many equal units as cover the CUs once.
// Several: no unit is longer than L blocks, and L is the smallest with which the units make r workgroups a CU; r is
// the one with the least modelled time: r full rounds of units or, where lengths leave the rounds ragged, the mean
// load of a CU and half a unit; two workgroups that share a CU take one and a half times as long as one, 1.35 times
// with one row tile, whose workgroups mostly wait for their keys (us a launch with 1.5 there, with 1.35, and with the same number of
// splits for all: 4 x 4096 keys of 1 row 21.8, 17.8, 19.3, of 16 rows 22.7, 20.3, 21.0, 6 x 4096 .. 1024 of 1 row 21.2, 17.5, 19.9,
// 6 x 1000 12.5, 11.2, 11.8).  A sequence
// gets units in proportion to its length, so that every workgroup has nearly the same share and the last round is
// full.  Against one number of splits for all sequences, chosen so that the longest share is half of a CU's average
// load (8B shape unless noted; us a launch): 4 x 32768 keys of 65 rows, 8 heads 397 -> 306 (576 workgroups were 2.25
// rounds), 6 blocks of ingestion at 2000 39.0 -> 29.0, 8 x 4096 .. 2048 keys of 33 rows 49.5 -> 39.1, 16 x 8192 .. 2048
// 104 -> 96, 8 x 8192 .. 2700 of 65 rows, 64 dims 68.5 -> 45.5, 16 x 17 rows 57 -> 48.5, 4 x 33 rows 29.1 -> 27.0 (two
// workgroups a CU counted as one: 30.9).  A merge of differing split counts reads them first and gets that back
// from fewer partials (16.5 -> 11.3, 11.0 -> 8.8, 14.0 -> 12.1 us in the first, second and fourth of these).
// kUnitFixed: a workgroup's start and finish cost about as much as three blocks.
constexpr int kUnitFixed = 3, kBatchSplits = 16;
int attn_bf16_units(const ts_model* m, int n_seqs, const int* n_keys, int max_M, AttnUnit* units, int* seq_splits) {
  const int G = m->cfg.n_q_heads / m->cfg.n_kv_heads, hb = heads_per_block(G);
  const int per_unit = m->cfg.n_kv_heads * (G / hb);
  int n_units = 0;
  auto cut = [&](int s, int want) {
    const int n_blk = (n_keys[s] + KB - 1) / KB, len = (n_blk + want - 1) / want;
    seq_splits[s] = (n_blk + len - 1) / len;
    for (int i = 0; i < seq_splits[s]; ++i, ++n_units) {
      units[n_units].seq = s;
      units[n_units].split = i;
      units[n_units].b0 = i * len;
      units[n_units].b1 = std::min(n_blk, (i + 1) * len);
    }
  };
  if (n_seqs == 1) {
    const int n_blk = (n_keys[0] + KB - 1) / KB, wg_per_cu = hb <= 2 ? 2 : 1;
    cut(0, std::min(std::min((wg_per_cu * m->n_cu + per_unit - 1) / per_unit, n_blk), kMergeMaxSplits));
    return n_units;
  }
  int longest = 0;
  long total = 0;
  for (int s = 0; s < n_seqs; ++s) {
    longest = std::max(longest, (n_keys[s] + KB - 1) / KB);
    total += (n_keys[s] + KB - 1) / KB;
  }
  const bool pairs = hb * (max_M > 48 ? 2 : 1) <= 4;     // up to four waves: two workgroups share a CU
  const double two = max_M <= 16 ? 1.35 : 1.5;           // ... and take so much longer than one
  const int per_round = std::max(1, m->n_cu / per_unit);
  auto count = [&](int len) {
    long u = 0;
    for (int s = 0; s < n_seqs; ++s) u += ((n_keys[s] + KB - 1) / KB + len - 1) / len;
    return u;
  };
  // partial sums grow with the split count: 16 of a sequence at most, more only if those leave CUs empty
  const int cap = std::min(std::max(kBatchSplits, (per_round + n_seqs - 1) / n_seqs), kMergeMaxSplits);
  const int r0 = (n_seqs + per_round - 1) / per_round, least = (longest + cap - 1) / cap;
  double best = 1e300;
  int best_len = longest;
  for (int r = r0; r < r0 + 4; ++r) {
    int lo = least, hi = longest;                        // count(hi) = n_seqs <= r * per_round
    while (lo < hi) {
      const int mid = (lo + hi) / 2;
      if (count(mid) <= (long)r * per_round) hi = mid;
      else lo = mid + 1;
    }
    const double unit = lo + kUnitFixed, rounds = pairs ? r / 2 * two + r % 2 : r;
    const double mean = (double)(total + kUnitFixed * count(lo)) / per_round * (pairs && r > 1 ? two / 2 : 1.0);
    const double cost = std::min(rounds * unit, mean + 0.5 * unit);
    if (cost < best) { best = cost; best_len = lo; }
  }
  for (int s = 0; s < n_seqs; ++s) cut(s, ((n_keys[s] + KB - 1) / KB + best_len - 1) / best_len);
  return n_units;
}
int attn_bf16_max_units(const ts_model* m, int n_seqs) { return std::max(std::max(kMergeMaxSplits, kBatchSplits * n_seqs), m->n_cu + n_seqs); }

void launch_attn_bf16(ts_model* m, const RowMeta& rm, int n_units, int layer, int max_M) {
  ProfScope ps(m, "attn_bf16");
  const ts_model_config& c = m->cfg;
  AttnArgs a;
  a.Qb = (const bf16_t*)m->Qb; a.row_anc = rm.anc; a.units = m->unit_dev;
  a.part_o = m->attn_part_o; a.part_ml = m->attn_part_ml;
  a.layer = layer; a.Hq = c.n_q_heads; a.Hkv = c.n_kv_heads; a.n_units = n_units; a.n_cu = m->n_cu;
  a.scale = (float)(1.4426950408889634 / sqrt((double)c.head_dim));   // 1/sqrt(hd) * log2(e)
  const int G = c.n_q_heads / c.n_kv_heads;
  const int hb = heads_per_block(G);
  dim3 grid((n_units * c.n_kv_heads + 7) / 8 * 8 * (G / hb));
  const int mt = (max_M + 15) / 16;
  if (c.head_dim == 128) launch_hd<128>(hb, mt, grid, m->stream, a);
  else launch_hd<64>(hb, mt, grid, m->stream, a);
}

// splits: the most of any row; row_part: where each row's are (nullptr: all rows have `splits`)
void launch_attn_merge(ts_model* m, int R, int splits, const int2* row_part) {
  ProfScope ps(m, "attn_merge");
  const ts_model_config& c = m->cfg;
  const size_t plane = (size_t)(m->ws_rows + TS_MROWS_PER_BLOCK) * act_ld(m->q_dim);
  const int slots = R * c.n_q_heads;
  if (merge_few(slots, splits)) {
    const int per_wg = 256 / (c.head_dim / 8);
    hipLaunchKernelGGL(k_attn_merge_few, dim3((slots + per_wg - 1) / per_wg), dim3(256), 0, m->stream, m->attn_part_o, m->attn_part_ml,
                       (f16_t*)m->Ab, plane, slots, c.n_q_heads, c.head_dim, splits, row_part, m->sat_count);
    return;
  }
  // R fits the second grid dimension: beyond 65535 rows there are more slots than merge_few leaves to this kernel
  auto merge = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(c.n_q_heads, R), dim3(256), 0, m->stream, m->attn_part_o, m->attn_part_ml,
                       (f16_t*)m->Ab, plane, c.n_q_heads, splits, row_part, m->sat_count);
  };
  if (c.head_dim == 128) row_part ? merge(k_attn_merge<128, true>) : merge(k_attn_merge<128, false>);
  else row_part ? merge(k_attn_merge<64, true>) : merge(k_attn_merge<64, false>);
}
