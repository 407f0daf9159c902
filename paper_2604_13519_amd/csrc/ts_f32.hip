// fp32 compute path (fp32 models: small decoders, a few rows per pass): projections and attention.
//
// At these sizes (weights of a projection about 1 MB, a pass of a few rows) nothing is bound by
// bandwidth or arithmetic: a launch costs one or two round trips through memory plus whatever it
// serialises.  Both kernels are therefore shaped to have every load of a workgroup's share in
// flight at once: K (or the keys) are spread over the waves of a workgroup and joined through LDS.
#include "ts_internal.h"
#include "ts_device_utils.h"

typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------
// out[R][N] = X[R][K] . W[N][K]^T on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32, fp32
// products and sums).  A workgroup owns MT x 16 rows and CT x 16 columns; its 8 waves take the
// 16-wide k chunks round robin.  A lane loads four consecutive k of one row (X) and of one column
// (W) - 16 bytes - and the four matrix instructions of a chunk take element e of both, so lane
// group g supplies k = 4g + e: a permutation of the chunk's k, the same on both sides.  No LDS
// until the end, when the waves' sums are added in the order wave 0, 1, ...
// SWIGLU (CT = 2): the fused gate/up weights alternate 16-row tiles, so the two column tiles are
// gate and up of the same features and the gated product is stored instead of the sums.
// Measured on the 2-layer 256-wide fp32 model (9 rows), against 16 x 64 tiles walking K alone through
// LDS: K = 1024 101 -> 5.3 us, K = 256 24 - 30 -> 4.0 us per launch.
// ---------------------------------------------------------------------------------
constexpr int kF32Waves = 8;

template <int MT, int CT, bool SWIGLU>
__global__ __launch_bounds__(64 * kF32Waves) void k_gemm_f32(const float* __restrict__ X, const float* __restrict__ W,
                                                              float* __restrict__ out, int R, int N, int K) {
  static_assert(!SWIGLU || CT == 2, "gate and up tiles alternate");
  constexpr int U = MT >= 4 ? 2 : 4;                 // chunks in flight per wave
  constexpr int NC = CT * 16;
  __shared__ float red[kF32Waves][MT * 16][NC + 4];     // +4: the four lane groups write 16 banks apart
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l15 = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * NC, m0 = blockIdx.y * (MT * 16);
  const int n_chunks = (K + 15) / 16;
  const float* xp[MT];
  const float* wp[CT];
#pragma unroll
  for (int m = 0; m < MT; ++m) xp[m] = X + (size_t)min(m0 + m * 16 + l15, R - 1) * K;    // rows past the end repeat the last
#pragma unroll
  for (int t = 0; t < CT; ++t) wp[t] = W + (size_t)min(n0 + t * 16 + l15, N - 1) * K;
  f32x4 acc[MT][CT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c = wave; c < n_chunks; c += kF32Waves * U) {
    f32x4 a[U][MT], b[U][CT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (c + u * kF32Waves) * 16 + g * 4;
      const bool in = k < K;                          // K is a multiple of 4: a lane's four k are all in or all out
      const int kc = in ? k : 0;
#pragma unroll
      for (int t = 0; t < CT; ++t) b[u][t] = *reinterpret_cast<const f32x4*>(wp[t] + kc);
#pragma unroll
      for (int m = 0; m < MT; ++m) a[u][m] = *reinterpret_cast<const f32x4*>(xp[m] + kc);
      if (!in) {                                      // both sides: 0 x inf would not vanish
#pragma unroll
        for (int t = 0; t < CT; ++t) b[u][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < MT; ++m) a[u][m] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int t = 0; t < CT; ++t)
            acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][m][e], b[u][t][e], acc[m][t], 0, 0, 0);
  }
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][m * 16 + g * 4 + r][t * 16 + l15] = acc[m][t][r];
  __syncthreads();
  auto total = [&](int row, int col) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) s += red[w][row][col];
    return s;
  };
  if (SWIGLU) {
    for (int i = tid; i < MT * 16 * 16; i += 64 * kF32Waves) {
      const int row = i / 16, col = i % 16;
      if (m0 + row < R && n0 + 16 + col < N) {
        const float gv = total(row, col), uv = total(row, 16 + col);
        out[(size_t)(m0 + row) * (N / 2) + blockIdx.x * 16 + col] = gv / (1.0f + expf(-gv)) * uv;
      }
    }
  } else {
    for (int i = tid; i < MT * 16 * NC; i += 64 * kF32Waves) {
      const int row = i / NC, col = i % NC;
      if (m0 + row < R && n0 + col < N) out[(size_t)(m0 + row) * N + n0 + col] = total(row, col);
    }
  }
}

// Row tiles per workgroup: all rows of a small pass in one workgroup (gate/up: up to 32 rows, whose two
// column tiles need twice the LDS; else up to 64), so that each weight is read once; larger passes
// (context ingestion) take blocks of that many rows.  One column tile per workgroup - 16 columns -
// keeps the narrow projections (256 columns: 16 workgroups) spread out.
void launch_gemm_f32(ts_model* m, const float* X, const float* W, float* out, int M, int N, int K, bool swiglu) {
  ProfScope ps(m, "gemm_f32");
  const int mt = M <= 16 ? 1 : (M <= 32 || swiglu ? 2 : 4);
  const dim3 block(64 * kF32Waves), grid((N + (swiglu ? 31 : 15)) / (swiglu ? 32 : 16), (M + mt * 16 - 1) / (mt * 16));
  if (swiglu) {
    if (mt == 1) hipLaunchKernelGGL((k_gemm_f32<1, 2, true>), grid, block, 0, m->stream, X, W, out, M, N, K);
    else hipLaunchKernelGGL((k_gemm_f32<2, 2, true>), grid, block, 0, m->stream, X, W, out, M, N, K);
  } else {
    if (mt == 1) hipLaunchKernelGGL((k_gemm_f32<1, 1, false>), grid, block, 0, m->stream, X, W, out, M, N, K);
    else if (mt == 2) hipLaunchKernelGGL((k_gemm_f32<2, 1, false>), grid, block, 0, m->stream, X, W, out, M, N, K);
    else hipLaunchKernelGGL((k_gemm_f32<4, 1, false>), grid, block, 0, m->stream, X, W, out, M, N, K);
  }
}

// ---------------------------------------------------------------------------------
// Tree-masked attention, fp32: one workgroup of 16 waves per (row, query head).  Key j < P is
// context (visible); key P + s is tree row s, visible iff s = 0 (root) or bit s-1 of the row's
// ancestor mask is set.  The row's scores live in LDS, and so does the page table: every K and V
// address is then known without a dependent load.
//  * scores: hd/4 lanes share a key, 16 bytes each (a K page row is contiguous), four keys per
//    lane group in flight;
//  * P.V: four lanes share a head dim, 16 bytes (4 tokens of the transposed V page) each; the
//    workgroup walks 4096 / (4 hd) pages at once.
// Bound by the latency of its few dependent steps; 45 -> 12.5 us at 9 rows x 4 heads x 521 keys
// (one thread per key walking hd alone before).
// ---------------------------------------------------------------------------------
constexpr int kAttnThreads = 1024;
size_t attn_f32_max_keys() { return 15000; }

__global__ __launch_bounds__(kAttnThreads) void k_attn_f32(const float* __restrict__ Qb, float* __restrict__ Ab,
                                                           const int32_t* __restrict__ row_seq, const uint64_t* __restrict__ row_anc,
                                                           const SeqDesc* __restrict__ seqs, int layer, int Hq, int Hkv, int hd,
                                                           float scale) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  __shared__ float red[kAttnThreads / 64];
  const int r = blockIdx.x, h = blockIdx.y, g = h / (Hq / Hkv), tid = threadIdx.x;
  const SeqDesc sd = seqs[row_seq[r]];
  const uint64_t anc = row_anc[r];
  const int T = sd.P + sd.M, n_pg = (T + 15) / 16;
  float* sc = smem;                       // [16 n_pg]: scores, then probabilities (0 past the last key)
  float* acc = sc + 16 * n_pg;            // [kAttnThreads / 4]
  int32_t* pt = reinterpret_cast<int32_t*>(acc + kAttnThreads / 4);    // [n_pg]
  const size_t page_elems = (size_t)Hkv * 16 * hd;
  const float* kl = (const float*)sd.k_pool + (size_t)layer * sd.n_pages * page_elems + (size_t)g * 16 * hd;
  const float* vl = (const float*)sd.v_pool + (size_t)layer * sd.n_pages * page_elems + (size_t)g * 16 * hd;
  for (int i = tid; i < n_pg; i += kAttnThreads) pt[i] = sd.page_table[i];
  const int lpk = hd / 4;                 // lanes per key (2 .. 32)
  const int sub = tid % lpk, kslot = tid / lpk, kstep = kAttnThreads / lpk;
  const float4 q = *reinterpret_cast<const float4*>(Qb + (size_t)r * Hq * hd + (size_t)h * hd + sub * 4);
  __syncthreads();
  float mx = -INFINITY;
  for (int j0 = kslot; j0 < 16 * n_pg; j0 += 4 * kstep) {
    float4 kv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = min(j0 + u * kstep, T - 1);
      kv[u] = *reinterpret_cast<const float4*>(kl + (size_t)pt[j >> 4] * page_elems + (size_t)(j & 15) * hd + sub * 4);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = j0 + u * kstep;
      float a = fmaf(q.x, kv[u].x, fmaf(q.y, kv[u].y, fmaf(q.z, kv[u].z, q.w * kv[u].w)));
      for (int o = lpk / 2; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
      const int s = j - sd.P;
      const bool vis = j < T && (s <= 0 || ((anc >> (s - 1)) & 1ull));
      const float v = vis ? a * scale : -INFINITY;
      if (sub == 0 && j < 16 * n_pg) sc[j] = v;
      mx = fmaxf(mx, v);
    }
  }
  mx = wave_max(mx);
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kAttnThreads / 64; ++w) mx = fmaxf(mx, red[w]);
  __syncthreads();
  float sum = 0.f;
  for (int j = tid; j < 16 * n_pg; j += kAttnThreads) {
    const float p = expf(sc[j] - mx);
    sc[j] = p;
    sum += p;
  }
  sum = wave_sum(sum);
  if ((tid & 63) == 0) red[tid >> 6] = sum;
  __syncthreads();
  sum = 0.f;
#pragma unroll
  for (int w = 0; w < kAttnThreads / 64; ++w) sum += red[w];
  const int tpp = 4 * hd;                 // threads per page
  const int parts = kAttnThreads / tpp, part = tid / tpp, dd = (tid % tpp) / 4, t4 = (tid & 3) * 4;
  float a = 0.f;
  for (int p0 = part; p0 < n_pg; p0 += 4 * parts) {
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v[u] = *reinterpret_cast<const float4*>(vl + (size_t)pt[min(p0 + u * parts, n_pg - 1)] * page_elems + (size_t)dd * 16 + t4);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int pg = p0 + u * parts;
      if (pg < n_pg) {
        const float4 p = *reinterpret_cast<const float4*>(sc + pg * 16 + t4);
        // slots that no visible key occupies never reach the sum, whatever they hold
        a = fmaf(p.x, p.x != 0.f ? v[u].x : 0.f, a);
        a = fmaf(p.y, p.y != 0.f ? v[u].y : 0.f, a);
        a = fmaf(p.z, p.z != 0.f ? v[u].z : 0.f, a);
        a = fmaf(p.w, p.w != 0.f ? v[u].w : 0.f, a);
      }
    }
  }
  a += __shfl_xor(a, 1, 64);
  a += __shfl_xor(a, 2, 64);
  if ((tid & 3) == 0) acc[part * hd + dd] = a;
  __syncthreads();
  if (tid < hd) {
    float o = 0.f;
    for (int p = 0; p < parts; ++p) o += acc[p * hd + tid];
    Ab[(size_t)r * Hq * hd + (size_t)h * hd + tid] = o / sum;
  }
}

void launch_attn_f32(ts_model* m, const RowMeta& rm, int R, int, int layer, int max_keys) {
  ProfScope ps(m, "attn_f32");
  const ts_model_config& c = m->cfg;
  const int n_pg = (max_keys + 15) / 16;
  const size_t shmem = (size_t)(16 * n_pg + kAttnThreads / 4 + n_pg) * sizeof(float);
  hipLaunchKernelGGL(k_attn_f32, dim3(R, c.n_q_heads), dim3(kAttnThreads), shmem, m->stream, (const float*)m->Qb, (float*)m->Ab,
                     rm.seq, rm.anc, m->seq_dev, layer, c.n_q_heads, c.n_kv_heads, c.head_dim, 1.0f / sqrtf((float)c.head_dim));
}
