// The tests' door to the planners and to single projection launches of libtoolspec_hip.so: a C entry that fills in the
// part of a model which a launch reads, so that a test can run every compiled variant, not only those a planner picks
// for the models it has.  No kernel of its own; links against the library.
#include "../../paper_2604_13519_amd/csrc/ts_internal.h"

extern "C" {

// Plan of a projection (id: shape of the skinny kernels, or 100 + 4 x row tiles + configuration of the many-row one).
void hook_plan(int n_cu, int R, int N, int K, int mode, long part_elems, int amax_parts, int* id, int* splits) {
  ts_model m{};
  m.n_cu = n_cu;
  m.part_elems = (size_t)part_elems;
  m.amax_parts = amax_parts;
  const GemmPlan p = gemm_bf16_plan(&m, R, N, K, mode);
  *id = p.shape;
  *splits = p.splits;
}

int hook_cols_per_group(int id) { return gemm_bf16_cols_per_group(id); }
int hook_chunk(int id) { return gemm_bf16_chunk(id); }

// One projection by the given plan (device pointers; the planes of X and of act hold ws_rows + TS_MROWS_PER_BLOCK rows).
// groups: partials per row that an arg-max launch wrote.
int hook_project(const uint16_t* X, const uint16_t* Wt, float* out, uint16_t* act, float* logits, float* aval, int32_t* aidx,
                 unsigned long long* sat, int ws_rows, int amax_parts, int R, int N, int K, int id, int splits, int mode, int* groups) {
  ts_model m{};
  m.ws_rows = ws_rows;
  m.amax_val = aval; m.amax_idx = aidx; m.amax_parts = amax_parts;
  m.sat_count = sat;
  launch_gemm_bf16(&m, X, Wt, out, R, N, K, GemmPlan{id, splits}, mode, logits, act);
  *groups = m.amax_used;
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? (int)e : (int)hipStreamSynchronize(nullptr);
}

int hook_max_units(int n_cu, int n_seqs) {
  ts_model m{};
  m.n_cu = n_cu;
  return attn_bf16_max_units(&m, n_seqs);
}

// Attention units of a pass: per unit (sequence, split, first block, last block + 1), and the splits of every sequence.
int hook_units(int n_cu, int hq, int hkv, int n_seqs, const int* n_keys, int max_M, int* units, int* splits) {
  ts_model m{};
  m.n_cu = n_cu;
  m.cfg.n_q_heads = hq;
  m.cfg.n_kv_heads = hkv;
  std::vector<AttnUnit> u(attn_bf16_max_units(&m, n_seqs));
  const int n = attn_bf16_units(&m, n_seqs, n_keys, max_M, u.data(), splits);
  for (int i = 0; i < n; ++i) {
    units[4 * i] = u[i].seq; units[4 * i + 1] = u[i].split; units[4 * i + 2] = u[i].b0; units[4 * i + 3] = u[i].b1;
  }
  return n;
}

}  // extern "C"
