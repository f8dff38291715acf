// Split-key attention on the matrix cores: bf16 storage with few current tokens, and fp32 storage (defined in
// attend_split.hip).
#pragma once
#include "esa_common.h"
#include "keyspace.h"

namespace esa {

bool attend_split_supported(int l_c, int h, int h_kv, int d, int dtype, int batch);
size_t attend_split_workspace_bytes(int l_c, int h, int h_kv, int d, int dtype, int batch);

struct SplitCall {
  int l_c, h, h_kv, d, dtype, batch;
  float scale;
  const void *k_sel, *v_sel;      // gathered rows (null: none, or an index list)
  int64_t sel_bs;
  void* out;
  int64_t out_bs;
  float* lse;
  void* ws;
  size_t ws_bytes;
  const void* turns = nullptr;    // not null: view a's keys are un-encoded and turned from position 0 on, by this table (kRopeTurns)
};
// Whether the kernel turns the n_keys local keys itself: bf16, all rows in one workgroup, which then reads each key once.
bool attend_split_turns_keys(int l_c, int h, int h_kv, int d, int dtype, int batch, int64_t n_keys);
// The slice counts and slots of the views are filled in by the launch.
// One call over the whole key sequence (one view), or over Section 3.2's two parts (view a: the local keys, b: the
// initial and selected ones; b may have no keys).
int launch_attend_split(const SplitCall& c, KeyView a, const KeyView* b, hipStream_t st);
// The two-call form: the early keys' partial results only; then the late keys (may be none) and the merge of both.
// early_keys: keys of the early part for the last current token, the same value in both calls.
int launch_attend_split_early(const SplitCall& c, KeyView early, int64_t early_keys, hipStream_t st);
int launch_attend_split_late(const SplitCall& c, KeyView late, int64_t late_keys, int64_t early_keys, hipStream_t st);

}  // namespace esa
