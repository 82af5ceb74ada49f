// A step of one-row groups run by one kernel: the table the kernel walks, and its launcher (chain.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <functional>
#include <vector>

#include "launch.hpp"

namespace sod2 {

enum ChainKind { CHAIN_GATHER = 0, CHAIN_GEMV, CHAIN_ATTN };
constexpr int CHAIN_MAX_STEPS = 144, CHAIN_MAX_EXT = 8, CHAIN_MAX_K = 4096, CHAIN_MAX_WG = 256;
constexpr int CHAIN_KEYS = 128;      // keys of one attention part

struct alignas(16) ChainStep {
  const void* w;                     // table / weights / cached keys
  const void* bias;                  // second table / bias / cached values
  const void* gamma; const void* beta;
  long long table_rows, table2_rows;
  int kind, n, k, ldw;               // n: results (attention: heads); ldw: elements between rows of w
  int rpw, seg_shift;                // rows per workgroup; log2 of the number of k segments of 512
  int src, res;                      // phases whose results are the input row and the residual, -1 none
  int act1, act2;
  float scale, eps;
  int out_ext, arg_ext, arg_i32;     // caller buffers the row / its arg-max go to, -1 none
  int idx_ext, idx_i32, idx2_ext, idx2_i32;
  int q_off, k_off, v_off;           // attention: where the query, new key and new value start in the row of src
  int lk_rel;                        // attention: keys relative to the launch's count
};

struct Chain {
  std::vector<ChainStep> steps;
  int workgroups = 0, n_ext = 0, lk0 = 0;
  int arrive_us = -1, polls = -1;      // limits of the waits between its workgroups, -1: the kernel's own
};

// The special stream handles besides NULL stay with the launches group by group, which ask the runtime nothing about a
// stream: not every runtime answers for them.
inline bool chain_takes(hipStream_t s) { return s != hipStreamLegacy && s != hipStreamPerThread; }
int chain_cus();
int chain_workgroups(hipStream_t s);
bool chain_build(const std::vector<Launch>& launches, int n_in, int n_out, const std::function<void*(const Ref&)>& at, int n_cu, int lk_grows,
                 Chain* out);
bool chain_fits(const Chain& c, void* const* ext);
void chain_launch(const Chain& c, void* const* ext, int lk, hipStream_t s);

}  // namespace sod2
