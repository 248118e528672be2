// Accepted-path commit (the step after verification): for every tree, the
// output of Def. def2 laid out for the next decoding cycle: the node indices
// of the accepted chain X^tau after the root, from the root down (the drafted
// positions whose cache entries are kept), and their tokens followed by Y.
#include <hip/hip_runtime.h>

#include "tv.h"
#include "tv_launch.h"

namespace {

// One wavefront per tree, bound by latency: a few hundred bytes a tree, read
// in one round of loads (links, status, accepted node and bonus token), then
// the chain is found in LDS by walking from the accepted node to the root
// (each step to a smaller index, so at most num_nodes steps) and its tokens
// are gathered and everything is written by all lanes; entries past the chain
// are -1. (One thread per tree, each step a
// load of its own, took 7.5 us for 64 trees against 4.8 us, 4.2 of which any kernel takes.)
constexpr int kWaves = 4;

__global__ void __launch_bounds__(64 * kWaves) commit_kernel(tv::CommitArgs a) {
  __shared__ int16_t link[kWaves][TV_MAX_NODES];   // parents, -1 where not smaller than the node
  __shared__ int16_t chain[kWaves][TV_MAX_NODES];  // from the accepted node up
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = static_cast<int>(blockIdx.x) * kWaves + wave;
  const bool live = b < a.batch;
  const int n1 = a.num_nodes, L = a.max_len;
  const size_t tree = static_cast<size_t>(live ? b : 0);
  const int status = a.status[tree], acc = a.accepted_node[tree], bonus = a.bonus_token[tree];
  for (int i = lane; i < n1; i += 64) {
    const int p = a.parents[tree * n1 + i];
    link[wave][i] = static_cast<int16_t>(p >= 0 && p < i ? p : -1);
  }
  __syncthreads();
  // length of the output, or the code of a tree that has none
  int depth = 0, len = 0;
  if (status == TV_TREE_OK) {
    bool bad = acc < 0 || acc >= n1;
    for (int x = acc; !bad && x > 0; ++depth) {
      if (lane == 0) chain[wave][depth] = static_cast<int16_t>(x);
      x = link[wave][x];
      bad = x < 0;
    }
    len = bad ? TV_COMMIT_INCONSISTENT : depth > L ? TV_COMMIT_OVERFLOW : depth + 1;
  }
  __syncthreads();
  if (!live) return;
  int32_t* pn = a.path_nodes + tree * L;
  int32_t* pt = a.path_tokens + tree * (L + 1);
  for (int i = lane; i <= L; i += 64) {
    const bool in = len > 0 && i < depth;
    const int x = in ? chain[wave][depth - 1 - i] : -1;
    if (i < L) pn[i] = x;
    pt[i] = in ? a.tokens[tree * n1 + x] : len > 0 && i == depth ? bonus : -1;
  }
  if (lane == 0) a.path_len[b] = len;
}

}  // namespace

namespace tv {

int launch_commit(const CommitArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(commit_kernel, dim3(static_cast<unsigned>((a.batch + kWaves - 1) / kWaves)),
                     dim3(64 * kWaves), 0, stream, a);
  return hipGetLastError() == hipSuccess ? TV_OK : TV_ERR_HIP;
}

}  // namespace tv
