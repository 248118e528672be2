// Accepted-path commit (the step after verification): for every tree, the
// output of Def. def2 laid out for the next decoding cycle: the node indices
// of the accepted chain X^tau after the root, from the root down (the drafted
// positions whose cache entries are kept), and their tokens followed by Y.
#include <hip/hip_runtime.h>

#include "tv.h"
#include "tv_launch.h"

namespace {

// kLanes lanes per tree of at most kNodes nodes. The links from the accepted
// node down are brought into LDS, kWindow nodes at a time, and the chain is
// found there by walking from the accepted node to the root (each step to a
// smaller index, so at most num_nodes steps); then its tokens are gathered and
// everything is written by all lanes; entries past the chain are -1.
//
// Few trees: bound by latency, so a wavefront a tree and all links at once, in
// the same round of loads as status, accepted node and bonus token. (One thread
// per tree, each step a load of its own, took 7.5 us for 64 trees against 4.8
// us, 4.2 of which any kernel takes.) Many trees: see kManyTrees below.
constexpr int kThreads = 256;

template <int kLanes, int kWindow, int kNodes>
__global__ void __launch_bounds__(kThreads) commit_kernel(tv::CommitArgs a) {
  constexpr int kTrees = kThreads / kLanes;
  __shared__ int16_t links[kTrees][kWindow];   // parents, -1 where not smaller than the node
  __shared__ int16_t chains[kTrees][kNodes];   // from the accepted node up
  const int lane = threadIdx.x % kLanes, sub = threadIdx.x / kLanes;
  const int b = static_cast<int>(blockIdx.x) * kTrees + sub;
  if (b >= a.batch) return;            // a tree's lanes are in one wavefront: no barriers here
  int16_t* link = links[sub];
  int16_t* chain = chains[sub];
  const int n1 = a.num_nodes, L = a.max_len;
  const size_t tree = static_cast<size_t>(b);
  const int status = a.status[tree], acc = a.accepted_node[tree], bonus = a.bonus_token[tree];
  auto ordered = [] {                  // LDS accesses of the wavefront, in program order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  auto load = [&](int from, int to) {
    ordered();
    for (int i = from + lane; i < to; i += kLanes) {
      const int p = a.parents[tree * n1 + i];
      link[i - from] = static_cast<int16_t>(p >= 0 && p < i ? p : -1);
    }
    ordered();
  };
  const bool all = kWindow == kNodes || n1 <= kWindow;
  if (all) load(0, n1);
  // length of the output, or the code of a tree that has none
  int depth = 0, len = 0;
  if (status == TV_TREE_OK) {
    int x = acc < n1 ? acc : -1;
    while (x > 0) {
      const int lo = all ? 0 : max(0, x + 1 - kWindow);
      if (!all) load(lo, x + 1);
      do {
        if (lane == 0) chain[depth] = static_cast<int16_t>(x);
        ++depth;
        x = link[x - lo];
      } while (x >= max(lo, 1));
    }
    len = x < 0 ? TV_COMMIT_INCONSISTENT : depth > L ? TV_COMMIT_OVERFLOW : depth + 1;
  }
  ordered();
  int32_t* pn = a.path_nodes + tree * L;
  int32_t* pt = a.path_tokens + tree * (L + 1);
  for (int i = lane; i <= L; i += kLanes) {
    const bool in = len > 0 && i < depth;
    const int x = in ? chain[depth - 1 - i] : -1;
    if (i < L) pn[i] = x;
    pt[i] = in ? a.tokens[tree * n1 + x] : len > 0 && i == depth ? bonus : -1;
  }
  if (lane == 0) a.path_len[b] = len;
}

// From about as many trees as the device holds wavefronts, the call is bound by
// what it issues and reads: two trees a wavefront, or sixteen very small ones,
// and windows of 128 links, so that a large tree reads only near its chain. (With
// a wavefront and all links for every tree, with one thread a tree, and now, us:
// 16384 trees of 65 nodes 5.5, 9.9, 4.2; of 1024 nodes with links up to 64 back
// 21, 28, 16, up to 7/8 of the index back 17, 9.2, 5.3; 200000 trees of 8 nodes
// 46, 44, 27.)
constexpr int kManyTrees = 8192, kManyWindow = 128, kSmallTree = 16;

template <int kLanes, int kWindow, int kNodes>
void run(const tv::CommitArgs& a, hipStream_t stream) {
  constexpr int kTrees = kThreads / kLanes;
  hipLaunchKernelGGL((commit_kernel<kLanes, kWindow, kNodes>),
                     dim3(static_cast<unsigned>((a.batch + kTrees - 1) / kTrees)), dim3(kThreads),
                     0, stream, a);
}

}  // namespace

namespace tv {

int launch_commit(const CommitArgs& a, hipStream_t stream) {
  if (a.batch < kManyTrees)
    run<64, TV_MAX_NODES, TV_MAX_NODES>(a, stream);
  else if (a.num_nodes <= kSmallTree && a.max_len < kSmallTree)
    run<4, kSmallTree, kSmallTree>(a, stream);
  else
    run<32, kManyWindow, TV_MAX_NODES>(a, stream);
  return hipGetLastError() == hipSuccess ? TV_OK : TV_ERR_HIP;
}

}  // namespace tv
