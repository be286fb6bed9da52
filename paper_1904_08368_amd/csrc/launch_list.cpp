// A recorded chain of kernel launches, enqueued again by one call.
//
// Replaying a HIP graph leaves the GPU idle for about 5 us between one replay and the next (measured as the difference between
// a graph that holds a network once and one that holds it two and four times: 5.0 to 5.7 us from 5 launches to 20), whatever the network;
// launches enqueued one by one leave no gap, as long as the host keeps ahead of the GPU.  From Python it does not at small
// batches (4.5 us a call); this loop over the launches of the captured graph does (2.1 to 2.6 us each) where passes are queued.  One after another,
// graph -> list: deep Q-network at batch 1 21.4 -> 16.3 to 18.4 us, ResNet-18 at batch 1 79.9 -> 74.9, at batch 32 224 -> 219, an Inception block of 32
// images 52.1 -> 46.5; int8 ResNet-18 at batch 1, whose 15 launches take the GPU 3.8 us each, 59.9 -> 57.2 to 58.6.
// The price is the host's time: 12 us for five launches and 32 to 49 for 15 to 20, where the graph's replay takes 18 and 13 to 30.  A GPU that
// idles when the pass comes waits for each launch in turn: waited for, the Q-network 38 -> 28 us, but ResNet-18 at batch 1 92 -> 92 to 94, int8
// 72 -> 69 to 87, MobileNet-v1 97 -> 108.  Which of the two a pass takes is the caller's choice (FusedNet.replay).
#include <memory>
#include <mutex>
#include <vector>

#include <dlfcn.h>
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace relay {

struct LaunchList {
  hipGraph_t copy = nullptr;                   // owns the argument blocks: the captured graph may go before the list
  std::vector<hipKernelNodeParams> launches;
  int device = 0;
  std::mutex issue;   // passes of threads that share the list follow one another whole
  ~LaunchList() {
    if (copy) (void)hipGraphDestroy(copy);
  }
};

namespace {
// Is this the host handle of a kernel of this library?  (Others stay in their graph: torch's, say, may read state that a replay of
// the graph renews.)
bool own_kernel(const void* func) {
  Dl_info here, there;
  return dladdr(reinterpret_cast<const void*>(&free_launch_list), &here) && dladdr(func, &there) && here.dli_fbase == there.dli_fbase;
}
}  // namespace

hipError_t make_launch_list(hipGraph_t graph, size_t most, LaunchList** out) {
  *out = nullptr;
  size_t n = 0, edges = 0;
  hipError_t e = hipGraphGetNodes(graph, nullptr, &n);
  if (e != hipSuccess) return e;
  if (n == 0 || n > most) return hipSuccess;
  auto l = std::make_unique<LaunchList>();
  if ((e = hipGetDevice(&l->device)) != hipSuccess) return e;
  if ((e = hipGraphClone(&l->copy, graph)) != hipSuccess) return e;
  std::vector<hipGraphNode_t> nodes(n);
  if ((e = hipGraphGetNodes(l->copy, nodes.data(), &n)) != hipSuccess) return e;
  if ((e = hipGraphGetEdges(l->copy, nullptr, nullptr, &edges)) != hipSuccess) return e;
  if (edges != n - 1) return hipSuccess;
  std::vector<hipGraphNode_t> from(n), to(n);
  if (edges && (e = hipGraphGetEdges(l->copy, from.data(), to.data(), &edges)) != hipSuccess) return e;
  // the first node is the one that nothing leads to; from it every node leads to one other
  hipGraphNode_t at = nullptr;
  for (hipGraphNode_t v : nodes) {
    bool led_to = false;
    for (size_t i = 0; i < edges; ++i) led_to |= to[i] == v;
    if (!led_to) {
      if (at) return hipSuccess;
      at = v;
    }
  }
  while (at && l->launches.size() < n) {
    hipGraphNodeType type;
    hipKernelNodeParams p{};
    if (hipGraphNodeGetType(at, &type) != hipSuccess || type != hipGraphNodeTypeKernel || hipGraphKernelNodeGetParams(at, &p) != hipSuccess ||
        !p.kernelParams || p.extra || !own_kernel(p.func)) return hipSuccess;
    l->launches.push_back(p);
    hipGraphNode_t next = nullptr;
    for (size_t i = 0; i < edges; ++i)
      if (from[i] == at) {
        if (next) return hipSuccess;   // two successors: not a chain
        next = to[i];
      }
    at = next;
  }
  if (l->launches.size() == n) *out = l.release();
  return hipSuccess;
}

hipError_t run_launch_list(LaunchList* l, hipStream_t st) {
  std::lock_guard<std::mutex> whole(l->issue);
  if (st) {
    hipStreamCaptureStatus capturing;
    const hipError_t c = hipStreamIsCapturing(st, &capturing);
    if (c != hipSuccess) return c;
    if (capturing != hipStreamCaptureStatusNone) return hipErrorStreamCaptureUnsupported;   // (as the launch of a graph)
  }
  int device = l->device;
  hipError_t e = hipGetDevice(&device);
  if (e == hipSuccess && device != l->device) e = hipSetDevice(l->device);
  for (size_t i = 0; e == hipSuccess && i < l->launches.size(); ++i) {
    const hipKernelNodeParams& p = l->launches[i];
    e = hipLaunchKernel(p.func, p.gridDim, p.blockDim, p.kernelParams, p.sharedMemBytes, st);
  }
  if (device != l->device) (void)hipSetDevice(device);
  return e;
}

void free_launch_list(LaunchList* l) { delete l; }

}  // namespace relay
