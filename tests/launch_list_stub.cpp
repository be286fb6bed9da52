// Host-only harness for launch_list.cpp: the HIP calls it makes, on graphs and streams that are plain structures, and one scenario per
// argument.  A destroyed graph overwrites the argument blocks of its nodes, so a list that still reads them launches other values.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

#include "../paper_1904_08368_amd/csrc/kernels.hpp"

namespace {
constexpr int kDead = 0x5ddd;

struct Node {
  hipGraphNodeType type = hipGraphNodeTypeKernel;
  void* func = nullptr;
  int arg = 0;
  void* args[1];
};
struct Graph {
  std::vector<Node*> nodes;
  std::vector<std::pair<int, int>> edges;
};
struct Launch {
  std::thread::id thread;
  void* func;
  int arg, device;
};

std::mutex g_lock;
std::vector<Launch> g_launches;
int g_graphs = 0;
thread_local int t_device = 0;
hipStreamCaptureStatus g_capture = hipStreamCaptureStatusNone;

void kernel_a() {}
void kernel_b() {}
void kernel_c() {}
void* const kKernels[] = {(void*)kernel_a, (void*)kernel_b, (void*)kernel_c};

Graph* chain(int n) {
  Graph* g = new Graph;
  ++g_graphs;
  for (int i = 0; i < n; ++i) {
    Node* v = new Node;
    v->func = kKernels[i % 3];
    v->arg = 100 + i;
    v->args[0] = &v->arg;
    g->nodes.push_back(v);
    if (i) g->edges.push_back({i - 1, i});
  }
  return g;
}

int fail(const char* what) {
  printf("FAILED: %s\n", what);
  return 1;
}

relay::LaunchList* make(Graph* g, size_t most = 64) {
  relay::LaunchList* l = nullptr;
  if (relay::make_launch_list(reinterpret_cast<hipGraph_t>(g), most, &l) != hipSuccess) fail("make_launch_list"), exit(1);
  return l;
}
hipStream_t stream() { return reinterpret_cast<hipStream_t>(&g_lock); }
}  // namespace

extern "C" {
hipError_t hipGraphGetNodes(hipGraph_t graph, hipGraphNode_t* nodes, size_t* n) {
  Graph* g = reinterpret_cast<Graph*>(graph);
  for (size_t i = 0; nodes && i < *n; ++i) nodes[i] = reinterpret_cast<hipGraphNode_t>(g->nodes[i]);
  *n = g->nodes.size();
  return hipSuccess;
}
hipError_t hipGraphGetEdges(hipGraph_t graph, hipGraphNode_t* from, hipGraphNode_t* to, size_t* n) {
  Graph* g = reinterpret_cast<Graph*>(graph);
  for (size_t i = 0; from && i < *n; ++i) {
    from[i] = reinterpret_cast<hipGraphNode_t>(g->nodes[g->edges[i].first]);
    to[i] = reinterpret_cast<hipGraphNode_t>(g->nodes[g->edges[i].second]);
  }
  *n = g->edges.size();
  return hipSuccess;
}
hipError_t hipGraphClone(hipGraph_t* copy, hipGraph_t graph) {
  Graph* g = reinterpret_cast<Graph*>(graph);
  Graph* c = new Graph;
  ++g_graphs;
  c->edges = g->edges;
  for (Node* v : g->nodes) {
    c->nodes.push_back(new Node(*v));
    c->nodes.back()->args[0] = &c->nodes.back()->arg;
  }
  *copy = reinterpret_cast<hipGraph_t>(c);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t graph) {   // (the nodes stay readable: what a list still reads of them is seen, not undefined)
  for (Node* v : reinterpret_cast<Graph*>(graph)->nodes) v->arg = kDead;
  --g_graphs;
  return hipSuccess;
}
hipError_t hipGraphNodeGetType(hipGraphNode_t node, hipGraphNodeType* type) {
  *type = reinterpret_cast<Node*>(node)->type;
  return hipSuccess;
}
hipError_t hipGraphKernelNodeGetParams(hipGraphNode_t node, hipKernelNodeParams* p) {
  Node* v = reinterpret_cast<Node*>(node);
  p->func = v->func;
  p->kernelParams = v->args;
  return hipSuccess;
}
hipError_t hipGetDevice(int* device) {
  *device = t_device;
  return hipSuccess;
}
hipError_t hipSetDevice(int device) {
  t_device = device;
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* status) {
  *status = g_capture;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* func, dim3, dim3, void** args, size_t, hipStream_t) {
  {
    std::lock_guard<std::mutex> hold(g_lock);
    g_launches.push_back({std::this_thread::get_id(), const_cast<void*>(func), *static_cast<int*>(args[0]), t_device});
  }
  std::this_thread::yield();
  return hipSuccess;
}
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  Graph* g = chain(5);
  if (!strcmp(what, "lifetime")) {
    relay::LaunchList* l = make(g);
    (void)hipGraphDestroy(reinterpret_cast<hipGraph_t>(g));
    if (!l || relay::run_launch_list(l, stream()) != hipSuccess || g_launches.size() != 5) return fail("run");
    for (int i = 0; i < 5; ++i)
      if (g_launches[i].func != kKernels[i % 3] || g_launches[i].arg != 100 + i) return fail("arguments of a destroyed graph were launched");
    relay::free_launch_list(l);
    if (g_graphs != 0) return fail("the copy outlives the list");
  } else if (!strcmp(what, "threads")) {
    relay::LaunchList* l = make(g);
    std::vector<std::thread> threads;
    for (int t = 0; t < 4; ++t)
      threads.emplace_back([l] {
        for (int i = 0; i < 200; ++i)
          if (relay::run_launch_list(l, stream()) != hipSuccess) abort();
      });
    for (auto& t : threads) t.join();
    if (g_launches.size() != 4 * 200 * 5) return fail("launches are missing");
    int turns = 0;
    for (size_t i = 0; i < g_launches.size(); ++i) {
      if (g_launches[i].arg != 100 + (int)(i % 5) || g_launches[i].thread != g_launches[i - i % 5].thread) return fail("a pass was not enqueued whole");
      turns += i >= 5 && i % 5 == 0 && g_launches[i].thread != g_launches[i - 5].thread;
    }
    printf("turns %d\n", turns);
  } else if (!strcmp(what, "capture")) {
    relay::LaunchList* l = make(g);
    for (hipStreamCaptureStatus s : {hipStreamCaptureStatusActive, hipStreamCaptureStatusInvalidated}) {
      g_capture = s;
      if (relay::run_launch_list(l, stream()) != hipErrorStreamCaptureUnsupported || !g_launches.empty()) return fail("enqueued into a capture");
    }
    g_capture = hipStreamCaptureStatusNone;
    if (relay::run_launch_list(l, stream()) != hipSuccess || g_launches.size() != 5) return fail("refused after the capture");
  } else if (!strcmp(what, "device")) {
    t_device = 2;
    relay::LaunchList* l = make(g);
    t_device = 1;
    if (relay::run_launch_list(l, nullptr) != hipSuccess || t_device != 1) return fail("the caller's device is not restored");
    for (const Launch& x : g_launches)
      if (x.device != 2) return fail("launched on another device than the capture's");
  } else if (!strcmp(what, "refused")) {
    const auto refused = [](Graph* h, size_t most = 64) {
      relay::LaunchList* l = make(h, most);
      (void)hipGraphDestroy(reinterpret_cast<hipGraph_t>(h));
      return l == nullptr;
    };
    if (!refused(chain(0))) return fail("an empty graph");
    if (refused(chain(64))) return fail("64 launches are a list");   // (its copy is the one that is left below)
    if (!refused(chain(65)) || !refused(chain(5), 4)) return fail("more launches than asked for");
    Graph* h = chain(4);
    h->nodes[2]->type = hipGraphNodeTypeMemset;
    if (!refused(h)) return fail("a memset");
    h = chain(4);
    h->nodes[3]->func = (void*)&strlen;
    if (!refused(h)) return fail("another library's kernel");
    h = chain(4);
    h->edges = {{0, 1}, {0, 2}, {1, 3}};
    if (!refused(h)) return fail("a fork");
    h = chain(4);
    h->edges = {{0, 2}, {1, 2}, {2, 3}};
    if (!refused(h)) return fail("two beginnings");
    h = chain(4);
    h->edges = {{1, 2}, {2, 3}, {3, 1}};
    if (!refused(h)) return fail("a cycle beside one node");
    if (g_graphs != 2) return fail("copies of refused graphs are left");
  } else {
    return fail("no such scenario");
  }
  printf("ok\n");
  return 0;
}
