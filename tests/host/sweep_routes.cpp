// The library's host side (nhp_api.cpp, nhp_batch.cpp, nhp_tables.cpp) over a
// runtime that launches nothing: memory is the host's, and every sweep launch is
// noted by the way it would go.  Checks what the host decides and what it keeps
// between calls; prints one line per finding ("name: value").
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <chrono>
#include <map>
#include <string>
#include <vector>

#include "nhp_internal.h"

namespace {

std::map<char*, size_t> g_memory;  // device allocations by address
int g_tracked = 0, g_full = 0, g_clears = 0, g_graphs = 0;
int g_fail_at = -1;  // shared launches until one fails
std::string g_wrong;

size_t room(const void* p) {
  char* c = (char*)const_cast<void*>(p);
  auto it = g_memory.upper_bound(c);
  if (it == g_memory.begin()) return 0;
  --it;
  return c < it->first + it->second ? (size_t)(it->first + it->second - c) : 0;
}

void wrong(const char* what) {
  if (g_wrong.empty()) g_wrong = what;
}

}  // namespace

// ---- the runtime ----
hipError_t hipMalloc(void** p, size_t n) {
  *p = calloc(1, n);
  g_memory[(char*)*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  g_memory.erase((char*)p);
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return (*p = calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { return free(p), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return memcpy(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { return memcpy(d, s, n), hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = nullptr, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { return *s = hipStreamCaptureStatusNone, hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { return *g = (hipGraph_t)&g_graphs, hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return *e = (hipGraphExec_t)&g_graphs, hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return g_graphs++, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return *e = nullptr, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }

// ---- the kernels' launchers ----
namespace nhp {

bool can_fuse(const DevPlan&) { return false; }
bool xmajor_wide(int) { return true; }
bool trackable(const DevPlan& d) { return d.nx >= 32; }
int set_knob(int, int) { return NHP_OK; }
int get_knob(int) { return 0; }
int set_section_steps(int, int) { return NHP_OK; }
bool soft_table_in_args(uint32_t) { return true; }
int render_blocks(int, int) { return 1; }
void schedule_passes(const uint8_t* s, int n, uint64_t first, uint64_t count, bool, std::vector<Pass>& out) {
  for (uint64_t k = first; k < first + count; k++) out.push_back(Pass{(int8_t)s[k % (uint64_t)n], -1});
}
// one row job, a tile per 64 x nt poses
int make_sweep_jobs(const DevPlan& d, Pass pass, SweepJob* row, SweepJob* xmaj, TrackState* ts) {
  *row = SweepJob{};
  *xmaj = SweepJob{};
  row->V = d.V;
  row->N = d.nx;
  row->L = d.nt;
  row->P = 32;
  row->blocks = (d.nx + 63) / 64 * d.nx;
  if (ts) {
    row->tr.mode = kTrackSkip;
    ts->last[(int)pass.mu] = ++ts->pass;
    ts->sweeps++;
  }
  return 1;
}

hipError_t launch_sweep(const DevPlan& d, Pass pass, hipStream_t, TrackState* ts) {
  SweepJob row, xm;
  (void)make_sweep_jobs(d, pass, &row, &xm, ts);
  (ts ? g_tracked : g_full)++;
  return hipSuccess;
}
hipError_t launch_sweep_part(const DevPlan& d, Pass pass, int, hipStream_t s, TrackState* ts) { return launch_sweep(d, pass, s, ts); }

// The tile list of a tracked launch, as its kernels keep it: all tiles listed
// from where the launch's counter stands, the other counter cleared.
hipError_t launch_sweep_batch(const SweepJob*, int, int total_blocks, int, bool, bool, bool, bool, int,
                              const TileLists* l, hipStream_t) {
  if (g_fail_at >= 0 && g_fail_at-- == 0) return hipErrorUnknown;
  (l ? g_tracked : g_full)++;
  if (!l) return hipSuccess;
  uint32_t& count = l->counters[l->which];
  if (count != 0) wrong("a list begins behind an older one's tiles");
  if (((size_t)count + (size_t)total_blocks) * sizeof(uint2) > room(l->list)) wrong("tiles listed past the list's memory");
  count += (uint32_t)total_blocks;
  l->counters[l->which ^ 1] = 0;
  return hipSuccess;
}
hipError_t launch_clear(uint32_t* words, size_t n, hipStream_t) {
  if (room(words) < 4 * n) wrong("a clear past its memory");
  memset(words, 0, 4 * n);
  return g_clears++, hipSuccess;
}
hipError_t launch_init(const DevPlan&, uint32_t, const StartTiles&, hipStream_t) { return hipSuccess; }
hipError_t launch_init_batch(const InitJob*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t launch_seed(const DevPlan&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_force_walls(const DevPlan&, hipStream_t) { return hipSuccess; }
hipError_t launch_render(const DevPlan&, const uint8_t*, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_render_batch(const RenderJob*, int, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_extract(const ExArgs&, bool, hipStream_t) { return hipSuccess; }
hipError_t launch_extract_batch(const ExArgs*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_soft_costs(const uint8_t*, uint32_t*, const uint8_t*, uint8_t*, uint32_t, uint8_t*, int, hipStream_t) {
  return hipSuccess;
}
hipError_t noalloc_extract_area(int, uint32_t**) { return hipErrorUnknown; }

}  // namespace nhp

// ---- what is asked of them ----
namespace {

nhp_plan* make_plan(uint32_t n, uint32_t nt) {
  nhp_params p{};
  p.nx = n;
  p.ntheta = nt;
  p.turn_radius = 9.0;
  p.half_cell = 1;
  for (int k = 0; k < 6; k++) {
    p.ct_q10[k] = 1024;
    p.gear_q8[k] = 256;
    p.schedule[k] = (uint8_t)k;
  }
  p.n_schedule = 6;
  nhp_plan* plan = nullptr;
  if (plan_create(&p, nullptr, 0, nullptr, &plan) != NHP_OK) {
    printf("error: %s\n", plan_last_error());
    exit(1);
  }
  static uint8_t image[1024 * 1024];
  render_cspace(plan, image, 0, 0, 0);
  return plan;
}

// A plan's or a call's route since the last question: t tracked, f in full
// (launched or replayed from a graph), - no sweep launched.
char route() {
  const char c = g_tracked ? (g_full || g_graphs ? 'x' : 't') : (g_full || g_graphs ? 'f' : '-');
  g_tracked = g_full = g_graphs = g_clears = 0;
  return c;
}

void failed_list_launch() {
  nhp_plan* plan[4];
  uint32_t start[12] = {}, steps[4] = {}, counts[4];
  for (int k = 0; k < 4; k++) {
    plan[k] = make_plan(256, 256);
    start[3 * k] = start[3 * k + 1] = 9;
    counts[k] = 6;
  }
  nhp_batch* b = nullptr;
  batch_create(4, nullptr, &b);
  for (int fail = 0; fail < 6; fail++) {
    batch_init(b, plan, start, 4);
    route();
    batch_advance(b, plan, steps, counts, 4);
    const char before = route();
    batch_init(b, plan, start, 4);
    g_fail_at = fail;
    const int rc = batch_advance(b, plan, steps, counts, 4);
    g_fail_at = -1;
    route();
    batch_init(b, plan, start, 4);
    const int after = batch_advance(b, plan, steps, counts, 4);
    printf("failure at launch %d: %c %d %d %c\n", fail, before, rc, after, route());
  }
  batch_destroy(b);
  for (nhp_plan* p : plan) plan_destroy(p);
}

char swept(nhp_plan* p, uint32_t cycles) {
  route();
  sweep_n_turns(p, 5, 5, 0, cycles);
  return route();
}

void whole_sweeps() {
  const struct {
    uint32_t n, nt, cycles[3];
  } asked[] = {{1024, 64, {1, 11, 12}}, {1024, 128, {4, 11, 12}}, {720, 136, {1, 3, 20}}, {512, 256, {1, 3, 20}}, {512, 248, {1, 20, 60}}};
  for (const auto& a : asked) {
    nhp_plan* p = make_plan(a.n, a.nt);
    printf("%ux%u:", a.n, a.nt);
    for (uint32_t c : a.cycles) printf(" %c", swept(p, c));
    printf("\n");
    plan_destroy(p);
  }
}

char resumed(nhp_plan* p, uint32_t cycles) {
  route();
  sweep_resume(p, cycles);
  return route();
}

void resumes() {
  nhp_plan* p = make_plan(512, 256);
  printf("after 2, 5 more: %c", swept(p, 2));
  printf(" %c\n", resumed(p, 5));
  printf("after 2, 6 more, 1 more: %c", swept(p, 2));
  printf(" %c", resumed(p, 6));
  printf(" %c\n", resumed(p, 1));
  sweep_one(p, 1);
  printf("after one maneuver, 7 more, 8 more: %c", resumed(p, 7));
  printf(" %c\n", resumed(p, 8));
  printf("after 0, 0, 3 more: %c", swept(p, 0));
  printf(" %c", resumed(p, 0));
  printf(" %c\n", resumed(p, 3));
  sweep_one(p, 1);
  resumed(p, 0);
  printf("after one maneuver and 0, 1 more: %c\n", resumed(p, 1));
  uint32_t* v;
  plan_device_ptrs(p, &v, nullptr);
  printf("handed out, 9, 1 more, 8 more: %c", swept(p, 9));
  printf(" %c", resumed(p, 1));
  printf(" %c\n", resumed(p, 8));
  plan_destroy(p);
  p = make_plan(1024, 64);
  printf("few headings, after 12, 1 more: %c", swept(p, 12));
  printf(" %c\n", resumed(p, 1));
  printf("after 11, 11 more, 12 more: %c", swept(p, 11));
  printf(" %c", resumed(p, 11));
  printf(" %c\n", resumed(p, 12));
  plan_destroy(p);
  p = make_plan(264, 1000);
  printf("64-step sections, after 12, 12 more: %c", swept(p, 12));
  printf(" %c\n", resumed(p, 12));
  plan_destroy(p);
}

double now() { return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count(); }

// A call that repeats an earlier one against hashing the bytes of its job table
// one by one, the fastest of 20 each.
void repeated_call() {
  constexpr int kPlans = 256;
  std::vector<nhp_plan*> plan(kPlans);
  std::vector<uint32_t> start(3 * kPlans, 5), steps(kPlans, 0), counts(kPlans, 6);
  for (nhp_plan*& p : plan) p = make_plan(32, 16);
  nhp_batch* b = nullptr;
  batch_create(kPlans, nullptr, &b);
  batch_init(b, plan.data(), start.data(), kPlans);
  double call = 1e9, bytes = 1e9;
  std::vector<unsigned char> table(kPlans * 6 * sizeof(nhp::SweepJob), 1);
  volatile uint64_t sink = 0;
  for (int k = 0; k < 20; k++) {
    double t = now();
    batch_advance(b, plan.data(), steps.data(), counts.data(), kPlans);
    call = std::min(call, now() - t);
    t = now();
    uint64_t h = 1469598103934665603ull;
    for (unsigned char c : table) h = (h ^ c) * 1099511628211ull;
    bytes = std::min(bytes, now() - t);
    sink = sink + h;
  }
  printf("route: %c\nfaster than its table's bytes: %s\n", route(), call < bytes ? "yes" : "no");
  fprintf(stderr, "call %.1f us, bytes %.1f us\n", call * 1e6, bytes * 1e6);
  batch_destroy(b);
  for (nhp_plan* p : plan) plan_destroy(p);
}

// batch_advance: cycles of one call each
std::string advance(nhp_batch* b, nhp_plan** plan, uint32_t n, int cycles) {
  static const uint32_t steps[64] = {};
  uint32_t counts[64];
  for (uint32_t& c : counts) c = 6;
  std::string out;
  for (int c = 0; c < cycles; c++) {
    if (batch_advance(b, plan, steps, counts, n) != NHP_OK) return plan_last_error();
    out += route();
  }
  return out;
}

char sweep(nhp_batch* b, nhp_plan** plan, uint32_t n, uint32_t cycles) {
  uint32_t start[3 * 64] = {}, n_cycles[64];
  for (uint32_t& c : n_cycles) c = cycles;
  for (uint32_t& s : start) s = 5;
  route();
  if (batch_sweep(b, plan, start, n_cycles, n) != NHP_OK) return '!';
  return route();
}

void shared_launches() {
  nhp_plan* plan[5];
  uint32_t start[15] = {};
  for (int k = 0; k < 4; k++) plan[k] = make_plan(256, 256);
  plan[4] = make_plan(16, 16);  // too small to be tracked
  for (uint32_t& s : start) s = 5;
  nhp_batch* b = nullptr;
  batch_create(5, nullptr, &b);
  batch_init(b, plan, start, 4);
  route();
  printf("four, 7 cycles: %s\n", advance(b, plan, 4, 7).c_str());
  printf("then one alone: %s\n", advance(b, plan, 1, 1).c_str());
  batch_init(b, plan, start, 4);
  printf("four, 5 cycles: %s\n", advance(b, plan, 4, 5).c_str());
  printf("then one alone, then all: %s", advance(b, plan, 1, 1).c_str());
  printf(" %s\n", advance(b, plan, 4, 1).c_str());
  batch_init(b, plan, start, 4);
  printf("two: %s\n", advance(b, plan, 2, 2).c_str());
  printf("with a small one: %c\n", sweep(b, plan + 1, 4, 8));
  printf("sweep of four, 1 cycle: %c\n", sweep(b, plan, 4, 1));
  printf("sweep of two, 7 and 8 cycles: %c", sweep(b, plan, 2, 7));
  printf(" %c\n", sweep(b, plan, 2, 8));
  printf("sweep of one, 15 and 16 cycles: %c", sweep(b, plan, 1, 15));
  printf(" %c\n", sweep(b, plan, 1, 16));
  uint32_t* v;
  plan_device_ptrs(plan[2], &v, nullptr);
  batch_init(b, plan, start, 4);
  route();
  printf("four, one handed out: %s\n", advance(b, plan, 4, 3).c_str());
  printf("sweep of four, one handed out: %c\n", sweep(b, plan, 4, 2));
  printf("four more, one handed out: %s\n", advance(b, plan, 4, 2).c_str());
  batch_destroy(b);
  for (nhp_plan* p : plan) plan_destroy(p);
}

void workgroups() {
  for (int P : {8, 32}) {
    printf("%d steps:", P);
    for (int w = 1; w <= 16; w++) printf(" %d", nhp::row_workgroups(w, P));
    printf("\n");
  }
}

void extract_wait() { printf("milliseconds at 2.4 GHz: %llu\n", (unsigned long long)(nhp::kLeastWaitClocks / 2400000)); }

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "failed_list_launch") failed_list_launch();
  if (what == "extract_wait") extract_wait();
  if (what == "repeated_call") repeated_call();
  if (what == "whole_sweeps") whole_sweeps();
  if (what == "row_workgroups") workgroups();
  if (what == "resumes") resumes();
  if (what == "shared_launches") shared_launches();
  printf("wrong: %s\n", g_wrong.empty() ? "nothing" : g_wrong.c_str());
  return 0;
}
