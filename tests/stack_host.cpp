// The bookkeeping of a layer stack (csrc/stack.hip) against a HIP of plain host memory: every copy is tracked from
// its call to its end, a chosen copy can be refused, and every launch of a layer's FFN is checked: each expert with rows
// must be found through the expert table, with its own bytes, in a slot whose copies have ended or are waited for.
// Exits with 0 and prints the number of checked launches.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

#include "../paper_2512_17073_amd/csrc/internal.h"

struct ihipStream_t { int issued = 0, done = 0, waits = 0; };      // copies queued and ended; last copy a stream waits for
struct ihipEvent_t { ihipStream_t* stream = nullptr; int seq = 0; };

static ihipStream_t* copy_stream = nullptr;
static std::map<const void*, int> copied;      // destination -> number of its last copy on the copy stream
static int refuse_in = 0;                      // 1: the next copy fails, 2: the one after it, ...

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "refused"; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = copy_stream = new ihipStream_t(); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { delete s; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { s->done = s->issued; return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t s) { return s->done == s->issued ? hipSuccess : hipErrorNotReady; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  if (e->stream == copy_stream && e->seq > s->waits) s->waits = e->seq;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = new ihipEvent_t(); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { e->stream = s; e->seq = s->issued; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { return !e->stream || e->seq <= e->stream->done ? hipSuccess : hipErrorNotReady; }
hipError_t hipEventSynchronize(hipEvent_t e) {
  if (e->stream && e->seq > e->stream->done) e->stream->done = e->seq;
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t s) {
  if (refuse_in > 0 && --refuse_in == 0) return hipErrorUnknown;
  memcpy(dst, src, n);
  if (s == copy_stream) copied[dst] = ++s->issued;
  return hipSuccess;
}
size_t moe_lrc_workspace_bytes(const moe_lrc_layer*, int) { return 256; }
}

#define REQUIRE(cond, ...) do { if (!(cond)) { printf(__VA_ARGS__); printf("\n"); exit(1); } } while (0)

constexpr int kExperts = 8, kBytes = 256;
static ihipStream_t compute;
static std::vector<std::vector<int>> wanted;   // [layer] the experts that receive rows
static int launches = 0, launched_ahead = 0;

namespace lrc {

int set_error(int code, const std::string&) { return code; }
void fill_algorithmic_stats(moe_lrc_layer*, const int32_t*) {}
void factor_section_bytes(const moe_lrc_layer*, int, int, size_t& a, size_t& b) { a = b = 0; }
void set_factor_ptrs(const moe_lrc_layer*, int, int mat, ExpertDesc& d, const uint8_t* a_base, const uint8_t*) {
  d.af[mat] = reinterpret_cast<const _Float16*>(a_base);
}

static bool in_place(const void* p, const uint8_t* own) {
  const auto it = copied.find(p);
  return it != copied.end() && (it->second <= copy_stream->done || it->second <= compute.waits) && memcmp(p, own, kBytes) == 0;
}
static bool ffn_would_be_right(const moe_lrc_layer* L) {
  for (int e : wanted[L->pool_index])
    if (!in_place(L->d_desc[e].codes[0], L->h_w + L->w_off[e]) || !in_place(L->d_desc[e].af[0], L->h_f + L->f_off[e])) return false;
  return true;
}

// what the library's does of a pooled layer's bookkeeping, with the counts of `wanted`
int forward_impl(moe_lrc_layer* L, const void*, int T, void*, void*, hipStream_t s, const void*) {
  bool ahead = false, complete = false;
  int rc = pool_begin(L, &ahead);
  if (rc) return rc;
  for (int e = 0; e < 2 * kExperts; ++e) L->h_stat[2 + e] = 0;
  for (int e : wanted[L->pool_index]) L->h_stat[2 + e] = L->h_stat[2 + kExperts + e] = 1;
  const RouteGuess g = pool_guess(L);
  if (g.layer) {
    const auto& next = wanted[L->pool_index + 1];
    for (int i = 0; i < T * g.layer->cfg.top_k; ++i) g.idx[i] = next[i % next.size()];
  }
  if ((rc = pool_counts_written(L, s))) return rc;
  const bool first = ahead && ffn_would_be_right(L);
  if ((rc = pool_stage(L, T, s, &complete))) return rc;
  REQUIRE(ahead && complete ? first : ffn_would_be_right(L), "layer %d: an FFN launch whose experts are not in place", L->pool_index);
  ++launches;
  launched_ahead += ahead;
  return MOE_LRC_OK;
}

}  // namespace lrc

// a stack of n layers with room for all experts; every expert's bytes differ
struct Fixture {
  std::vector<moe_lrc_layer*> layers;
  moe_lrc_stack* stack = nullptr;
  explicit Fixture(int n, bool prefetch) {
    for (int l = 0; l < n; ++l) {
      auto* L = new moe_lrc_layer();
      L->cfg.hidden = 64; L->cfg.n_experts = kExperts; L->cfg.top_k = 2; L->cfg.top_n = 2; L->cfg.rank = 8; L->cfg.max_tokens = 4;
      L->cfg.residency = MOE_LRC_POOLED; L->device = 0; L->n_total = kExperts; L->gate_set = true;
      L->routed.w_bytes = L->routed.f_bytes = kBytes;
      L->h_w = (uint8_t*)malloc(kExperts * kBytes); L->h_f = (uint8_t*)malloc(kExperts * kBytes);
      for (int i = 0; i < kExperts * kBytes; ++i) { L->h_w[i] = uint8_t(16 * l + i / kBytes); L->h_f[i] = uint8_t(128 + 16 * l + i / kBytes); }
      for (int e = 0; e < kExperts; ++e) { L->w_off.push_back(e * kBytes); L->f_off.push_back(e * kBytes); }
      L->h_desc.resize(kExperts);
      L->d_desc = (lrc::ExpertDesc*)calloc(kExperts, sizeof(lrc::ExpertDesc));
      L->h_stat = (int32_t*)calloc(2 + 2 * kExperts, 4);
      L->mat_set.assign(3 * kExperts, 1); L->mat_q3.assign(3 * kExperts, 0);
      layers.push_back(L);
    }
    copied.clear(); compute = ihipStream_t(); refuse_in = 0;
    REQUIRE(moe_lrc_stack_create(layers.data(), n, n * kExperts, prefetch ? MOE_LRC_STACK_PREFETCH : 0, &stack) == MOE_LRC_OK, "create");
  }
  // one step; ended: whether the copies end before the next one begins; refuse: the copy of the step that fails
  int step(std::vector<std::vector<int>> experts, bool ended = true, int refuse = 0) {
    wanted = experts; refuse_in = refuse;
    char x[4 * 64 * 2];
    const int rc = moe_lrc_stack_step(stack, x, 2, x, nullptr, &compute);
    refuse_in = 0;
    if (ended) copy_stream->done = copy_stream->issued;
    return rc;
  }
};

int main() {
  // (copies of an expert: its weights, then its factors; then the table.)  Refused: the second expert's weights or
  // factors, while the first one's copies are under way; then the table itself
  for (int refuse = 1; refuse <= 5; ++refuse) {
    Fixture f(1, false);
    for (int i = 0; i < 2; ++i) REQUIRE(f.step({{0, 1}}) == MOE_LRC_OK, "step");
    REQUIRE(f.step({{2, 3}}, false, refuse) != MOE_LRC_OK, "a refused copy must be reported");
    REQUIRE(f.step({{2}}, false) == MOE_LRC_OK, "step");
    REQUIRE(f.step({{0, 1}}, false) == MOE_LRC_OK, "step");
    for (int i = 0; i < 3; ++i) REQUIRE(f.step({{2, 3}}, i > 0) == MOE_LRC_OK, "step");
    moe_lrc_stack_destroy(f.stack);
  }
  // the same for copies ahead of the second layer (after the first one's own, and its table)
  for (int refuse = 1; refuse <= 10; ++refuse) {
    Fixture f(2, true);
    for (int i = 0; i < 2; ++i) REQUIRE(f.step({{0, 1}, {4, 5}}) == MOE_LRC_OK, "step");
    REQUIRE(f.step({{2, 3}, {6, 7}}, false, refuse) != MOE_LRC_OK, "a refused copy must be reported");
    REQUIRE(f.step({{0, 2}, {6}}, false) == MOE_LRC_OK, "step");
    for (int i = 0; i < 3; ++i) REQUIRE(f.step({{2, 3}, {6, 7}}, i > 0) == MOE_LRC_OK, "step");
    moe_lrc_stack_destroy(f.stack);
  }
  REQUIRE(launched_ahead > 0, "no launch before the counts");
  printf("%d launches, %d before the counts\n", launches, launched_ahead);
  return 0;
}
