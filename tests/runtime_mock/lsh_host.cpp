// The host side of lsh.hip on the mocked runtime: query batches of an index
// whose shape the test gives (its arrays are never read).
#include <cstring>

#include "mock_launch.h"

#include "lsh.hip"

namespace stag {
void exclusive_scan(Workspace& ws, int64_t n) {
  uint64_t* tot = nullptr;
  (void)ws.alloc(&tot, (size_t)ceil_div(n, 1024));
}
stag_status exclusive_scan_u32(const uint32_t*, uint64_t*, int64_t n, Workspace& ws, hipStream_t) {
  exclusive_scan(ws, n);
  return STAG_OK;
}
stag_status radix_sort_pairs_u32(const uint32_t*, const uint32_t*, uint32_t*, uint32_t*, int64_t, int, Workspace&,
                                 hipStream_t) {
  return STAG_OK;
}
stag_status e2lsh_launch(const float*, int64_t, int, const double*, int, const double*, int, int, int32_t*, uint64_t*,
                         hipStream_t) {
  return STAG_OK;
}
int e2lsh_reg_dim(int d) { return d <= 64 ? 64 : 0; }
stag_status e2lsh_regroup(const float*, int, int, int, Workspace&, double**, int*, hipStream_t) { return STAG_OK; }
stag_status zero_async(void*, size_t, hipStream_t) { return STAG_OK; }
}  // namespace stag

using namespace stag;

namespace {
struct Span {
  int64_t q0, count;
};
std::vector<Span> g_combined;  // queries whose join results were taken
int64_t g_cur = 0;             // queries of the batch being set up
int64_t g_tasks = 0;           // tasks that a query makes
size_t g_peak = 0;
}  // namespace

extern "C" {
void* lsh_index(int d, int K1, int J, int L, int K, int64_t slots) {
  auto* idx = new stag_lsh_index();
  idx->d = d;
  idx->dx = (int)round_up(d, 4);
  idx->dreg = e2lsh_reg_dim(d);
  idx->dg = idx->dreg > 0 ? idx->dreg : d;
  idx->nch = (int)ceil_div(K, 8);
  idx->prm.n = 1000;
  idx->prm.shape.K1 = K1;
  idx->prm.shape.J = J;
  idx->prm.shape.L = L;
  idx->prm.shape.K = K;
  idx->nseg = (int64_t)K1 * J;
  idx->ntab = idx->nseg * L;
  idx->total_slots = slots;
  return idx;
}
// `tiles` column tiles of dense segments (walked indexes: d > 128 or L > 32).
void lsh_dense(void* idx, int tiles) {
  auto* x = static_cast<stag_lsh_index*>(idx);
  x->dense_tiles = tiles;
  x->dlevels = reinterpret_cast<uint64_t*>(64);
}
int lsh_sample(void* idx, void* stream, int64_t n, int s) {
  auto* x = static_cast<stag_lsh_index*>(idx);
  x->prm.n = n;
  mock::launches().clear();
  auto* p = reinterpret_cast<int64_t*>((uintptr_t)1 << 42);
  return (int)lsh_sample_edges(x, s, 1, p, p, (double*)p, nullptr, (hipStream_t)stream);
}
void lsh_free(void* idx) { delete static_cast<stag_lsh_index*>(idx); }

void lsh_members(void* idx, int64_t members) { static_cast<stag_lsh_index*>(idx)->M = members; }
uint64_t lsh_pairs(void* idx, int64_t m) { return lsh_pair_bytes(static_cast<stag_lsh_index*>(idx), m); }

// A query of m rows (pair_bytes > 0: with at most that many); tasks: join
// tasks that every query makes.
int lsh_query(void* idx, void* stream, int64_t m, int64_t tasks, uint64_t pair_bytes) {
  g_combined.clear();
  mock::launches().clear();
  g_tasks = tasks;
  mock::hooks()["locate_queries"] = [](void** a) { g_cur = mock::arg<int64_t>(a, 2); };
  mock::hooks()["combine_groups"] = [](void** a) { g_combined.push_back({mock::arg<int64_t>(a, 8), mock::arg<int64_t>(a, 2)}); };
  mock::readback() = [](void* p, size_t n) {
    const uint64_t v = (uint64_t)(g_cur * g_tasks);
    if (n == sizeof(v)) std::memcpy(p, &v, n);
  };
  const float* Q = reinterpret_cast<const float*>((uintptr_t)1 << 40);
  double* S = reinterpret_cast<double*>((uintptr_t)1 << 41);
  if (pair_bytes > 0) return (int)lsh_query_within((stag_lsh_index*)idx, Q, m, S, pair_bytes, (hipStream_t)stream);
  return (int)stag_lsh_index_query((stag_lsh_index*)idx, Q, m, S, (hipStream_t)stream);
}
int64_t lsh_combined(int64_t* q0, int64_t* count, int64_t cap) {
  for (size_t k = 0; k < g_combined.size() && (int64_t)k < cap; ++k) {
    q0[k] = g_combined[k].q0;
    count[k] = g_combined[k].count;
  }
  return (int64_t)g_combined.size();
}
uint32_t lsh_bucket_tasks(uint32_t nq, uint32_t nm) { return bucket_tasks(nq, nm); }
// Threads of the largest launch, and how many launches a kernel had.
int64_t launch_threads(void) {
  int64_t t = 0;
  for (const auto& l : mock::launches())
    t = std::max(t, (int64_t)l.grid.x * l.grid.y * l.grid.z * l.block.x);
  return t;
}
int64_t launch_count(const char* name) {
  int64_t c = 0;
  for (const auto& l : mock::launches()) c += l.name.find(name) != std::string::npos;
  return c;
}
}  // extern "C"
