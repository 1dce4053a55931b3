// The library's own host code against a HIP runtime made of host memory: this
// program defines the HIP calls that libdaso.so makes, and stands a host model
// behind hipLaunchKernel that does what the kernels do with the statistics scratch.
// A step launch writes, for each bucket and workgroup, how many of the
// bucket's elements that workgroup has; a statistics launch sums them.  So every
// bucket's statistics come out as its element count exactly if the launches' tables,
// places and order are right.  No access leaves its buffer unnoticed.  No GPU.
// Usage: launch_model <scenario>.  Exit status 0 when every expectation holds.
#include <dlfcn.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <random>
#include <string>
#include <vector>

#include "daso_launch.h"

static int failures = 0;
#define EXPECT(cond)                                                                           \
  do {                                                                                         \
    if (!(cond)) {                                                                             \
      if (++failures < 20) std::fprintf(stderr, "%s, line %d: %s\n", what.c_str(), __LINE__, #cond); \
    }                                                                                          \
  } while (0)

static std::string what;  // the call under test
static std::map<const void*, std::string> kernel_names;
static std::map<const void*, size_t> symbol_bytes;
static std::map<const char*, size_t> buffers;  // "device" memory: begin -> bytes
static size_t allocated = 0;
static bool capturing = false;
static int mallocs = 0, mallocs_in_capture = 0, steps = 0, passes = 0;
static uint32_t last_block = 0, last_lds = 0;

static bool inside(const void* p, size_t bytes) {
  auto it = buffers.upper_bound(static_cast<const char*>(p));
  if (it == buffers.begin()) return false;
  --it;
  return static_cast<const char*>(p) + bytes <= it->first + it->second;
}

static void* new_buffer(size_t bytes) {
  char* p = static_cast<char*>(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
  buffers[p] = bytes;
  return p;
}

// ------------------------------------------------------------- the two kernels
static void sum_buckets(const daso::SlicePartial* partials, const daso::BucketSlots* table, daso_bucket_stats* stats,
                        uint32_t nb) {
  EXPECT(inside(table, nb * sizeof(*table)));
  for (uint32_t i = 0; i < nb; ++i) {
    daso_bucket_stats r = {0.0, 0.0, 0};
    EXPECT(table[i].end == table[i].first || inside(partials + table[i].first, static_cast<size_t>(table[i].end - table[i].first) * sizeof(*partials)));
    for (int64_t j = table[i].first; j < table[i].end; ++j) {
      r.grad_sq += partials[j].grad_sq;
      r.delta_sq += partials[j].delta_sq;
      r.nonfinite += partials[j].nonfinite;
    }
    EXPECT(inside(stats + table[i].out, sizeof(r)));
    const daso_bucket_stats& was = stats[table[i].out];
    if (table[i].add) r = {was.grad_sq + r.grad_sq, was.delta_sq + r.delta_sq, was.nonfinite + r.nonfinite};
    stats[table[i].out] = r;
  }
}

static void model_buckets(const daso::StepArgs& a) {
  for (int i = 0; i < a.nb && a.stats != nullptr; ++i) {
    const int64_t count = a.start[i + 1] - a.start[i];
    EXPECT(inside(a.stats + a.out[i], sizeof(*a.stats)) && inside(a.table + i, sizeof(*a.table)));
    daso_bucket_stats r = {static_cast<double>(count), 2.0 * static_cast<double>(count), static_cast<uint64_t>(count)};
    const daso_bucket_stats& was = a.stats[a.out[i]];
    if (i == 0 && a.cont) r = {was.grad_sq + r.grad_sq, was.delta_sq + r.delta_sq, was.nonfinite + r.nonfinite};
    a.stats[a.out[i]] = r;
    a.table[i] = daso::BucketSlots{0, 0, a.out[i], 1};
  }
}

static void model_step(const daso::StepArgs& a, int waves) {
  if (a.stats == nullptr) return;
  const int shift = daso::super_shift(waves);
  for (int i = 0; i < a.nb; ++i) {
    const int64_t bs = a.start[i], be = a.start[i + 1];
    const int64_t first = a.slot0 + daso::slot_of((bs >> shift) - a.sb0, i);
    EXPECT(inside(a.table + i, sizeof(*a.table)));
    a.table[i] = daso::BucketSlots{first, be > bs ? a.slot0 + daso::slot_of(((be - 1) >> shift) - a.sb0, i) + 8 : first, a.out[i],
                                   i == 0 ? a.cont : 0};
    for (int64_t sb = bs >> shift; be > bs && sb <= (be - 1) >> shift; ++sb)
      for (int w = 0; w < 8; ++w) {
        int64_t count = 0;
        for (int k = 0; k < waves; ++k) {
          const int64_t p = (sb << shift) + (k * 8 + w) * daso::kPiece;
          count += std::max<int64_t>(0, std::min(be, p + daso::kPiece) - std::max(bs, p));
        }
        daso::SlicePartial* s = a.partials + a.slot0 + daso::slot_of(sb - a.sb0, i) + w;
        EXPECT(inside(s, sizeof(*s)));
        *s = daso::SlicePartial{static_cast<double>(count), 2.0 * static_cast<double>(count), static_cast<uint64_t>(count)};
      }
  }
  if (a.done == nullptr) return;
  EXPECT(inside(a.done, 4) && *a.done == 0);
  for (int i = 0; i < a.nb; ++i) sum_buckets(a.partials, a.table + i, a.stats, 1);
}

// ------------------------------------------------------------- the HIP calls
extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  kernel_names[host] = name;
}
void __hipRegisterVar(void**, void* var, char*, char*, int, size_t size, int, int) { symbol_bytes[var] = size; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { return *d = 0, hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes) {
  ++mallocs;
  if (capturing) return ++mallocs_in_capture, hipErrorStreamCaptureUnsupported;
  allocated += bytes;
  *p = new_buffer(bytes);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* symbol) {
  static std::map<const void*, void*> made;
  if (!made.count(symbol)) made[symbol] = new_buffer(symbol_bytes.at(symbol));
  *p = made[symbol];
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t) {
  // the dispatch packet holds the work-items of each dimension in 32 bits
  EXPECT(uint64_t(grid.x) * block.x < (uint64_t(1) << 32) && uint64_t(grid.y) * block.y < (uint64_t(1) << 32));
  EXPECT(grid.x >= 1 && grid.y >= 1 && grid.z == 1 && grid.y < 65536 && lds <= 160 * 1024);
  const std::string& name = kernel_names.at(f);
  if (name.find("step_kernel") != std::string::npos) {
    const daso::StepArgs& a = **reinterpret_cast<daso::StepArgs**>(args);
    EXPECT(int64_t(grid.x) * grid.y >= a.nslices && a.nb >= 1 && a.nb <= daso::kLaunchBuckets);
    model_step(a, static_cast<int>(block.x) / 64);
    last_block = block.x;
    last_lds = static_cast<uint32_t>(lds);
    ++steps;
  } else if (name.find("bucket_kernel") != std::string::npos) {
    const daso::StepArgs& a = **reinterpret_cast<daso::StepArgs**>(args);
    EXPECT(grid.x == static_cast<uint32_t>(a.nb) && (a.stats == nullptr ? block.x == 64 : grid.y == 1 && block.x == 256));
    model_buckets(a);
    ++steps;
  } else if (name.find("stats_kernel") != std::string::npos) {
    const daso::StatsArgs& a = **reinterpret_cast<daso::StatsArgs**>(args);
    sum_buckets(a.partials, a.table, a.stats, grid.x);
    ++passes;
  } else {
    *static_cast<uint32_t*>(*reinterpret_cast<void**>(args[0])) = 0;  // clear_counter_kernel
  }
  return hipSuccess;
}
}  // extern "C"

// ------------------------------------------------------------------- the calls
static int (*fused)(const daso_sync_args*, hipStream_t);
static int (*fused_noalloc)(const daso_sync_args*, hipStream_t);

struct Call {
  int32_t g, P;
  std::vector<daso_bucket> buckets;
  bool noalloc = false;
  uint32_t flags = 0;
};

static int64_t elements(const std::vector<daso_bucket>& b) {
  int64_t n = 0;
  for (const auto& k : b) n += k.numel;
  return n;
}

// One call with statistics, checked bucket by bucket; returns the status.
static int run(const Call& c, hipStream_t stream) {
  const auto fake = [](int k) { return reinterpret_cast<void*>((uint64_t(1) << 62) + (uint64_t(k) << 40)); };
  const int64_t n = elements(c.buckets);
  std::vector<const float*> grads;
  std::vector<const uint16_t*> stale;
  for (int r = 0; r < c.g; ++r) grads.push_back(static_cast<float*>(fake(r)));
  for (int r = 0; r < c.P; ++r) stale.push_back(static_cast<uint16_t*>(fake(64 + r)));
  auto* stats = static_cast<daso_bucket_stats*>(new_buffer(c.buckets.size() * sizeof(daso_bucket_stats)));
  std::memset(static_cast<void*>(stats), 0xFF, c.buckets.size() * sizeof(daso_bucket_stats));
  daso_sync_args s;
  std::memset(&s, 0, sizeof(s));
  s.n = n;
  s.g = c.g;
  s.P = c.P;
  s.grads = grads.data();
  if (c.flags & DASO_EXCHANGE_F32) s.stale_f32 = reinterpret_cast<const float* const*>(stale.data());
  else s.stale = stale.data();
  s.params = static_cast<float*>(fake(130));
  s.momentum = static_cast<float*>(fake(131));
  s.buckets = c.buckets.data();
  s.nbuckets = static_cast<int32_t>(c.buckets.size());
  s.lr = 0.1f;
  s.mu = 0.9f;
  s.flags = c.flags;
  s.stats = stats;
  const int rc = (c.noalloc ? fused_noalloc : fused)(&s, stream);
  if (rc == DASO_OK)
    for (size_t k = 0; k < c.buckets.size(); ++k) {
      const auto want = c.buckets[k].numel;
      EXPECT(stats[k].grad_sq == static_cast<double>(want) && stats[k].delta_sq == 2.0 * static_cast<double>(want) &&
             stats[k].nonfinite == static_cast<uint64_t>(want));
    }
  buffers.erase(reinterpret_cast<char*>(stats));
  std::free(stats);
  return rc;
}

static std::vector<daso_bucket> even(int64_t n, int64_t size) {
  std::vector<daso_bucket> b;
  for (int64_t s = 0; s < n; s += size) b.push_back({s, std::min(size, n - s), static_cast<int32_t>(b.size() % 3), 0});
  return b;
}

static hipStream_t stream_at(int k) { return reinterpret_cast<hipStream_t>(static_cast<uintptr_t>(0x1000 + 64 * k)); }

static const std::pair<int, int> kShapes[] = {{4, 8}, {8, 32}, {4, 0}, {3, 5}, {9, 40}, {8, 16}};

// Random tables through both entry points, eager and captured after an eager call.
static void random_tables() {
  std::mt19937_64 rng(5);
  for (int trial = 0; trial < 300; ++trial) {
    Call c{kShapes[trial % 6].first, kShapes[trial % 6].second, {}};
    const int64_t n = 1 + static_cast<int64_t>(rng() % (trial % 5 ? 200000 : 5000000));
    int64_t pos = 0;
    while (pos < n) {
      const int64_t size = std::min<int64_t>(n - pos, static_cast<int64_t>(rng() % (1 + n / (1 + static_cast<int64_t>(rng() % 300)))));
      c.buckets.push_back({pos, size, static_cast<int32_t>(rng() % 4), 0});
      pos += size;
      if (c.buckets.size() > 3000) {
        c.buckets.push_back({pos, n - pos, 1, 0});
        pos = n;
      }
    }
    std::shuffle(c.buckets.begin(), c.buckets.end(), rng);
    what = "random table " + std::to_string(trial);
    EXPECT(run(c, stream_at(trial % 3)) == DASO_OK);
    capturing = true;
    EXPECT(run(c, stream_at(trial % 3)) == DASO_OK);
    capturing = false;
    c.noalloc = true;
    EXPECT(run(c, stream_at(trial % 3)) == DASO_OK);
  }
}

// A table so long that one statistics launch for all buckets would overflow the
// dispatch packet, and whose partials would fill a gigabyte.
static void long_table() {
  what = "4,200,000 buckets of one element";
  Call c{4, 2, even(4200000, 1)};
  EXPECT(run(c, stream_at(0)) == DASO_OK);
  for (size_t k = 0, pos = 0; k < c.buckets.size(); ++k) {  // every other launch with a large one
    c.buckets[k].start = static_cast<int64_t>(pos);
    c.buckets[k].numel = k % 256 == 5 ? 600 : 1;
    pos += static_cast<size_t>(c.buckets[k].numel);
  }
  EXPECT(run(c, stream_at(0)) == DASO_OK);
  EXPECT(allocated <= (size_t(64) << 20));
}

// A captured call that follows an eager one over as many elements on its stream finds
// room in the workspace, whatever its buckets and stream counts are: it must not allocate.
static void capture() {
  const std::vector<std::vector<daso_bucket>> tables = {
      even(30000001, 30000001), even(30000001, 6553600), even(30000001, 7001), even(30000001, 261), even(8000000, 97)};
  int stream = 10;
  for (const auto& warm : kShapes)
    for (const auto& shape : kShapes)
      for (size_t first = 0; first < 4; ++first) {
        const hipStream_t st = stream_at(stream++);
        what = "warm-up g=" + std::to_string(warm.first) + " table " + std::to_string(first);
        EXPECT(run(Call{warm.first, warm.second, tables[first]}, st) == DASO_OK);
        capturing = true;
        for (size_t k = 0; k < tables.size(); ++k) {
          what = "captured g=" + std::to_string(shape.first) + " P=" + std::to_string(shape.second) + " table " +
                 std::to_string(k) + " after g=" + std::to_string(warm.first) + " table " + std::to_string(first);
          EXPECT(run(Call{shape.first, shape.second, tables[k]}, st) == DASO_OK);
        }
        capturing = false;
        EXPECT(mallocs_in_capture == 0);
        mallocs_in_capture = 0;
      }
}

// The no-alloc entry point's array, no larger than its documented size, with more partials than it
// holds: of many buckets, of one bucket, of both.
static void fixed_array() {
  const int64_t big = (static_cast<int64_t>(DASO_NOALLOC_SCRATCH_BYTES) - 256 - 260) / 24 * 2048;  // at the limit
  for (const auto& shape : {std::pair<int, int>{4, 8}, {1, 0}, {9, 40}}) {
    for (int k = 0; k < 4; ++k) {
      Call c{shape.first, shape.second, {}, true};
      int64_t pos = 0;
      const auto add = [&](int64_t numel) {
        c.buckets.push_back({pos, numel, 1, 0});
        pos += numel;
      };
      if (k != 1) add(2047);
      if (k >= 1) add(big - (k == 1 ? 4096 : 80 * 2048));
      add(0);
      for (int i = 0; i < (k == 0 ? 170000 : k == 1 ? 0 : 300); ++i) add(i % 100 == 7 && i < 80000 ? 1001 : 1 + i % 3);
      what = "no-alloc, table " + std::to_string(k) + ", g=" + std::to_string(shape.first);
      steps = 0;
      EXPECT(run(c, stream_at(0)) == DASO_OK);
      EXPECT(k == 0 ? steps >= 170000 / 128 : steps >= 3);
      if (k == 1) {
        add(8192);
        EXPECT(run(c, stream_at(0)) == DASO_ENOSPACE);
      }
    }
  }
  for (const auto& s : symbol_bytes) EXPECT(s.second <= DASO_NOALLOC_SCRATCH_BYTES);
  EXPECT(symbol_bytes.size() == 1);
}

// The workgroup and LDS that the step's shapes are launched with, as "g P threads lds", and
// those of the longest short call and of the shortest beyond.
static void shapes() {
  for (int g : {4, 8})
    for (int P : {2, 4, 8, 16, 32}) {
      EXPECT(run(Call{g, P, even(25557032, 6553600)}, stream_at(0)) == DASO_OK);
      std::printf("shape %d %d %u %u\n", g, P, last_block, last_lds);
      for (int64_t n : {daso::kShortCall, daso::kShortCall + 1}) {
        EXPECT(run(Call{g, P, even(n, n)}, stream_at(0)) == DASO_OK);
        std::printf("%s %d %d %u %u\n", n > daso::kShortCall ? "shape" : "short", g, P, last_block, last_lds);
      }
    }
}

int main(int argc, char** argv) {
  if (argc != 3) return 2;
  void* lib = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
  if (lib == nullptr) return std::fprintf(stderr, "%s\n", dlerror()), 2;
  fused = reinterpret_cast<decltype(fused)>(dlsym(lib, "daso_fused_sync_step"));
  fused_noalloc = reinterpret_cast<decltype(fused_noalloc)>(dlsym(lib, "daso_fused_sync_step_noalloc"));
  const std::string scenario = argv[2];
  if (scenario == "random_tables") random_tables();
  else if (scenario == "long_table") long_table();
  else if (scenario == "capture") capture();
  else if (scenario == "fixed_array") fixed_array();
  else if (scenario == "shapes") shapes();
  else return 2;
  if (failures == 0) std::printf("launch model ok: %d step launches, %d statistics passes\n", steps, passes);
  return failures == 0 ? 0 : 1;
}
