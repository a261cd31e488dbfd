// Scenarios over the library's host code with a HIP runtime of the host alone
// (fake_hip.h): what each call launches, allocates and waits for.  Takes the
// scenario's name; prints "ok" and exits 0, or names the first failure.
#include "fake_hip.h"

using namespace fake;

#define CHECK(cond)                                                          \
  do {                                                                       \
    if (!(cond)) {                                                           \
      printf("FAIL line %d: %s\n", __LINE__, #cond);                         \
      for (const Launch& l : launches)                                       \
        printf("  %s grid %u %u block %u\n", l.kernel.c_str(), l.grid.x, l.grid.y, l.block.x); \
      return 1;                                                              \
    }                                                                        \
  } while (0)

template <typename T>
T* fk(uintptr_t off = 0) {
  return reinterpret_cast<T*>(uintptr_t(0x10000) + off);
}
int64_t ld_of(int64_t n_f) { return (n_f + 63) / 64 * 16; }

int two_way(int64_t n_v, int64_t n_f, hipStream_t s = nullptr, const ccc_opts* o = nullptr) {
  return ccc_2way(fk<uint8_t>(), n_v, n_f, ld_of(n_f), fk<int32_t>(), fk<double>(), fk<int32_t>(),
                  o, s);
}
int select2(int64_t n_v, int64_t n_f, const ccc_opts* o = nullptr) {
  const ccc_selection sel{fk<int64_t>(), fk<double>(), nullptr, 100, fk<unsigned long long>()};
  return ccc_2way_select(fk<uint8_t>(), n_v, n_f, ld_of(n_f), 0.5, &sel, fk<int32_t>(), o, nullptr);
}
int select3(int64_t n_v, int64_t n_f, const ccc_opts* o = nullptr) {
  const ccc_selection sel{fk<int64_t>(), fk<double>(), nullptr, 100, fk<unsigned long long>()};
  return ccc_3way_select(fk<uint8_t>(), n_v, n_f, ld_of(n_f), 0.5, &sel, fk<int32_t>(), o, nullptr);
}
int block(int64_t n_a, int64_t n_b, int64_t n_f, const ccc_opts* o = nullptr) {
  return ccc_2way_block(fk<uint8_t>(), n_a, ld_of(n_f), fk<uint8_t>(), n_b, ld_of(n_f), n_f,
                        fk<int32_t>(), fk<int32_t>(), fk<int32_t>(0x100000), fk<double>(), o,
                        nullptr);
}

// Tiles of `side` of the triangle of n rows, of which the last has no pair.
int64_t squares(int64_t n, int64_t side) {
  const int64_t T = (n + side - 1) / side, rows = (n - 1 + side - 1) / side;
  return rows * T - rows * (rows - 1) / 2;
}

// The launches of the kernel named by `part` cover workgroups 0 .. total - 1, in order.
bool covers(const char* part, int64_t total) {
  int64_t next = 0;
  for (const Launch& l : launches)
    if (is(l, part)) {
      if (l.pair.tile_base != next) return false;
      next += l.grid.x;
    }
  return next == total;
}

// Every call whose sizes are accepted has launches that the runtime accepts.
int launch_limits() {
  ccc_opts pop = ccc_default_opts(), i8 = ccc_default_opts();
  pop.path = CCC_PATH_POPCOUNT;
  i8.operands = CCC_OPERANDS_INT8;
  for (const ccc_opts* o : {(const ccc_opts*)nullptr, (const ccc_opts*)&i8, (const ccc_opts*)&pop}) {
    for (int64_t n : {2000, 185344, 185345, 200000, 524289, 700000}) {
      for (int64_t n_f : {1000, 1025, 9000}) {
        launches.clear();
        CHECK(select2(n, n_f, o) == CCC_OK);
        if (!o && n_f == 1000) CHECK(covers("mfma2_split_kernel", squares(n, 32)));
        if (o == &pop) CHECK(covers("pop2_kernel", squares(n, 64)));
      }
    }
    launches.clear();
    CHECK(block(100000000, 3, 40, o) == CCC_OK);  // rows past 2^32 / 64
    CHECK(block(3, 100000000, 40, o) == CCC_OK);
    launches.clear();
    CHECK(select3(8200, 100, o) == CCC_OK);
    int64_t next = 0;  // of the last kernel, the one that every data takes
    for (const Launch& l : launches)
      if (l.kernel == launches.back().kernel) {
        CHECK(l.base == next && l.count == l.grid.x);
        next += l.count;
      }
    CHECK(next > (int64_t(1) << 24));
  }
  for (int s : {2, 3, 4}) {
    launches.clear();
    CHECK(ccc_2way_multi(fk<uint8_t>(), 400000, 100, 112, s, fk<int32_t>(), nullptr, fk<int32_t>(),
                         nullptr, nullptr) == CCC_OK);
  }
  return 0;
}

// The workspace of the last 2-way call: its flag and its operands.
const Launch* last_tiles() {
  for (size_t k = launches.size(); k-- > 0;)
    if (is(launches[k], "mfma2_")) return &launches[k];
  return nullptr;
}

// A capture shares its workspace with no other capture, no other stream and no
// eager call, and what it was given stays where it is.
int captures() {
  std::vector<const void*> flags, ops;
  auto call = [&](int s, unsigned long long id, int64_t n_v) {
    if (id) capture[stream(s)] = id;
    const int st = two_way(n_v, 2000, stream(s));
    capture.clear();
    if (st != CCC_OK) return false;
    for (const void* f : flags)
      if (f == last_tiles()->pair.flag) return false;
    for (const void* z : ops)
      if (z == last_tiles()->pair.za) return false;
    flags.push_back(last_tiles()->pair.flag);
    ops.push_back(last_tiles()->pair.za);
    return true;
  };
  CHECK(call(1, 0, 300));
  CHECK(call(1, 7, 300));   // beside the stream's eager calls
  CHECK(call(1, 8, 300));   // another capture on the stream
  CHECK(call(1, 9, 300));
  CHECK(call(2, 9, 300));   // a fork of that capture
  CHECK(call(2, 0, 300));
  const long f0 = frees;
  CHECK(call(1, 9, 3000));  // outgrown within the capture: nodes hold the old one
  CHECK(frees == f0);
  const size_t held = flags.size() - 1;
  CHECK(call(1, 0, 6000));  // the eager call's own buffer alone goes
  for (size_t k = 1; k < held; ++k) {
    bool found = false;
    for (auto& a : allocated)
      if (a.first <= (uintptr_t)flags[k] && (uintptr_t)flags[k] < a.first + a.second) found = true;
    CHECK(found);
  }
  // graphs that are no more give their buffers back, behind a wait; others stay
  for (unsigned long long id = 100; id < 140; ++id) {
    CHECK(call(1, id, 300));
    if (id != 120) destroy_graph(id);
    CHECK(call(3, 0, 200 + (int)id));  // eager
    flags.pop_back();  // (its buffer is the same every time)
    ops.pop_back();
    CHECK(allocated.size() < 24);
  }
  const void* live = flags[flags.size() - 20];
  CHECK(graphs.count(120) == 1);
  bool found = false;
  for (auto& a : allocated) found |= a.first <= (uintptr_t)live && (uintptr_t)live < a.first + a.second;
  CHECK(found);
  ccc_release_workspace();
  CHECK(allocated.empty() && used == 0);
  destroy_graph(120);  // later than its buffer
  CHECK(call(1, 0, 300));
  return 0;
}

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  int r = 2;
  if (what == "launch_limits") r = launch_limits();
  if (what == "captures") r = captures();
  if (r == 2) printf("no such scenario\n");
  if (r == 0) printf("ok\n");
  return r;
}
