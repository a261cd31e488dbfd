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
        if (!o && n > 2000 && n_f < 1100) CHECK(covers("mfma2_operand_kernel", squares(n, 64)));
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

bool is_allocated(const void* p) {
  for (auto& a : allocated)
    if (a.first <= (uintptr_t)p && (uintptr_t)p < a.first + a.second) return true;
  return false;
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
  auto call = [&](int s, unsigned long long id, int64_t n_v, bool grows = false) {
    if (id) capture[stream(s)] = id;
    const int st = two_way(n_v, 2000, stream(s));
    capture.clear();
    if (st != CCC_OK) return false;
    for (const void* f : flags)
      if (!grows && f == last_tiles()->pair.flag) return false;
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
  CHECK(call(1, 9, 3000, true));  // outgrown within the capture: nodes hold the old one
  CHECK(frees == f0);
  const size_t held = flags.size() - 1;
  CHECK(call(1, 0, 6000, true));  // the eager call's own buffer alone goes
  CHECK(frees == f0 + 1);
  for (size_t k = 1; k < held; ++k) CHECK(is_allocated(flags[k]) && is_allocated(ops[k]));
  // graphs that are no more give their buffers back, behind a wait; others stay
  for (unsigned long long id = 100; id < 140; ++id) {
    CHECK(call(1, id, 300));
    if (id != 120) destroy_graph(id);
    CHECK(call(3, 0, 200 + (int)id, true));  // eager
    flags.pop_back();  // (its buffer is the same every time)
    ops.pop_back();
    CHECK(allocated.size() < 48);
  }
  CHECK(graphs.count(120) == 1);
  CHECK(is_allocated(flags[flags.size() - 20]) && is_allocated(ops[flags.size() - 20]));
  ccc_release_workspace();
  CHECK(allocated.empty() && used == 0);
  destroy_graph(120);  // later than its buffer
  CHECK(call(1, 0, 300));
  return 0;
}

int64_t operand_bytes(int64_t n_v, int64_t n_f) { return ccc::operand_bytes(n_v, n_f); }
bool on_operands() { return last_tiles()->pair.za != nullptr; }

// On a card that is nearly full a call takes the packed rows at once: no waits,
// no failed allocation, and nobody's buffers go; with room again it takes
// operands.  They never take more than half of what is free.
int nearly_full() {
  for (int s = 1; s <= 3; ++s) CHECK(two_way(400, 4000, stream(s)) == CCC_OK && on_operands());
  const long f0 = frees, s0 = syncs, m0 = mallocs;
  const size_t whole = card;
  card = used + (size_t(20) << 20);
  const auto before = allocated;
  for (int rep = 0; rep < 3; ++rep)
    for (int s = 1; s <= 3; ++s) {
      CHECK(operand_bytes(3000, 40000) > (int64_t(20) << 20));
      CHECK(two_way(3000, 40000, stream(s)) == CCC_OK && !on_operands());
      CHECK(two_way(2000, 25000, stream(s)) == CCC_OK && !on_operands());  // past half
    }
  CHECK(block(3000, 3000, 20000) == CCC_OK && !on_operands());  // (a workspace of its own)
  CHECK(ccc_2way_multi(fk<uint8_t>(), 3000, 20000, 20000, 4, fk<int32_t>(), nullptr,
                       fk<int32_t>(), nullptr, stream(2)) == CCC_OK);
  CHECK(frees == f0 && syncs == s0 && failed == 0 && mallocs == m0 + 1);
  for (auto& a : before) CHECK(allocated.count(a.first) == 1);
  CHECK(two_way(400, 4000, stream(2)) == CCC_OK && on_operands());  // fits what it has
  card = whole;
  CHECK(two_way(3000, 40000, stream(2)) == CCC_OK && on_operands());
  // what a call cannot do without evicts what no graph holds
  card = used + (size_t(4) << 20);
  launches.clear();
  CHECK(ccc_2way(fk<uint8_t>(), 600000, 40, 16, fk<int32_t>(), nullptr, nullptr, nullptr,
                 stream(3)) == CCC_OK);  // 9.6 MB of counts
  CHECK(failed == 1);
  return 0;
}

// Forty streams in turn: once each has its workspace, no call waits or allocates;
// streams without end do not add up, and seldom wait.
int many_streams() {
  for (int rep = 0; rep < 4; ++rep) {
    const long s0 = syncs, m0 = mallocs;
    for (int s = 1; s <= 40; ++s) {
      CHECK(two_way(400, 4000, stream(s)) == CCC_OK && on_operands());
      CHECK(select3(40, 100) == CCC_OK);
    }
    if (rep) CHECK(syncs == s0 && mallocs == m0);
  }
  const long s0 = syncs;
  for (int s = 100; s < 1100; ++s) {
    CHECK(two_way(400, 4000, stream(s)) == CCC_OK && on_operands());
    CHECK(allocated.size() <= 2 * 130);
  }
  CHECK(syncs - s0 <= 20);
  ccc_release_workspace();
  CHECK(allocated.empty());
  return 0;
}

// The 2-way tiles that calls take, by form and size.
int shapes() {
  ccc_opts acc = ccc_default_opts(), fin = ccc_default_opts();
  acc.flags = CCC_ACCUMULATE;
  fin.flags = CCC_FINALIZE;
  auto split = [] { return is(*last_tiles(), "mfma2_split"); };
  auto staged64 = [] { return is(*last_tiles(), "mfma2_operand_kernel") && is(*last_tiles(), "ELi2ELi2ELi4E"); };
  auto tables = [](int64_t n_v, int64_t n_f) {
    return ccc_2way(fk<uint8_t>(), n_v, n_f, ld_of(n_f), fk<int32_t>(), nullptr, fk<int32_t>(),
                    nullptr, nullptr);
  };
  // dense triangles with CCC rows: small tiles while small or short
  CHECK(two_way(3000, 4000) == CCC_OK && split());
  CHECK(two_way(9000, 1000) == CCC_OK && split());
  CHECK(two_way(5000, 4000) == CCC_OK && staged64());
  // the other forms: larger tiles earlier, and however short the fields
  CHECK(select2(2100, 20000) == CCC_OK && split());
  CHECK(select2(2400, 300) == CCC_OK && staged64());
  CHECK(select2(30000, 1000) == CCC_OK && staged64());
  CHECK(tables(3000, 300) == CCC_OK && staged64());
  CHECK(tables(8000, 1000) == CCC_OK && staged64());
  CHECK(block(1024, 4000, 4000, &fin) == CCC_OK && staged64());
  CHECK(block(256, 1000000, 1000, &fin) == CCC_OK && !split());
  CHECK(block(1000, 1000, 4000, &fin) == CCC_OK && split());
  CHECK(block(8000, 8000, 256, &acc) == CCC_OK && staged64());
  CHECK(block(8000, 8000, 8192, &acc) == CCC_OK && staged64());
  CHECK(block(1500, 1500, 8192, &acc) == CCC_OK && split());
  // beside the staged tiles, complete data's: 32 x 32 (1) or 128 x 256 (0)
  auto small_complete = [&](int status) {
    int one_plane = 0, small = 0;
    for (const Launch& l : launches) {
      one_plane += is(l, "mfma2_complete_operand");
      small += is(l, "mfma2_split_kernel");
    }
    launches.clear();
    return status != CCC_OK || one_plane + small != 1 ? -1 : small;
  };
  launches.clear();
  CHECK(small_complete(block(1700, 1700, 1000, &fin)) == 1);
  CHECK(small_complete(block(6000, 6000, 1000, &fin)) == 1);
  CHECK(small_complete(block(6000, 6000, 2000, &fin)) == 0);
  CHECK(small_complete(block(4096, 50000, 1000, &fin)) == 0);
  CHECK(small_complete(block(6000, 6000, 1000)) == 0);  // tables alone
  CHECK(small_complete(select2(3000, 8000)) == 1 && small_complete(select2(5000, 1000)) == 0);
  CHECK(small_complete(select2(2400, 16000)) == 1);
  CHECK(small_complete(tables(3000, 300)) == 0 && small_complete(tables(3000, 16000)) == 1);
  return 0;
}

// Whether the complete-data tiles of the last call stream their tables (Out 3) or not (0).
int streams() {
  const Launch* complete = nullptr;
  for (const Launch& l : launches)
    if (is(l, "mfma2_complete_operand")) complete = &l;
  if (!complete) return -1;
  return is(*complete, "OutE3") ? 1 : is(*complete, "OutE0") ? 0 : -1;
}
int streamed_tables() {
  ccc_opts fin = ccc_default_opts();
  fin.flags = CCC_FINALIZE;
  auto rect = [&](int64_t n_b, int64_t n_f) {
    launches.clear();
    return block(12000, n_b, n_f, &fin) == CCC_OK ? streams() : -2;
  };
  CHECK(rect(12000, 1500) == 0 && rect(12000, 3000) == 1 && rect(12000, 4000) == 1);
  CHECK(rect(12004, 4000) == 1 && rect(12001, 4000) == 0 && rect(12001, 16000) == 1);
  launches.clear();
  CHECK(two_way(16384, 8000) == CCC_OK && streams() == 0);
  launches.clear();
  CHECK(two_way(16384, 16384) == CCC_OK && streams() == 1);
  return 0;
}

// Which 3-way calls take the complete-data form.
int small_triples() {
  auto general_alone = [](int64_t n_v, int64_t n_f) {
    launches.clear();
    if (ccc_3way(fk<uint8_t>(), n_v, n_f, ld_of(n_f), fk<int32_t>(), fk<double>(), fk<int32_t>(),
                 nullptr, nullptr) != CCC_OK)
      return -1;
    for (const Launch& l : launches)
      if (is(l, "mfma3_complete")) return 0;
    return 1;
  };
  CHECK(general_alone(60, 2000) == 1 && general_alone(180, 200000) == 1);    // one turn
  CHECK(general_alone(200, 20000) == 1 && general_alone(200, 100000) == 0);  // two turns
  CHECK(general_alone(228, 20000) == 1 && general_alone(228, 40000) == 0);
  CHECK(general_alone(260, 1000) == 1 && general_alone(260, 10000) == 0);
  return 0;
}

// Where exact sums need the field-split tiles, large calls take the packed rows,
// complete data its one-plane tiles on operands.
int long_fields() {
  const int64_t most = 1864135;  // 9 n_f <= 2^24
  CHECK(two_way(8000, most) == CCC_OK && on_operands());
  launches.clear();
  CHECK(two_way(8000, most + 1) == CCC_OK && is(*last_tiles(), "12mfma2_kernel"));
  bool one_plane = false;
  for (const Launch& l : launches) one_plane |= is(l, "mfma2_complete_operand");
  CHECK(one_plane);
  CHECK(two_way(2400, 4000000) == CCC_OK && on_operands() && is(*last_tiles(), "split"));
  CHECK(block(40, 8000, 2000000) == CCC_OK && on_operands());
  CHECK(block(4000, 4000, 2000000) == CCC_OK && is(*last_tiles(), "12mfma2_kernel"));
  ccc_opts acc = ccc_default_opts();
  acc.flags = CCC_ACCUMULATE;
  CHECK(block(4000, 4000, 2000000, &acc) == CCC_OK && !on_operands());
  ccc_problem p{fk<uint8_t>(), 4000, 1900000, ld_of(1900000), fk<int32_t>(), fk<double>(),
                fk<int32_t>()};
  launches.clear();
  CHECK(ccc_2way_many(&p, 1, nullptr, nullptr) == CCC_OK);
  for (const Launch& l : launches) CHECK(!is(l, "operands_many"));
  return 0;
}

// A row range lays out the rows from its first tile on, no more.
int row_ranges() {
  const int64_t n_v = 100000, n_f = 10000;
  for (int64_t i0 : {0, 255, 256, 50000, 98976, 99990}) {
    ccc_release_workspace();
    launches.clear();
    CHECK(ccc_2way_rows(fk<uint8_t>(), n_v, n_f, ld_of(n_f), i0, i0 + 8, fk<int32_t>(),
                        fk<double>(), fk<int32_t>(), nullptr, nullptr) == CCC_OK);
    const Launch& p = launches[0];
    CHECK(is(p, "15operands_kernel"));
    const int64_t first = p.job.set[0].first, step = p.job.steps * 1024;
    CHECK(first == i0 / 256 * 16);
    const uintptr_t z = (uintptr_t)p.job.set[0].z;
    CHECK((uintptr_t)last_tiles()->pair.za + first * step == z);
    // what the blocks from `first` on take is there
    auto it = allocated.find(z);
    const int64_t need = (n_v / 16 - first) * step;
    CHECK(it != allocated.end() && (int64_t)it->second >= need);
    CHECK((int64_t)it->second <= need + (int64_t(16) << 20));
  }
  return 0;
}

// A block whose sides share counts adds to them one side after the other.
int shared_counts() {
  ccc_opts acc = ccc_default_opts();
  acc.flags = CCC_ACCUMULATE;
  auto passes = [&](int64_t n_a, int64_t n_b, int64_t offset) {
    launches.clear();
    int32_t* c = fk<int32_t>();
    if (ccc_2way_block(fk<uint8_t>(), n_a, 256, fk<uint8_t>(), n_b, 256, 1000, fk<int32_t>(), c,
                       c + 4 * offset, fk<double>(), &acc, nullptr) != CCC_OK)
      return -1;
    int k = 0;
    for (const Launch& l : launches)
      if (is(l, "15operands_kernel")) {
        ++k;
        if (l.job.set[0].blocks == 0 || (k == 2 && l.job.set[1].blocks != 0)) return -2;
      }
    return k;
  };
  CHECK(passes(100, 100, 0) == 2);   // the same counts
  CHECK(passes(100, 50, 99) == 2);   // one entry shared
  CHECK(passes(100, 50, 100) == 1);  // none
  return 0;
}

// A batch built under one operand limit is not replayed under another.
int batch_limits() {
  ccc_problem p{fk<uint8_t>(), 1000, 2000, ld_of(2000), fk<int32_t>(), fk<double>(), fk<int32_t>()};
  auto built = [&](const char* limit) {  // launches of a build: -1 on operands, 1 on packed rows
    if (limit)
      setenv("CCC_OPERAND_LIMIT", limit, 1);
    else
      unsetenv("CCC_OPERAND_LIMIT");
    launches.clear();
    if (ccc_2way_many(&p, 1, nullptr, nullptr) != CCC_OK) return 9;
    for (const Launch& l : launches)
      if (is(l, "operands_many")) return -1;
    return launches.empty() ? 0 : 1;
  };
  CHECK(built("0") == 1);
  CHECK(built("17179869184") == -1);  // 2^34, 0 in 32 bits
  CHECK(built("4294967296") == -1);
  CHECK(built("0") == 0 && built("17179869184") == 0);  // replays
  CHECK(built(nullptr) == 0);  // the default is 2^34
  return 0;
}

// CCC_SPLIT forces whole numbers in its range and nothing else.
int forced_splits() {
  auto workgroups = [](const char* split) -> int64_t {
    if (split)
      setenv("CCC_SPLIT", split, 1);
    else
      unsetenv("CCC_SPLIT");
    launches.clear();
    if (two_way(384, 250000) != CCC_OK) return -1;
    for (const Launch& l : launches)
      if (is(l, "mfma2_split_kernel")) return l.grid.x;
    return -2;
  };
  const int64_t tiles = 78, own = workgroups(nullptr);
  CHECK(own == tiles * 6);
  CHECK(workgroups("1") == tiles && workgroups("3") == tiles * 3 && workgroups("64") == tiles * 64);
  for (const char* bad : {"", "0", "-3", "65", "1000000", "3x", "abc"}) CHECK(workgroups(bad) == own);
  return 0;
}

// Over all streams and batches the library holds at most 16 GiB of operands.
int held() {
  const size_t limit = size_t(16) << 30, rest = size_t(64) << 20;
  int on = 0;
  for (int s = 1; s <= 12; ++s) {
    CHECK(two_way(65536, 200000, stream(s)) == CCC_OK);  // 3.3 GB
    on += on_operands();
    CHECK(used <= limit + rest);
  }
  CHECK(on == 5);
  std::vector<ccc_problem> p(1, ccc_problem{fk<uint8_t>(), 40000, 100000, ld_of(100000),
                                            fk<int32_t>(), fk<double>(), fk<int32_t>()});
  for (int k = 0; k < 6; ++k) {  // 1 GB each
    p[0].tables = fk<int32_t>(1024 * k);
    CHECK(ccc_2way_many(p.data(), 1, nullptr, nullptr) == CCC_OK);
    CHECK(used <= limit + rest);
  }
  ccc_release_workspace();
  CHECK(used == 0);
  for (int k = 0; k < 6; ++k) {
    p[0].tables = fk<int32_t>(1024 * k);
    CHECK(ccc_2way_many(p.data(), 1, nullptr, nullptr) == CCC_OK);
  }
  CHECK(used > size_t(5) << 30);  // operands again
  // what a graph held is free again soon after it is gone
  ccc_release_workspace();
  for (unsigned long long id = 200; id < 203; ++id) {
    capture[stream(1)] = id;
    CHECK(two_way(65536, 300000, stream(1)) == CCC_OK && on_operands());  // 4.9 GB each
    capture.clear();
  }
  CHECK(two_way(65536, 300000, stream(2)) == CCC_OK && !on_operands());
  destroy_graph(201);
  CHECK(two_way(65536, 300000, stream(2)) == CCC_OK && on_operands());
  return 0;
}

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  int r = 2;
  if (what == "launch_limits") r = launch_limits();
  if (what == "captures") r = captures();
  if (what == "nearly_full") r = nearly_full();
  if (what == "held") r = held();
  if (what == "many_streams") r = many_streams();
  if (what == "shapes") r = shapes();
  if (what == "streamed_tables") r = streamed_tables();
  if (what == "small_triples") r = small_triples();
  if (what == "long_fields") r = long_fields();
  if (what == "row_ranges") r = row_ranges();
  if (what == "shared_counts") r = shared_counts();
  if (what == "batch_limits") r = batch_limits();
  if (what == "forced_splits") r = forced_splits();
  if (r == 2) printf("no such scenario\n");
  if (r == 0) printf("ok\n");
  return r;
}
