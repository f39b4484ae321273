// CPU driver of the work-item tables (built and run by tests/test_host_split.py): the C ABI's
// source with the device memory calls replaced by host memory, whose allocations can be made
// to fail.  No kernel is launched.
#include "../paper_2605_26347_amd/csrc/wf_abi.cpp"

#include <cstdio>
#include <cstdlib>
#include <set>

static std::set<void*> g_live;
static int g_fail_at = -1;   // allocations until one fails; -1: none does
static bool g_failed = false;

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  if (g_fail_at == 0) {
    g_failed = true;
    return hipErrorOutOfMemory;
  }
  if (g_fail_at > 0) --g_fail_at;
  *p = std::malloc(n);
  g_live.insert(*p);
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (g_live.erase(p) != 1) {
    std::printf("free of an unknown block\n");
    std::exit(1);
  }
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  if (n) std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  if (n) std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "out of memory"; }
}

#define CHECK(c)                                              \
  if (!(c)) {                                                 \
    std::printf("line %d: %s\n", __LINE__, #c);               \
    std::exit(1);                                             \
  }

// One channel: rows of every patch class in a few tiles of 32 cells, in two bins.
static void fill(wf_op& op, std::vector<int> rows_of) {
  op.tile = 32;
  op.halo = 18;
  op.max_tsh = 1;
  op.Kx = op.Ky = 256;
  op.chans.resize(1);
  ChanOp& ch = op.chans[0];
  ch.P = 2;
  std::vector<uint32_t> meta, voff;
  std::vector<uint8_t> trow;
  const int sides[NCLS] = {9, 15, 21, 27, 31, 37};
  int64_t at = 0;
  uint32_t rnd = 1;
  for (int p = 0; p < ch.P; ++p)
    for (int c = 0; c < NCLS; ++c)
      for (size_t t = 0; t < rows_of.size(); ++t) {
        int tv, tu;
        tile_unmorton((uint32_t)t, &tv, &tu);
        RowGroup g{};
        g.voff = at;
        g.row0 = (int32_t)meta.size();
        g.nrows = rows_of[t];
        g.u0 = tu * op.tile - op.halo;
        g.v0 = tv * op.tile - op.halo;
        g.bin = p;
        g.cls = c;
        ch.groups.push_back(g);
        for (int r = 0; r < rows_of[t]; ++r) {
          rnd = rnd * 1664525u + 1013904223u;
          const int T = sides[c], off = (T - 1) / 2;
          meta.push_back(pack_meta((int)(rnd >> 27) + op.halo - off,
                                   (int)((rnd >> 22) & 31) + op.halo - off, T));
          trow.push_back((uint8_t)T);
          at += T * T;
        }
      }
  ch.nrows = (int64_t)meta.size();
  voff.resize(meta.size());
  std::vector<WorkItem> wis;
  ch.bin_tsh.assign(ch.P, 0);
  split_items(ch, trow.data(), meta.data(), 1024, op.tile, op.halo, wis, voff.data(),
              meta.data(), nullptr);
  auto up = [](DevBuf& b, const void* p, size_t n) {
    CHECK(dalloc(b, n) == WF_OK);
    std::memcpy(b.p, p, n);
  };
  up(ch.meta, meta.data(), 4 * meta.size());
  up(ch.voff, voff.data(), 4 * voff.size());
  up(ch.work, wis.data(), sizeof(WorkItem) * wis.size());
  CHECK(schedule_rows(ch, wis, meta.data(), nullptr) == WF_OK);
}

static bool held(const DevBuf& b, size_t bytes) {
  return b.p && g_live.count(b.p) && b.bytes >= bytes;
}

// Items and pieces cover each row of the channel once, within their tables.
static void covered(const ChanOp& ch) {
  CHECK(held(ch.work, sizeof(WorkItem) * ch.nwork));
  std::vector<int> hit(ch.nrows, 0);
  const WorkItem* wk = (const WorkItem*)ch.work.p;
  for (int64_t i = 0; i < ch.nwork; ++i)
    for (int r = 0; r < wk[i].nrows; ++r) ++hit[wk[i].row0 + r];
  for (int h : hit) CHECK(h == 1);
  std::fill(hit.begin(), hit.end(), 0);
  const WorkItem* pc = (const WorkItem*)ch.pieces.p;
  for (size_t k = 0; k < ch.pc_n.size(); ++k) {
    if (ch.pc_n[k] == 0) continue;
    CHECK(held(ch.pieces, sizeof(WorkItem) * (ch.pc_0[k] + ch.pc_n[k])));
    for (int i = ch.pc_0[k]; i < ch.pc_0[k] + ch.pc_n[k]; ++i)
      for (int r = 0; r < pc[i].nrows; ++r) ++hit[pc[i].row0 + r];
  }
  for (int h : hit) CHECK(h == 1);
}

// A re-split that runs out of memory, at each of its allocations, leaves the split in use.
static void failed_resplit() {
  wf_op op;
  fill(op, {3000, 70, 1, 500});
  ChanOp& ch = op.chans[0];
  covered(ch);
  const ItemTables was = ch;
  const std::vector<uint32_t> meta((uint32_t*)ch.meta.p, (uint32_t*)ch.meta.p + ch.nrows);
  const std::vector<int8_t> wide(ch.P, 1);
  const size_t blocks = g_live.size();
  int fails = 0;
  for (int k = 0;; ++k) {
    g_fail_at = k;
    g_failed = false;
    const wf_status st = retune_channel(&op, 0, 256, wide.data());
    g_fail_at = -1;
    if (!g_failed) {
      CHECK(st == WF_OK);
      break;
    }
    ++fails;
    CHECK(st == WF_ENOMEM);
    CHECK(g_live.size() == blocks);
    CHECK(ch.work.p == was.work.p && ch.pieces.p == was.pieces.p);
    CHECK(ch.pc_0 == was.pc_0 && ch.pc_n == was.pc_n && ch.nwork == was.nwork);
    CHECK(ch.cls_wi0 == was.cls_wi0 && ch.cls_nwi == was.cls_nwi);
    CHECK(ch.bin_tsh == was.bin_tsh && ch.max_rows == was.max_rows);
    CHECK(std::equal(meta.begin(), meta.end(), (uint32_t*)ch.meta.p));
    covered(ch);
  }
  CHECK(fails >= 2);
  CHECK(ch.max_rows == 256 && ch.bin_tsh == wide);
  CHECK(g_live.size() == blocks);
  covered(ch);
}

int main() {
  failed_resplit();
  std::printf("host split ok\n");
  return 0;
}
