// CPU driver of host decisions and of the work-item tables (built and run by
// tests/test_host_split.py): the C ABI's source with the device memory calls replaced by host
// memory, whose allocations can be made to fail.  No kernel is launched.
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
hipError_t hipMemset(void* d, int v, size_t n) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t)1;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t)1;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "out of memory"; }
}

#define CHECK(c)                                              \
  if (!(c)) {                                                 \
    std::printf("line %d: %s\n", __LINE__, #c);               \
    std::exit(1);                                             \
  }

// One channel: rows of every patch class in a few tiles of 32 cells, in two bins.
static void fill(wf_op& op, std::vector<int> rows_of, wf_store store = WF_STORE_F32) {
  op.opt.store = store;
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
  CHECK(schedule_rows(ch, wis, meta.data(), op.opt.store, nullptr) == WF_OK);
}

static bool held(const DevBuf& b, size_t bytes) {
  return b.p && g_live.count(b.p) && b.bytes >= bytes;
}

static const CutItem* cuts_of(const ChanOp& ch) {
  return (const CutItem*)((const char*)ch.pieces.p + ch.cuts_at);
}
static const CutPart* parts_of(const ChanOp& ch) {
  return (const CutPart*)((const char*)ch.pieces.p + ch.parts_at);
}

// Items and pieces cover each row of the channel once, within their tables.
static void covered(const ChanOp& ch) {
  CHECK(held(ch.work, sizeof(WorkItem) * ch.nwork));
  std::vector<int> hit(ch.nrows, 0);
  const WorkItem* wk = (const WorkItem*)ch.work.p;
  for (int64_t i = 0; i < ch.nwork; ++i)
    for (int r = 0; r < wk[i].nrows; ++r) ++hit[wk[i].row0 + r];
  for (int h : hit) CHECK(h == 1);
  const WorkItem* pc = (const WorkItem*)ch.pieces.p;
  const size_t nk = ch.pc_n.size() / 2;   // de-gridding's, then the scattering kernels'
  for (size_t use = 0; use < 2; ++use) {
    std::fill(hit.begin(), hit.end(), 0);
    for (size_t k = use * nk; k < (use + 1) * nk; ++k) {
      if (ch.pc_n[k] == 0) continue;
      CHECK(held(ch.pieces, sizeof(WorkItem) * (ch.pc_0[k] + ch.pc_n[k])));
      for (int i = ch.pc_0[k]; i < ch.pc_0[k] + ch.pc_n[k]; ++i)
        for (int r = 0; r < pc[i].nrows; ++r) ++hit[pc[i].row0 + r];
    }
    for (int h : hit) CHECK(h == 1);
  }
}

// Each cut item is covered by its pieces: their boxes inside its box, their slots apart and inside
// the buffer, and nothing but pieces of whole items adds into the grid by itself.
static void cut_items_meet(const ChanOp& ch) {
  const WorkItem* wk = (const WorkItem*)ch.work.p;
  const WorkItem* pc = (const WorkItem*)ch.pieces.p;
  const CutItem* cuts = cuts_of(ch);
  const CutPart* parts = parts_of(ch);
  struct B {
    int u0, v0, w, h;
  };
  auto box = [](int32_t b) {
    const uint32_t x = (uint32_t)b;
    return B{(int)(x & 255), (int)((x >> 8) & 255), (int)((x >> 16) & 255), (int)(x >> 24)};
  };
  const size_t nk = ch.pc_n.size() / 2;
  int64_t largest = 0;
  for (size_t bin = 0; bin < ch.cut_n.size(); ++bin) {
    // pieces of the bin by slot; the items that they come from
    std::vector<std::pair<int, const WorkItem*>> by_slot;
    size_t whole = 0;
    for (int c = 0; c < NCLS; ++c)
      for (int i = 0; i < ch.pc_n[nk + bin * NCLS + c]; ++i) {
        const WorkItem& p = pc[ch.pc_0[nk + bin * NCLS + c] + i];
        if (p.bin >= 0) by_slot.push_back({p.bin, &p});
        else ++whole;
      }
    std::sort(by_slot.begin(), by_slot.end());
    size_t at = 0;
    int64_t cells = 0, items = 0;
    CHECK(held(ch.pieces, ch.cuts_at + sizeof(CutItem) * (ch.cut_0[bin] + ch.cut_n[bin])));
    for (int i = 0; i < ch.cut_n[bin]; ++i) {
      const CutItem& it = cuts[ch.cut_0[bin] + i];
      const B ib = box(it.box);
      CHECK(it.nparts > 1);
      CHECK(held(ch.pieces, ch.parts_at + sizeof(CutPart) * (it.part0 + it.nparts)));
      CHECK(box_lines(it.box) <= ch.cut_lines[bin]);
      int rows = 0;
      const WorkItem* from = nullptr;
      for (int j = 0; j < it.nparts; ++j, ++at) {
        const CutPart& q = parts[it.part0 + j];
        CHECK(at < by_slot.size() && by_slot[at].first == q.slot && q.slot == cells);
        const WorkItem& p = *by_slot[at].second;
        CHECK(p.box == q.box && p.u0 == it.u0 && p.v0 == it.v0);
        const B b = box(q.box);
        CHECK(b.u0 >= ib.u0 && b.v0 >= ib.v0 && b.u0 + b.w <= ib.u0 + ib.w &&
              b.v0 + b.h <= ib.v0 + ib.h);
        for (int64_t k = 0; k < ch.nwork; ++k)
          if (p.row0 >= wk[k].row0 && p.row0 < wk[k].row0 + wk[k].nrows) {
            CHECK(!from || from == &wk[k]);
            from = &wk[k];
          }
        rows += p.nrows;
        cells += (int64_t)b.w * b.h;
      }
      CHECK(from && rows == from->nrows && it.box == from->box);
      ++items;
    }
    CHECK(at == by_slot.size());
    int64_t in_bin = 0;
    for (int64_t k = 0; k < ch.nwork; ++k) in_bin += wk[k].bin == (int)bin;
    CHECK(items + (int64_t)whole == in_bin);
    largest = std::max(largest, cells);
  }
  CHECK(largest == ch.sum_cells);
}

// A re-split that runs out of memory, at each of its allocations, leaves the split in use.
static void failed_resplit() {
  wf_op op;
  fill(op, {3000, 70, 1, 500});
  ChanOp& ch = op.chans[0];
  covered(ch);
  cut_items_meet(ch);
  CHECK(ch.cut_n[0] > 0);
  op.br.resize(2);
  CHECK(grow_sums(&op) == WF_OK);
  const double rows = 1e6;   // the channel's other bytes
  ch.info.mem_g_bytes = rows + item_bytes(ch);
  const ItemTables was = ch;
  const void* sums = op.br[1].sums.p;
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
    CHECK(ch.info.mem_g_bytes == rows + item_bytes(was));
    CHECK(ch.work.p == was.work.p && ch.pieces.p == was.pieces.p);
    CHECK(ch.pc_0 == was.pc_0 && ch.pc_n == was.pc_n && ch.nwork == was.nwork);
    CHECK(ch.cls_wi0 == was.cls_wi0 && ch.cls_nwi == was.cls_nwi);
    CHECK(op.br[0].sums.bytes == op.br[1].sums.bytes && op.br[1].sums.p == sums);
    CHECK(sizeof(double2) * ch.sum_cells <= op.br[1].sums.bytes);
    CHECK(ch.bin_tsh == was.bin_tsh && ch.max_rows == was.max_rows);
    CHECK(std::equal(meta.begin(), meta.end(), (uint32_t*)ch.meta.p));
    covered(ch);
  }
  CHECK(fails >= 2);
  CHECK(ch.max_rows == 256 && ch.bin_tsh == wide);
  CHECK(item_bytes(ch) != item_bytes(was) && ch.info.mem_g_bytes == rows + item_bytes(ch));
  CHECK(item_bytes(ch) >= sizeof(WorkItem) * 2.0 * ch.nwork);   // items and their pieces
  CHECK(g_live.size() == blocks);
  covered(ch);
  cut_items_meet(ch);
  CHECK(held(op.br[0].sums, sizeof(double2) * ch.sum_cells));
  CHECK(held(op.br[1].sums, sizeof(double2) * ch.sum_cells));
}

// A lane taken before a re-split launches on the buffers that the re-split left.
static void lane_after_resplit() {
  wf_op op;
  fill(op, {200, 70, 1, 100});
  ChanOp& ch = op.chans[0];
  op.br.resize(1);
  CHECK(grow_sums(&op) == WF_OK);
  const Lane L = lane_of(&op, 0, nullptr);
  const size_t was = op.br[0].sums.bytes;
  const std::vector<int8_t> wide(ch.P, 1);
  CHECK(retune_channel(&op, 0, 1024, wide.data()) == WF_OK);
  CHECK(op.br[0].sums.bytes > was);
  const RowPieces pc = pieces_of(&op, ch, 0, L, true);
  CHECK(pc.sums == op.br[0].sums.p && g_live.count(pc.sums));
  CHECK(g_live.count((void*)pc.items) && pc.cuts == cuts_of(ch));
}

// Branches that run out of memory, at each of their allocations, leave a complete first one.
static void failed_branches() {
  wf_op op;
  fill(op, {3000, 70, 1, 500});
  op.shape = wf_image_shape{128, 128, 1e-5};
  ChanOp& ch = op.chans[0];
  ch.bin_nrows.assign(ch.P, 1);
  ch.bin_taps.assign(ch.P, 1);
  ch.active_tile_frac.assign(ch.P, 1.0);
  CHECK(set_branches(&op, 1) == WF_OK);
  const Branch one = op.br[0];
  const size_t blocks = g_live.size(), grid = sizeof(float2) * 256 * 256;
  auto whole = [&](const Branch& b) {
    return held(b.X, grid) && held(b.Y, grid) && held(b.A, grid / 2) &&
           held(b.sums, sizeof(double2) * ch.sum_cells);
  };
  CHECK(whole(one) && ch.sum_cells > 0);
  for (int k = 0;; ++k) {
    g_fail_at = k;
    g_failed = false;
    const wf_status st = set_branches(&op, 2);
    g_fail_at = -1;
    if (!g_failed) {
      CHECK(st == WF_OK && k == 5);   // grids, half image, partial sums, image sum
      break;
    }
    CHECK(st == WF_ENOMEM && g_live.size() == blocks);
    CHECK(op.nbranch == 1 && op.br.size() == 1 && op.br[0].X.p == one.X.p && whole(op.br[0]));
    CHECK(op.segs.size() == 1 && op.segs[0].branch == 0 && op.segs[0].direct);
    CHECK(op.segs[0].bins.size() == 2);
  }
  CHECK(op.nbranch == 2 && whole(op.br[0]) && whole(op.br[1]));
}

// Few rows, rows in one item, items at the pieces' smallest size, and many items.
static void pieces_of_items() {
  for (const std::vector<int>& rows : {std::vector<int>{1}, {64}, {65}, {1025}, {0, 63, 64, 129},
                                       {5000, 1, 1, 700, 64, 65, 2000, 333}}) {
    for (wf_store store : {WF_STORE_F32, WF_STORE_F16}) {
      wf_op op;
      fill(op, rows, store);
      covered(op.chans[0]);
      cut_items_meet(op.chans[0]);
    }
  }
}

// The FP32 series of the modulation serve the long rows only, and there within their bounds.
static void modulation_form() {
  for (int nx = 8; nx <= 8192; nx *= 2)
    for (int ny : {8, 512, 8192}) {
      const wf_image_shape small{nx, ny, 1e-5};
      CHECK(series_modulation(small, 2 * nx, 100.0) == (nx >= 1024));
      CHECK(!series_modulation(small, 2 * nx, 1e11));
    }
  CHECK(!series_modulation(wf_image_shape{1024, 1024, 2e-4}, 2048, 0.0));
}

int main() {
  modulation_form();
  pieces_of_items();
  failed_resplit();
  lane_after_resplit();
  failed_branches();
  std::printf("host split ok\n");
  return 0;
}
