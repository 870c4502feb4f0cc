// rlx_batch.hip -- batched generation: planner and one fused kernel.
//
// A batch is a list of requests, each a window [start, start + count) of one
// stream (values counted from field 0 of the record's current step).  The
// planner (host) cuts every request into segments of at most `seg_blocks`
// generator steps and groups segments of the same luxury level into work
// items of 64 lanes (64 / G segments of G lanes each).  One kernel then
// runs one wave per item; inside an item every segment is run by G lanes
// exactly as the plain kernel runs a record: lane l starts at the segment's
// block l (skip by 16-bit windows, section 2.4), then takes every G-th block
// with the multiplier A^G, converts (section 2.3) and stores through LDS.
// Records are only read.
//
// Segments are sorted by length (longest first) inside a level and items by
// cost, and the hardware dispatches waves in item order, so late waves get
// short items (longest-processing-time order); long requests are cut so
// that no item dominates the launch.  One wave per item (or a part of one,
// item_share), rather than persistent waves popping items from a counter,
// keeps the kernel's registers low: 118 VGPRs and 4 waves per SIMD.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "rlx.h"
#include "rlx_arith.hpp"
#include "rlx_device.hpp"
#include "rlx_internal.hpp"
#include "rlx_mfma.hpp"
#include "rlx_share.hpp"

using namespace rlx;
using namespace rlx::host;

namespace {

constexpr int MAX_LEVELS = 16;

// One segment: blocks block .. block + nblocks - 1 of record `state` (block 0
// is the record's current LCG state); field f of block block + t has output
// index jbase + 12 t + f and is written when that index is in [lo, hi).
struct Segment {
  uint64_t state;
  uint64_t block;
  int64_t jbase;
  int64_t lo;
  int64_t hi;
  uint32_t nblocks;
  uint32_t slot;  // luxury-level slot
};
static_assert(sizeof(Segment) == 48, "segment descriptor layout");

// Work item: segments seg0 .. seg0 + nseg - 1, all of level `slot`.
struct Item {
  uint32_t seg0;
  uint32_t nseg;
  uint32_t slot;
  uint32_t cost;  // longest segment, in blocks
};
static_assert(sizeof(Item) == 16, "item descriptor layout");

// Device-side header of a plan.  Everything a launch depends on that can
// change between updates lives here (not in kernel arguments), so a launch
// captured in a HIP graph replays whatever the plan holds at replay time.
struct Header {
  uint32_t reserved;
  uint32_t n_items;  // a multiple of GROUP; that many Items follow, then the Segments
  uint32_t pad[2];
  const uint32_t* C[MAX_LEVELS];  // folded multipliers A^(2^g) of each level
  const uint32_t* W[MAX_LEVELS];  // 16-bit window tables A^(j 65536^i) of each level
  const uint32_t* M[MAX_LEVELS];  // matrix-core step operands of each level
  uint32_t p[MAX_LEVELS];
};
static_assert(sizeof(Header) % 16 == 0, "items and segments stay aligned behind the header");

template <Out K, int LGS, bool MF>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(MF ? 3 : 4))) void k_batch(
    const rlx_state* __restrict__ st, const Header* __restrict__ hdr, uint64_t* __restrict__ out,
    uint32_t* __restrict__ err) {
  // header, items and segments lie one after the other (upload)
  const Item* __restrict__ items = reinterpret_cast<const Item*>(hdr + 1);
  const Segment* __restrict__ segs = reinterpret_cast<const Segment*>(items + hdr->n_items);
  constexpr uint32_t G = 1u << LGS;
  constexpr bool SHARED = MF && LGS >= 5;  // a segment's lanes fill half-waves
  __shared__ __align__(16) uint64_t stage[BLOCK * SLOT_VALUES];
  __shared__ mf_v4i af_lds[MF ? MF_FRAGS * 64 : 1];
  const uint32_t tid_blk = threadIdx.x;
  const uint32_t lane = tid_blk & (WAVE - 1);
  const uint32_t team = lane >> LGS;
  const uint32_t l = lane & (G - 1);
  const uint32_t n_items = __builtin_amdgcn_readfirstlane(hdr->n_items);
  {
    // Waves part n_items + it, part < share, share item `it`; the item count is
    // read here, so a captured launch shares out whatever an update left, and
    // waves past the parts exit at once.  All first parts come first: short
    // items have no others, and a launch of them is then the unshared one with
    // empty waves behind it (with an item's waves side by side 1000 requests
    // of 1024 values took 17 us against 10.6).
    const uint32_t wave = __builtin_amdgcn_readfirstlane(blockIdx.x * (BLOCK / WAVE) + tid_blk / WAVE);
    const uint32_t share = item_share(n_items, gridDim.x * (BLOCK / WAVE));
    if (wave >= n_items * share) return;  // the whole block: items come in groups of four
    const uint32_t part = wave / n_items, it = wave % n_items;
    // MF: the block stages its level's matrix-core operands for A^G in LDS;
    // its items (group_items) and the waves that share one have one level.
    // (With mixed blocks, whose waves read their operands through the L1 and
    // so had the loop a second time in the code, 8192 requests up to 2^14
    // values took 47 us against 43, 3000 up to 2^18 123 us against 119, and
    // the kernel 146 VGPRs against 118.)
    const Item item = items[it];
    const uint32_t slot = __builtin_amdgcn_readfirstlane(item.slot);
    const uint32_t per = part_blocks(item.cost, LGS, share);
    if (part != 0) {
      // the parts of the block's four items are all empty
      bool empty = true;
      for (uint32_t q = 0; q < BLOCK / WAVE; ++q) {
        const uint32_t cost = items[it - it % (BLOCK / WAVE) + q].cost;
        empty = empty && part * part_blocks(cost, LGS, share) >= cost;
      }
      if (empty) return;
    }
    if constexpr (MF) {
      mf_stage_operands(af_lds, hdr->M[slot] + (size_t)LGS * MF_LEVEL_WORDS, tid_blk, BLOCK);
      __syncthreads();
    }
    const uint32_t* __restrict__ ctabs = hdr->C[slot];
    const uint32_t* __restrict__ wtabs = hdr->W[slot];
    const uint32_t p = __builtin_amdgcn_readfirstlane(hdr->p[slot]);
    bool active = team < item.nseg;
    uint32_t si = item.seg0 + team;
    uint32_t nblocks = 0;
    uint32_t x[NW];
    uint64_t first = 0;  // this lane's first block: the segment's first + l
    // this wave's part of every segment: blocks from..from + nblocks - 1
    uint32_t from = 0;
    uint32_t w = 0;
    if (active) {
      const Segment& sg = segs[si];
      from = part * per;
      nblocks = from < sg.nblocks ? (sg.nblocks - from < per ? sg.nblocks - from : per) : 0u;
      active = nblocks != 0;
      if (SHARED || active) {
        // one half-wave is one segment if SHARED, so its lanes agree
        uint32_t pos, sp;
        uint32_t bad = 0;
        if constexpr (SHARED) {
          w = load_record_word(st, sg.state, true, tid_blk & 31u, pos, sp);
          bad = check_record_word(st, sg.state, w, 0u, sp, p);
        } else {
          load_record(st, sg.state, x, pos, sp);
          if (sp != p) bad |= RLX_ERR_BAD_P;
          if (geq_m(x)) bad |= RLX_ERR_BAD_X;
        }
        if (bad) {
          if (l == 0) atomicOr(err, bad);
          active = false;
        }
        first = sg.block + from + l;
      }
    }
    if (!__any(active)) return;
    if constexpr (SHARED) {
      // X_l = A^first X_0: the lowest 16-bit digit of `first` by the shared
      // product, the rest (segments that start past 65 536 steps) by windows
      uint32_t y[NW];
      mf_v4i b[6];
      if (!active) first = 0;
      load_words(wtabs + (size_t)(first & (WIN_COLS - 1u)) * NW, y);
      mf_shared_operands(y, b);
      uint8_t* const lds = reinterpret_cast<uint8_t*>(stage + (size_t)(tid_blk - lane) * SLOT_VALUES);
      mf_shared_digits(w, lds, lane);
      mf_shared_product<LGS == 6>(lds, b, x, lane);
      wave_sync();
      skip_windows(x, first & ~(uint64_t)(WIN_COLS - 1u), wtabs);
    } else {
      if (!active) {
        set_one(x);
        first = 0;
      }
      skip_windows(x, first, wtabs);
    }
    const uint32_t* __restrict__ ctab = ctabs + (size_t)LGS * FOLD_ROW_WORDS;
    // Output window of the segment: base[u] for u < span, with the
    // segment's first field at u = rel (rel >= -11; span < 2^30 because
    // segments hold at most 2^26 blocks).  Read after the lane set-up (the
    // index is made opaque so the load is not merged with the one above),
    // which keeps the window out of registers during it.
    asm volatile("" : "+v"(si));
    uint64_t* base = out;
    uint32_t span = 0;
    int32_t rel = 0;
    if (active) {
      const Segment& sg = segs[si];
      const int64_t jbase = sg.jbase + (int64_t)FIELDS * from;
      const int64_t lo = sg.lo > jbase ? sg.lo : jbase;
      const int64_t end = jbase + (int64_t)FIELDS * nblocks;
      const int64_t hi = sg.hi < end ? sg.hi : end;
      base = out + lo;
      span = hi > lo ? (uint32_t)(hi - lo) : 0u;
      rel = (int32_t)(jbase - lo);
    }
    for (uint32_t k = 0;; ++k) {
      const uint32_t t = l + (k << LGS);
      const bool live = active && t < nblocks;
      if (!__any(live)) break;
      convert_to_lds<K>(x, stage + (size_t)tid_blk * SLOT_VALUES, false);
      const int32_t u0 = rel + (int32_t)(FIELDS * (t - l));
      group_store<LGS>(stage, tid_blk, l, u0, span, active, base);
      if (__any(live && t + G < nblocks)) {
        if constexpr (MF) {
          mfma_step_split<MF_CROSS_LDS>(x, MfFromArray{af_lds, lane}, false);
        } else {
          step(x, constant_table(ctab), false, SgprBarrier());
        }
      }
    }
  }
}

// A plan's upload from its pinned staging, on the stream's own queue: a copy
// engine's hand-over to and from the compute queue costs about 20 us between
// two launches, this about 5 (256 requests up to 65 536 values, planning
// included: 39 us, now 21.5).
__global__ __launch_bounds__(BLOCK) void k_upload(const uint4* __restrict__ src, uint4* __restrict__ dst, uint32_t n) {
  const uint32_t i = blockIdx.x * BLOCK + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

}  // namespace

// ---------------------------------------------------------------------------
// host: the plan

struct rlx_plan {
  int device = 0;
  uint32_t lanes = 0, lg = 0;
  uint64_t seg_blocks = 0;
  uint64_t cap = 0;  // segments (and items, with MAX_EMPTY more) the device buffers hold
  Header* d_hdr = nullptr;  // header, items, segments: one buffer, one copy per upload
  Header* h_hdr = nullptr;  // staging for it: pinned, coherent (k_upload reads it)
  hipEvent_t uploaded = nullptr;
  uint64_t n_segs = 0, n_items = 0, total = 0;
  uint64_t extent = 0, records = 0;
};

namespace {

struct Planned {
  std::vector<Segment> segs;
  std::vector<Item> items;
  std::vector<uint32_t> ps;  // luxury level of each slot
  uint64_t total = 0;
  uint64_t extent = 0, records = 0;  // output elements and records the requests need
};

// Segments are laid out level by level; inside a level, the full segments
// (seg_blocks steps) in request order, then the partial ones (at most one per
// request) by decreasing length.  Items take 64/G consecutive segments of one
// level and run longest first.  Only the partial segments and the items that
// hold them are sorted, so planning is linear in the number of segments.
int plan_requests(const rlx_request* reqs, uint64_t n, uint32_t lg, uint64_t seg_blocks, Planned* out) {
  Planned pl;
  std::vector<uint32_t> slot_of(n, 0);
  std::vector<uint64_t> full_n, part_n;  // per level
  for (uint64_t r = 0; r < n; ++r) {
    const rlx_request& q = reqs[r];
    if (q.reserved != 0 || !valid_p(q.p)) return RLX_EINVAL;
    if (q.count == 0) continue;
    if (q.start > UINT64_MAX - q.count) return RLX_EINVAL;
    if (q.out_offset > (uint64_t)INT64_MAX / 2 || q.count > (uint64_t)INT64_MAX / 2) return RLX_EINVAL;
    uint32_t slot = 0;
    while (slot < pl.ps.size() && pl.ps[slot] != q.p) ++slot;
    if (slot == pl.ps.size()) {
      if (pl.ps.size() == MAX_LEVELS) return RLX_EINVAL;
      pl.ps.push_back(q.p);
      full_n.push_back(0);
      part_n.push_back(0);
    }
    slot_of[r] = slot;
    const uint64_t nb = (q.start % FIELDS + q.count + FIELDS - 1) / FIELDS;
    full_n[slot] += nb / seg_blocks;
    part_n[slot] += (nb % seg_blocks) != 0;
    pl.total += q.count;
    pl.extent = std::max(pl.extent, q.out_offset + q.count);
    pl.records = std::max(pl.records, q.state == UINT64_MAX ? q.state : q.state + 1);
  }
  const size_t levels = pl.ps.size();
  std::vector<uint64_t> full_at(levels), part_at(levels), part_end(levels);
  uint64_t total_segs = 0;
  for (size_t k = 0; k < levels; ++k) {
    full_at[k] = total_segs;
    part_at[k] = total_segs + full_n[k];
    total_segs += full_n[k] + part_n[k];
    part_end[k] = total_segs;
  }
  if (total_segs > 0xFFFFFFFFull) return RLX_EINVAL;
  pl.segs.resize(total_segs);
  for (uint64_t r = 0; r < n; ++r) {
    const rlx_request& q = reqs[r];
    if (q.count == 0) continue;
    const uint32_t slot = slot_of[r];
    const uint64_t b0 = q.start / FIELDS;
    const uint64_t f0 = q.start % FIELDS;
    const uint64_t nb = (f0 + q.count + FIELDS - 1) / FIELDS;
    for (uint64_t k = 0; k * seg_blocks < nb; ++k) {
      const uint64_t len = std::min<uint64_t>(seg_blocks, nb - k * seg_blocks);
      Segment& sg = pl.segs[len == seg_blocks ? full_at[slot]++ : part_at[slot]++];
      sg.state = q.state;
      sg.block = b0 + k * seg_blocks;
      sg.jbase = (int64_t)q.out_offset + (int64_t)(FIELDS * k * seg_blocks) - (int64_t)f0;
      sg.lo = (int64_t)q.out_offset;
      sg.hi = (int64_t)(q.out_offset + q.count);
      sg.nblocks = (uint32_t)len;
      sg.slot = slot;
    }
  }
  for (size_t k = 0; k < levels; ++k) {
    std::stable_sort(pl.segs.begin() + (part_end[k] - part_n[k]), pl.segs.begin() + part_end[k],
                     [](const Segment& a, const Segment& b) { return a.nblocks > b.nblocks; });
  }
  // items: those that start with a full segment (cost seg_blocks) first, in
  // level order, then the rest by decreasing cost
  const uint32_t per_item = WAVE >> lg;  // segments per 64-lane item
  std::vector<Item> rest;
  pl.items.reserve(total_segs / per_item + 2 * levels);
  for (size_t k = 0, i = 0; k < levels; ++k) {
    const uint64_t end = part_end[k];
    while (i < end) {
      Item it;
      it.seg0 = (uint32_t)i;
      it.slot = (uint32_t)k;
      it.cost = pl.segs[i].nblocks;
      it.nseg = (uint32_t)std::min<uint64_t>(per_item, end - i);
      i += it.nseg;
      if (it.cost == seg_blocks) {
        pl.items.push_back(it);
      } else {
        rest.push_back(it);
      }
    }
  }
  std::stable_sort(rest.begin(), rest.end(), [](const Item& a, const Item& b) { return a.cost > b.cost; });
  pl.items.insert(pl.items.end(), rest.begin(), rest.end());
  *out = std::move(pl);
  return RLX_OK;
}

// The items of a plan in launch order, regrouped so that the four items of a
// block have one level and its operands are staged once: the items that start
// with a full segment (level by level already) and the rest (by decreasing
// cost over all levels) each keep their order within a level; a level's items
// are taken when four have come up, and those left at the end of each part
// with empty items to make four.  Returns the items written: a multiple of
// four, at most items.size() + MAX_EMPTY.
constexpr size_t GROUP = BLOCK / WAVE;
constexpr size_t MAX_EMPTY = 2 * (GROUP - 1) * MAX_LEVELS;

size_t group_items(const std::vector<Item>& items, uint32_t full_cost, Item* out) {
  size_t n = 0, k = 0;
  for (int part = 0; part < 2; ++part) {
    Item held[MAX_LEVELS][GROUP];
    size_t have[MAX_LEVELS] = {};
    for (; k < items.size() && (part == 1 || items[k].cost == full_cost); ++k) {
      const uint32_t s = items[k].slot;
      held[s][have[s]++] = items[k];
      if (have[s] == GROUP) {
        for (const Item& it : held[s]) out[n++] = it;
        have[s] = 0;
      }
    }
    for (uint32_t s = 0; s < (uint32_t)MAX_LEVELS; ++s) {
      if (have[s] == 0) continue;
      for (size_t q = 0; q < GROUP; ++q) out[n++] = q < have[s] ? held[s][q] : Item{0, 0, s, 0};
    }
  }
  return n;
}

// Larger uploads (some 16 000 segments) go through the copy engine: their
// planning takes the host over 0.8 ms, beside which its hand-over is nothing.
constexpr size_t UPLOAD_KERNEL_BYTES = 1u << 20;
static_assert(sizeof(Segment) % sizeof(uint4) == 0, "uploads are whole 16-byte words");

int upload(rlx_plan* plan, const Planned& pl, hipStream_t s) {
  if (pl.segs.size() > plan->cap || pl.items.size() > plan->cap) return RLX_EINVAL;
  if (pl.ps.size() > MAX_LEVELS) return RLX_EINVAL;
  Header hd{};
  for (size_t k = 0; k < pl.ps.size(); ++k) {
    Tables t;
    const int rc = tables(pl.ps[k], s, &t);
    if (rc) return rc;
    hd.C[k] = t.C;
    hd.W[k] = t.W;
    hd.M[k] = t.P;
    hd.p[k] = pl.ps[k];
  }
  // the previous upload must have left the staging buffers
  if (hipEventSynchronize(plan->uploaded) != hipSuccess) return RLX_EHIP;
  Item* const items = reinterpret_cast<Item*>(plan->h_hdr + 1);
  const size_t n_items = group_items(pl.items, (uint32_t)plan->seg_blocks, items);
  hd.n_items = (uint32_t)n_items;
  *plan->h_hdr = hd;
  if (!pl.segs.empty())
    std::memcpy(reinterpret_cast<Segment*>(items + n_items), pl.segs.data(), pl.segs.size() * sizeof(Segment));
  const size_t bytes = sizeof(Header) + n_items * sizeof(Item) + pl.segs.size() * sizeof(Segment);
  if (bytes <= UPLOAD_KERNEL_BYTES) {
    const uint32_t quads = (uint32_t)(bytes / sizeof(uint4));
    k_upload<<<(quads + BLOCK - 1) / BLOCK, BLOCK, 0, s>>>(reinterpret_cast<const uint4*>(plan->h_hdr),
                                                          reinterpret_cast<uint4*>(plan->d_hdr), quads);
    if (hipGetLastError() != hipSuccess) return RLX_EHIP;
  } else if (hipMemcpyAsync(plan->d_hdr, plan->h_hdr, bytes, hipMemcpyHostToDevice, s) != hipSuccess) {
    return RLX_EHIP;
  }
  if (hipEventRecord(plan->uploaded, s) != hipSuccess) return RLX_EHIP;
  plan->n_segs = pl.segs.size();
  plan->n_items = pl.items.size();
  plan->total = pl.total;
  plan->extent = pl.extent;
  plan->records = pl.records;
  return RLX_OK;
}

void free_plan(rlx_plan* p) {
  if (!p) return;
  if (p->d_hdr) (void)hipFree(p->d_hdr);
  if (p->h_hdr) (void)hipHostFree(p->h_hdr);
  if (p->uploaded) (void)hipEventDestroy(p->uploaded);
  delete p;
}

// The plan's tables and descriptors live on the device it was created on.
bool on_plan_device(const rlx_plan* plan) {
  int dev;
  return hipGetDevice(&dev) == hipSuccess && dev == plan->device;
}

template <Out K>
int plan_launch(rlx_plan* plan, const rlx_state* states, void* out, void* stream) {
  if (!plan) return RLX_EINVAL;
  if (!on_plan_device(plan)) return RLX_EINVAL;
  if (!states || !out || !aligned(states, 16) || !aligned(out, 8)) return RLX_EINVAL;
  hipStream_t s = as_stream(stream);
  uint32_t* err;
  int rc = error_word(s, &err);
  if (rc) return rc;
  // One wave per item of a full plan (items never outnumber the segment
  // capacity, plus the empty ones), and for small plans more (item_share).
  // The grid depends only on the capacity, so a captured launch stays valid
  // after updates; waves past the current item count exit.
  const uint64_t waves =
      std::max<uint64_t>(plan->cap + MAX_EMPTY, std::min<uint64_t>(SHARE_WAVES, plan->cap * MAX_SHARE));
  const uint64_t blocks = (waves + (BLOCK / WAVE) - 1) / (BLOCK / WAVE);
  if (blocks == 0 || blocks > 0x7FFFFFFFull) return RLX_EINVAL;
  uint64_t* o = reinterpret_cast<uint64_t*>(out);
  const bool mf = rlx_step_kernel() == RLX_STEP_MFMA;
#define RLX_BATCH(L)                                                                                      \
  case L:                                                                                                 \
    if (mf) {                                                                                             \
      k_batch<K, L, true><<<(unsigned)blocks, BLOCK, 0, s>>>(states, plan->d_hdr, o, err);                \
    } else {                                                                                              \
      k_batch<K, L, false><<<(unsigned)blocks, BLOCK, 0, s>>>(states, plan->d_hdr, o, err);               \
    }                                                                                                     \
    break;
  switch (plan->lg) {
    RLX_BATCH(0) RLX_BATCH(1) RLX_BATCH(2) RLX_BATCH(3) RLX_BATCH(4) RLX_BATCH(5) RLX_BATCH(6)
    default: return RLX_EINVAL;
  }
#undef RLX_BATCH
  return launch_status();
}

}  // namespace

extern "C" {

int rlx_plan_create(rlx_plan** plan, const rlx_request* reqs, uint64_t n, uint32_t lanes, uint64_t seg_blocks,
                    uint64_t capacity_segments, void* stream) try {
  if (!plan) return RLX_EINVAL;
  *plan = nullptr;
  if (n > 0 && !reqs) return RLX_EINVAL;
  if (lanes == 0 || lanes > (uint32_t)WAVE || (lanes & (lanes - 1)) != 0) return RLX_EINVAL;
  if (seg_blocks == 0 || seg_blocks > RLX_MAX_SEG_BLOCKS) return RLX_EINVAL;
  // a plan never holds more than 2^32 - 1 segments (the planner's limit)
  if (capacity_segments > 0xFFFFFFFFull) return RLX_EINVAL;
  const uint32_t lg = (uint32_t)__builtin_ctz(lanes);
  Planned pl;
  int rc = plan_requests(reqs, n, lg, seg_blocks, &pl);
  if (rc) return rc;
  rlx_plan* p = new (std::nothrow) rlx_plan();
  if (!p) return RLX_ENOMEM;
  if (hipGetDevice(&p->device) != hipSuccess) {
    free_plan(p);
    return RLX_EHIP;
  }
  p->lanes = lanes;
  p->lg = lg;
  p->seg_blocks = seg_blocks;
  p->cap = std::max<uint64_t>({capacity_segments, (uint64_t)pl.segs.size(), 1});
  const size_t bytes = sizeof(Header) + (p->cap + MAX_EMPTY) * sizeof(Item) + p->cap * sizeof(Segment);
  if (hipMalloc(&p->d_hdr, bytes) != hipSuccess || hipHostMalloc(&p->h_hdr, bytes, hipHostMallocCoherent) != hipSuccess) {
    free_plan(p);
    return RLX_ENOMEM;
  }
  if (hipEventCreateWithFlags(&p->uploaded, hipEventDisableTiming) != hipSuccess ||
      hipEventRecord(p->uploaded, as_stream(stream)) != hipSuccess) {
    free_plan(p);
    return RLX_EHIP;
  }
  rc = upload(p, pl, as_stream(stream));
  if (rc) {
    free_plan(p);
    return rc;
  }
  *plan = p;
  return RLX_OK;
} catch (const std::bad_alloc&) {
  return RLX_ENOMEM;
}

int rlx_plan_update(rlx_plan* plan, const rlx_request* reqs, uint64_t n, void* stream) try {
  if (!plan || (n > 0 && !reqs)) return RLX_EINVAL;
  if (!on_plan_device(plan)) return RLX_EINVAL;
  Planned pl;
  int rc = plan_requests(reqs, n, plan->lg, plan->seg_blocks, &pl);
  if (rc) return rc;
  return upload(plan, pl, as_stream(stream));
} catch (const std::bad_alloc&) {
  return RLX_ENOMEM;
}

int rlx_plan_info(const rlx_plan* plan, uint64_t* segments, uint64_t* items, uint64_t* total_values) {
  if (!plan) return RLX_EINVAL;
  if (segments) *segments = plan->n_segs;
  if (items) *items = plan->n_items;
  if (total_values) *total_values = plan->total;
  return RLX_OK;
}

int rlx_plan_needs(const rlx_plan* plan, uint64_t* extent, uint64_t* records) {
  if (!plan) return RLX_EINVAL;
  if (extent) *extent = plan->extent;
  if (records) *records = plan->records;
  return RLX_OK;
}

int rlx_plan_generate_f64(rlx_plan* plan, const rlx_state* states, double* out, void* stream) {
  return plan_launch<Out::F64>(plan, states, out, stream);
}

int rlx_plan_generate_u64(rlx_plan* plan, const rlx_state* states, uint64_t* out, void* stream) {
  return plan_launch<Out::U64>(plan, states, out, stream);
}

int rlx_plan_generate_f32(rlx_plan* plan, const rlx_state* states, float* out, void* stream) {
  return plan_launch<Out::F32>(plan, states, out, stream);
}

int rlx_plan_dry_run(const rlx_request* reqs, uint64_t n, uint32_t lanes, uint64_t seg_blocks,
                     uint64_t* n_segments, uint64_t* n_items, uint64_t* total_values, uint64_t* segments,
                     uint64_t max_segments) try {
  if (n > 0 && !reqs) return RLX_EINVAL;
  if (lanes == 0 || lanes > (uint32_t)WAVE || (lanes & (lanes - 1)) != 0) return RLX_EINVAL;
  if (seg_blocks == 0 || seg_blocks > RLX_MAX_SEG_BLOCKS) return RLX_EINVAL;
  Planned pl;
  const int rc = plan_requests(reqs, n, (uint32_t)__builtin_ctz(lanes), seg_blocks, &pl);
  if (rc) return rc;
  if (n_segments) *n_segments = pl.segs.size();
  if (n_items) *n_items = pl.items.size();
  if (total_values) *total_values = pl.total;
  if (segments) {
    uint64_t row = 0;
    for (const Item& it : pl.items) {
      for (uint32_t k = 0; k < it.nseg && row < max_segments; ++k, ++row) {
        const Segment& sg = pl.segs[it.seg0 + k];
        uint64_t* r = segments + 6 * row;
        r[0] = sg.state;
        r[1] = sg.block;
        r[2] = (uint64_t)sg.jbase;
        r[3] = (uint64_t)sg.lo;
        r[4] = (uint64_t)sg.hi;
        r[5] = (uint64_t)sg.nblocks | ((uint64_t)sg.slot << 32);
      }
    }
  }
  return RLX_OK;
} catch (const std::bad_alloc&) {
  return RLX_ENOMEM;
}

int rlx_plan_destroy(rlx_plan* plan) {
  if (!plan) return RLX_OK;
  const bool ok = hipDeviceSynchronize() == hipSuccess;
  free_plan(plan);
  return ok ? RLX_OK : RLX_EHIP;
}

}  // extern "C"
