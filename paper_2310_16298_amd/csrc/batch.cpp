// Batched launch: many grids of uneven sizes advanced together, one
// persistent launch per kernel group and step (declared in stencil.h).
#include <algorithm>
#include <cstring>
#include <map>
#include <new>
#include <set>
#include <tuple>
#include <vector>

#include "kernels_rows3d.hpp"
#include "runtime.hpp"

using namespace stencil;

namespace {

struct Group {
  Kernel k;                     // shared kernel (items = 0 here; per grid in the table)
  std::vector<BatchGrid> grids;
  int64_t total = 0;            // work items over the group's grids
  unsigned blocks = 0;          // persistent workgroups of one launch
  const BatchGrid* d_table = nullptr;
};

// The grids whose plans the library time-blocked (time block T) with the
// same T-step kernel.  A run advances them in launches of at most T steps:
// by_size[s] lists the groups (one per kernel) that advance s steps in one
// launch, s = 1 .. T (s = 1: the plans' one-step kernels).
struct TbClass {
  int T = 1;
  std::vector<std::vector<size_t>> by_size;
};

// Launch sizes of a class's run of `steps` steps: the fewest launches of at
// most T steps whose count has the parity of `steps` (every grid of the
// batch then ends in buffer steps % 2), sizes as even as possible.
std::vector<int> tb_schedule(int64_t steps, int T) {
  std::vector<int> sizes;
  if (steps <= 0) return sizes;
  int64_t L = (steps + T - 1) / T;
  if ((L & 1) != (steps & 1)) ++L;  // L <= steps: steps >= 2 whenever the parity needs one more launch
  const int64_t base = steps / L, extra = steps % L;
  for (int64_t l = 0; l < L; ++l) sizes.push_back((int)(base + (l < extra ? 1 : 0)));
  return sizes;
}

}  // namespace

struct stencil_batch_s {
  int device = -1;
  int32_t count = 0;
  std::vector<Group> groups;
  std::vector<size_t> plain;      // groups of one step per launch: `steps` launches each
  std::vector<TbClass> classes;   // time-blocked grids
  void* d_tables = nullptr;
  std::vector<hipStream_t> side;  // one stream per group beyond the first
  hipEvent_t fork = nullptr;
  std::vector<hipEvent_t> join;
  GraphCache graphs;

  ~stencil_batch_s() {
    for (hipStream_t s : side) (void)hipStreamDestroy(s);
    for (hipEvent_t e : join) (void)hipEventDestroy(e);
    if (fork) (void)hipEventDestroy(fork);
    if (d_tables) (void)hipFree(d_tables);
  }
};

namespace {

stencil_status_t launch_group(const Group& g, int parity, hipStream_t s) {
  BatchArgs b;
  b.table = g.d_table;
  b.ngrids = (int32_t)g.grids.size();
  b.total = (int32_t)g.total;
  b.launch = parity & 1;
  b.pad = 0;
  return g.k.launch_batch(b, g.blocks, s) == hipSuccess ? STENCIL_OK : STENCIL_EHIP;
}

// Steps t = 0 .. steps-1 of every plain group, the scheduled launches of
// every time-blocked class; each plain group and each class on its own
// stream, forked from and joined back into `s`.
stencil_status_t enqueue_batch(stencil_batch_s* b, int64_t steps, hipStream_t s) {
  const size_t slots = b->plain.size() + b->classes.size();
  if (slots > 1) {
    if (hipEventRecord(b->fork, s) != hipSuccess) return STENCIL_EHIP;
    for (size_t k = 1; k < slots; ++k)
      if (hipStreamWaitEvent(b->side[k - 1], b->fork, 0) != hipSuccess) return STENCIL_EHIP;
  }
  size_t slot = 0;
  for (size_t gi : b->plain) {
    const hipStream_t st = slot == 0 ? s : b->side[slot - 1];
    ++slot;
    for (int64_t t = 0; t < steps; ++t) {
      const stencil_status_t e = launch_group(b->groups[gi], (int)(t & 1), st);
      if (e != STENCIL_OK) return e;
    }
  }
  for (const TbClass& c : b->classes) {
    const hipStream_t st = slot == 0 ? s : b->side[slot - 1];
    ++slot;
    const std::vector<int> sizes = tb_schedule(steps, c.T);
    for (size_t l = 0; l < sizes.size(); ++l)
      for (size_t gi : c.by_size[sizes[l]]) {
        const stencil_status_t e = launch_group(b->groups[gi], (int)(l & 1), st);
        if (e != STENCIL_OK) return e;
      }
  }
  for (size_t k = 1; k < slots; ++k) {
    if (hipEventRecord(b->join[k - 1], b->side[k - 1]) != hipSuccess) return STENCIL_EHIP;
    if (hipStreamWaitEvent(s, b->join[k - 1], 0) != hipSuccess) return STENCIL_EHIP;
  }
  return STENCIL_OK;
}

struct Span {
  uintptr_t lo, hi;
};

}  // namespace

extern "C" {

stencil_status_t stencil_batch_create(const stencil_plan_t* plans, void* const* buf0, void* const* buf1,
                                      int32_t count, stencil_batch_t* out) {
  if (!out) return STENCIL_EINVAL;
  *out = nullptr;
  if (!plans || !buf0 || !buf1 || count < 1) return STENCIL_EINVAL;
  stencil_batch_s* b = nullptr;
  try {
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess) return STENCIL_EHIP;
    std::vector<Span> spans;
    spans.reserve(2 * (size_t)count);
    for (int32_t i = 0; i < count; ++i) {
      const stencil_plan_s* p = plans[i];
      if (!p || !buf0[i] || !buf1[i]) return STENCIL_EINVAL;
      if (p->device != device) return STENCIL_EINVAL;
      // an explicit time block is rejected; one the library chose advances
      // its grid up to T steps per launch (a time-blocked class below)
      if (p->rs.time_block > 1 && !p->rs.tb_auto) return STENCIL_EUNSUPPORTED;
      spans.push_back({(uintptr_t)buf0[i], (uintptr_t)buf0[i] + p->grid_bytes});
      spans.push_back({(uintptr_t)buf1[i], (uintptr_t)buf1[i] + p->grid_bytes});
    }
    std::sort(spans.begin(), spans.end(), [](const Span& x, const Span& y) { return x.lo < y.lo; });
    for (size_t k = 1; k < spans.size(); ++k)
      if (spans[k].lo < spans[k - 1].hi) return STENCIL_EALIAS;

    b = new (std::nothrow) stencil_batch_s();
    if (!b) return STENCIL_ENOMEM;
    b->device = device;
    b->count = count;
    std::map<const void*, size_t> by_kernel;                       // plain group by batched kernel
    std::map<std::pair<const void*, int>, size_t> by_class;         // class by (T-step kernel, T)
    std::map<std::tuple<size_t, int, const void*>, size_t> by_cgroup;  // group by (class, size, kernel)
    auto add_grid = [&](size_t gi, const KArgs& a, const Kernel& k) {
      Group& g = b->groups[gi];
      BatchGrid e;
      std::memset(&e, 0, sizeof(e));
      e.args = a;
      e.first = (int32_t)g.total;
      e.phase = 0;
      e.limit = 2;  // launches 0 and 1 (the launch parity) always advance every grid
      g.grids.push_back(e);
      g.total += k.items;
      return g.total <= (int64_t(1) << 31) - 1;
    };
    auto new_group = [&](const Kernel& k) {
      b->groups.emplace_back();
      b->groups.back().k = k;
      return b->groups.size() - 1;
    };
    struct Plain {
      KArgs a;
      Kernel k;
      double flops = 0.0;  // per point
      int64_t frag = -1;   // offset of outer-product fragments of the batch's own
    };
    std::vector<uint8_t> frags;  // those fragments
    std::map<const stencil_plan_s*, int64_t> frag_of;
    struct FragUse {
      size_t group, grid;
      int64_t frag;
    };
    std::vector<FragUse> frag_uses;
    std::vector<Plain> plain;  // grids of one step per launch
    // columns per lane (3D: grids) and shares of the waves of the gathers, by class
    std::vector<int> columns(count, 0), share(count, 1);
    std::vector<double> points(count, 0.0);  // of the grid's class
    std::map<std::pair<Picker, int>, std::vector<int32_t>> members;
    for (int32_t i = 0; i < count; ++i) {
      const Resolved& rs = plans[i]->rs;
      if (rs.family == FAM_TB2D) members[{rs.pick_batch, rs.time_block}].push_back(i);
      if (rs.family == FAM_GATHER2D || rs.family == FAM_GATHER3D || rs.family == FAM_TB3D)
        members[{rs.pick, 1}].push_back(i);
    }
    for (const auto& m : members) {
      std::vector<const Resolved*> grids;
      double bytes = 0.0;
      for (int32_t i : m.second) {
        grids.push_back(&plans[i]->rs);
        bytes += (double)plans[i]->grid_bytes;
      }
      // a grid's part of the class's bytes; 3D also their number, by which small
      // grids take a workgroup each
      const bool d2 = grids[0]->info.ndim == 2;
      for (int32_t i : m.second) share[i] = std::max(1, (int)(2048.0 * (double)plans[i]->grid_bytes / bytes));
      for (int32_t i : m.second) points[i] = bytes / (grids[0]->info.dtype == STENCIL_F64 ? 8.0 : 4.0);
      const int nc = d2 ? rs2d_batch_cut(grids, share.data(), m.second.data()) : (int)grids.size();
      for (int32_t i : m.second) columns[i] = nc;
    }
    // one-step gathers of all taps merge by type and dimension
    std::map<std::pair<int, int>, std::set<int>> mergeable;
    for (int32_t i = 0; i < count; ++i) {
      const Resolved& rs = plans[i]->rs;
      if ((rs.family == FAM_GATHER2D || rs.family == FAM_GATHER3D || rs.family == FAM_TB3D) && rs.frag.empty())
        mergeable[{rs.info.ndim, rs.info.dtype}].insert(2 * rs.info.radius + (rs.info.shape != STENCIL_STAR ? 1 : 0));
    }
    // One step of 2D grids beside other classes: orders 1 and 2 walk, in one launch of
    // all of them; a class of order 3 or 4 joins it only where it is small, as the
    // merged walk is slow for its weights (us a step, merged / a kernel each, FP32 zero
    // halo, from order 3 on: 16 grids of 128^2 of 2 / 3 / 8 stencils 12.9 / 11.1, 13.2 / 14.9,
    // 15.1 / 28, two of 512^2 of 2 / 3 / 4 16.2 / 10.7, 17.0 / 14.6, 18.1 / 18.7, 16 of 256^2 of
    // 2 / 4 / 8 21.8 / 11.8, 26.9 / 19.8, 34 / 29; orders 1 and 2: two of 512^2 of 3 stencils 9.0 / 14.3,
    // eight of 2 11.3 / 12.6).
    const int classes = (int)members.size();
    for (int32_t i = 0; i < count; ++i) {
      const Resolved& rs = plans[i]->rs;
      const int T = rs.tb_auto ? rs.time_block : 1;
      bool placed = false;
      if (T > 1) {
        // the kernels of launches of 1 .. T steps, picked for a grid among
        // many; a grid whose buffers do not take a time-blocked kernel, or
        // that has none there, runs one step per launch
        std::vector<Kernel> ks(T + 1);
        std::vector<KArgs> as(T + 1);
        bool ok = true;
        for (int sz = 1; sz <= T && ok; ++sz) {
          ks[sz] = plan_kernel(rs, buf0[i], buf1[i], &as[sz], sz, rs.pick_batch, columns[i], share[i],
                               sz > 1 || classes > 3 ? classes : 1);
          ok = ks[sz].launch_batch && ks[sz].items >= 1;
        }
        if (ok) {
          auto cit = by_class.find({ks[T].batch_id, T});
          if (cit == by_class.end()) {
            cit = by_class.emplace(std::make_pair(ks[T].batch_id, T), b->classes.size()).first;
            b->classes.emplace_back();
            b->classes.back().T = T;
            b->classes.back().by_size.resize(T + 1);
          }
          const size_t ci = cit->second;
          for (int sz = 1; sz <= T; ++sz) {
            auto git = by_cgroup.find({ci, sz, ks[sz].batch_id});
            if (git == by_cgroup.end()) {
              git = by_cgroup.emplace(std::make_tuple(ci, sz, ks[sz].batch_id), new_group(ks[sz])).first;
              b->classes[ci].by_size[sz].push_back(git->second);
            }
            if (!add_grid(git->second, as[sz], ks[sz])) {
              delete b;
              return STENCIL_EUNSUPPORTED;
            }
          }
          placed = true;
        }
      }
      if (placed) continue;
      plain.emplace_back();
      plain.back().flops = rs.info.executed_flops_per_point;
      int kinds = (int)mergeable[{rs.info.ndim, rs.info.dtype}].size();
      if (rs.info.ndim == 2 && rs.info.radius >= 3) kinds = points[i] < 1.0e5 * classes ? classes : 1;
      plain.back().k =
          plan_kernel(rs, buf0[i], buf1[i], &plain.back().a, 1, nullptr, columns[i], share[i], kinds);
      if (rs.auto_rows) {
        // the gather that AUTO chose for the grid alone, or the outer products
        KArgs m;
        const Picker outer = find_mfma3d_b4(rs.info.radius, true);
        const Kernel k = plan_kernel(rs, buf0[i], buf1[i], &m, 1, outer, 0, share[i]);
        KArgs whole = rs.args;
        whole.in = buf0[i];
        whole.out = buf1[i];
        whole.share = share[i];
        if (k.launch_batch && outer_products_better_many(whole, rs.info.radius)) {
          auto it = frag_of.find(plans[i]);
          if (it == frag_of.end()) {
            const std::vector<uint8_t> f = box3d_b4_fragments(rs);
            it = frag_of.emplace(plans[i], (int64_t)frags.size()).first;
            frags.insert(frags.end(), f.begin(), f.end());
            frags.resize((frags.size() + 255) / 256 * 256);
          }
          plain.back().a = m;
          plain.back().k = k;
          plain.back().frag = it->second;
        }
      }
      if (!plain.back().k.launch_batch || plain.back().k.items < 1) {
        delete b;
        return STENCIL_EINTERNAL;
      }
    }
    // the grids of the costliest items first: the last items to end are short
    std::stable_sort(plain.begin(), plain.end(), [](const Plain& x, const Plain& y) { return x.flops > y.flops; });
    // plain grids by kernel, or by the kernel several of theirs merge into
    std::map<const void*, std::set<const void*>> kinds;
    for (const Plain& p : plain)
      if (p.k.merged_id) kinds[p.k.merged_id].insert(p.k.batch_id);
    for (Plain& p : plain) {
      if (p.k.merged_id && kinds[p.k.merged_id].size() > 1) {
        p.k.batch_id = p.k.merged_id;
        p.k.launch_batch = p.k.launch_merged;
      }
      auto it = by_kernel.find(p.k.batch_id);
      if (it == by_kernel.end()) {
        it = by_kernel.emplace(p.k.batch_id, new_group(p.k)).first;
        b->plain.push_back(it->second);
      }
      if (p.frag >= 0) frag_uses.push_back({it->second, b->groups[it->second].grids.size(), p.frag});
      if (!add_grid(it->second, p.a, p.k)) {
        delete b;
        return STENCIL_EUNSUPPORTED;
      }
    }
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) {
      delete b;
      return STENCIL_EHIP;
    }
    size_t table_entries = 0;
    for (Group& g : b->groups) {
      int occ = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, g.k.batch_id, g.k.threads, 0) != hipSuccess || occ < 1)
        occ = 1;
      const int64_t cap = (int64_t)occ * cus;
      g.blocks = (unsigned)std::min<int64_t>(g.total, cap);
      table_entries += g.grids.size();
    }
    const size_t frag_at = (table_entries * sizeof(BatchGrid) + 255) / 256 * 256;
    if (hipMalloc(&b->d_tables, frag_at + frags.size()) != hipSuccess) {
      delete b;
      return STENCIL_ENOMEM;
    }
    char* const d_frags = static_cast<char*>(b->d_tables) + frag_at;
    for (const FragUse& u : frag_uses) b->groups[u.group].grids[u.grid].args.frag = d_frags + u.frag;
    if (!frags.empty() && hipMemcpy(d_frags, frags.data(), frags.size(), hipMemcpyHostToDevice) != hipSuccess) {
      delete b;
      return STENCIL_EHIP;
    }
    std::vector<BatchGrid> host;
    host.reserve(table_entries);
    for (Group& g : b->groups) {
      g.d_table = reinterpret_cast<const BatchGrid*>(b->d_tables) + host.size();
      host.insert(host.end(), g.grids.begin(), g.grids.end());
    }
    if (hipMemcpy(b->d_tables, host.data(), host.size() * sizeof(BatchGrid), hipMemcpyHostToDevice) != hipSuccess) {
      delete b;
      return STENCIL_EHIP;
    }
    const size_t slots = b->plain.size() + b->classes.size();
    if (slots > 1) {
      if (hipEventCreateWithFlags(&b->fork, hipEventDisableTiming) != hipSuccess) {
        delete b;
        return STENCIL_EHIP;
      }
      for (size_t g = 1; g < slots; ++g) {
        hipStream_t s = nullptr;
        hipEvent_t e = nullptr;
        if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) {
          delete b;
          return STENCIL_EHIP;
        }
        b->side.push_back(s);
        if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
          delete b;
          return STENCIL_EHIP;
        }
        b->join.push_back(e);
      }
    }
    *out = b;
    return STENCIL_OK;
  } catch (const std::bad_alloc&) {
    delete b;
    return STENCIL_ENOMEM;
  } catch (...) {
    delete b;
    return STENCIL_EINTERNAL;
  }
}

stencil_status_t stencil_batch_run_steps(stencil_batch_t batch, int64_t steps, void* stream, int32_t* result_index) {
  if (!batch || steps < 0) return STENCIL_EINVAL;
  try {
    const stencil_status_t d = check_device(batch->device);
    if (d != STENCIL_OK) return d;
    const hipStream_t s = (hipStream_t)stream;
    stencil_status_t st = batch->graphs.run(batch, nullptr, steps, s, [&](hipStream_t cs) {
      return enqueue_batch(batch, steps, cs);
    });
    if (st == STENCIL_EUNSUPPORTED) st = enqueue_batch(batch, steps, s);
    if (st != STENCIL_OK) return st;
    if (result_index) *result_index = (int32_t)(steps & 1);
    return STENCIL_OK;
  } catch (...) {
    return STENCIL_EINTERNAL;
  }
}

stencil_status_t stencil_batch_info(stencil_batch_t batch, int32_t* groups, int64_t* items, int64_t* blocks) {
  if (!batch) return STENCIL_EINVAL;
  int64_t it = 0, bl = 0;
  for (const Group& g : batch->groups) {
    it += g.total;
    bl += g.blocks;
  }
  if (groups) *groups = (int32_t)batch->groups.size();
  if (items) *items = it;
  if (blocks) *blocks = bl;
  return STENCIL_OK;
}

stencil_status_t stencil_batch_destroy(stencil_batch_t batch) {
  try {
    delete batch;
    return STENCIL_OK;
  } catch (...) {
    return STENCIL_EINTERNAL;
  }
}

}  // extern "C"
