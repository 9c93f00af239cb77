// Reads of a level step's input arrays against the memory a call carves for
// them, over external workspaces of every depth: the host's own carve and choice
// of levels, with a made-up index and no device.  Prints
// "<cases> <cases beyond by the slot's plain index> <cases beyond>".
#include "gt_api.cpp"

#include <stdio.h>

namespace {

// Largest entry index a level step reads for head level h (dense input), by
// the kernels' index or by the slot's plain one; entries are carved for
// nt x fr_cap of them.
bool beyond(const Index& ix, const Batch& b, bool plain) {
  const int64_t bcap = b.fr_cap >> b.nb;
  const uint32_t last = (uint32_t)(int64_t(1) << (b.head - b.nb)) - 1;
  const uint32_t slot = (uint32_t)((buckets_used(&ix, &b) - 1) * b.nt + b.nt - 1);
  const size_t at = plain ? (size_t)slot * bcap + last : gt::input_entry(true, slot, bcap, last);
  return at >= (size_t)b.nt * (size_t)b.fr_cap;
}

}  // namespace

int main() {
  long cases = 0, plain = 0, bad = 0;
  const int fmts[] = {GT_POOL_F32, GT_POOL_MAX_F32, GT_POOL_BF16, GT_POOL_FP8E4M3};
  for (int depth = 7; depth <= 26; ++depth)  // (shallower: refused)
    for (int fill = 1; fill <= 4; ++fill)
      for (int dp : {128, 1024, 2048})
        for (int fmt : fmts) {
          gt_index ix;
          ix.depth = depth;
          ix.cap = int64_t(1) << depth;
          ix.n = std::max<int64_t>(1, ix.cap * fill / 4 - (fill < 4 ? 1 : 0));
          ix.d = ix.dp = ix.pw = dp;
          ix.n_cu = 256;
          ix.formats = (uint32_t)fmt;
          for (int nq : {1, 33, 200, 1024, 4100, 32768})
            for (int state = -2; state < depth; ++state) {
              // state: -2 an explicit head as deep as it can be, -1 the first
              // call, else a later call's head by its last frontier
              ix.head_level = state == -2 ? depth - 2 : -1;
              int64_t need = 0, least = 0;
              if (gt_call_bytes(&ix, nq, (gt_pool)fmt, 0, 0, &need, &least) != GT_OK) return 1;
              gt_batch b;
              b.ix = &ix;
              if (carve_budget(&ix, &b, reinterpret_cast<void*>(uintptr_t(1) << 40), (size_t)least, nq, fmt,
                               1024, true) != GT_OK)
                return 2;
              const CallShape c = call_shape(&ix, nq, fmt);
              b.kind = 1;
              b.fmt = c.wf;
              b.maxpool = c.maxp;
              b.nq = nq;
              b.nt = (nq + c.tq - 1) / c.tq;
              b.tq = c.tq;
              b.n_epoch = ix.n;
              if (state >= 0) {
                b.have_last = true;
                b.last_walk_fmt = b.fmt;
                b.last_maxpool = b.maxpool;
                b.last_walk_nt = b.nt;
                b.last_n_epoch = ix.n;
                b.last_dl = state;
                for (int l = 0; l < GT_MAX_LEVELS; ++l)  // full frontiers: the first level moves down
                  b.last_entries[l] = l < 40 ? (unsigned long long)b.nt << l : 0;
              }
              choose_levels(&ix, &b);
              if (b.sub_top >= 0 || b.dense_last >= 0 || b.head > depth - 2) continue;  // no dense input
              ++cases;
              plain += beyond(ix, b, true);
              bad += beyond(ix, b, false);
            }
        }
  printf("%ld %ld %ld\n", cases, plain, bad);
  return 0;
}
