// Dependencies between the entries of a chain laid out per XCD, and their placement in columns (see st_chain_deps.cpp).
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "st_host.h"
#include "st_internal.h"

namespace st {

bool chain_ops_disjoint(const TenantDev& T, const TenantDev& P);
bool chain_reads(const TenantDev& T, const TenantDev& P);
bool chain_reads_exactly(const TenantDev& T, const TenantDev& P);
// Flags of the tiles of P that write what T's tiles of index tile_m read; T reads P's output exactly.
ChainDep chain_local_range(const TenantDev& T, const TenantDev& P, uint32_t tile_m);

// List scheduling of one XCD's entries on its columns, in the planner's clocks.  An entry in a shared column runs beside
// another on the same compute unit.
class ChainDealer {
 public:
  explicit ChainDealer(bool shared_too);
  size_t columns() const { return shared_too_ ? 2 * kKind : kKind; }
  size_t earliest(double ready, double cost) const {                       // the column where an entry would end first
    const size_t e = first_[0][1], s = kKind + first_[1][1];
    return shared_too_ && finish(s, ready, cost) < finish(e, ready, cost) ? s : e;
  }
  void place(size_t column, double ready, double cost);
  double ends(size_t column) const { return free_[column]; }              // when the column's last entry ends
 private:
  static constexpr size_t kKind = kChainColumns;
  static constexpr double kSharedFactor = 1.15;
  double finish(size_t c, double ready, double cost) const { return std::max(free_[c], ready) + (c < kKind ? cost : cost * kSharedFactor); }
  bool shared_too_;
  double free_[2 * kKind] = {};
  uint8_t first_[2][kKind];      // per kind a tree over its columns: [1] is the one that is free first, node n holds the first of nodes 2n and 2n + 1
};

}  // namespace st
