// Instances of the scatter that sums a table of pair counts, for one and two choices.
#include "route_table.h"

namespace tamoe {

void launch_route_table_few(const RouteArgs& a, const RowPolicies& how, hipStream_t st) {
    if (a.k == 1) launch_table_of<1>(a, how, st);
    else launch_table_of<2>(a, how, st);
}

}  // namespace tamoe
