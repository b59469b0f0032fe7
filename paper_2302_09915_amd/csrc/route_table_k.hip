// Instances of the scatter that sums a table of pair counts, for three choices and more.
#include "route_table.h"

namespace tamoe {

void launch_route_table_many(const RouteArgs& a, const RowPolicies& how, hipStream_t st) {
    if (a.k == 3) launch_table_of<3>(a, how, st);
    else if (a.k == 4) launch_table_of<4>(a, how, st);
    else launch_table_of<0>(a, how, st);
}

}  // namespace tamoe
