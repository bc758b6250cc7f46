// The host's side of the conjugate-gradient loop (solve.hip): when it waits for the residual of an iteration, and when it launches
// the next one first.
#pragma once
#include <algorithm>

namespace f3m {

// Whether the next iteration may be launched before the residual of the one under way is known.  A wait costs the solver some 30 us an
// iteration, a product launched for nothing costs all of it (0.7 ms at 1e7 points), so: not where that iteration may be the
// last one.  seen: iterations whose residual is known; known, before: the last two residuals.  The residual under way is taken to
// fall as the last one did; ten times the limit leaves room for steps that fall faster.
inline bool cg_may_go_ahead(int seen, double before, double known, double limit) {
    if (!(limit > 0.0)) return true;    // only max_iter ends the solve
    if (seen < 1) return false;         // nothing known of how it falls
    return known * std::min(1.0, known / before) > 10.0 * limit;
}

// launch(k): iteration k on its way, k = 0 .. max_iter - 1.  look(k, &residual): waits for its residual; true: it was the last.
// At most one iteration is under way that has not been looked at when another is launched; all launched ones are looked at
// unless one of them is the last.
template <class Launch, class Look>
void cg_iterate(int max_iter, double first, double limit, Launch &&launch, Look &&look) {
    double before = first, known = first;
    int seen = 0;
    for (int k = 0; k < max_iter; ++k) {
        launch(k);
        while (seen <= k) {
            if (seen == k && k + 1 < max_iter && cg_may_go_ahead(seen, before, known, limit)) break;
            double residual = 0.0;
            if (look(seen, &residual)) return;
            before = known;
            known = residual;
            ++seen;
        }
    }
}

}  // namespace f3m
