// The rules of wht_route.h for the tests, as a library that the host compiler builds: which kernel a call of a size runs on, and
// where the sizes lie at which it changes.  Not part of the layer's library.
#include <stddef.h>

#include "wht_route.h"
#include "wht_validate.h"

using namespace wht;

static bool rows_for(int32_t dtype, int32_t d, int32_t butterfly, Rows* rows) {
    Width w{};
    if (check_dims(1, d, dtype, &w) != WHT_OK) return false;
    const int bytes = dtype == WHT_DTYPE_F32 ? 4 : 2;
    if (w.twelve) *rows = {Sched::Twelve, w.logd - 4, bytes};
    else *rows = {bytes == 2 && w.logd >= 10 && !butterfly ? Sched::Matrix : Sched::Wave, w.logd, bytes};
    return true;
}

extern "C" {

// out: 0 y, 1 with the residual, 2 with the statistic.  The steps of the route into mib[8] and way[8]; their number, or -1.
int wht_query_forward_steps(int32_t dtype, int32_t d, int32_t butterfly, int32_t out, double* mib, int32_t* way) {
    Rows rows{};
    if (!rows_for(dtype, d, butterfly, &rows)) return -1;
    const Route r = forward_route(rows, static_cast<Out>(out));
    int n = 0;
    for (; n < 8 && (n == 0 || r.step[n].mib > 0); ++n) {
        mib[n] = r.step[n].mib;
        way[n] = static_cast<int32_t>(r.step[n].way);
    }
    return n;
}
int wht_query_forward(int32_t dtype, int32_t d, int32_t butterfly, int32_t out, int64_t N) {
    Rows rows{};
    if (!rows_for(dtype, d, butterfly, &rows)) return -1;
    const Out o = static_cast<Out>(out);
    const Way way = forward_way(rows, o, N * d * rows.bytes);
    return forward_reaches(rows, o, way) ? static_cast<int>(way) : -1;
}
int wht_query_dx_through(int32_t dtype, int32_t d, int32_t grads, int64_t N) {
    Rows rows{};
    if (!rows_for(dtype, d, 0, &rows)) return -1;
    return dx_through(rows, grads != 0, N * d * rows.bytes);
}
int wht_query_sums_store(int32_t dtype, int32_t d, int32_t dx) {
    Rows rows{};
    return rows_for(dtype, d, 0, &rows) ? static_cast<int>(sums_store(rows, dx != 0)) : -1;
}
int wht_query_takes_few(int32_t dtype, int32_t d, int64_t N, int32_t over_alpha) {
    Rows rows{};
    if (!rows_for(dtype, d, 0, &rows)) return -1;
    return takes_few_backward(rows, N, over_alpha != 0);
}
int64_t wht_query_few_elements(int32_t dtype, int32_t d) {
    Rows rows{};
    return rows_for(dtype, d, 0, &rows) ? few_backward_elements(rows) : -1;
}

}  // extern "C"
