// The launch plan of the 16-bit attention path behind a C function, for the host tests.
#include "cf_plan.h"

extern "C" void probe_plan(int n_q_heads, int n_kv_heads, int batch, int max_tq, int seg_stride, int64_t max_kv_tokens, size_t given, int64_t* out) {
    const cf::attn::Plan p = cf::attn::make_plan(n_q_heads, n_kv_heads, batch, max_tq, seg_stride, max_kv_tokens, given);
    const int64_t v[] = {p.wide, p.nrb, p.groups, p.n_rg, p.nsplit, p.units, p.slots, (int64_t)p.total, cf::attn::wide_grid_ok(n_kv_heads, p)};
    std::copy(v, v + 9, out);
}
