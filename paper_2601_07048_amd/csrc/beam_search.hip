// beamSearch kernel (Alg. 1 / Alg. 2 of the paper, fused as in Sec. 4.1 and
// App. B): one wavefront serves one query for its whole life.
//
// Per expansion ("hop") the wavefront
//   1. picks the closest unexpanded frontier entry u (ballot over registers),
//   2. reads adjacency row adj[u] with one coalesced 4R-byte load,
//   3. drops ids it has seen before with a small table in LDS: sets of two
//      16-bit tags of a permuted id (set and tag together name the id exactly),
//      or full ids when the index is too large for that.  A table that only
//      ever forgets has no false positives, so the frontier sequence equals
//      that of an exact visited set -- the filter changes the number of distance
//      evaluations, never the result,
//   4. gathers the surviving neighbours' records (vector or RaBitQ code) with
//      16-byte loads, T lanes per record, several records in flight per lane,
//   5. reduces the partial distances inside each T-lane group,
//   6. merges the new (distance,id) keys into the sorted frontier, which lives
//      in registers (one key per lane per 64 entries): every candidate that
//      beats the current worst entry is broadcast once, every lane counts how
//      many candidates precede its entries, and one LDS scatter/gather applies
//      the permutation.  Keys are 64-bit (ordered distance, id, expanded flag),
//      so the order is the strict total order (distance, id).
#include "beam_launch.h"

namespace jx {

hipError_t launch_beam_search(int kind, int qbits, const BeamArgs& a, hipStream_t st, char* kernel_name) {
    if (kernel_name) kernel_name[0] = 0;
    if (a.nq <= 0) return hipSuccess;
    bool done = false;
    const hipError_t e = launch_beam_ahead(kind, qbits, a, st, kernel_name, &done);  // small batches
    if (e != hipSuccess || done) return e;
    const hipError_t es = launch_beam_sketch(kind, a, st, kernel_name, &done);
    if (es != hipSuccess || done) return es;
    if (a.vis_cap) return launch_beam_visited(kind, a, st, kernel_name);
    if (a.flags & (JX_FLAG_TILED_LOADS | JX_FLAG_QPW_2 | JX_FLAG_QPW_4 | JX_FLAG_WAVES_2 | JX_FLAG_WAVES_4))
        return launch_beam_variant(kind, a, st, kernel_name);
    switch (kind) {
        case K_U8: return launch_shape<K_U8, 0>(a, st, kernel_name);
        case K_F32: return launch_shape<K_F32, 0>(a, st, kernel_name);
        case K_F16: return launch_shape<K_F16, 0>(a, st, kernel_name);
        case K_RQ4:
        case K_RQ1: return launch_beam_codes(kind, qbits, a, st, kernel_name);
    }
    return hipErrorInvalidValue;
}

}  // namespace jx
