// noalloc.hip -- st_check_edges_noalloc: the discretised edge check of
// st_check_edges for callers that cannot allocate (code under HIP graph
// capture, tight serving loops).  The one-kernel check keeps its state in LDS,
// so there is no work area at all: calls on different streams or threads are
// independent, and whatever lanes st_set_tuning chose for st_check_edges do not
// apply.  The limit on the number of edges is that of the work area the call once
// had, kept so that it refuses what it always refused.
#include "st_internal.hpp"

using namespace st;

extern "C" int st_check_edges_noalloc(st_problem *p, int64_t E, const float *xa, const float *xb,
                                      uint8_t *free_out, int32_t *first_hit, void *stream) {
    if (!p || E < 0 || (E > 0 && (!xa || !xb || !free_out))) {
        set_error("st_check_edges_noalloc: bad arguments");
        return ST_EINVAL;
    }
    if (E > ST_NOALLOC_MAX_EDGES) {
        set_error("st_check_edges_noalloc: %lld edges exceed the call's limit of %lld edges (what its former fixed "
                  "work area held)", (long long)E, (long long)ST_NOALLOC_MAX_EDGES);
        return ST_EINVAL;
    }
    ST_HIP(launch_check_edges_flat(p->sc, E, xa, xb, free_out, first_hit, (hipStream_t)stream));
    return ST_OK;
}
