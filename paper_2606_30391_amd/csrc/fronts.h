// fronts.h -- internal interface of fronts.hip (the placement search of 8 x 16 tables over
// candidate fronts), called by the placement entry points in festina.hip.
#pragma once

#include <cstddef>
#include <cstdint>

#include "festina.h"

namespace festina_fronts {

struct Layout {
  size_t host_cnt, hosts, rowle, dc_positive, row_max, info, pool_used, front, total;
  int32_t buckets;               // n_waves * n_models
  int32_t cap, pool_steps;       // front steps per bucket (both SM-level ranges), and in the pool
  int32_t chunk;                 // requests per workgroup of the choosing kernel
};

// Too few requests per (wave, model) for fronts to pay.
bool sparse(long long buckets, long long R);

// Workspace layout when these shapes take the front search; false: they do not.
bool layout(const festina_lut *L, const festina_gpus *G, const festina_requests *Q, Layout *o);

// The launches of one call on a checked workspace of lay.total bytes; ev_begin / ev_end (or
// nullptr) are recorded around all three: each of them rules candidates out.
festina_status launch(const festina_lut *L, const festina_gpus *G, const festina_requests *Q,
                      const festina_placements *out, const Layout &lay, char *ws, void *stream, void *ev_begin,
                      void *ev_end);

}  // namespace festina_fronts
