// Traceback of the memory-indexed table (dual.hip).
#pragma once

#include "rc_internal.h"
#include "schedule.h"

namespace rcdp {

// Chain traced back through the table of launch_dual from st->t_sel /
// st->m_sel, and its strategy re-evaluated (Eq. 1, Eq. 2) into out; chain[F]
// is scratch.
hipError_t launch_dual_trace(rc_family f, int32_t B, int32_t W, int objective, const uint32_t* D,
                             DevStatus* st, int32_t* chain, const ScheduleOut& out,
                             hipStream_t s);

}  // namespace rcdp
