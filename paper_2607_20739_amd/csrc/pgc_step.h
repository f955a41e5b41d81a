// The step of include/pgc.h with the gradient kernel's block partial sums at a
// caller-chosen device address.  Internal to the library.
#pragma once

#include <cstddef>
#include <cstdint>

#include "pgc.h"

namespace pgc {

// pgc_step with the linear models' block partials at `partials` (device, 8-byte
// aligned; at least linear_partials_bytes(ctx) bytes), or in the bound workspace
// when `partials` is null.  Same checks, errors and effects as pgc_step.
int step_impl(pgc_ctx* ctx, const void* X, const void* y, float* w, const uint8_t* straggler_mask,
              float lr, float* partials);

// The most bytes of block partials that a step of the configured context (a linear
// model) writes.
size_t linear_partials_bytes(const pgc_ctx* ctx);
// The bytes by which pgc_step_noalloc takes (up to PGC_NOALLOC_SCRATCH_BYTES) or refuses
// the configured context: those of the partials on a grid of about 1,024 blocks, not on
// the grid that a step launches.  The grid of every shape that is taken fits.
size_t noalloc_rule_bytes(const pgc_ctx* ctx);

bool context_is_configured(const pgc_ctx* ctx);
bool context_has_workspace(const pgc_ctx* ctx);
bool context_is_linear(const pgc_ctx* ctx);

// Records `msg` as the context's last error and returns `status`.
int set_error(pgc_ctx* ctx, int status, const char* msg);

}  // namespace pgc
