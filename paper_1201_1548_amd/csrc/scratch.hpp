// Bytes of the scratch array past BIRES_NOALLOC_SCRATCH_BYTES: metadata that a call
// needs beside the buffers that count against the documented size (the queue of
// blocks to recompute, at most one word per 64 values of [P][D], and the rows'
// slack), so that the largest calls keep fitting.
#pragma once
#include <stddef.h>

namespace bires {
constexpr size_t NOALLOC_MARGIN = (size_t)512 << 10;
}
