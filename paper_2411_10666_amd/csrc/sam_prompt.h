// Launcher of the prompt kernel (sam_prompt.hip).
#pragma once
#include "sam_device.h"
#include "sam_ingest.h"

namespace sam {

// Fresh sequences (launch_reset before) take their prompts.  host_offsets: [n_seqs + 1], the host's
// copy of offsets.  most: what a prompt may have by the time the kernel runs, or 0 if the host's copy
// holds for sure.
hipError_t launch_ingest(const StaticView &S, const BatchView &B, const int32_t *seq_map,
                         int n_seqs, const int32_t *tokens, const int64_t *offsets,
                         const int64_t *host_offsets, int64_t most, hipStream_t stream);

}  // namespace sam
