// Launcher of the prompt kernel (sam_prompt.hip).
#pragma once
#include "sam_device.h"

namespace sam {

// Fresh sequences (launch_reset before) take their prompts; no prompt is longer than max_tokens.
hipError_t launch_ingest(const StaticView &S, const BatchView &B, const int32_t *seq_map,
                         int n_seqs, const int32_t *tokens, const int64_t *offsets,
                         int64_t max_tokens, hipStream_t stream);

}  // namespace sam
