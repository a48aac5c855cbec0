// Launcher of the prompt kernel (sam_prompt.hip).
#pragma once
#include "sam_device.h"

namespace sam {

// What the host knows of the prompts' lengths.
struct PromptSizes {
    int64_t longest;     // what the launch is made for
    int64_t most;        // what a prompt may have when the kernel runs: more than `longest` where
                         // the host has not read the device's offsets itself (a captured call that
                         // is replayed with other prompts)
};

// Fresh sequences (launch_reset before) take their prompts.
hipError_t launch_ingest(const StaticView &S, const BatchView &B, const int32_t *seq_map,
                         int n_seqs, const int32_t *tokens, const int64_t *offsets,
                         const PromptSizes &sizes, hipStream_t stream);

}  // namespace sam
