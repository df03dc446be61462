// Declarations shared by the library's own sources (not part of the C ABI).
#pragma once

#include <cstdint>

#include "iqa.h"

namespace iqa {

// iqa_batch_describe with the per-pair geometry of tuned kind `kind`
// (IQA_TUNE_BATCH: the ragged-batch geometry; IQA_TUNE_SERVE: the server's;
// kDescribeOdd: iqa_odd_batch_describe).
constexpr int kDescribeOdd = -1;
iqa_status describe_pairs(const iqa_pair *pairs, int64_t count, void *descs,
                          int64_t *total_units, int kind);

// iqa_tiles_batched_inline for up to kArgsMax pairs, as many as 4 KiB of kernel
// arguments hold.
constexpr int64_t kArgsMax = 31;
iqa_status tiles_batched_args(const void *descs_host, int64_t count, int64_t total_units,
                              int64_t waves, void *stream);

}  // namespace iqa
