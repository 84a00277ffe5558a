// hb_tile.h -- tables and launcher of the row-by-tree tile kernel (hb_tile.hip).
#pragma once

#include "hb_device.h"

namespace hb {

// Without a tree split the tile kernel takes batches from this size on: its launch
// rules were measured from 50,000 rows up. It is no limit of the kernel, which
// gives every CU a workgroup of 64 rows from 16,384 rows on.
constexpr int kTileMinRowsPerCu = 192;
// With a workspace, batches up to this size may have their trees split by the
// tile kernel (measured from 1,100 to 16,384 rows). The batches between the two
// keep the kernels they had before the tile kernel; where trees are deeper than
// 10, that is the general one.
constexpr int64_t kTileSplitMaxRows = 16384;

// Launches the tile kernel with the fp32 tile's tables, or the rank tile's
// (may be null) where its estimated time is less. Returns HB_OK, an error, or
// 1 when no shape fits or the batch is too small.
int launch_tile(bool perfect, const EnsembleDev &e, const TileDev &tile, const TileDev *rank, const int32_t *leaf_id,
                int leaf_slots, int levels, const int32_t *tree_depth, const float *X, int64_t n_rows, float *scores,
                int32_t *leaf_ids, const Launch &ws, hipStream_t stream, std::string *err);

}  // namespace hb
