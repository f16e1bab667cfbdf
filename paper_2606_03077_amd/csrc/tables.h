// Constants and table formats shared by the host code and the HIP kernels of libra:
// everything the device code reads from the plan workspace is laid out here.
#pragma once

#include <cstdint>

#include "libra.h"

namespace libra {

constexpr int kPage = LIBRA_PAGE_SIZE;     // tokens per page
constexpr int kDim = LIBRA_HEAD_DIM;       // channels per head
constexpr int kTileElems = kPage * kDim;   // bf16 elements per (page, head) tile
constexpr int kTileBytes = kTileElems * 2; // 4 KiB
constexpr int kUnitInts = LIBRA_UNIT_INTS;

// Unit record fields (int32), in table order.
enum UnitField : int {
  U_B = 0, U_G, U_KV0, U_KV1, U_Q0, U_Q1, U_SPLIT, U_NSPLIT, U_PART, U_ROW0, U_KIND, U_PRIOR
};
constexpr int kKindSingle = 0;
constexpr int kKindChunk = 1;
constexpr int kNumXcds = 8;  // MI355X: workgroup w is dispatched to XCD w % 8
constexpr int kChunkStepKeys = 64;  // keys per step of a query tile's cost (plan rule step 9)
constexpr int kChunkRows = 256;  // most (token, head) rows of one query tile
constexpr int kTileRows = 128;   // rows of a fine tile: a query tile is one or two of them
constexpr int kTileStepKeys = 32;  // keys per step of the chunk kernel on fine tiles

// What a workgroup of the chunk launch takes: a query tile (wide form, kChunkRows rows), or a
// fine tile (narrow form, kTileRows rows), which is half h of a query tile over the keys that
// it sees (of tiles of one half each; of both halves of every tile; or as a table lists them,
// query tile << 1 | h), or, where they fit in one wave, over all keys or a split, as a record
// of the fine-tile table has it.
enum ChunkForm : int { kUnits = 0, kFirstHalves, kBothHalves, kListedHalves, kFineTiles };

// Fine tiles: rows [128 h, 128 h + 128) of the query tile [q0, q1) of (sequence b, KV head g),
// T_GH = g | h << 16, over keys [kv0, kv1): all of them, or split `part` of n.
enum TileField : int { T_B = 0, T_GH, T_Q0, T_Q1, T_ROW0, T_PRIOR, T_KV0, T_KV1, T_PART, T_NSPLIT };
constexpr int kTileInts = 10;

// Append cache-write table: one record per (sequence, page) the new tokens touch.
enum WriteField : int { W_B = 0, W_PAGE, W_SLOT0, W_SLOT1, W_ROW, W_PAD0, W_PAD1, W_PAD2 };
constexpr int kWriteInts = 8;

// Split-merge table: one record per (sequence, KV head) whose KV range was split.
enum MergeField : int { M_B = 0, M_G, M_N, M_PART, M_ROW, M_PAD0, M_PAD1, M_PAD2 };
constexpr int kMergeInts = 8;

// Merge table of split fine tiles: one record per tile of rows (T_GH as above).
enum ChunkMergeField : int { CM_GH = 0, CM_Q0, CM_N, CM_PART, CM_ROW0, CM_Q1, CM_PAD0, CM_PAD1 };

}  // namespace libra
