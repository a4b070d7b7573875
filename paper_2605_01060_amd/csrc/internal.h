// Internal declarations shared by the library's translation units.
#pragma once

#include <stdint.h>

#include <string>

#include "surge.h"

namespace surge {

// Thread-local error message of the last failing call.
surge_status fail(surge_status code, const char* fmt, ...);
void clear_error();

// SuperBatch formation (Alg. 1), host only.  Appends to the output vectors.
struct PlanSB {
  int64_t text_begin, text_end, seg_begin, seg_end;
};
struct PlanSeg {
  int64_t first_text, count, row_offset;
  int32_t partition;
};
surge_status plan_superbatches(const int64_t* part_offsets, int32_t n_parts, int64_t b_min,
                               int64_t n_max, int32_t policy, void (*emit_sb)(void*, const PlanSB&),
                               void (*emit_seg)(void*, const PlanSeg&), void* ctx,
                               int64_t* n_sbs, int64_t* n_segs);

// Host-side check of an encoder description.
surge_status validate_desc(const surge_encoder_desc* desc);

// bf16 bits of a float, nearest value with ties to even (host side).
uint16_t f32_to_bf16_rne(float f);

// Up to 32 consecutive rows of one text: the text's first token row and
// (text length << 7 | block index), so a kernel needs no second load to know
// its rows.  Text lengths are in [1, 4096].
struct RowBlock {
  uint32_t beg;
  uint32_t len_block;
};

// The work list of a chunk: every 32-row block of every text (the
// attention's query blocks, the embedding's row blocks), longest text first,
// ties in text order.  cu [n_texts + 1]; row numbers count from cu[0].
// count_row_blocks gives the list's length (at most cu[n] - cu[0]).
int64_t count_row_blocks(const int64_t* cu, int64_t n_texts);
void fill_row_blocks(const int64_t* cu, int64_t n_texts, RowBlock* items);

}  // namespace surge
