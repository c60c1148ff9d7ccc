// The forms that ordinary calls take keep as many rows in flight as the split
// counts on; checked by the compiler.
#include "../../paper_1910_03517_amd/csrc/apply_split.h"

using namespace rc;
static_assert(rows_in_flight(kMapDirect, 3, true) == kSplitRows, "8-bit RGB with statistics");
static_assert(rows_in_flight(kMapDirect, 1, false) == kSplitRows, "gray, maps blended between blocks");
static_assert(rows_in_flight(kMapCross, 3, true) == kSplitRows, "3x3 maps");
static_assert(rows_in_flight(kMapWide, 1, true) == kSplitRows, "16-bit cameras");
static_assert(rows_in_flight(kMapWide, 1, false) == kSplitRows, "16-bit cameras without statistics");
static_assert(rows_in_flight(kMapTable, 3, false) == kSplitRows, "8-bit RGB without statistics");
static_assert(rows_in_flight(kMapTable, 1, false) == kSplitRows, "8-bit gray without statistics");

int main() { return 0; }
