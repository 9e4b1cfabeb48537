// Radius neighbours of a range of points on the matrix cores (search.hip).
#pragma once

#include "geom.h"

namespace pirrt {

// What the search kernels report back; cleared by the packing kernel of each search
// (`outside` stays set: points never change).
struct SearchState {
  int32_t outside;  // some point lies outside the unit cube
  int32_t most;     // largest candidate count of a list that was too short (0: none was)
  int32_t listed;   // largest candidate count of a row past kSearchRowMax (0: none; not where wide)
  int32_t wide;     // wide finish: some row has more than kSearchRowMax candidates
  int32_t crowded;  // some list holds more than SearchArgs::crowd candidates
  int64_t nnz;      // entries of all rows
};

constexpr int kSearchRowMax = 512;     // candidates a row may have in the finish by 32 lanes
constexpr int64_t kSearchWindow = 1 << 18;  // ids the finish by a workgroup orders together
constexpr int kSearchRecord = 32;      // bytes of a point's packed record
constexpr int kSearchPad = 256;        // records of room past the last point
constexpr int kSearchMaxChunks = 64;
constexpr int64_t kSearchGroups = 1024;   // workgroups that fill the chip (4 waves each)
constexpr int32_t kSearchWideRows = 65536;  // rows from which a wave takes four blocks of them

struct SearchArgs {
  int d;
  int64_t n_old, n;       // rows of points n_old .. n - 1
  int64_t row0;           // first row of this slab
  int32_t rows;           // rows of this slab
  double radius;
  const double* pts;
  ObsView obs;
  const uint4* rec;       // packed records, kSearchRecord bytes each
  int32_t nch;            // candidate lists per row (chunks of earlier points)
  int64_t chunk;          // earlier points per chunk (a multiple of kSearchPad; wide: at most kSearchWindow)
  int32_t cap;            // room of one candidate list
  int32_t crowd;          // candidates from which a list speaks against less room
  int32_t* cand;          // [rows][nch][cap] candidate ids; the finished rows replace them
  int32_t* cnt;           // [rows][nch] candidates per list
  float* ccost;           // [rows][nch * cap] costs of the finished rows
  int32_t* deg;           // [rows] entries of the finished rows
  bool wide;              // rows finished by a workgroup each
  SearchState* state;
  SearchState* report;    // pinned host memory: *state at the end
};

// Packs points [first, n) and clears the state's counters.
void launch_search_pack(int d, int64_t first, int64_t n, const double* pts, uint4* rec, SearchState* state,
                        hipStream_t s);
// Candidates, then the exact distance and segment tests: rows sorted by neighbour id in
// cand / ccost at stride nch * cap, their lengths in deg.
void launch_search(const SearchArgs& a, hipStream_t s);
// The finished rows of a slab into CSR: row_ptr[row0 + i], col / cost from entry `base`
// on (written only when the total fits `capacity`; either may be NULL), the total into
// report->nnz.  off: rows + 1 int64 of scratch, scan: scan scratch for rows.
void launch_search_rows(const SearchArgs& a, int64_t base, int64_t capacity, int64_t* row_ptr, int32_t* col,
                        float* cost, int64_t* off, void* scan, hipStream_t s);

}  // namespace pirrt
