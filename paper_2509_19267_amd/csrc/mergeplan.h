// Chunks of the nonzero-balanced residual pass (spmv.hip, mp_chunks): the
// host's plan, and the one index that the device forms from it without a
// look at the chunk's rows.  Plain C++, shared by both sides.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace rg {

constexpr int64_t MP_CH = 256;   // nonzeros per chunk

// Chunk c holds nonzeros [c*MP_CH, (c+1)*MP_CH); it owns the rows whose
// first nonzero position lies in it (empty rows: the position of the next
// nonzero; trailing empty rows: the last chunk): rs[c] .. rs[c+1]-1.  A chunk
// that owns no rows has rs[c] == rs[c+1], which is `rows` where the last row
// runs into it.  Rows running past their chunk are listed with their first
// and last chunk.
struct MergeRows {
  std::vector<int32_t> rs, xrow, xcs, xce;
  int64_t nchunk = 0, maxrows = 0, maxlen = 0;   // of a chunk; of a row
};
inline MergeRows merge_rows(const int64_t *rp, int64_t rows) {
  MergeRows p;
  const int64_t nnz = rp[rows];
  p.nchunk = std::max<int64_t>(1, (nnz + MP_CH - 1) / MP_CH);
  p.rs.resize(p.nchunk + 1);
  for (int64_t c = 0; c < p.nchunk; ++c)
    p.rs[c] = (int32_t)(std::lower_bound(rp, rp + rows, c * MP_CH) - rp);
  p.rs[p.nchunk] = (int32_t)rows;
  for (int64_t c = 0; c < p.nchunk; ++c)
    p.maxrows = std::max<int64_t>(p.maxrows, p.rs[c + 1] - p.rs[c]);
  for (int64_t r = 0; r < rows; ++r) {
    p.maxlen = std::max<int64_t>(p.maxlen, rp[r + 1] - rp[r]);
    if (rp[r + 1] == rp[r]) continue;
    const int64_t cs = rp[r] / MP_CH, ce = (rp[r + 1] - 1) / MP_CH;
    if (ce > cs) {
      p.xrow.push_back((int32_t)r);
      p.xcs.push_back((int32_t)cs);
      p.xce.push_back((int32_t)ce);
    }
  }
  return p;
}

// The row whose bounds a lane of a chunk owning [rs, re) loads ahead: its
// first owned one, else a row that there is (ptr[rows + 1] is not).
constexpr int64_t mp_first_row(int64_t rs, int64_t re, int64_t lane,
                               int64_t rows) {
  const int64_t r = rs + lane < re ? rs + lane : rs;
  return r < rows ? r : rows - 1;
}

}  // namespace rg
