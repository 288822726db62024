// Who publishes, reads and leaves in each step of the in-register tridiagonal
// reduction's exchange (tridiag.hip).  Plain integer rules without device code,
// so that a model of the exchange can be built from them on the host.
//
// In step i (column i), a workgroup of rows r0 .. r0 + kTridiagRows - 1 writes
// its words of slot i & 1 with epoch i + 1, one per row right of column i, then
// either leaves or waits until every such word of the slot has that epoch.
#pragma once

namespace bitsmoe {

constexpr int kTridiagRows = 8;  // rows per workgroup

// Step i has an exchange (the last one has a single entry and needs none).
constexpr bool tridiag_exchanges(int n, int i) { return i + 2 < n; }
// The word of row r is written, and read by everybody who stays, in step i.
constexpr bool tridiag_word_live(int n, int i, int r) { return r > i && r < n; }
// After publishing in step i the workgroup leaves without reading: it has no
// row right of column i + 1, so nothing that it would form from the words
// concerns a row of its own.  (The workgroup of row n - 1 stays to the end.)
//
// This is also what makes two slots enough.  The slot of step i is written
// again in step i + 2, by a workgroup that has read every word of step i + 1,
// one per row r > i + 1.  A workgroup that reads in step i has such a row, and
// publishes it in step i + 1, after all its reads of step i.  So no word is
// overwritten while somebody still waits for it.  (One that read in its last
// step could be: it has no word in step i + 1 for the others to wait for.)
constexpr bool tridiag_leaves(int n, int i, int r0) {
  return r0 + kTridiagRows < n && r0 + kTridiagRows <= i + 2;
}

}  // namespace bitsmoe
