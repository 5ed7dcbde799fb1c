// Where the pivoting panel (pivchol.hip) keeps the entries of its columns in
// LDS, and why its steps need no barrier for them beyond the one they have.
//
// A panel is kPanel steps.  Step j reads the entries 0 .. j - 1 of the pivot's
// column and then writes entry j of every column.  Entry t of a column sits in
// slot t mod (sh + 1), sh = kPanel (every entry has its own) or kPanelHalf.
// Between the barrier before step j's reads and the one before step j + 1's
// the waves run freely: the wave that owns the pivot's column may have written
// entry j before another wave has read the column.  So step j's own slot must
// hold nothing that the step reads straight from the slots, and every entry
// read there must still be in its slot.
//
// With sh = kPanelHalf the slots come round: step 16 writes the slot past the
// first half, and step 17 is the first to write over an entry of it.  From that
// step on the first half is read from a copy that the column's owner posts from
// its registers behind a barrier of its own, and the slots are read for the
// second half alone.  (With sh slots and not sh + 1, step 16 would write over
// entry 0 while other waves read it.)
#pragma once

namespace lev {

constexpr int kPanel = 32;
constexpr int kPanelHalf = 16;

// Slots of a column, an odd number: the columns' writes spread over the banks.
constexpr int panel_stride(int sh) { return sh + 1; }
constexpr int panel_slot(int sh, int t) { return t % panel_stride(sh); }
// Whether step j reads the first half from the posted copy.
constexpr bool panel_posted(int sh, int j) { return sh < kPanel && j > kPanelHalf; }

constexpr bool panel_slots_hold(int sh) {
  for (int j = 0; j < kPanel; ++j)
    for (int t = panel_posted(sh, j) ? kPanelHalf : 0; t < j; ++t)
      for (int later = t + 1; later <= j; ++later)  // j: this step's own write
        if (panel_slot(sh, later) == panel_slot(sh, t)) return false;
  return true;
}
static_assert(panel_slots_hold(kPanel) && panel_slots_hold(kPanelHalf), "a step writes over an entry that it reads");

}  // namespace lev
