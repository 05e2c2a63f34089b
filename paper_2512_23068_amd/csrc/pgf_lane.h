// Channels of the lanes of k_scan_m: plain arithmetic, shared with the host
// test of the ownership.  A wave that begins at channel d0 has 16 lane columns
// of nc consecutive channels each.
#pragma once

namespace pgf {

// First channel of lane column c: lanes past the last channel are moved back
// onto the last nc (onto channel 0 with fewer than nc channels in all) and
// compute those again.
constexpr int lane_first(int D, int nc, int d0, int c) {
    return D < nc ? 0 : (d0 + nc * c < D - nc ? d0 + nc * c : D - nc);
}

// Leading channels of a lane that belong to the wave before: only where fewer
// than nc channels are left for the wave (all its lanes are then moved back).
// That wave alone reads and writes their state and writes their outputs: in
// the sequential evaluation the exit state replaces the entry state, and
// nothing orders the two waves.
constexpr int wave_skip(int D, int nc, int d0) {
    return D >= nc && d0 > D - nc ? d0 - (D - nc) : 0;
}

// Whether a lane stores its channel number j (of nc).
constexpr bool lane_stores(int D, int skip, int j) { return j >= skip && j < D; }

}  // namespace pgf
