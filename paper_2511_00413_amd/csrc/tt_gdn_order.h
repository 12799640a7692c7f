// In which order the workgroups of a gated delta rule walk take the segments of the chunk program.  (Plain C++: the kernels and host code.)
#pragma once

namespace tt {

// Forward walks take the segments as the schedule lists them: level by level, the longest of a level first.  The reverse walk takes the
// last level first, and a level's segments in their order; with n_levels = 0 (more levels than a launch lists) the list backwards.
// In both a segment comes behind all that it waits for: a forward walk for the saver of the state that it starts from (an earlier
// level), the reverse walk for the readers of the states that it saves (later levels).
constexpr int reverse_walk_segment(int place, int n_segments, int n_levels, const int* level_off) {
  const int seg = n_segments - 1 - place;
  for (int l = 0; l < n_levels; l++)
    if (seg >= level_off[l] && seg < level_off[l + 1]) return level_off[l] + level_off[l + 1] - 1 - seg;
  return seg;
}

}  // namespace tt
