// launch_shape.hpp -- how many waves a run of n_traj trajectories takes, and how they are laid out (host
// arithmetic only; valid for every count up to 2^64 - 1).
#pragma once

#include <algorithm>
#include <cstdint>

namespace fpt {

// Waves of one trajectory per lane (the rounding up must not overflow).
inline uint64_t wave_count(uint64_t n_traj) { return n_traj / 64 + (n_traj % 64 != 0); }

// Spread a run of less than a trajectory per lane of the full grid (`grid` blocks of `block` threads): one
// block per CU of just the waves it needs.  Larger runs keep the full grid.
inline void spread_run(uint64_t n_traj, int cu_count, int &grid, int &block)
{
    const uint64_t waves = wave_count(n_traj), cus = (uint64_t)cu_count;
    if (waves >= (uint64_t)grid * (uint64_t)(block / 64)) return;
    const uint64_t per_cu = std::min<uint64_t>((waves + cus - 1) / cus, (uint64_t)(block / 64));
    block = 64 * (int)per_cu;
    grid = (int)std::min<uint64_t>((uint64_t)grid, (waves + per_cu - 1) / per_cu);
}

}  // namespace fpt
