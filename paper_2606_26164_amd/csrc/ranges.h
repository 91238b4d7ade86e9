// Index arithmetic of launches over very many rows.  Plain constexpr C++, so
// that it can be compiled and checked without a GPU.
#pragma once

namespace chisao {

// Work units of a launch are counted in 64 bits: d = 1 rows fit a GPU's memory
// beyond 2^31, and a population's probes (samples times probes) do as well.
using unit_t = long long;
constexpr unit_t units_of(int jobs, int centres) { return jobs > 0 && centres > 0 ? (unit_t)jobs * centres : 0; }
// the first unit of a wave, and the one after u
constexpr unit_t first_unit(unsigned block, int waves, int wave) { return (unit_t)block * waves + wave; }
constexpr unit_t next_unit(unit_t u, unsigned blocks, int waves) { return u + (unit_t)blocks * waves; }

// Launches with one workgroup per tile and no loop (the small-mixture and
// central-difference kernels on caller memory: up to four threads a row) take
// at most this many rows; a larger call is a sequence of such launches.  HIP
// refuses 2^32 threads or more, and a row's index fits 32 bits here.
constexpr int kLaunchRows = 1 << 29, kThreadsPerRow = 4;
static_assert((unit_t)kLaunchRows * kThreadsPerRow + 1024 < 1ll << 32, "threads of a launch");
// rows of the next launch when `left` are left: even parts, so that every
// launch of a call of many rows is one of many rows
constexpr int launch_rows(int left) {
    const unit_t parts = ((unit_t)left + kLaunchRows - 1) / kLaunchRows;
    return parts <= 1 ? left : (int)(((unit_t)left + parts - 1) / parts);
}

}  // namespace chisao
