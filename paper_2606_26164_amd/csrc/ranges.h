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

}  // namespace chisao
