// dcs_graph.hip -- random graphs G(n, m) and G(n, p) (Sec. 7: generating
// such a graph is sampling from its n(n-1)/2 possible edges, without
// replacement for G(n, m) and by Bernoulli sampling for G(n, p)).
//
// The edge with index k (0-based) is the pair (u, v), v < u, with
// k = u(u-1)/2 + v: edges ordered by u, then v.  The sampler's kernels write
// each value as its pair (edge_pair), so the edge list keeps the sample's
// order and needs neither a pass of its own nor a buffer beyond the caller's.
// (2^28 edges on 2^26 vertices: a separate decoding pass, 16 bytes an edge at
// 4.7 TB/s, took 0.91 ms.)
#include <stdint.h>

#include "../../include/dcs.h"
#include "dcs_host.hpp"

namespace {

// Edges of a graph on n vertices, or an error if n(n-1)/2 exceeds the
// largest universe of the sampler used (max_N).
int32_t edge_universe(uint64_t n_vertices, uint64_t max_N, uint64_t* N) {
  if (n_vertices > (1ull << 32)) return DCS_EINVAL;
  const uint64_t e = n_vertices < 2 ? 0 : n_vertices * (n_vertices - 1) / 2;
  if (e > max_N) return DCS_EINVAL;
  *N = e;
  return DCS_OK;
}

}  // namespace

extern "C" {

int32_t dcs_sample_edges_gnm(uint64_t n_vertices, uint64_t m, uint64_t seed,
                             const dcs_params* params, uint32_t* uv_dev, void* stream) {
  uint64_t N = 0;
  if (edge_universe(n_vertices, DCS_MAX_UNIVERSE, &N) != DCS_OK || m > N) return DCS_EINVAL;
  if (m > 0 && (uv_dev == nullptr || (reinterpret_cast<uintptr_t>(uv_dev) & 7u) != 0))
    return DCS_EINVAL;
  if (m == 0) return DCS_OK;
  return dcs::host::sample_tree(0, m, N, seed, params, reinterpret_cast<uint64_t*>(uv_dev),
                                nullptr, 0, stream, false, true);
}

int32_t dcs_sample_edges_gnp(uint64_t n_vertices, double p, uint64_t seed,
                             const dcs_params* params, uint32_t* uv_dev, uint64_t capacity,
                             uint64_t* count_dev, void* stream) {
  uint64_t N = 0;
  if (edge_universe(n_vertices, DCS_MAX_BERNOULLI_UNIVERSE, &N) != DCS_OK) return DCS_EINVAL;
  if (capacity > 0 && (uv_dev == nullptr || (reinterpret_cast<uintptr_t>(uv_dev) & 7u) != 0))
    return DCS_EINVAL;
  return dcs::host::sample_bernoulli(p, N, seed, params, reinterpret_cast<uint64_t*>(uv_dev),
                                     capacity, count_dev, nullptr, 0, stream, true);
}

}  // extern "C"
