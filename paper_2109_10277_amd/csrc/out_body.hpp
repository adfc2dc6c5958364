// Device-side body of the slice outputs: full planes, the row y = 0 or the axis
// node, on node arrays with their zero boundary.
#pragma once

#include "common.hpp"
#include "kernels.hpp"

namespace qsp {
namespace out_detail {

// Workgroups output id takes: 1024 nodes each of a plane, one for a row or a
// node.
__host__ __device__ inline int out_wgs(const Geom& g, const OutCopy& c, int id) {
  return c.kind[id] == 0 ? ((g.nx + 1) * (g.ny + 1) + 4 * kBlock - 1) / (4 * kBlock) : 1;
}

// Workgroup wg of output id.  32-bit arithmetic: a plane is below 2^23 nodes.
__device__ __forceinline__ void out_copy(const Geom& g, const OutCopy& c, int id, int wg) {
  const int kind = c.kind[id];
  const int nx = g.nx, ny = g.ny;
  const unsigned int w = static_cast<unsigned int>(nx + 1);
  const unsigned int total = kind == 0 ? w * static_cast<unsigned int>(ny + 1) : (kind == 1 ? w : 1u);
  const unsigned int e0 = static_cast<unsigned int>(wg) * 4 * kBlock + threadIdx.x;
  const unsigned int end = kind == 0 ? min(total, (static_cast<unsigned int>(wg) + 1) * 4 * kBlock) : total;
  for (unsigned int e = e0; e < end; e += kBlock) {
    int i, j;
    if (kind == 0) {
      j = static_cast<int>(e / w);
      i = static_cast<int>(e - static_cast<unsigned int>(j) * w);
    } else if (kind == 1) {
      i = static_cast<int>(e);
      j = ny / 2;
    } else {
      i = nx / 2;
      j = ny / 2;
    }
    const bool stored = i < nx && j < ny;
    const bool interior = i > 0 && j > 0 && i < nx && j < ny;
    double v = 0.0;
    if (stored) {
      const unsigned int o = static_cast<unsigned int>(j * nx + i);
      v = c.is_double[id] ? load_at(static_cast<const double*>(c.src[id]), o)
                          : static_cast<double>(load_at(static_cast<const float*>(c.src[id]), o));
      if (c.src2[id]) v += load_at(c.src2[id], o);
    }
    if (interior) {
      if (c.add_beam[id]) v -= c.beam_amp * c.bgx[i] * c.bgy[j];
      if (c.add_ion[id]) v += c.ionx ? c.n0 * c.ionx[i] * c.iony[j] : c.n0;
    }
    if (c.is_double[id])
      static_cast<double*>(c.dst[id])[e] = v;
    else
      static_cast<float*>(c.dst[id])[e] = static_cast<float>(v);
  }
}

// Workgroup b of all outputs together (none: b beyond the last).
__device__ __forceinline__ void out_copy_all(const Geom& g, const OutCopy& c, int b) {
  for (int id = 0; id < c.count; ++id) {
    const int n = out_wgs(g, c, id);
    if (b < n) {
      out_copy(g, c, id, b);
      return;
    }
    b -= n;
  }
}

inline int out_wgs_all(const Geom& g, const OutCopy& c) {
  int n = 0;
  for (int id = 0; id < c.count; ++id) n += out_wgs(g, c, id);
  return n;
}

}  // namespace out_detail
}  // namespace qsp
