// How the settling pass of a gradient that was read once fetches a listed float4 group (qa_settle.h).  Without headers of
// the GPU: the kernels and the tests on the CPU run the same lines.
#ifndef QA_OPEN_GROUP_H
#define QA_OPEN_GROUP_H

#include <stdint.h>

#if defined(__HIPCC__)
#define QA_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define QA_HOST_DEVICE inline
#endif

namespace qa {

// Group `group` of the `live` components from g on; those beyond are 0.  Quad: four floats x, y, z, w.
template <typename Quad>
QA_HOST_DEVICE Quad load_group(const float* g, uint32_t group, uint32_t live) {
  if (4 * group + 4 <= live) return *reinterpret_cast<const Quad*>(g + 4 * group);
  Quad q = {0.0f, 0.0f, 0.0f, 0.0f};                     // the row's last group; what follows it belongs to nobody
  if (4 * group < live) q.x = g[4 * group];
  if (4 * group + 1 < live) q.y = g[4 * group + 1];
  if (4 * group + 2 < live) q.z = g[4 * group + 2];
  return q;
}

}  // namespace qa

#endif
