// Arithmetic of the walked attention's work split, shared by the kernels and the host launcher.  Plain C++ without HIP
// types, so that it can also be compiled and checked on a CPU.
#pragma once

#ifdef __HIPCC__
#define RS_HD __host__ __device__ __forceinline__
#else
#define RS_HD inline
#endif

namespace rs {

constexpr int ATT_BT = 64;        // positions per workgroup and pass

// Start of the pass that is requested while the pass at t0 (of a slice that ends before t_end) is multiplied.  It stays on
// the slice's grid of whole passes: V pieces are 16-byte loads of 8 positions, which are aligned only at starts that are a
// multiple of 8.  The last pass requests itself once more (its lines are in the cache; the values are not used).
RS_HD int walk_next_pass(int t0, int t_end) { return t0 + ATT_BT < t_end ? t0 + ATT_BT : t0; }

}  // namespace rs
