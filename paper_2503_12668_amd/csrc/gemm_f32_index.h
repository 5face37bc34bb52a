// Which k a load of the float32 kernels (gemm_f32.hip) starts at, counted from the row's or the piece's first: plain arithmetic,
// so that a host program can walk through every load of a launch (tests/test_f32_gemm_bounds.py does).
#pragma once
#if defined(__HIPCC__) || defined(__HIP__)
#define ZO2_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define ZO2_HOST_DEVICE inline
#endif

namespace zo2 {

// Slab kt of nk, slabs of `slab` k, the four k from `chunk` on in it; K is a multiple of 8.  A slab past the last one is the last again.
// Where the four lie past the end of the row, and their place in LDS is to hold zeros, the address is that of the row's first four.
ZO2_HOST_DEVICE bool f32_chunk_inside(int kt, int nk, int slab, int chunk, int K) { return (kt < nk ? kt : nk - 1) * slab + chunk < K; }
ZO2_HOST_DEVICE int f32_chunk_at(int kt, int nk, int slab, int chunk, int K) {
    return f32_chunk_inside(kt, nk, slab, chunk, K) ? (kt < nk ? kt : nk - 1) * slab + chunk : 0;
}

}  // namespace zo2
