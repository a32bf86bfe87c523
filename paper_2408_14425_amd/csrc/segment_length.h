// segment_length.h -- lengths of a segment table that are scaled after they are
// stored (the path per projected cell of an inclined ray; Osborne & Sannikov,
// arXiv:2408.14425, Sec. 3.1). An FP32 length times the FP32 scale rounds three
// times where a walk rounds its FP64 product once, so a table of scaled lengths
// also keeps what the FP32 length left out.
#pragma once

#if defined(__HIPCC__)
#define RCX_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define RCX_HOST_DEVICE inline
#endif

namespace rcx {

// what (float)len leaves out of len
RCX_HOST_DEVICE float length_rest(double len) { return (float)(len - (double)(float)len); }
// len x scale, rounded once (of the FP64 length, 2^-48 of it may be missing)
RCX_HOST_DEVICE float scaled_length(float len, float rest, double scale)
{
    return (float)(((double)len + (double)rest) * scale);
}

}  // namespace rcx
