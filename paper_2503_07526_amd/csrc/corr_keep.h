// corr_keep.h -- copy of one push's samples of a group to the row where they wait.
#ifndef CORR_KEEP_H
#define CORR_KEEP_H

#include <hip/hip_runtime.h>

#include "corr_internal.h"

namespace corr {

inline int64_t keep_wide(const KeepRow &k)
{
    return (reinterpret_cast<uintptr_t>(k.src) | reinterpret_cast<uintptr_t>(k.dst)) % 16 == 0;
}

// Copy of a push's samples of a group to its waiting row: 16-byte words where
// both ends are aligned, else 4-byte ones (every sample type is a multiple of
// 4 bytes).
// Thread i0 of `stride`.
__device__ __forceinline__ void keep_row(const KeepRow &k, int64_t i0, int64_t stride)
{
    if (k.wide) {
        const uint4 *s = static_cast<const uint4 *>(k.src);
        uint4 *d = static_cast<uint4 *>(k.dst);
        const int64_t n = k.bytes / 16;
        for (int64_t i = i0; i < n; i += stride) d[i] = s[i];
        const int64_t t = n * 4 + i0; // the last 0 .. 3 words
        if (t < k.bytes / 4) static_cast<uint32_t *>(k.dst)[t] = static_cast<const uint32_t *>(k.src)[t];
    } else {
        const uint32_t *s = static_cast<const uint32_t *>(k.src);
        uint32_t *d = static_cast<uint32_t *>(k.dst);
        for (int64_t i = i0; i < k.bytes / 4; i += stride) d[i] = s[i];
    }
}

} // namespace corr

#endif
