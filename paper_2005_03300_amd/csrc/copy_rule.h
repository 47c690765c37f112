// Host-only helper, free of HIP so that it can be tested by itself.
#pragma once
#include <cstddef>
#include <cstdint>

namespace gcn {

// What the runtime says of an address: the kind of memory, its GPU, and the allocation that the address lies in.
struct MemoryOf {
    bool device = false;
    int gpu = -1;
    uintptr_t base = 0;
    size_t size = 0;
};

// Whether a kernel on GPU `runs_on`, launched while `current` is, can copy an array of a matrix on GPU `matrix` to the `bytes` at
// dst, in 16-byte pieces.  Everything else (a matrix, a destination or a stream of another GPU, whose memory a kernel reaches with
// peer access only; memory of the host; a range that no one allocation holds; an odd address) is the runtime's copy, which takes or refuses it.
inline bool kernel_copies(int matrix, int current, int runs_on, const MemoryOf& of, uintptr_t dst, size_t bytes) {
    if (matrix != current || runs_on != current || !of.device || of.gpu != current || dst % 16 != 0) return false;
    return dst >= of.base && bytes <= of.size && dst - of.base <= of.size - bytes;
}

}  // namespace gcn
