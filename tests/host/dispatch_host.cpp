// Host build of the launch rules (csrc/dispatch.hpp) for the CPU tests: plain g++, nothing is launched.
#include "../../paper_2605_21325_amd/csrc/dispatch.hpp"

using namespace triinv;

// Whether a kernel with this kind of map argument (words: 0 offsets, else that many for lengths) is launched on sequences of these lengths, which
// are (packed) known by the lengths alone or else by offset arrays.
template <class Map> static int launched(const ChunkMap& map) { return launch_kernel(true, static_cast<void (*)(int, Map)>(nullptr), dim3(1), dim3(64), 0, nullptr, 1, map); }
extern "C" int dispatch_launched(int words, bool packed, const int64_t* lens, uint32_t n_seq, int64_t total)
{
    const ChunkMap map = packed ? ChunkMap{total, 0u, n_seq, nullptr, nullptr, lens} : ChunkMap{total, 0u, n_seq, lens, lens};
    return words == 0 ? launched<OffsetMap>(map) : words == 12 ? launched<KernelMap<12>>(map) : launched<KernelMap<24>>(map);
}
extern "C" bool dispatch_lengths_in_arguments(int method, bool refine) { return lengths_in_arguments(method, refine); }
