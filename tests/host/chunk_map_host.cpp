// Host build of the chunk map (csrc/chunk_map.hpp) for the CPU tests: plain g++, no GPU.
#include "../../paper_2605_21325_amd/csrc/chunk_map.hpp"

extern "C" void chunk_map_locate(int C, int64_t Tlen_or_total, uint32_t cps, uint32_t n_seq, const int64_t* cu_seqlens,
                                 const int64_t* cu_chunks, uint32_t bc, int64_t* tok0, int* valid)
{
    const triinv::ChunkMap map{Tlen_or_total, cps, n_seq, cu_seqlens, cu_chunks};
    triinv::ChunkPos p;
    switch (C) {
    case 16: p = triinv::locate_chunk<16>(map, bc); break;
    case 32: p = triinv::locate_chunk<32>(map, bc); break;
    case 64: p = triinv::locate_chunk<64>(map, bc); break;
    default: p = triinv::locate_chunk<128>(map, bc); break;
    }
    *tok0 = p.tok0;
    *valid = p.valid;
}

// The packed layout: lengths in a kernel's argument of 12 or 24 words.  False if it does not take them.
template <int WORDS> static bool locate_packed(int C, int64_t total, uint32_t n_seq, const int64_t* lens, uint32_t bc, int64_t* tok0, int* valid)
{
    using namespace triinv;
    if (!KernelMap<WORDS>::bits_of(lens, (int)n_seq)) return false;
    const KernelMap<WORDS> map(ChunkMap{total, 0u, n_seq, nullptr, nullptr, lens});
    const ChunkPos p = C == 16 ? locate_chunk<16>(map, bc) : C == 32 ? locate_chunk<32>(map, bc) : C == 64 ? locate_chunk<64>(map, bc) : locate_chunk<128>(map, bc);
    *tok0 = p.tok0;
    *valid = p.valid;
    return true;
}
extern "C" bool chunk_map_locate_packed(int words, int C, int64_t total, uint32_t n_seq, const int64_t* lens, uint32_t bc, int64_t* tok0, int* valid)
{
    return words == 12 ? locate_packed<12>(C, total, n_seq, lens, bc, tok0, valid) : locate_packed<24>(C, total, n_seq, lens, bc, tok0, valid);
}

// The other layouts as a kernel gets them.
extern "C" void chunk_map_locate_argument(int C, int64_t Tlen_or_total, uint32_t cps, uint32_t n_seq, const int64_t* cu_seqlens,
                                          const int64_t* cu_chunks, uint32_t bc, int64_t* tok0, int* valid)
{
    const triinv::InvMap map(triinv::ChunkMap{Tlen_or_total, cps, n_seq, cu_seqlens, cu_chunks});
    const triinv::ChunkPos p = C == 64 ? triinv::locate_chunk<64>(map, bc) : triinv::locate_chunk<128>(map, bc);
    *tok0 = p.tok0;
    *valid = p.valid;
}
