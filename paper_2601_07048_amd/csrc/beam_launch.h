// Launch of the one-wavefront beamSearch kernels, shared by the translation units that hold their instances
// (beam_search.hip: stored vectors; beam_codes.hip: RaBitQ codes).
#pragma once
#include <stdio.h>
#include "beam_kernels.h"

namespace jx {

// largest batch that takes two expansions per round: beyond it the machine is full several times over and a search is
// bound by bandwidth, not by the lifetime of a query
static constexpr long long PAIR_MAX_QUERIES = 32768;

template <int KIND, int T, int CPL, int QB>
static hipError_t launch_nreg(const BeamArgs& a, hipStream_t st, char* name) {
    const int nreg = (a.L + 63) / 64;
    const int H = a.hash_slots;
    dim3 grid((unsigned)((a.nq + JX_BEAM_WPB - 1) / JX_BEAM_WPB)), block(JX_BEAM_WPB * 64);
    if constexpr (CPL <= 2 && (KIND == K_U8 || KIND == K_RQ4 || KIND == K_RQ1)) {
        // batches that do not fill the machine several times over are bound by the lifetime of a query: two
        // expansions per round (JX_FLAG_NO_PAIR switches it off).  Not for float vectors: their searches are bound by
        // bandwidth, and the dropped second lists cost 12 % at d = 200, L = 128.
        // measured: +2..6 % for records of one 128-byte line from L = 64 (-3 % at L = 32); -8..-11 % for the 496- and
        // 208-byte records of d = 960 / 1536 codes, whose searches run at 7 TB/s and pay for every dropped list
        // uint8 with one or two frontier registers and the tag table: that table's own loop (MODE 1) with its row read ahead is ahead
        // of the pair, pair / one expansion, us, L = 64 / 96 / 128: 20,000 x 128, 10,000 queries 249 / 232, 420 / 388, 550 / 508;
        // 300,000 283 / 267, 420 / 403, 514 / 494; 1M 421 / 382, 579 / 546, 697 / 666, 32,768 queries 1,192 / 1,052, 1,512 / 1,387,
        // 1,813 / 1,663, 1,000 181 / 164, 250 / 241, 285 / 275, four 91 / 91, 142 / 134, 172 / 165 (300,000 114 / 112, 140 / 140).
        // With four registers the pair wins (10,000 on 1M, L = 256 1,252 / 1,393), and with full ids in up to 10,000 queries (1M,
        // L = 96, 1,000 queries 266 / 294, 10,000 709 / 720, 32,768 1,957 / 1,835)
        const bool alone = KIND == K_U8 && nreg <= 2 && beam_mode<KIND, T, CPL, 2, QB>(a) == 1;
        if (nreg <= 4 && a.L >= 64 && a.R <= 64 && a.ds.rec_stride <= 128 && a.nq <= PAIR_MAX_QUERIES && H > 0 && !alone &&
            !(a.flags & JX_FLAG_NO_PAIR)) {
            const int pn = nreg <= 1 ? 1 : (nreg <= 2 ? 2 : 4);
            const size_t sh = (size_t)pn * 64 * 8 + 128 * 8 + 128 * 4 + (size_t)H * (a.tag_bits ? 2 : 4);
            dim3 pgrid((unsigned)a.nq), pblock(64);
            if (name) snprintf(name, 96, "beam_search_pair_kernel<%d,%d,%d,%d,%d>", KIND, T, CPL, pn, QB);
            if (pn == 1)
                hipLaunchKernelGGL((beam_search_pair_kernel<KIND, T, CPL, 1, QB>), pgrid, pblock, sh, st, a);
            else if (pn == 2)
                hipLaunchKernelGGL((beam_search_pair_kernel<KIND, T, CPL, 2, QB>), pgrid, pblock, sh, st, a);
            else
                hipLaunchKernelGGL((beam_search_pair_kernel<KIND, T, CPL, 4, QB>), pgrid, pblock, sh, st, a);
            return hipGetLastError();
        }
    }
#define JX_LAUNCH(NR)                                                                                   \
    {                                                                                                   \
        size_t sh = ((size_t)query_lds_bytes<KIND, T, CPL, QB>() + (size_t)mirror_entries<NR>() * 8 + 64 * 8 + 64 * 4 + (size_t)H * (a.tag_bits ? 2 : 4)) * JX_BEAM_WPB; \
        const int mode = beam_mode<KIND, T, CPL, NR, QB>(a);                                            \
        auto kern = mode == 2 ? beam_search_kernel<KIND, T, CPL, NR, QB, has_mode<KIND, T, CPL, NR>(2) ? 2 : 0> \
                              : (mode ? beam_search_kernel<KIND, T, CPL, NR, QB, has_mode<KIND, T, CPL, NR>(1) ? 1 : 0> \
                                      : beam_search_kernel<KIND, T, CPL, NR, QB, 0>);                   \
        if (sh > 48 * 1024) {                                                                           \
            hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh); \
            if (e != hipSuccess) return e;                                                              \
        }                                                                                               \
        if (name) snprintf(name, 96, "beam_search_kernel<%d,%d,%d,%d,%d,%d>", KIND, T, CPL, NR, QB, mode); \
        hipLaunchKernelGGL(kern, grid, block, sh, st, a);                                               \
        return hipGetLastError();                                                                       \
    }
    if (nreg <= 1) JX_LAUNCH(1)
    if (nreg <= 2) JX_LAUNCH(2)
    if constexpr (KIND == K_RQ1 || KIND == K_RQ4) {
        // code searches run wide beams (L = 192, 384 are sweep points): 3 and 6 frontier registers per lane
        if (nreg == 3) JX_LAUNCH(3)
    }
    if (nreg <= 4) JX_LAUNCH(4)
    if constexpr (KIND == K_RQ1 || KIND == K_RQ4) {
        if (nreg <= 6) JX_LAUNCH(6)
    }
    JX_LAUNCH(8)
#undef JX_LAUNCH
}

// Record-to-lane mapping.  Default: two 16-byte chunks per lane for records of at most 64 chunks -- a record is then
// covered by half as many lanes as it has chunks, so twice as many candidates share one instruction and the in-group
// reduction is one step shorter (1-bit codes with B_q = 8: one chunk per lane, the eight bit planes of a second
// chunk would not fit the registers); larger records: all 64 lanes, 2 to 6 chunks each.  JX_FLAG_LANES_WIDE: one
// chunk per lane.  JX_FLAG_LANES_NARROW: four chunks per lane (uint8 records of at most 8 chunks, float32 records of
// at most 32).
template <int KIND, int QB>
static hipError_t launch_shape(const BeamArgs& a, hipStream_t st, char* name) {
    const int nch = a.ds.nch;
    const bool wide = (a.flags & JX_FLAG_LANES_WIDE) != 0, narrow = (a.flags & JX_FLAG_LANES_NARROW) != 0;
    if constexpr (KIND == K_U8) {
        if (narrow && nch <= 8) return launch_nreg<KIND, 2, 4, QB>(a, st, name);
    }
    if constexpr (KIND == K_F32) {
        if (narrow && nch <= 32) return launch_nreg<KIND, 8, 4, QB>(a, st, name);
    }
    if constexpr (KIND == K_RQ1 && QB == 4) {
        // 9 to 12 code chunks (1-bit codes of d = 1536: 208-byte records): 4 lanes x 3 code chunks, meta chunk read
        // by every lane -- 16 records per pass and no idle chunk slot
        if (!wide && !narrow && a.ds.meta_chunk > 8 && a.ds.meta_chunk <= 12) return launch_nreg<KIND, 4, 3, QB>(a, st, name);
    }
    const bool two = !wide && nch <= 64 && !(KIND == K_RQ1 && (QB == 8 || nch > 16));
    if (two) {
        if constexpr (KIND == K_RQ1) {
            // 8 lanes x 2 chunks with the four bit planes of both chunks in registers (measured 10 % faster than
            // 16 x 1 at L = 64..128)
            return launch_nreg<KIND, 8, 2, QB>(a, st, name);
        } else {
            if (nch <= 8) return launch_nreg<KIND, 4, 2, QB>(a, st, name);
            if (nch <= 16) return launch_nreg<KIND, 8, 2, QB>(a, st, name);
            if (nch <= 32) return launch_nreg<KIND, 16, 2, QB>(a, st, name);
            return launch_nreg<KIND, 32, 2, QB>(a, st, name);
        }
    }
    if (nch <= 8) return launch_nreg<KIND, 8, 1, QB>(a, st, name);
    if (nch <= 16) return launch_nreg<KIND, 16, 1, QB>(a, st, name);
    if (nch <= 32) return launch_nreg<KIND, 32, 1, QB>(a, st, name);
    if (nch <= 64) return launch_nreg<KIND, 64, 1, QB>(a, st, name);
    if constexpr (KIND == K_RQ1) {
        return hipErrorInvalidValue;
    } else {
        if (nch <= 128) return launch_nreg<KIND, 64, 2, QB>(a, st, name);
        if constexpr (KIND == K_RQ4) {
            return hipErrorInvalidValue;
        } else {
            if (nch <= 256) return launch_nreg<KIND, 64, 4, QB>(a, st, name);
            if (nch <= 384) return launch_nreg<KIND, 64, 6, QB>(a, st, name);
            return hipErrorInvalidValue;
        }
    }
}

}  // namespace jx
