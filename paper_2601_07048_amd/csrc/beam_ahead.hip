// beamSearch for batches that leave the machine mostly idle: a team of wavefronts per query that reads ahead.
//
// Such a batch takes as long as its longest search, and a search is a chain of dependent expansions: select, row,
// filter, gather, distances, merge.  With long records most of a link is the gather and the arithmetic of one
// wavefront, which issues an instruction every four to five cycles whatever the rest of the machine does (d = 960
// float32: 8,000 cycles an expansion).  Here wavefront 0 owns frontier, visited table and merge, as in
// beam_search_kernel.  When the entry it has to expand next has not been fetched, it asks for the S closest unexpanded
// entries at once; all wavefronts then read those rows, evaluate the neighbours that the visited table does not hold
// and leave ids and keys in S slots of LDS.  Wavefront 0 goes on expanding from the slots, in the order Alg. 1
// prescribes, until the next entry is missing again.  An entry fetched early keeps its slot while it is among the S
// closest, so nearly all of what is fetched is used.  Distances do not depend on when they are taken, and the filter is
// applied at the expansion (which evaluates what the table held when the row was read and has forgotten since), so
// frontier sequence, results and counters are those of beam_search_kernel, float sums to the last bit (the same
// record-to-lane mapping); what is fetched beyond them costs bandwidth, which such a batch does not use.
#include <stdio.h>
#include "beam_kernels.h"

namespace jx {

#define JX_AHEAD_S 2  // expansions fetched together: 4 is no faster (-2..+1 %) and takes twice the wavefronts, 8 loses

// records in flight per lane group: 8 loads of 16 bytes per lane, 16 where a record takes 4 chunks of every lane
template <int T, int CPL>
constexpr int ahead_u() {
    constexpr int G = 64 / T;
    constexpr int U0 = CPL <= 2 ? 8 / CPL : (CPL == 3 ? 2 : (CPL == 4 ? 4 : 2));
    return U0 < 64 / G ? U0 : 64 / G;
}
// wavefronts per query: as many as the S rows have batches of records, at most 16
template <int T, int CPL>
constexpr int ahead_waves() {
    constexpr int chunks = JX_AHEAD_S * 64 / (64 / T * ahead_u<T, CPL>());
    return chunks < 4 ? 4 : (chunks > 16 ? 16 : chunks);
}

// rows of at most 64 entries only (the launcher checks)
template <int KIND, int T, int CPL, int NREG, int QB, int NW>
__global__ void __launch_bounds__(NW * 64) beam_search_ahead_kernel(BeamArgs a) {
    constexpr int S = JX_AHEAD_S;
    constexpr int G = 64 / T;
    constexpr int U = ahead_u<T, CPL>();
    constexpr int GU = G * U;
    constexpr int FCAP = mirror_entries<NREG>();
    constexpr int QL = query_lds_bytes<KIND, T, CPL, QB>();
    extern __shared__ __align__(16) unsigned char smem[];
    const int wave = threadIdx.x >> 6;
    const int lane = lane_id();
    const int g = lane / T, lig = lane % T;
    const int64_t qi = blockIdx.x;
    if (qi >= a.nq) return;  // the whole workgroup leaves

    const int H = a.hash_slots;
    const int tag_bits = a.tag_bits;
    const uint32_t id_mask = tag_bits ? ((1u << (tag_bits + 30 - __builtin_clz((uint32_t)H))) - 1u) : 0u;
    uint64_t* fr = reinterpret_cast<uint64_t*>(smem + QL);
    uint64_t* keys = fr + FCAP;                                     // [S][64] of the neighbours whose bit is set in have
    uint64_t* have = keys + S * 64;                                 // [S]
    uint64_t* late_key = have + S;                                  // [64]
    uint32_t* ids = reinterpret_cast<uint32_t*>(late_key + 64);     // [S][64] rows
    uint32_t* late_id = ids + S * 64;                               // [64]
    uint32_t* part_id = late_id + 64;                               // [NW][64]
    uint32_t* ctrl = part_id + NW * 64;                             // [0] slots to fill, then their numbers, then the vertices
    uint32_t* tab = ctrl + 4 * S;

    for (int i = threadIdx.x; i < (tag_bits ? H / 2 : H); i += NW * 64) tab[i] = JX_NONE_ID;
    for (int i = threadIdx.x; i < FCAP; i += NW * 64) fr[i] = JX_EMPTY_KEY;

    QueryRegs<KIND, CPL, QB> q;
    load_query<KIND, T, CPL, QB>(q, a.ds, qi + (qi >= a.q_skip ? 1 : 0), lig, reinterpret_cast<uint4*>(smem));

    uint64_t fk[NREG];
#pragma unroll
    for (int r = 0; r < NREG; r++) fk[r] = JX_EMPTY_KEY;
    int count = 0;
    uint64_t worst = JX_EMPTY_KEY;  // see frontier_merge
    const int L = a.L;
    const bool full = (sep_meta<KIND, CPL>() ? a.ds.meta_chunk : a.ds.nch) == T * CPL;
    uint32_t hops = 0, evals = 0;
    uint32_t slot_v[S];  // wavefront 0: the vertex whose row and keys slot j holds
#pragma unroll
    for (int j = 0; j < S; j++) slot_v[j] = JX_NONE_ID;

    // visited filter, see beam_search_body: the table's word for v and whether it lacks v; v entered into it
    auto unseen = [&](const uint32_t v, uint32_t& slot, uint32_t& word) -> bool {
        if (v == JX_NONE_ID) return false;
        if (tag_bits) {
            const uint32_t h = (v * 0x9E3779B1u) & id_mask, tag = h & ((1u << tag_bits) - 1u);
            slot = h >> tag_bits;
            word = tab[slot];
            return (word & 0xFFFFu) != tag && (word >> 16) != tag;
        }
        if (!H) return true;
        slot = __umulhi(v * 0x9E3779B1u, (uint32_t)H);
        word = tab[slot];
        return word != v;
    };
    auto mark = [&](const uint32_t v, const uint32_t slot, const uint32_t word) {
        if (tag_bits)
            tab[slot] = (word << 16) | (((v * 0x9E3779B1u) & id_mask) & ((1u << tag_bits) - 1u));
        else if (H)
            tab[slot] = v;
    };

    __syncthreads();
    if (wave == 0) {  // seed: the entry vertex
        if (lane == 0) {
            ids[0] = a.entry;
            if (tag_bits) {
                const uint32_t h = (a.entry * 0x9E3779B1u) & id_mask;
                tab[h >> tag_bits] = 0xFFFF0000u | (h & ((1u << tag_bits) - 1u));
            } else if (H) {
                tab[__umulhi(a.entry * 0x9E3779B1u, (uint32_t)H)] = a.entry;
            }
        }
        wave_sync();
        eval_batch<KIND, T, CPL, QB, 1>(q, a.ds, 0, 1, ids, keys, g, lig);
        wave_sync();
        if (lane == 0) {
            fk[0] = keys[0];
            fr[0] = keys[0];
        }
        wave_sync();
        count = 1;
        evals = 1;
    }

    for (;;) {
        if (wave == 0) {
            int nreq = 0;
            for (;;) {
                uint64_t um[NREG];
#pragma unroll
                for (int r = 0; r < NREG; r++) um[r] = ballot((fk[r] & 1ull) == 0ull);
                // ---- 1. closest unexpanded entry
                int sel_r = -1, sel_lane = 0;
                uint64_t ukey = 0;
#pragma unroll
                for (int r = 0; r < NREG; r++)
                    if (sel_r < 0 && um[r] != 0ull) {
                        sel_r = r;
                        sel_lane = __builtin_ctzll(um[r]);
                        ukey = readlane64(fk[r], sel_lane);
                    }
                if (sel_r < 0) break;  // nothing to fetch: the search is over
                const uint32_t u = key_id(ukey);
                int s = -1;
#pragma unroll
                for (int j = 0; j < S; j++)
                    if (slot_v[j] == u) s = j;
                if (s < 0) {
                    // ---- ask for the closest unexpanded entries that no slot holds, in place of what is not among them
                    uint32_t want[S];
                    bool keep[S], cached[S];
#pragma unroll
                    for (int i = 0; i < S; i++) {
                        want[i] = JX_NONE_ID;
                        keep[i] = cached[i] = false;
                        bool found = false;
#pragma unroll
                        for (int r = 0; r < NREG; r++)
                            if (!found && um[r] != 0ull) {
                                want[i] = key_id(readlane64(fk[r], __builtin_ctzll(um[r])));
                                um[r] &= um[r] - 1ull;
                                found = true;
                            }
                    }
#pragma unroll
                    for (int i = 0; i < S; i++)
#pragma unroll
                        for (int j = 0; j < S; j++)
                            if (want[i] != JX_NONE_ID && slot_v[j] == want[i]) keep[j] = cached[i] = true;
#pragma unroll
                    for (int i = 0; i < S; i++) {
                        bool placed = want[i] == JX_NONE_ID || cached[i];
#pragma unroll
                        for (int j = 0; j < S; j++)
                            if (!placed && !keep[j]) {
                                slot_v[j] = want[i];
                                keep[j] = placed = true;
                                if (lane == 0) {
                                    ctrl[1 + nreq] = (uint32_t)j;
                                    ctrl[1 + S + nreq] = want[i];
                                }
                                nreq++;
                            }
                    }
                    break;
                }
                // ---- 2. expand it from its slot
#pragma unroll
                for (int r = 0; r < NREG; r++)
                    if (r == sel_r && lane == sel_lane) fk[r] |= 1ull;
                hops++;
#pragma unroll
                for (int j = 0; j < S; j++)
                    if (j == s) slot_v[j] = JX_NONE_ID;
                const uint32_t v = ids[s * 64 + lane];
                const uint64_t got = have[s];
                const bool mine = (got >> lane) & 1ull;
                uint64_t vkey = mine ? keys[s * 64 + prefix_count(got)] : JX_EMPTY_KEY;
                uint32_t slot = 0, word = 0;
                bool is_new = unseen(v, slot, word);
                if (is_new) mark(v, slot, word);
                wave_sync();
                const uint64_t late = ballot(is_new && !mine);
                if (late) {
                    if (is_new && !mine) late_id[prefix_count(late)] = v;
                    wave_sync();
                    const int n = __builtin_popcountll(late);
                    for (int s0 = 0; s0 < n; s0 += GU) eval_batch<KIND, T, CPL, QB, U, false>(q, a.ds, s0, n, late_id, late_key, g, lig);
                    wave_sync();
                    if (is_new && !mine) vkey = late_key[prefix_count(late)];
                    wave_sync();
                }
                const int n_new = __builtin_popcountll(ballot(is_new));
                evals += (uint32_t)n_new;
                wave_sync();
                if (n_new) frontier_merge<NREG>(fk, fr, count, worst, L, is_new ? vkey : JX_EMPTY_KEY, 64, lane);
            }
            if (lane == 0) ctrl[0] = (uint32_t)nreq;
        }
        __syncthreads();
        const int nreq = (int)ctrl[0];
        if (nreq == 0) break;  // every wavefront reads the same value: the barriers stay matched
        uint32_t row[S];
#pragma unroll
        for (int i = 0; i < S; i++) {
            row[i] = JX_NONE_ID;
            if (i < nreq && lane < a.R) row[i] = a.adj[(size_t)ctrl[1 + S + i] * (size_t)a.R + lane];
        }
        int turn = 0;  // batches of records are dealt to the wavefronts in turn
#pragma unroll
        for (int i = 0; i < S; i++) {
            if (i >= nreq) break;
            const int at = (int)ctrl[1 + i] * 64;
            uint32_t slot, word;
            const bool want = unseen(row[i], slot, word);
            const uint64_t wm = ballot(want);
            const int n = __builtin_popcountll(wm), rank = prefix_count(wm);
            if (wave == 0) {
                ids[at + lane] = row[i];
                if (lane == 0) have[ctrl[1 + i]] = wm;
            }
            for (int s0 = 0; s0 < n; s0 += GU, turn++) {
                if (turn % NW != wave) continue;
                uint32_t* part = part_id + wave * 64;
                if (want && rank >= s0 && rank < s0 + GU) part[rank - s0] = row[i];
                wave_sync();
                const int m = n - s0 < GU ? n - s0 : GU;
                if (full)
                    eval_batch<KIND, T, CPL, QB, U, true>(q, a.ds, 0, m, part, keys + at + s0, g, lig);
                else
                    eval_batch<KIND, T, CPL, QB, U, false>(q, a.ds, 0, m, part, keys + at + s0, g, lig);
                wave_sync();
            }
        }
        __syncthreads();
    }

    if (wave != 0) return;
    write_results<KIND, NREG>(a, qi, fk, count, lane, hops, evals);
}

// ------------------------------------------------------------------ launch

// Batches whose teams are resident at once, four wavefronts per SIMD.  Against the one-wavefront kernels, L = 16 / 64 /
// 128, 64 queries: float32 d = 960 355 / 895 / 1463 -> 138 / 292 / 602 us, 200 115 / 227 / 422 -> 71 / 161 / 291;
// binary16 d = 960 294 / 627 / 1178 -> 108 / 224 / 406; 4-bit codes of d = 960 237 / 377 / 539 -> 220 / 328 / 462.  Whole
// searches on codes of d = 1536, L = 16 / 64 / 128 / 200: 1 bit, B_q = 4 215 / 322 / 512 / 832 -> 211 / 308 / 467 / 692, B_q
// = 8 266 / 435 / 683 / 1034 -> 239 / 356 / 550 / 818; 2 bits, B_q = 4 302 / 523 / 832 / 1234 -> 231 / 354 / 540 / 790.  Beyond
// the limit a second round of teams costs more than the team gains (without the filter at the fetch: d = 960 float32, 512
// queries, L = 128 1637 -> 1803 us; 4-bit codes, 1,024 queries 591 -> 804).
#define JX_AHEAD_WAVES 4096
#define JX_AHEAD_QUERIES 512

template <int KIND, int T, int CPL, int QB>
static hipError_t launch_ahead_shape(const BeamArgs& a, hipStream_t st, char* name, bool* done) {
    constexpr int NW = ahead_waves<T, CPL>();
    if (a.nq * NW > JX_AHEAD_WAVES || a.nq > JX_AHEAD_QUERIES) return hipSuccess;
    *done = true;
    const int nreg = (a.L + 63) / 64;
    const size_t sh0 = (size_t)query_lds_bytes<KIND, T, CPL, QB>() + JX_AHEAD_S * (64 * 12 + 8 + 16) + 64 * 12 + NW * 64 * 4 +
                       (size_t)a.hash_slots * (a.tag_bits ? 2 : 4);
#define JX_LAUNCH(NR)                                                                                                 \
    {                                                                                                                 \
        const size_t sh = sh0 + mirror_entries<NR>() * 8;                                                             \
        auto kern = beam_search_ahead_kernel<KIND, T, CPL, NR, QB, NW>;                                          \
        if (sh > 48 * 1024) {                                                                                         \
            hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh); \
            if (e != hipSuccess) return e;                                                                            \
        }                                                                                                             \
        if (name) snprintf(name, 96, "beam_search_ahead_kernel<%d,%d,%d,%d,%d,%d>", KIND, T, CPL, NR, QB, NW); \
        hipLaunchKernelGGL(kern, dim3((unsigned)a.nq), dim3(NW * 64), sh, st, a);                                     \
        return hipGetLastError();                                                                                     \
    }
    if (nreg <= 1) JX_LAUNCH(1)
    if (nreg <= 2) JX_LAUNCH(2)
    JX_LAUNCH(4)
#undef JX_LAUNCH
}

// The record-to-lane mapping of the one-wavefront kernels.  Records of at most 512 bytes on 16 or fewer lanes stay with
// them: there the merge is the longest part of a link, and handing over through LDS and barriers costs more than the
// gather (128-byte uint8 vectors 87 -> 117 us at L = 64, 64 queries, float32 d = 128 128 -> 129, binary16 92 -> 115).
template <int KIND, int QB>
static hipError_t launch_ahead_kind(const BeamArgs& a, hipStream_t st, char* name, bool* done) {
    const int nch = a.ds.nch;
    if constexpr (KIND == K_RQ1) {
        if constexpr (QB == 4) {
            if (a.ds.meta_chunk > 8 && a.ds.meta_chunk <= 12) return launch_ahead_shape<KIND, 4, 3, QB>(a, st, name, done);
            if (nch <= 16) return hipSuccess;
        } else {
            if (nch <= 8) return hipSuccess;
            if (nch <= 16) return launch_ahead_shape<KIND, 16, 1, QB>(a, st, name, done);
        }
        if (nch <= 32) return launch_ahead_shape<KIND, 32, 1, QB>(a, st, name, done);
        if (nch <= 64) return launch_ahead_shape<KIND, 64, 1, QB>(a, st, name, done);
    } else if constexpr (KIND == K_RQ4) {
        if (nch <= 16) return hipSuccess;
        if (nch <= 32) return launch_ahead_shape<KIND, 16, 2, QB>(a, st, name, done);
        if (nch <= 64) return launch_ahead_shape<KIND, 32, 2, QB>(a, st, name, done);
        if (nch <= 128) return launch_ahead_shape<KIND, 64, 2, QB>(a, st, name, done);
    } else {
        if (nch <= 32) return hipSuccess;
        if (nch <= 64) return launch_ahead_shape<KIND, 32, 2, QB>(a, st, name, done);
        if (nch <= 128) return launch_ahead_shape<KIND, 64, 2, QB>(a, st, name, done);
        if (nch <= 256) return launch_ahead_shape<KIND, 64, 4, QB>(a, st, name, done);
        if (nch <= 384) return launch_ahead_shape<KIND, 64, 6, QB>(a, st, name, done);
    }
    return hipSuccess;
}

hipError_t launch_beam_ahead(int kind, int qbits, const BeamArgs& a, hipStream_t st, char* name, bool* done) {
    *done = false;
    const uint32_t prune_flags = JX_FLAG_NO_INCR_PRUNE | JX_FLAG_NO_GRAM | JX_FLAG_GRAM_U8;
    // not for expansion lists (insertion): early in a build nearly every neighbour has been seen, and a link is the merge
    // (d = 960 float32, 24 points 122 -> 170 us, 142 points 294 -> 309)
    if (a.R > 64 || a.L > 256 || a.vis_cap || (a.flags & ~prune_flags)) return hipSuccess;
    // nor for rows so short that handing over costs more than their gather and arithmetic (one query, R = 16 / 32 / 64: 4-bit
    // codes of d = 960 at L = 200 0.86 / 0.98 / 1.29 times as fast, 1-bit codes of d = 1536 0.88 / 0.94 / 1.10, at L = 100 0.95
    // / 1.02 / 1.06; float32 d = 200 at L = 256 0.94 / 1.4 / 2.0, d = 960 1.4 and more)
    if (kind == K_RQ4 || kind == K_RQ1) {
        if (a.R <= 16 || (a.R <= 32 && a.L > 128)) return hipSuccess;
    } else if (a.R <= 16 && a.L > 128 && a.ds.nch <= 64) {
        return hipSuccess;
    }
    switch (kind) {
        case K_F32: return launch_ahead_kind<K_F32, 0>(a, st, name, done);
        case K_F16: return launch_ahead_kind<K_F16, 0>(a, st, name, done);
        case K_RQ4: return qbits == 8 ? launch_ahead_kind<K_RQ4, 8>(a, st, name, done) : launch_ahead_kind<K_RQ4, 4>(a, st, name, done);
        case K_RQ1: return qbits == 8 ? launch_ahead_kind<K_RQ1, 8>(a, st, name, done) : launch_ahead_kind<K_RQ1, 4>(a, st, name, done);
    }
    return hipSuccess;
}

}  // namespace jx
