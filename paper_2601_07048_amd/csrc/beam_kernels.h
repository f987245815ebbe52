// beamSearch kernels shared by the translation units that launch them (beam_search.hip: the production
// instances; beam_variants.hip: the ablation instances).
#pragma once
#include "jx_distance.h"

namespace jx {

// Tuning constants (compile-time; the values are the optima measured on gfx950 at N = 1M, 10,000 queries):
// 16-byte loads in flight per lane for the exact uint8, 1-bit and 4-bit kernels, and the
// waves per SIMD the small exact kernels are held to.
#ifndef JX_UMAX_EXACT
#define JX_UMAX_EXACT 8
#endif
#ifndef JX_UMAX_RQ1
#define JX_UMAX_RQ1 8
#endif
#ifndef JX_UMAX_RQ4
#define JX_UMAX_RQ4 8
#endif
#ifndef JX_WPE_RQ1
#define JX_WPE_RQ1 5  // wavefronts per SIMD the 1-bit kernel with its query planes in LDS is held to (96 VGPRs)
#endif
#ifndef JX_WPE_EXACT
#define JX_WPE_EXACT 6
#endif

// Results of one query: the first out_k frontier entries that are not logically deleted (Sec. 4.6: deleted vertices
// are traversed but never returned), then padding; the expansion and evaluation counters.
template <int KIND, int NREG>
__device__ __forceinline__ void write_results(const BeamArgs& a, const int64_t qi, const uint64_t (&fk)[NREG], const int count,
                                              const int lane, const uint32_t hops, const uint32_t evals) {
    int base_pos = 0;
#pragma unroll
    for (int r = 0; r < NREG; r++) {
        const int p = r * 64 + lane;
        const uint64_t k = fk[r];
        const uint32_t id = key_id(k);
        bool keep = p < count;
        if (keep && a.deleted) keep = a.deleted[id] == 0;
        const uint64_t km = ballot(keep);
        const int pos = base_pos + prefix_count(km);
        if (keep && pos < a.out_k) {
            const uint32_t dc = key_dist(k);
            float d;
            if constexpr (KIND == K_U8)
                d = (float)dc;
            else
                d = ordered_to_f32(dc);
            a.out_ids[qi * a.out_k + pos] = id;
            a.out_dist[qi * a.out_k + pos] = d;
        }
        base_pos += __builtin_popcountll(km);
    }
    for (int p = base_pos + lane; p < a.out_k; p += 64) {
        a.out_ids[qi * a.out_k + p] = JX_NONE_ID;
        a.out_dist[qi * a.out_k + p] = __builtin_inff();
    }
    if (a.stats && lane == 0) {
        // 64 stripes of counters, one 128-byte line each: ten thousand same-address atomics would serialise
        unsigned long long* sp = a.stats + (size_t)(qi & 63) * 16;
        atomicAdd(&sp[0], (unsigned long long)hops);
        atomicAdd(&sp[1], (unsigned long long)evals);
    }
}

// Entries of the LDS mirror of the frontier: the binary search wants a power of two
template <int NREG>
constexpr int mirror_entries() {
    int m = 64;
    while (m < NREG * 64) m *= 2;
    return m;
}

// Merge step: candidates ck (one per lane, lane < n) into the sorted frontier (registers fk: entry p in lane p % 64,
// register p / 64; mirror fr in LDS, unused slots hold the largest key).  Every candidate finds its rank among the
// frontier entries by binary search in the mirror, all candidates at once (this also recognises an id that is in
// the frontier already).  A candidate that lands in register r (rank / 64 == r) precedes every entry of the higher
// registers and none of the lower ones, so only register r's lanes have to compare against it: the candidates are
// broadcast one by one per register, which makes the step cost O(inserted) instead of O(inserted x registers).
// One LDS scatter / gather applies the permutation; the tail beyond L is dropped.
// That chain of dependent LDS reads is about 1,300 cycles.  Up to MERGE_FEW candidates (an expansion inserts 4 to 7 on
// average) go in one by one without LDS instead, about 150 cycles each; broadcasting and ranking them with ballots but
// moving the frontier through LDS once took 1,400.  With three and more registers per lane an insertion moves them all,
// and the chain is the shorter way (L = 256, 10,000 queries, ten one by one: 1256 -> 1341 us).
template <int NREG>
constexpr int MERGE_FEW = NREG == 1 ? 10 : (NREG == 2 ? 8 : 0);  // frontier_merge: candidates inserted one by one

template <int NREG>
__device__ __forceinline__ void frontier_merge(uint64_t (&fk)[NREG], uint64_t* fr, int& count, uint64_t& worst, const int L,
                                               const uint64_t ck, const int n, const int lane) {
    constexpr int FCAP = NREG * 64;
    constexpr int MIR = mirror_entries<NREG>();
    const uint64_t ckm = ck | 1ull;
    // worst = entry L - 1 of the frontier with the flag bit set (all ones while the frontier is not full): kept in
    // a register from merge to merge, so that the usual expansion, which inserts nothing, reads no LDS here
    bool beats = lane < n && ckm < worst;
    uint64_t todo = ballot(beats);
    if (todo == 0ull) return;  // nothing enters the frontier (the common case late in a search)
    if (MERGE_FEW<NREG> > 0 && __builtin_popcountll(todo) <= MERGE_FEW<NREG>) {  // (a constant: no such code at all where 0)
        // few candidates (the usual case): one after the other, ranked with a ballot per frontier register and moved
        // in with a one-lane shift; the mirror is written and not waited for
        int n_ins = 0;
        while (todo) {
            const int j = __builtin_ctzll(todo);
            todo &= todo - 1ull;
            const uint64_t s = readlane64(ckm, j);
            int rank = 0;
            uint64_t same = 0;
#pragma unroll
            for (int r = 0; r < NREG; r++) {
                rank += __builtin_popcountll(ballot((fk[r] | 1ull) < s));
                same |= ballot((fk[r] | 1ull) == s);
            }
            if (same) continue;  // in the frontier already (the visited table forgot it)
            n_ins++;
#pragma unroll
            for (int r = NREG - 1; r >= 0; r--) {
                const uint64_t in = r ? readlane64(fk[r ? r - 1 : 0], 63) : 0ull;
                const uint64_t up = wave_shift_up(fk[r], in);
                const int p = r * 64 + lane;
                fk[r] = p < rank ? fk[r] : (p == rank ? s - 1ull : up);
            }
        }
        if (n_ins == 0) return;
#pragma unroll
        for (int r = 0; r < NREG; r++) {
            if (r * 64 + lane >= L) fk[r] = JX_EMPTY_KEY;  // truncate to the beam width
            fr[r * 64 + lane] = fk[r];
            if (r == (L - 1) >> 6) worst = readlane64(fk[r], (L - 1) & 63) | 1ull;
        }
        wave_sync();
        count = count + n_ins < L ? count + n_ins : L;
        return;
    }
    // many (the first expansions of a search): all ranks at once by binary search in the mirror
    uint32_t pos = 0;
#pragma unroll
    for (int step = MIR / 2; step >= 1; step >>= 1)
        if ((fr[pos + step - 1] | 1ull) < ckm) pos += step;
    // an id that is already in the frontier (the visited table forgot it) is dropped
    beats = beats && ((fr[pos] | 1ull) != ckm);
    const uint64_t sm = ballot(beats);
    if (sm == 0ull) return;
    const int n_ins = __builtin_popcountll(sm);
    uint32_t shift[NREG];
    uint32_t crank = 0, below = 0;
#pragma unroll
    for (int r = 0; r < NREG; r++) {
        uint64_t m = NREG == 1 ? sm : ballot(beats && (pos >> 6) == (uint32_t)r);
        shift[r] = below;  // candidates of the lower registers precede every entry of this one
        below += (uint32_t)__builtin_popcountll(m);
        const uint64_t mine = fk[r] | 1ull;
        while (m) {
            const int j = __builtin_ctzll(m);
            m &= m - 1;
            const uint64_t s = readlane64(ckm, j);
            shift[r] += (s < mine) ? 1u : 0u;
            crank += (s < ckm) ? 1u : 0u;  // over all registers' loops: rank among the inserted candidates
        }
    }
    wave_sync();  // all binary-search reads of fr[] are done
#pragma unroll
    for (int r = 0; r < NREG; r++) {
        uint32_t np = (uint32_t)(r * 64 + lane) + shift[r];
        if (np < (uint32_t)FCAP) fr[np] = fk[r];
    }
    if (beats) {
        uint32_t np = pos + crank;
        if (np < (uint32_t)FCAP) fr[np] = ck;
    }
    wave_sync();
#pragma unroll
    for (int r = 0; r < NREG; r++) {
        fk[r] = fr[r * 64 + lane];
        if (r * 64 + lane >= L) {  // truncate to the beam width
            fk[r] = JX_EMPTY_KEY;
            fr[r * 64 + lane] = JX_EMPTY_KEY;
        }
    }
    wave_sync();
    count = count + n_ins < L ? count + n_ins : L;
#pragma unroll
    for (int r = 0; r < NREG; r++)
        if (r == (L - 1) >> 6) worst = readlane64(fk[r], (L - 1) & 63) | 1ull;
}

// The expansion list of one query (Alg. 1's set V; what Alg. 4 hands to robustPrune): its first vis_cap entries in expansion
// order, sorted by (distance, id), those not logically deleted, written to out_ids / out_dist [qi][out_k] and padded with
// JX_NONE / +inf.  While the search runs, 64 expansions at a time stand in a register (visited_add) and then in the query's own
// part of the two output arrays, vis_cap / 2 keys each (visited_slot).  In LDS the list took 4 of 10 KB at L = 128 and with that
// a third of the wavefronts a CU can hold (200,000 x 128 uint8 built in 22.3 -> 18.8 ms, 60,000 x 128 float32 20.8 -> 19.2, 32
// points into 50,000 uint8 249 -> 231 us); a store at every expansion is waited for by the next gather (249 -> 299).
__device__ __forceinline__ uint64_t* visited_slot(const BeamArgs& a, const int64_t qi, const uint32_t i) {
    const uint32_t half = (uint32_t)a.vis_cap / 2;
    return i < half ? reinterpret_cast<uint64_t*>(a.out_ids + qi * a.out_k) + i : reinterpret_cast<uint64_t*>(a.out_dist + qi * a.out_k) + (i - half);
}

__device__ __forceinline__ void visited_add(const BeamArgs& a, const int64_t qi, uint64_t& vk, const uint32_t hops, const uint64_t key, const int lane) {
    vk = lane == (int)(hops & 63u) ? key : vk;
    if ((hops & 63u) == 63u && hops < (uint32_t)a.vis_cap) *visited_slot(a, qi, hops - 63u + (uint32_t)lane) = vk;
}

// Every entry of the final frontier has been expanded, and an expanded vertex that is not in it was pushed out by closer
// ones: it lies behind all of them.  So the list is the frontier, which is sorted, and then those pushed out, which are few
// (hops - L, a handful at L = 128) and are sorted in LDS (list: room for vis_cap keys, where the visited table was).  Only a
// search of more than vis_cap expansions has to sort them all.
template <int KIND, int NREG>
__device__ __forceinline__ void write_visited(const BeamArgs& a, const int64_t qi, const uint64_t (&fk)[NREG], const int count,
                                              const uint64_t worst, const uint64_t vk, uint64_t* list, const uint32_t hops, const int lane) {
    const bool whole = hops <= (uint32_t)a.vis_cap;
    const int n = whole ? (int)hops : a.vis_cap;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // the keys stored below are read back by other lanes
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    wave_sync();
    int m = 0;
    for (int i0 = 0; i0 < n; i0 += 64) {
        const uint64_t k = i0 + 64 <= n ? *visited_slot(a, qi, (uint32_t)(i0 + lane)) : vk;
        const bool out = i0 + lane < n && (!whole || k > worst);
        const uint64_t om = ballot(out);
        if (out) list[m + prefix_count(om)] = k;
        m += __builtin_popcountll(om);
    }
    int cap = 1;
    while (cap < m) cap <<= 1;
    for (int i = m + lane; i < cap; i += 64) list[i] = JX_EMPTY_KEY;
    wave_sync();
    for (int k = 2; k <= cap; k <<= 1) {  // a bitonic network
        for (int j = k >> 1; j >= 1; j >>= 1) {
            for (int p = lane; p < cap / 2; p += 64) {
                const int i = ((p & ~(j - 1)) << 1) | (p & (j - 1));  // p with a zero bit inserted at bit log2(j)
                const int o = i | j;
                const uint64_t x = list[i], y = list[o];
                const bool up = (i & k) == 0;
                if ((x > y) == up) {
                    list[i] = y;
                    list[o] = x;
                }
            }
            wave_sync();
        }
    }
    int base_pos = 0;
    auto put = [&](const uint64_t k, bool keep) {
        const uint32_t id = key_id(k);
        if (keep && a.deleted) keep = a.deleted[id] == 0;
        const uint64_t km = ballot(keep);
        const int pos = base_pos + prefix_count(km);
        if (keep && pos < a.out_k) {
            const uint32_t dc = key_dist(k);
            float d;
            if constexpr (KIND == K_U8)
                d = (float)dc;
            else
                d = ordered_to_f32(dc);
            a.out_ids[qi * a.out_k + pos] = id;
            a.out_dist[qi * a.out_k + pos] = d;
        }
        base_pos += __builtin_popcountll(km);
    };
    if (whole) {
#pragma unroll
        for (int r = 0; r < NREG; r++) put(fk[r], r * 64 + lane < count);
    }
    for (int p0 = 0; p0 < m; p0 += 64) put(list[p0 + lane < m ? p0 + lane : 0], p0 + lane < m);
    for (int p = base_pos + lane; p < a.out_k; p += 64) {
        a.out_ids[qi * a.out_k + p] = JX_NONE_ID;
        a.out_dist[qi * a.out_k + p] = __builtin_inff();
    }
}

// LDS behind the candidate buffers: the visited table, and after the search what the expansion list has to sort
inline size_t table_bytes(const BeamArgs& a) {
    const size_t t = (size_t)a.hash_slots * (a.tag_bits ? 2 : 4), v = (size_t)a.vis_cap * 8;
    return t > v ? t : v;
}

// Records in flight per lane group of the wide instances, for batches of at most two wavefronts per SIMD: 48 records at
// once (a row has about 36 new neighbours), in at most 160 registers
template <int T, int CPL>
constexpr int wide_u() {
    constexpr int G = 64 / T;
    constexpr int want = (48 + G - 1) / G, fit = 160 / (4 * CPL);
    return want < fit ? want : fit;
}

// Not where the usual form covers a row already (four lanes per record)
template <int T, int CPL>
constexpr bool has_wide() {
    return 64 / T * wide_u<T, CPL>() > 64 / T * (8 / CPL > 0 ? 8 / CPL : 1) && T > 4;
}
// Beyond 1,536 queries the registers of the wide instances cost more residency than the loads in flight gain.  L = 128,
// 1,000 queries: d = 128 float32 343 -> 270 us, d = 960 2220 -> 1930, its 4-bit codes 679 -> 599; as insertion search
// (expansion lists) d = 960, 1,060 points 1233 -> 940 us.
static constexpr long long WIDE_MAX_QUERIES = 1536;

// Whether two wavefronts of a wide instance fit a SIMD: at most 256 registers each, as compiled (160 of loads in flight leave
// room for the fewest frontier registers only)
template <int KIND, int T, int CPL, int NREG, int QB>
constexpr bool wide_two_resident() {
    if (4 * CPL * wide_u<T, CPL>() < 160) return true;
    return CPL > 1 && NREG <= (QB == 8 ? 1 : 2);
}

// Largest batch of a wide instance.  One wavefront per SIMD ends at 1,024 queries: the next waits for a whole search (binary16
// d = 960 and float32 d = 200 at L = 200, 8-bit codes at L = 128 from 1,060 to 1,536 queries 1.3 to 1.5 times as long).
// Records of 64 lanes x 4 or 6 chunks are bound by bandwidth earlier: float32 d = 960 at L = 64 / 128, gain at 1,152 / 1,280 /
// 1,536 queries 1.00 / 1.00 / 0.97, d = 1,536 0.94 / 0.91 / 0.92, but at L = 24 1.11 / 1.07 / 1.03 and 1.08 / 1.07 / 1.03;
// insert calls of 1,280 and 1,536 points, expansion lists of d = 1,536, 7.81 and 8.67 ms with them, 7.58 and 8.56 without
template <int KIND, int T, int CPL, int NREG, int QB>
inline long long wide_max_queries(int L) {
    if (!wide_two_resident<KIND, T, CPL, NREG, QB>()) return 1024;
    if (CPL >= 4 && T == 64 && L > 32) return CPL == 4 ? 1280 : 1024;
    return WIDE_MAX_QUERIES;
}

// Whether the instances of a shape with NREG frontier registers exist (MODE of beam_search_body)
template <int KIND, int T, int CPL, int NREG>
constexpr bool has_mode(int mode) {
    return mode == 0 || (mode == 1 && NREG < 6) || (mode == 2 && has_wide<T, CPL>() && (NREG < 6 || KIND != K_RQ1));
}

// The form of a batch.  Figures: as many times as fast as the general form.
//   2  wide: where a row may hold more neighbours than the usual form keeps in flight, and more than 16 unless a record takes
//      four chunks of every lane (R = 16, one query, L = 200: float32 d = 96 0.95, d = 200 0.92, d = 960 1.4).  With six
//      and eight frontier registers the merge is the longest part: not for bit planes (0.88 to 1.00), and others only where
//      rows are long or records are (L = 300, R = 16 / 64: float32 d = 96 0.90 / 1.06, d = 960 1.13 / 1.24)
//   1  the tag table's own loop.  It costs six or eight wavefronts' worth of registers the seventh or the fifth, and with six
//      and eight frontier registers it gains nothing (0.93 to 1.01).  Short records with three or four frontier registers
//      pay for the lost wavefront beyond 4,096 queries (256-byte uint8 and binary16, L = 200, 4,500 queries 0.78, 10,000
//      0.89, 2,500 1.03); longer ones wait for memory (0.98 to 1.10)
template <int KIND, int T, int CPL, int NREG, int QB>
inline int beam_mode(const BeamArgs& a) {
    if (a.tag_bits == 0 || a.R > 64) return 0;
    constexpr int usual = 64 / T * (8 / CPL > 0 ? 8 / CPL : 1);  // records in flight
    constexpr int rows = CPL >= 4 || usual > 16 ? usual : 16;
    if (has_mode<KIND, T, CPL, NREG>(2) && a.R > rows && a.nq <= wide_max_queries<KIND, T, CPL, NREG, QB>(a.L) &&
        (NREG < 6 || a.R > 32 || a.ds.nch > 64))
        return 2;
    if (NREG >= 6 || (NREG >= 3 && a.ds.rec_stride <= 256 && a.nq > 4096)) return 0;
    return 1;
}

// One query per wavefront, WPB wavefronts (queries) per workgroup; TILED selects the element-strided loads of the
// load ablation (jx_distance.h); VIS returns the expansion list instead of the frontier (BeamArgs::vis_cap).
template <int KIND, int T, int CPL, int NREG, int QB, int WPB, bool TILED, bool VIS = false, int MODE = 0>
__device__ __forceinline__ void beam_search_body(const BeamArgs& a) {
    constexpr int G = 64 / T;
    constexpr int UMAX = MODE == 3 ? 4 : (KIND == K_RQ1) ? JX_UMAX_RQ1 : ((KIND == K_U8) ? JX_UMAX_EXACT : ((KIND == K_RQ4) ? JX_UMAX_RQ4 : 8));  // 16-byte loads in flight per lane (the 1-bit path keeps its bit planes in registers)
    constexpr int U0 = (UMAX / CPL) > 0 ? (UMAX / CPL) : 1;
    constexpr bool FAST = MODE != 0;
    constexpr int U = MODE == 2 ? wide_u<T, CPL>() : (U0 < (64 / G) ? U0 : (64 / G));  // records in flight per lane group
    constexpr int FCAP = mirror_entries<NREG>();  // entries of the LDS mirror of the frontier
    extern __shared__ __align__(16) unsigned char smem[];
    const int wave = threadIdx.x >> 6;
    const int lane = lane_id();
    const int g = lane / T, lig = lane % T;
    const int64_t qi = (int64_t)blockIdx.x * WPB + wave;
    if (qi >= a.nq) return;  // whole wavefront leaves; there is no block-level barrier below

    const int H = a.hash_slots;
    const int tag_bits = a.tag_bits;  // > 0: 16-bit entries (slot and tag together name the id exactly)
    const uint32_t id_mask = tag_bits ? ((1u << (tag_bits + 30 - __builtin_clz((uint32_t)H))) - 1u) : 0u;  // H / 2 sets
    constexpr int QL = query_lds_bytes<KIND, T, CPL, QB>();  // query bit planes kept in LDS (jx_distance.h)
    const size_t per_wave = (size_t)QL + (size_t)FCAP * 8 + 64 * 8 + 64 * 4 + (size_t)H * (tag_bits ? 2 : 4);  // (VIS: one wavefront per workgroup)
    unsigned char* my = smem + per_wave * wave;
    uint64_t* fr = reinterpret_cast<uint64_t*>(my + QL);
    uint64_t* cand_key = fr + FCAP;
    uint32_t* cand_id = reinterpret_cast<uint32_t*>(cand_key + 64);
    uint32_t* tab = cand_id + 64;

    for (int i = lane; i < (tag_bits ? H / 2 : H); i += 64) tab[i] = JX_NONE_ID;
    for (int i = lane; i < FCAP; i += 64) fr[i] = JX_EMPTY_KEY;

    QueryRegs<KIND, CPL, QB> q;
    load_query<KIND, T, CPL, QB, TILED>(q, a.ds, qi + (qi >= a.q_skip ? 1 : 0), lig, reinterpret_cast<uint4*>(my));

    uint64_t fk[NREG];
#pragma unroll
    for (int r = 0; r < NREG; r++) fk[r] = JX_EMPTY_KEY;
    int count = 0;
    uint64_t worst = JX_EMPTY_KEY;  // see frontier_merge
    const int L = a.L;
    const bool full = (sep_meta<KIND, CPL>() ? a.ds.meta_chunk : a.ds.nch) == T * CPL;  // wave-uniform: no chunk slot is idle
    uint32_t hops = 0, evals = 0;
    uint64_t vk = 0;  // VIS: see visited_add

    // seed: the entry vertex
    if (lane == 0) {
        cand_id[0] = a.entry;
        if (tag_bits) {
            const uint32_t h = (a.entry * 0x9E3779B1u) & id_mask;
            tab[h >> tag_bits] = 0xFFFF0000u | (h & ((1u << tag_bits) - 1u));
        } else if (H) {
            tab[__umulhi(a.entry * 0x9E3779B1u, (uint32_t)H)] = a.entry;
        }
    }
    wave_sync();
    eval_batch<KIND, T, CPL, QB, 1, false, TILED>(q, a.ds, 0, 1, cand_id, cand_key, g, lig);
    wave_sync();
    if (lane == 0) {
        fk[0] = cand_key[0];
        fr[0] = cand_key[0];
    }
    wave_sync();
    count = 1;
    evals = 1;

    if constexpr (FAST) {
        // tag table, rows of one 64-entry block: the same loop without the general form's branches (a lone wavefront
        // issues an instruction every four to five cycles, so they are latency), and with the row of the second closest
        // unexpanded entry read ahead, behind the gathers of this expansion: it is the next one to be expanded unless a
        // new candidate overtakes it.  Cycles of an expansion, 128-byte vectors, L = 32, 1,000 queries: select and row
        // 480, filter 330, gather and distances 1,250, merge 1,220.  With the one-by-one merge (frontier_merge), before
        // -> after: N = 1M, L = 16, one query 37.6 -> 33.0 us, 1,000 queries 92 -> 80, 10,000 177 -> 168
        const uint32_t* my_adj = a.adj + (lane < a.R ? lane : 0);
        uint32_t row_u = a.entry, row_v = my_adj[(size_t)a.entry * (uint32_t)a.R];
        for (;;) {
            // ---- 1. the two closest unexpanded entries
            uint64_t ukey = 0;
            uint32_t u2 = 0;
            int sel_r = -1, sel_lane = 0;
            bool have2 = false;
#pragma unroll
            for (int r = 0; r < NREG; r++) {
                uint64_t m = ballot((fk[r] & 1ull) == 0ull);
                if (sel_r < 0 && m != 0ull) {
                    sel_r = r;
                    sel_lane = __builtin_ctzll(m);
                    ukey = readlane64(fk[r], sel_lane);
                    m &= m - 1ull;
                }
                if (!have2 && m != 0ull) {
                    have2 = true;
                    u2 = readlane32((uint32_t)fk[r], __builtin_ctzll(m)) >> 1;
                }
            }
            if (sel_r < 0) break;
            const uint32_t u = key_id(ukey);
#pragma unroll
            for (int r = 0; r < NREG; r++) fk[r] |= (r == sel_r && lane == sel_lane) ? 1ull : 0ull;
            if constexpr (VIS) {
                visited_add(a, qi, vk, hops, ukey | 1ull, lane);
            }
            hops++;
            // ---- 2. adjacency row
            if (row_u != u) row_v = my_adj[(size_t)u * (uint32_t)a.R];
            const uint32_t v = lane < a.R ? row_v : JX_NONE_ID;
            // ---- 3. visited filter (see the general form); padding finds its own tag in no set and is masked
            const uint32_t h = (v * 0x9E3779B1u) & id_mask;
            const uint32_t tag = h & ((1u << tag_bits) - 1u);
            const uint32_t w = tab[h >> tag_bits];
            row_u = have2 ? u2 : u;
            row_v = my_adj[(size_t)row_u * (uint32_t)a.R];
            const bool is_new = v != JX_NONE_ID && (w & 0xFFFFu) != tag && (w >> 16) != tag;
            const uint64_t nm = ballot(is_new);
            if (nm == 0ull) continue;
            const int n_new = __builtin_popcountll(nm);
            if (is_new) {
                tab[h >> tag_bits] = (w << 16) | tag;
                cand_id[prefix_count(nm)] = v;
            }
            wave_sync();
            // ---- 4./5. gather + distances
            if (full) {
                for (int s0 = 0; s0 < n_new; s0 += G * U)
                    eval_batch<KIND, T, CPL, QB, U, true, TILED>(q, a.ds, s0, n_new, cand_id, cand_key, g, lig);
            } else {
                for (int s0 = 0; s0 < n_new; s0 += G * U)
                    eval_batch<KIND, T, CPL, QB, U, false, TILED>(q, a.ds, s0, n_new, cand_id, cand_key, g, lig);
            }
            evals += n_new;
            wave_sync();
            const uint64_t ck = lane < n_new ? cand_key[lane] : JX_EMPTY_KEY;
            wave_sync();
            // ---- 6. merge into the sorted frontier
            frontier_merge<NREG>(fk, fr, count, worst, L, ck, n_new, lane);
        }
    } else
    for (;;) {
        // ---- 1. closest unexpanded entry
        int sel_r = -1, sel_lane = 0;
#pragma unroll
        for (int r = 0; r < NREG; r++) {
            uint64_t m = ballot((fk[r] & 1ull) == 0ull);
            if (sel_r < 0 && m != 0ull) {
                sel_r = r;
                sel_lane = __builtin_ctzll(m);
            }
        }
        if (sel_r < 0) break;
        uint32_t u = 0;
#pragma unroll
        for (int r = 0; r < NREG; r++) {
            if (r == sel_r) {
                const uint64_t ukey = readlane64(fk[r], sel_lane);
                u = key_id(ukey);
                if (lane == sel_lane) fk[r] |= 1ull;
                if constexpr (VIS) {
                    visited_add(a, qi, vk, hops, ukey | 1ull, lane);
                }
            }
        }
        hops++;
        const uint32_t* row = a.adj + (size_t)u * (size_t)a.R;
        for (int rb = 0; rb < a.R; rb += 64) {
            // ---- 2. adjacency row (coalesced)
            uint32_t v = JX_NONE_ID;
            if (rb + lane < a.R) v = row[rb + lane];
            bool is_new = false;
            // ---- 3. visited filter
            if (v != JX_NONE_ID) {
                if (tag_bits) {
                    // ids below 2^b, b = log2(sets) + tag_bits: multiplying by an odd constant permutes them, so the
                    // set (high bits) and the tag (low bits) of the product identify the id.  Two tags per set in one
                    // 32-bit word, most recent first: one LDS read finds both, one write installs the new one
                    const uint32_t h = (v * 0x9E3779B1u) & id_mask;
                    const uint32_t tag = h & ((1u << tag_bits) - 1u);
                    const uint32_t w = tab[h >> tag_bits];
                    is_new = (w & 0xFFFFu) != tag && (w >> 16) != tag;
                    if (is_new) tab[h >> tag_bits] = (w << 16) | tag;
                } else if (H) {
                    uint32_t h = __umulhi(v * 0x9E3779B1u, (uint32_t)H);
                    is_new = tab[h] != v;
                    if (is_new) tab[h] = v;
                } else {
                    // no filter (Alg. 2 as printed): every neighbour is evaluated; one that is still in the frontier
                    // is recognised by the merge, one that has left it cannot come back (its key is above the worst)
                    is_new = true;
                }
            }
            uint64_t nm = ballot(is_new);
            if (ballot(v != JX_NONE_ID) == 0ull) break;  // rows are filled from the left
            const int n_new = __builtin_popcountll(nm);
            if (n_new == 0) continue;
            if (is_new) cand_id[prefix_count(nm)] = v;
            wave_sync();
            // ---- 4./5. gather + distances
            if (full) {
                for (int s0 = 0; s0 < n_new; s0 += G * U)
                    eval_batch<KIND, T, CPL, QB, U, true, TILED>(q, a.ds, s0, n_new, cand_id, cand_key, g, lig);
            } else {
                for (int s0 = 0; s0 < n_new; s0 += G * U)
                    eval_batch<KIND, T, CPL, QB, U, false, TILED>(q, a.ds, s0, n_new, cand_id, cand_key, g, lig);
            }
            evals += n_new;
            wave_sync();
            uint64_t ck = lane < n_new ? cand_key[lane] : JX_EMPTY_KEY;
            wave_sync();
            // ---- 6. merge into the sorted frontier
            frontier_merge<NREG>(fk, fr, count, worst, L, ck, n_new, lane);
        }
    }

    if constexpr (VIS) {
        write_visited<KIND, NREG>(a, qi, fk, count, worst, vk, reinterpret_cast<uint64_t*>(tab), hops, lane);
        if (a.stats && lane == 0) {
            unsigned long long* sp = a.stats + (size_t)(qi & 63) * 16;
            atomicAdd(&sp[0], (unsigned long long)hops);
            atomicAdd(&sp[1], (unsigned long long)evals);
        }
    } else {
        write_results<KIND, NREG>(a, qi, fk, count, lane, hops, evals);
    }
}

// MODE 1: tag table and R <= 64; 2: the same with more records in flight (see beam_search_body)
template <int KIND, int T, int CPL, int NREG, int QB, int MODE>
__global__ void __launch_bounds__(JX_BEAM_WPB * 64) __attribute__((amdgpu_waves_per_eu(MODE == 2 ? 1 : ((KIND <= K_F32 || KIND == K_F16) && NREG <= 2 && CPL <= 2) ? JX_WPE_EXACT : ((query_in_lds<KIND, CPL, QB>() && NREG <= 4) ? JX_WPE_RQ1 : 1), 8)))
beam_search_kernel(BeamArgs a) {
    beam_search_body<KIND, T, CPL, NREG, QB, JX_BEAM_WPB, false, false, MODE>(a);
}

// Ablation instances (exact distances): WPB queries per workgroup, element-strided ("tiled") loads.
template <int KIND, int T, int CPL, int NREG, int WPB, bool TILED>
__global__ void __launch_bounds__(WPB * 64) __attribute__((amdgpu_waves_per_eu((NREG <= 2 && CPL <= 2) ? JX_WPE_EXACT : 1, 8)))
beam_search_variant_kernel(BeamArgs a) {
    beam_search_body<KIND, T, CPL, NREG, 0, WPB, TILED>(a);
}

// Insertion with the expansion list as candidate set (exact distances; see BeamArgs::vis_cap).  Five wavefronts per SIMD by
// registers (six spill: 22.3 -> 23.8 ms for 200,000 x 128 uint8).  MODE 3: half as many records in flight and six, for batches
// that fill the card more than once
template <int KIND, int T, int CPL, int NREG, int MODE>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(MODE == 3 ? 6 : (MODE != 2 && CPL <= 2 ? 5 : 1), 8))) beam_search_visited_kernel(BeamArgs a) {
    beam_search_body<KIND, T, CPL, NREG, 0, 1, false, true, MODE>(a);
}

// ------------------------------------------------------------------ two expansions per round
//
// A search over a 10,000-query batch lasts about two query lifetimes, and a lifetime is a chain of dependent
// expansions: select, row, filter, gather, merge.  This variant overlaps two links of the chain without changing
// the sequence Alg. 1 prescribes.  Besides the closest unexpanded entry u1 it takes the second closest, u2, reads
// both rows, filters row(u1) and then row(u2) through the visited table (in that order: what the sequential search
// would do if u2 came next), and gathers both candidate lists in one batch.  The candidates of u1 are merged; if u2
// is still the closest unexpanded entry -- no candidate of u1 overtook or evicted it, the usual case -- its
// expansion has happened exactly as it would have, and its candidates are merged too.  Otherwise the table words
// that row(u2) changed are restored, its candidates are dropped, and the search goes on from the merged frontier.
// Frontier sequence, results and the expansion / evaluation counts are those of the one-at-a-time search; a
// dropped list costs its gather.

// rows of at most 64 entries only (the launcher checks)
template <int KIND, int T, int CPL, int NREG, int QB>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(((KIND <= K_F32 || KIND == K_F16) && NREG <= 2 && CPL <= 2) ? JX_WPE_EXACT : 1, 8)))
beam_search_pair_kernel(BeamArgs a) {
    constexpr int G = 64 / T;
    constexpr int U0 = (8 / CPL) > 0 ? (8 / CPL) : 1;
    constexpr int U = U0 < (64 / G) ? U0 : (64 / G);
    constexpr int FCAP = mirror_entries<NREG>();
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = lane_id();
    const int g = lane / T, lig = lane % T;
    const int64_t qi = blockIdx.x;
    if (qi >= a.nq) return;

    const int H = a.hash_slots;
    const int tag_bits = a.tag_bits;
    const uint32_t id_mask = tag_bits ? ((1u << (tag_bits + 30 - __builtin_clz((uint32_t)H))) - 1u) : 0u;
    uint64_t* fr = reinterpret_cast<uint64_t*>(smem);
    uint64_t* cand_key = fr + FCAP;                                     // [128]
    uint32_t* cand_id = reinterpret_cast<uint32_t*>(cand_key + 128);    // [128]
    uint32_t* tab = cand_id + 128;

    for (int i = lane; i < (tag_bits ? H / 2 : H); i += 64) tab[i] = JX_NONE_ID;
    for (int i = lane; i < FCAP; i += 64) fr[i] = JX_EMPTY_KEY;

    QueryRegs<KIND, CPL, QB> q;
    load_query<KIND, T, CPL, QB>(q, a.ds, qi + (qi >= a.q_skip ? 1 : 0), lig);

    uint64_t fk[NREG];
#pragma unroll
    for (int r = 0; r < NREG; r++) fk[r] = JX_EMPTY_KEY;
    int count = 0;
    uint64_t worst = JX_EMPTY_KEY;  // see frontier_merge
    const int L = a.L;
    const bool full = a.ds.nch == T * CPL;
    uint32_t hops = 0, evals = 0;

    if (lane == 0) {
        cand_id[0] = a.entry;
        if (tag_bits) {
            const uint32_t h = (a.entry * 0x9E3779B1u) & id_mask;
            tab[h >> tag_bits] = 0xFFFF0000u | (h & ((1u << tag_bits) - 1u));
        } else {
            tab[__umulhi(a.entry * 0x9E3779B1u, (uint32_t)H)] = a.entry;
        }
    }
    wave_sync();
    eval_batch<KIND, T, CPL, QB, 1>(q, a.ds, 0, 1, cand_id, cand_key, g, lig);
    wave_sync();
    if (lane == 0) {
        fk[0] = cand_key[0];
        fr[0] = cand_key[0];
    }
    wave_sync();
    count = 1;
    evals = 1;

    // visited filter: true if v has not been seen; installs it; slot / old word returned for a possible restore
    auto filter = [&](const uint32_t v, uint32_t& slot, uint32_t& old) -> bool {
        bool is_new = false;
        slot = 0;
        old = 0;
        if (v != JX_NONE_ID) {
            if (tag_bits) {
                const uint32_t h = (v * 0x9E3779B1u) & id_mask;
                const uint32_t tag = h & ((1u << tag_bits) - 1u);
                slot = h >> tag_bits;
                old = tab[slot];
                is_new = (old & 0xFFFFu) != tag && (old >> 16) != tag;
                if (is_new) tab[slot] = (old << 16) | tag;
            } else {
                slot = __umulhi(v * 0x9E3779B1u, (uint32_t)H);
                old = tab[slot];
                is_new = old != v;
                if (is_new) tab[slot] = v;
            }
        }
        return is_new;
    };

    for (;;) {
        // ---- the two closest unexpanded entries
        uint64_t um[NREG];
#pragma unroll
        for (int r = 0; r < NREG; r++) um[r] = ballot((fk[r] & 1ull) == 0ull);
        int r1 = -1, l1 = 0;
#pragma unroll
        for (int r = 0; r < NREG; r++)
            if (r1 < 0 && um[r] != 0ull) {
                r1 = r;
                l1 = __builtin_ctzll(um[r]);
                um[r] &= um[r] - 1ull;
            }
        if (r1 < 0) break;
        int r2 = -1, l2 = 0;
#pragma unroll
        for (int r = 0; r < NREG; r++)
            if (r2 < 0 && um[r] != 0ull) {
                r2 = r;
                l2 = __builtin_ctzll(um[r]);
            }
        uint32_t u1 = 0;
        uint64_t key2 = JX_EMPTY_KEY;
#pragma unroll
        for (int r = 0; r < NREG; r++) {
            if (r == r1) {
                u1 = readlane32((uint32_t)fk[r], l1) >> 1;
                if (lane == l1) fk[r] |= 1ull;
            }
            if (r == r2) key2 = readlane64(fk[r], l2);
        }
        const bool have2 = r2 >= 0;
        // ---- both rows, both filters (row 1 first), one gather
        uint32_t v1 = JX_NONE_ID, v2 = JX_NONE_ID;
        if (lane < a.R) v1 = a.adj[(size_t)u1 * (size_t)a.R + lane];
        if (have2 && lane < a.R) v2 = a.adj[(size_t)key_id(key2) * (size_t)a.R + lane];
        uint32_t slot1, old1, slot2, old2;
        const bool new1 = filter(v1, slot1, old1);
        const uint64_t nm1 = ballot(new1);
        const bool new2 = filter(v2, slot2, old2);
        const uint64_t nm2 = ballot(new2);
        const int n1 = __builtin_popcountll(nm1), n2 = __builtin_popcountll(nm2);
        uint64_t ck1 = JX_EMPTY_KEY, ck2 = JX_EMPTY_KEY;
        if (n1 + n2 > 0) {
            if (new1) cand_id[prefix_count(nm1)] = v1;
            if (new2) cand_id[n1 + prefix_count(nm2)] = v2;
            wave_sync();
            const int ntot = n1 + n2;
            if (full) {
                for (int s0 = 0; s0 < ntot; s0 += G * U)
                    eval_batch<KIND, T, CPL, QB, U, true>(q, a.ds, s0, ntot, cand_id, cand_key, g, lig);
            } else {
                for (int s0 = 0; s0 < ntot; s0 += G * U)
                    eval_batch<KIND, T, CPL, QB, U, false>(q, a.ds, s0, ntot, cand_id, cand_key, g, lig);
            }
            wave_sync();
            if (lane < n1) ck1 = cand_key[lane];
            if (lane < n2) ck2 = cand_key[n1 + lane];
            wave_sync();
        }
        // ---- expansion of u1
        hops++;
        evals += n1;
        if (n1 > 0) frontier_merge<NREG>(fk, fr, count, worst, L, ck1, n1, lane);
        if (!have2) continue;
        // ---- is u2 what comes next?
        int rn = -1, ln = 0;
#pragma unroll
        for (int r = 0; r < NREG; r++) {
            const uint64_t m = ballot((fk[r] & 1ull) == 0ull);
            if (rn < 0 && m != 0ull) {
                rn = r;
                ln = __builtin_ctzll(m);
            }
        }
        bool ok = false;
#pragma unroll
        for (int r = 0; r < NREG; r++) {
            if (r == rn) {
                ok = readlane64(fk[r], ln) == key2;
                if (ok && lane == ln) fk[r] |= 1ull;
            }
        }
        if (ok) {
            hops++;
            evals += n2;
            if (n2 > 0) frontier_merge<NREG>(fk, fr, count, worst, L, ck2, n2, lane);
        } else {
            if (new2) tab[slot2] = old2;  // as if row(u2) had never been looked at
            wave_sync();
        }
    }

    write_results<KIND, NREG>(a, qi, fk, count, lane, hops, evals);
}

}  // namespace jx
