// Workgroup-wide exact top-k by radix selection, with the lower index winning
// ties and the survivors emitted in ascending index order (Alg. 1 of the paper
// names only TopK; the tie rule and the order are this library's contract).
//
// Keys are 32-bit unsigned with "smaller key = better".  A non-negative float
// orders like its bit pattern, so "k smallest norms" uses the bits as they are
// and "k largest scores" uses their complement.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_utils.h"

namespace vitcop {

constexpr int SEL_THREADS = 1024, SEL_WAVES = SEL_THREADS / 64;
constexpr int SEL_DIGIT = 10, SEL_LIST = 64;
constexpr int SEL_MAX_CHUNKS = 16;                   // keys per thread: at most 16384 keys

struct SelectShared {
    alignas(16) unsigned hist[1 << SEL_DIGIT];       // (read and cleared 16 bytes at a time)
    alignas(16) unsigned count_of[SEL_MAX_CHUNKS * SEL_WAVES];       // survivors of a wavefront's 64 keys, by chunk
    alignas(8) uint2 list[SEL_LIST];                 // key, index
    alignas(16) unsigned low[SEL_WAVES];
    alignas(16) unsigned high[SEL_WAVES];
    unsigned n_list, digit, kk, count;
};

// keys: n entries in LDS, entry i written by thread i % SEL_THREADS (so nothing waits for them here).  Writes
// out[r] = base + i for the r-th survivor in index order.  Must be called by all SEL_THREADS threads of the workgroup.
//
// The workgroup is alone on its CU and every step is a latency between two barriers, so there are few of them.  The keys
// are counted in 512 to 1024 bins of equal width between the smallest and the largest, a power of two wide; the bin that
// holds the one looked for is counted again the same way until at most 64 keys are in question, and those rank themselves
// against each other.  One count and the ranking, five barriers, are the rule: the bins follow the keys' range wherever
// it lies (a digit of ten bits below the bits that all keys share, used before, wasted most of its bins where the range
// crosses a power of two, and took a second pass).  Scans run in vector registers, positions come from ballots, a thread
// keeps its keys in registers.  Launches on log-normal norms, us, before and now: 576 in one part 8.1, 4.5; in 32 parts
// 6.8, 5.5; four samples of 2880 in 32 parts 12.5, 9.6; 6272 in four parts 13.0, 9.0; 16384 27.8, 18.5; the filter's
// finalize, 576 patches x 16 heads, 7.0, 5.7.
//
// C: keys a thread holds in registers, at least ceil(n / SEL_THREADS).
template <int C>
__device__ __forceinline__ void block_select_held(const unsigned* keys, int n, int keep, int32_t* out, int base,
                                                  SelectShared& sh) {
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    unsigned key[C];
    bool valid[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int i = c * SEL_THREADS + tid;
        valid[c] = i < n;
        key[c] = valid[c] ? keys[i] : 0u;
    }
    // keys below theta survive, and the first `need` of those equal to it; of the listed ones those whose bit is set
    unsigned theta = 0, need = 0, listed = 0;
    if (keep > 0) {
        auto least = [](unsigned a, unsigned b) { return min(a, b); };
        auto most = [](unsigned a, unsigned b) { return max(a, b); };
        unsigned lo = ~0u, hi = 0u;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            lo = valid[c] ? min(lo, key[c]) : lo;
            hi = max(hi, key[c]);                                // (past the end: 0)
        }
        lo = wave_reduce(lo, ~0u, least);
        hi = wave_reduce(hi, 0u, most);
        if (lane == 0) {
            sh.low[wv] = lo;
            sh.high[wv] = hi;
        }
        static_assert(1 << SEL_DIGIT == SEL_THREADS, "a bin a thread");
        sh.hist[tid] = 0;
        if (tid == 0) sh.n_list = 0;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < SEL_WAVES; w += 4) {
            const uint4 a = *reinterpret_cast<const uint4*>(sh.low + w), b = *reinterpret_cast<const uint4*>(sh.high + w);
            lo = min(min(lo, min(a.x, a.y)), min(a.z, a.w));
            hi = max(max(hi, max(b.x, b.y)), max(b.z, b.w));
        }
        // the keys of [first, first + range] hold the one of rank kk (from 1) among them
        unsigned first = lo, range = hi - lo, kk = (unsigned)keep;
        for (;;) {
            if (range == 0) {                                    // they are all equal
                theta = first;
                need = kk;
                break;
            }
            const int shift = max(0, 32 - __builtin_clz(range) - SEL_DIGIT);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const unsigned off = key[c] - first, bin = off >> shift;
                const bool live = valid[c] && off <= range;
                // the lanes that agree with the first live lane are counted with one atomic, the others add individually
                const unsigned long long live_mask = __builtin_amdgcn_ballot_w64(live);
                if (live_mask != 0) {
                    const int leader = __builtin_ctzll(live_mask);
                    const unsigned b0 = __builtin_amdgcn_readlane(bin, leader);
                    const unsigned long long same = __builtin_amdgcn_ballot_w64(live && bin == b0);
                    const bool alone = bin != b0;
                    if (live && (alone || lane == leader))
                        atomicAdd(&sh.hist[bin], alone ? 1u : (unsigned)__builtin_popcountll(same));
                }
            }
            __syncthreads();
            if (tid < 64) {                                      // 16 bins a lane; cleared for a next count
                uint4* bins = reinterpret_cast<uint4*>(sh.hist) + 4 * tid;
                unsigned c[16], s = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint4 v = bins[q];
                    c[4 * q] = v.x; c[4 * q + 1] = v.y; c[4 * q + 2] = v.z; c[4 * q + 3] = v.w;
                    bins[q] = make_uint4(0, 0, 0, 0);
                }
#pragma unroll
                for (int q = 0; q < 16; ++q) s += c[q];
                const unsigned incl = wave_scan(s, 0u, [](unsigned a, unsigned b) { return a + b; });
                if (kk > incl - s && kk <= incl) {
                    unsigned below = incl - s, at = 0, digit = 0;
                    bool found = false;
#pragma unroll
                    for (int q = 0; q < 16; ++q) {
                        if (!found && kk <= below + c[q]) {
                            found = true;
                            digit = q;
                            at = c[q];
                        }
                        if (!found) below += c[q];
                    }
                    sh.digit = 16u * tid + digit;
                    sh.kk = kk - below;
                    sh.count = at;
                }
            }
            __syncthreads();
            const unsigned skipped = sh.digit << shift, count = sh.count;
            first += skipped;
            range = min(range - skipped, (1u << shift) - 1u);
            kk = sh.kk;
            if (count == kk) {                                   // all of the bin survive
                theta = first + range;
                need = (unsigned)n;
                break;
            }
            if (count <= SEL_LIST) {
                unsigned mine = 0;                               // my keys of the bin, a bit each
#pragma unroll
                for (int c = 0; c < C; ++c)
                    if (valid[c] && key[c] - first <= range) {
                        sh.list[atomicAdd(&sh.n_list, 1u)] = make_uint2(key[c], (unsigned)(c * SEL_THREADS + tid));
                        mine |= 1u << c;
                    }
                __syncthreads();
                while (mine != 0) {
                    const int c = __builtin_ctz(mine);
                    mine &= mine - 1;
                    const unsigned i = (unsigned)(c * SEL_THREADS + tid), k = keys[i];
                    unsigned rank = 0;
                    for (unsigned j = 0; j < count; ++j) {
                        const uint2 o = sh.list[j];
                        rank += o.x < k || (o.x == k && o.y < i);
                    }
                    if (rank < kk) listed |= 1u << c;
                }
                theta = first;
                break;
            }
        }
    }

    // positions: a wavefront's survivors of every chunk are counted, then added up over the chunks and wavefronts before
    unsigned sure = 0, equal = 0;                                // a bit for each of my keys
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const bool s = valid[c] && (key[c] < theta || (listed >> c & 1u)), e = valid[c] && key[c] == theta && need != 0;
        sure |= (unsigned)s << c;
        equal |= (unsigned)e << c;
        const unsigned both = (unsigned)__builtin_popcountll(__builtin_amdgcn_ballot_w64(s)) |
                              (unsigned)__builtin_popcountll(__builtin_amdgcn_ballot_w64(e)) << 16;      // (n <= 16384)
        if (lane == 0) sh.count_of[c * SEL_WAVES + wv] = both;
    }
    __syncthreads();
    static_assert(SEL_MAX_CHUNKS * SEL_WAVES == 256 && SEL_WAVES == 16, "four counts a lane");
    uint4 cnt = make_uint4(0, 0, 0, 0);
    if (4 * lane < C * SEL_WAVES) cnt = reinterpret_cast<const uint4*>(sh.count_of)[lane];
    const unsigned four = cnt.x + cnt.y + cnt.z + cnt.w;
    unsigned before = wave_scan(four, 0u, [](unsigned a, unsigned b) { return a + b; }) - four;
    if ((wv & 3) > 0) before += cnt.x;
    if ((wv & 3) > 1) before += cnt.y;
    if ((wv & 3) > 2) before += cnt.z;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const unsigned at = __builtin_amdgcn_readlane(before, 4 * c + (wv >> 2));
        const bool s = sure >> c & 1u, e = equal >> c & 1u;
        const unsigned long long ms = __builtin_amdgcn_ballot_w64(s), me = __builtin_amdgcn_ballot_w64(e);
        auto ahead = [](unsigned long long m) {                  // set bits of the lanes before this one
            return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
        };
        const unsigned lb = (at & 0xFFFFu) + ahead(ms), eb = (at >> 16) + ahead(me);
        if (s || (e && eb < need)) out[lb + min(eb, need)] = base + c * SEL_THREADS + tid;
    }
}
__device__ __forceinline__ void block_select_emit(const unsigned* keys, int n, int keep, int32_t* out, int base,
                                                  SelectShared& sh) {
    if (n <= SEL_THREADS) block_select_held<1>(keys, n, keep, out, base, sh);
    else if (n <= 3 * SEL_THREADS) block_select_held<3>(keys, n, keep, out, base, sh);
    else if (n <= 8 * SEL_THREADS) block_select_held<8>(keys, n, keep, out, base, sh);
    else block_select_held<SEL_MAX_CHUNKS>(keys, n, keep, out, base, sh);
}

}  // namespace vitcop
