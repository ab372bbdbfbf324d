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

namespace vitcop {

constexpr int SEL_THREADS = 1024;

constexpr int SEL_DIGIT = 10, SEL_LIST = 64;

struct SelectShared {
    alignas(16) unsigned hist[1 << SEL_DIGIT];       // (read and cleared 16 bytes at a time)
    unsigned list[SEL_LIST];
    unsigned low[SEL_THREADS / 64], high[SEL_THREADS / 64];
    unsigned wave_tot[SEL_THREADS / 64];
    unsigned n_list, prefix, kk, count;
};

// keys: n entries in LDS.  Writes out[r] = base + i for the r-th survivor in
// index order.  Must be called by all SEL_THREADS threads of the workgroup.
//
// The workgroup is alone on its CU and every step is a latency between two barriers, so there are few of them: digits of
// ten bits, the first right below the bits that all keys share (scores of one sample share their exponent: the
// high digits would say nothing and all threads would count in the same bins), and as soon as at most 64 keys share the
// prefix of the one looked for, one wavefront compares them directly.  One digit and the comparison, i.e. six
// barriers, are the rule (four digits of eight bits took fourteen: 4 samples of 2880 norms 9.1 -> 7.7 us a launch, one
// of 6272 in four partial sums 15.0 -> 12.0).
__device__ inline void block_select_emit(const unsigned* keys, int n, int keep, int32_t* out,
                                         int base, SelectShared& sh) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    unsigned theta = 0, need = 0;            // keys below theta survive, and the first `need` of those equal to it
    if (keep > 0) {
        unsigned lo = ~0u, hi = 0u;
        for (int i = tid; i < n; i += SEL_THREADS) {
            lo = min(lo, keys[i]);
            hi = max(hi, keys[i]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo = min(lo, __shfl_xor(lo, o, 64));
            hi = max(hi, __shfl_xor(hi, o, 64));
        }
        if (lane == 0) {
            sh.low[wv] = lo;
            sh.high[wv] = hi;
        }
        for (int i = tid; i < 1 << SEL_DIGIT; i += SEL_THREADS) sh.hist[i] = 0;
        if (tid == 0) sh.n_list = 0;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < SEL_THREADS / 64; ++w) {
            lo = min(lo, sh.low[w]);
            hi = max(hi, sh.high[w]);
        }
        // the keys that share `prefix` above their low `bits` bits hold the one of rank kk among them
        int bits = lo == hi ? 0 : 32 - __builtin_clz(lo ^ hi);
        unsigned prefix = (unsigned)((uint64_t)lo >> bits << bits), kk = (unsigned)keep;
        for (;;) {
            if (bits == 0) {                                     // they are all equal
                theta = prefix;
                need = kk;
                break;
            }
            const int width = min(bits, SEL_DIGIT), shift = bits - width;
            const uint64_t above = (uint64_t)prefix >> bits;
            for (int i0 = 0; i0 < n; i0 += SEL_THREADS) {        // uniform trip count: ballots below
                const int i = i0 + tid;
                const unsigned k = i < n ? keys[i] : 0u;
                const bool live = i < n && (uint64_t)k >> bits == above;
                const unsigned dgt = (k >> shift) & ((1u << width) - 1u);
                // the lanes that agree with the first live lane are counted with one atomic, the others add individually
                const unsigned long long live_mask = __builtin_amdgcn_ballot_w64(live);
                if (live_mask != 0) {
                    const int leader = __builtin_ctzll(live_mask);
                    const unsigned d0 = __builtin_amdgcn_readlane(dgt, leader);
                    const unsigned long long same = __builtin_amdgcn_ballot_w64(live && dgt == d0);
                    if (lane == leader) atomicAdd(&sh.hist[d0], (unsigned)__builtin_popcountll(same));
                    else if (live && dgt != d0) atomicAdd(&sh.hist[dgt], 1u);
                }
            }
            __syncthreads();
            if (tid < 64) {                                      // 16 bins a lane; cleared for a next digit
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
                unsigned incl = s;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const unsigned t = __shfl_up(incl, o, 64);
                    if (tid >= o) incl += t;
                }
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
                    sh.prefix = prefix | (16u * tid + digit) << shift;
                    sh.kk = kk - below;
                    sh.count = at;
                }
            }
            __syncthreads();
            prefix = sh.prefix;
            kk = sh.kk;
            bits = shift;
            const unsigned count = sh.count;
            if (count == kk) {                                   // all that share the prefix survive
                theta = prefix | (unsigned)(((uint64_t)1 << bits) - 1);
                need = (unsigned)n;
                break;
            }
            if (count <= SEL_LIST) {
                for (int i = tid; i < n; i += SEL_THREADS) {
                    const unsigned k = keys[i];
                    if ((uint64_t)k >> bits == (uint64_t)prefix >> bits) sh.list[atomicAdd(&sh.n_list, 1u)] = k;
                }
                __syncthreads();
                if (tid < 64) {
                    const unsigned key = tid < (int)count ? sh.list[tid] : ~0u;
                    unsigned less = 0, equal = 0;
                    for (unsigned j = 0; j < count; ++j) {
                        const unsigned other = __builtin_amdgcn_readlane(key, j);
                        less += other < key;
                        equal += other == key;
                    }
                    if (tid < (int)count && kk > less && kk <= less + equal) {      // (equal keys agree)
                        sh.prefix = key;
                        sh.kk = kk - less;
                    }
                }
                __syncthreads();
                theta = sh.prefix;
                need = sh.kk;
                break;
            }
        }
    }

    const int ipt = (n + SEL_THREADS - 1) / SEL_THREADS;
    const int lo = min(n, tid * ipt), hi = min(n, lo + ipt);
    unsigned less = 0, eq = 0;
    for (int i = lo; i < hi; ++i) {
        unsigned k = keys[i];
        less += k < theta;
        eq += k == theta;
    }
    // exclusive scan of (less, eq) packed in 16+16 bits (n <= 16384)
    unsigned packed = less | (eq << 16), incl = packed;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        unsigned t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) sh.wave_tot[wv] = incl;
    __syncthreads();
    unsigned woff = 0;
    for (int w = 0; w < wv; ++w) woff += sh.wave_tot[w];
    unsigned excl = incl - packed + woff;
    unsigned lb = excl & 0xFFFFu, eb = excl >> 16;
    for (int i = lo; i < hi; ++i) {
        unsigned k = keys[i];
        if (k < theta) {
            out[lb + min(eb, need)] = base + i;
            ++lb;
        } else if (k == theta) {
            if (eb < need) out[lb + eb] = base + i;
            ++eb;
        }
    }
}

}  // namespace vitcop
