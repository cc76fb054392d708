// k-SAT kernels for gfx950.
//
// Work decomposition.  One workgroup owns one group of 4 replicas for the
// whole launch.  Their spins live in LDS as a byte per variable (bit j =
// replica j of the group), next to the complement table, so "literal is
// true" is a single byte load whatever the literal's sign:
//   lds[v]       = x_v        (positive literal of v)
//   lds[N + v]   = NOT x_v    (negative literal of v)
//   lds[2N]      = 0          (absent literal: never true)
//   lds[2N + 1]  = all ones   (padding slot: clause counts as satisfied)
// The energy change of flipping x_i (section "Nonequilibrium inhomogeneous
// sampling over subgraphs" uses single-variable Metropolis moves; CNF energy
// as in subsection "4-SAT Problems Near Computational Phase Transitions") is
//   dE = sum over clauses a of i with every other literal false of
//        (+1 if i's literal in a is currently true, -1 otherwise),
// computed for the 4 replicas at once: the OR of the other literals' bytes
// is a 4-bit "satisfied by others" mask, spread into four byte lanes of a
// 32-bit accumulator (SIMD within a register).
// A wave handles up to 64 variables of one colour class;
// classes are conflict-free, so all lanes update concurrently and the result
// equals the sequential colour-major order.  The instance (per-variable
// clause records) streams from L2/MALL, shared by every workgroup.
#include <climits>
#include <cstdlib>
#include <type_traits>

#include "nmc_internal.h"
#include "nmc_philox.h"

namespace nmc {

namespace {

__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_xor(v, off, 64);
    return v;
}

// Sum over each group of 2^lg lanes (lg wave-uniform, at most 6), returned to
// every lane of the group: swaps within quads, the mirrors within half-rows
// and rows (register moves, no LDS crossbar), then shuffles across rows.
// Sums mod 2^32, so the order does not matter.
__device__ __forceinline__ uint32_t lane_group_sum(uint32_t x, int lg) {
    if (lg >= 1)
        x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    if (lg >= 2)
        x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    if (lg >= 3)
        x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, false);  // row_half_mirror
    if (lg >= 4)
        x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, false);  // row_mirror
    if (lg >= 5)
        x += (uint32_t)__shfl_xor((int)x, 16, 64);
    if (lg >= 6)
        x += (uint32_t)__shfl_xor((int)x, 32, 64);
    return x;
}

__device__ __forceinline__ uint32_t spread4(uint32_t f) {
    // bit j of f (j < 4) -> bit 8j; no carries for f < 16
    return (f * 0x00204081u) & 0x01010101u;
}

// Compiler-only barrier: memory operations are not moved across it, so
// prefetch loads stay where they are issued and their waits stay at first use.
__device__ __forceinline__ void issue_fence() { __asm__ volatile("" ::: "memory"); }

typedef __attribute__((address_space(3))) const uint8_t lds_cu8;
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef int i32x4 __attribute__((ext_vector_type(4)));

// Byte at LDS address a.  The sweep kernel declares no static LDS, so its
// dynamic LDS block starts at address 0 and spin-table offsets are addresses.
__device__ __forceinline__ uint32_t lds_load_u8(uint32_t a) { return *(lds_cu8 *)(uintptr_t)a; }
__device__ __forceinline__ void lds_store_u8(uint32_t a, uint32_t v) { *(lds_u8 *)(uintptr_t)a = (uint8_t)v; }

// The three gathered bytes and the sign mask of one clause slot (below).
__device__ __forceinline__ void slot_gather(uint2 r, uint32_t (&x)[3], uint32_t &sm) {
    x[0] = lds_load_u8(r.x & kAddrMask);
    x[1] = lds_load_u8(__builtin_amdgcn_alignbit(r.y, r.x, kAddrBits) & kAddrMask);
    x[2] = lds_load_u8(__builtin_amdgcn_ubfe(r.y, 2 * kAddrBits - 32, kAddrBits));
    sm = (uint32_t)__builtin_amdgcn_sbfe(r.y, 3 * kAddrBits - 32, 1);
}

// One clause slot: r.x bits 0..16 and r.y bits 0..1 / 2..18 hold the spin-table
// addresses of the clause's three other literals, r.y bit 19 whether the
// lane's own literal in the clause is negated.  Adds spread(sat) xor sign.
__device__ __forceinline__ uint32_t slot_step(uint32_t acc, uint2 r) {
    const uint32_t a0 = r.x & kAddrMask;
    const uint32_t a1 = __builtin_amdgcn_alignbit(r.y, r.x, kAddrBits) & kAddrMask;
    const uint32_t a2 = __builtin_amdgcn_ubfe(r.y, 2 * kAddrBits - 32, kAddrBits);
    const uint32_t sm = (uint32_t)__builtin_amdgcn_sbfe(r.y, 3 * kAddrBits - 32, 1);
    const uint32_t sat = lds_load_u8(a0) | lds_load_u8(a1) | lds_load_u8(a2);
    return (spread4(sat) ^ sm) + acc;
}

__global__ void ksat_init_kernel(KsatDev I, KsatRepDev R, uint32_t key0, uint32_t key1) {
    const size_t total = (size_t)R.n_groups * I.n;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (size_t)gridDim.x * blockDim.x) {
        const int g = (int)(idx / I.n);
        const int v = (int)(idx % I.n);
        const int nact = min(kGroup, R.n_rep - g * kGroup);
        const uint4 u = philox4x32_10((uint32_t)v, 0u, (uint32_t)g, kStreamKsatInit, key0, key1);
        uint32_t b = (u.x >> 31) | ((u.y >> 31) << 1) | ((u.z >> 31) << 2) | ((u.w >> 31) << 3);
        b &= (1u << nact) - 1u;
        R.xs[idx] = (uint8_t)b;
        R.best_xs[idx] = (uint8_t)b;
    }
}

// Full energy count of every replica of one group (one workgroup per group).
__global__ void ksat_recount_kernel(KsatDev I, const uint8_t *xs, int n_rep, int32_t *energy_out) {
    extern __shared__ __align__(16) uint8_t smem[];
    const int n = I.n, g = blockIdx.x, tid = threadIdx.x;
    const int nact = min(kGroup, n_rep - g * kGroup);
    const uint32_t amask = (1u << nact) - 1u;
    uint8_t *xt = smem;
    int *red = (int *)(smem + align_up(2 * n + 2, 16));
    for (int v = tid; v < n; v += blockDim.x) {
        const uint32_t b = xs[(size_t)g * n + v] & amask;
        xt[v] = (uint8_t)b;
        xt[n + v] = (uint8_t)(~b & amask);
    }
    if (tid == 0) {
        xt[2 * n] = 0;
        xt[2 * n + 1] = (uint8_t)amask;
    }
    if (tid < kGroup)
        red[tid] = 0;
    __syncthreads();
    int c0 = 0, c1 = 0, c2 = 0, c3 = 0;
    for (int a = tid; a < I.m; a += blockDim.x) {
        const uint4 ad = reinterpret_cast<const uint4 *>(I.clause_addr)[a];
        const uint32_t sat = xt[ad.x] | xt[ad.y] | xt[ad.z] | xt[ad.w];
        const uint32_t f = ~sat & amask;
        c0 += f & 1;
        c1 += (f >> 1) & 1;
        c2 += (f >> 2) & 1;
        c3 += (f >> 3) & 1;
    }
    c0 = wave_sum(c0);
    c1 = wave_sum(c1);
    c2 = wave_sum(c2);
    c3 = wave_sum(c3);
    if ((tid & 63) == 0) {
        atomicAdd(&red[0], c0);
        atomicAdd(&red[1], c1);
        atomicAdd(&red[2], c2);
        atomicAdd(&red[3], c3);
    }
    __syncthreads();
    if (tid < nact)
        energy_out[g * kGroup + tid] = red[tid];
}

__global__ void ksat_reset_tallies_kernel(KsatRepDev R) {
    const int total = R.n_groups * kGroup;
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < total; r += gridDim.x * blockDim.x) {
        R.best[r] = R.energy[r];
        R.first_hit[r] = -1;
    }
}

// Arrays that no kernel writes, read at wave-uniform indexes into scalar
// registers.
template <class T>
__device__ __forceinline__ T scalar_read(const T *p, int i) {
    typedef const T __attribute__((address_space(4))) *cp;
    return ((cp)(uintptr_t)p)[i];
}

// The three gathered bytes of a sweep-layout record, and their union (as 32-bit
// words: the compiler is kept from forming it in 16 bits and extending it).
struct SlotBytes {
    uint32_t x[3];
};
struct SlotPair {
    SlotBytes a, b;
};
__device__ __forceinline__ SlotBytes slot_bytes(uint32_t lo, uint32_t hi) {
    // the third address: the words' high bytes, and bit 16 (byte 2) of the first
    return {{lds_load_u8(lo & kAddrMask), lds_load_u8(hi & kAddrMask),
             lds_load_u8(__builtin_amdgcn_perm(hi, lo, 0x0C020703u))}};
}
__device__ __forceinline__ uint32_t slot_sat(SlotBytes b) {
    __asm__("" : "+v"(b.x[0]), "+v"(b.x[1]), "+v"(b.x[2]));
    return b.x[0] | b.x[1] | b.x[2];
}

// cnt[j] += set bits of the nibbles of w at replica j.
__device__ __forceinline__ void count_nibbles(uint32_t (&cnt)[4], uint32_t w) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
        cnt[j] += (uint32_t)__builtin_popcount(w & (0x11111111u << j));
}

__device__ __forceinline__ uint32_t pack_counts(const uint32_t (&c)[4]) {
    return c[0] + (c[1] << 8) + (c[2] << 16) + (c[3] << 24);
}

// n_sweeps full sweeps of every colour class for the replicas of item g, by
// the whole workgroup, with smem = the workgroup's dynamic LDS block.
// GPW = 1: the 4 replicas of group g.  GPW = 2: the 8 replicas of groups 2g
// and 2g + 1, held in one spin byte per variable (first group in bits 0..3),
// so every clause record, address decode and LDS gather serves 8 replicas;
// the random words and every result are those of the groups run one by one.
//
// Bound: a class step (one chunk per wave, then a barrier) takes the LDS
// gathers of all waves (3.8 cycles each, two thirds of the time) and one
// decision.  The sweep layout serves both: chunks of a class have one length (a
// heavy variable's last clauses are walked by its light neighbour's lane;
// lengths of 28 to 60 slots at degree 40 left early waves waiting), a slot takes
// 6 vector instructions instead of 9 (signs are words of their own, satisfied
// slots are collected as nibbles and counted 8 at a time, an address takes one
// instruction), chunk descriptors are read as scalars one chunk ahead and the
// first records before the class barrier.  N = 50,000, 1024 replicas: 285 -> 257
// us per sweep; 4096 replicas of N = 20,000: 577 -> 490; 3-SAT N = 30,000, 512
// replicas: 86 -> 71.  Tried: the generator's rounds spread over the slot loop
// (263, small instances slower), one loop for whole and short blocks (copies of
// the records in flight: 255 where this loop took 240), rows past a short block
// left out (263).
template <int GPW>
__device__ __forceinline__ void sweep_group(const KsatDev &I, const KsatRepDev &R, const SweepCall &C, const int g,
                                            uint8_t *smem) {
    constexpr int NR = kGroup * GPW;  // replicas of the item
    const int n = I.n;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & 63, nwaves = nthr >> 6;
    const int wave_u = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tab_words = C.n_classes * C.stride;

    uint8_t *xt = smem;
    uint32_t *tl = (uint32_t *)(smem + align_up(2 * n + 2, 16));
    int *red = (int *)(tl + align_up(tab_words, 4));  // [0..NR) dE sums, [NR] improved mask

    const int g0 = g * GPW;  // first group of the item
    const int r0 = g0 * kGroup;
    const int nact = min(NR, R.n_rep - r0);
    const uint32_t amask = (1u << nact) - 1u;
    const bool second = GPW == 2 && g0 + 1 < R.n_groups;  // the item's second group exists
    // per-temperature tables (tempering): the item's replicas share one row
    const uint32_t *tab = C.tab + (C.reps_per_row > 0 ? (size_t)(r0 / C.reps_per_row) * tab_words : 0);

    // spin tables x and not-x from the group rows; rows and tables are
    // 16-byte aligned when N is a multiple of 16, then moved 16 bytes a lane
    uint8_t *xg = R.xs + (size_t)g0 * n;
    const bool wide = (n & 15) == 0;
    if (wide) {
        const uint32_t m4 = amask * 0x01010101u;
        for (int w = tid; w < n / 16; w += nthr) {
            uint4 b = reinterpret_cast<const uint4 *>(xg)[w];
            if (GPW == 2 && second) {
                // the second group's nibbles (values below 16) move to bits 4..7 of each byte
                const uint4 h = reinterpret_cast<const uint4 *>(xg + n)[w];
                b.x |= h.x << 4;
                b.y |= h.y << 4;
                b.z |= h.z << 4;
                b.w |= h.w << 4;
            }
            b.x &= m4;
            b.y &= m4;
            b.z &= m4;
            b.w &= m4;
            reinterpret_cast<uint4 *>(xt)[w] = b;
            reinterpret_cast<uint4 *>(xt + n)[w] = make_uint4(~b.x & m4, ~b.y & m4, ~b.z & m4, ~b.w & m4);
        }
    } else {
        for (int v = tid; v < n; v += nthr) {
            uint32_t b = xg[v];
            if (GPW == 2 && second)
                b |= (uint32_t)xg[n + v] << 4;
            b &= amask;
            xt[v] = (uint8_t)b;
            xt[n + v] = (uint8_t)(~b & amask);
        }
    }
    if (tid == 0) {
        xt[2 * n] = 0;
        xt[2 * n + 1] = (uint8_t)amask;
    }
    if (tid < 16)
        red[tid] = 0;
    int E = 0, best = 0, fh = -1;
    if (tid < nact) {
        E = R.energy[r0 + tid];
        best = R.best[r0 + tid];
        fh = R.first_hit[r0 + tid];
        if (C.check_start && fh < 0 && E <= C.target)
            fh = (int)C.t0;
    }
    __syncthreads();

    uint32_t n_acc = 0;  // flips this lane accepted in this call
    // the instance's records, with room for the reads ahead of the last chunk
    const __amdgpu_buffer_rsrc_t recs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(I.bl_rec), 0, (int)I.bl_rec_bytes, kBufferWord3);
    auto sign_at = [&](uint32_t at) { return __builtin_amdgcn_raw_buffer_load_b32(recs, lane * 4, (int)at, 0); };
    auto row_at = [&](uint32_t at, int row) -> uint4 {
        const uint32_t to = at + (uint32_t)(kBlockSign + row * kBlockRow);
        return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(recs, lane * 16, (int)to, 0));
    };
    // the four waves of a SIMD at four priorities: chunks of one length would
    // otherwise all gather, then all decide (264 -> 257 us per sweep)
    switch (wave_u >> 2 & 3) {
    case 0: __builtin_amdgcn_s_setprio(3); break;
    case 1: __builtin_amdgcn_s_setprio(2); break;
    case 2: __builtin_amdgcn_s_setprio(1); break;
    default: __builtin_amdgcn_s_setprio(0);
    }
    // A wave takes every nwaves-th chunk of a class.  While it works on one, the
    // next one's descriptor is known (class next_c, chunk next_h), so that its
    // first block can be read in time; after a sweep's last chunk (next_c =
    // n_colors) that is the first one again.
    int next_c = 0, next_h = wave_u, end_h = scalar_read(I.bl_color, 1);
    auto skip = [&] {  // to the first chunk at or after next_h
        while (next_h >= end_h && ++next_c < I.n_colors) {
            next_h = end_h + wave_u;
            end_h = scalar_read(I.bl_color, next_c + 1);
        }
    };
    skip();
    const int first_c = next_c, first_h = next_h, first_end = end_h;
    const i32x4 *infos = reinterpret_cast<const i32x4 *>(I.bl_info);
    i32x4 info = {0, 0, 0, 0}, next = {0, 0, 0, 0};
    int lane_word = -1, chunk_c = first_c;  // the chunk at hand
    uint32_t sign = 0;
    uint4 q[4];
    auto advance = [&] {
        if (next_c == I.n_colors) {
            next_c = first_c;
            next_h = first_h;
            end_h = first_end;
        }
        next_h += nwaves;
        skip();
        if (next_c == I.n_colors)
            next_h = first_h;
        next = scalar_read(infos, next_h);
    };
    // a block, with what follows one shorter than 8 slots (after the last one
    // zeros); not used
    auto read_block = [&](uint32_t at) {
        sign = (uint32_t)sign_at(at);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            q[i] = row_at(at, i);
    };
    auto lane_words = [&](int h) { return I.bl_var[(size_t)h * kChunk + lane]; };
    if (first_c < I.n_colors) {
        info = scalar_read(infos, first_h);
        lane_word = lane_words(first_h);
        read_block((uint32_t)info.x);
        advance();
    }
    for (int s = 0; s < C.n_sweeps; ++s) {
        const uint32_t t = C.t0 + (uint32_t)s;
        const uint32_t *tg = tab + (size_t)s * C.sweep_words;
        for (int i = tid; i < tab_words; i += nthr)
            tl[i] = tg[i];
        __syncthreads();

        int dsum[NR];
#pragma unroll
        for (int j = 0; j < NR; ++j)
            dsum[j] = 0;
        for (int cur = 0;;) {
            // (a wave joins the barriers of the classes it has no chunk in)
            for (; cur < chunk_c; ++cur)
                __syncthreads();
            if (chunk_c == I.n_colors)
                break;
            {
                const int nslot = info.y, lg = info.z, ws = info.w, lw = lane_word;
                const int v = lw < 0 ? -1 : (lw & 0xFFFFF);
                // the variable's class is needed after the slot loop; load it now
                const int cl = (C.var_cls && v >= 0) ? (int)C.var_cls[v] : 0;
                // 8 slots at a time: a word of nibbles (two words for two
                // groups), one per slot, whose xor with the signs has a bit set
                // where the slot's own literal is positive and another is true,
                // or negated and none is; cnt adds those bits up per replica,
                // cnf those of the slots from ws on, which in an odd lane are its
                // neighbour's.  The next block's records are in flight.
                uint32_t cnt[GPW][4] = {}, cnf[GPW][4] = {};
                uint32_t word[GPW];
                auto pair = [&](const uint4 &q) {
                    const SlotBytes b0 = slot_bytes(q.x, q.y), b1 = slot_bytes(q.z, q.w);
                    return SlotPair{b0, b1};
                };
                auto add = [&](const SlotPair &p) {
                    const uint32_t x0 = slot_sat(p.a), x1 = slot_sat(p.b);
                    if constexpr (GPW == 1) {
                        word[0] = (word[0] << 4) | x0;
                        word[0] = (word[0] << 4) | x1;
                    } else {
                        word[0] = (((word[0] << 4) | (x0 & 0xFu)) << 4) | (x1 & 0xFu);
                        word[GPW - 1] = (((word[GPW - 1] << 4) | (x0 >> 4)) << 4) | (x1 >> 4);
                    }
                };
                // the block's slots past ws are its low f nibbles
                auto count = [&](uint32_t sg, int f) {
#pragma unroll
                    for (int k = 0; k < GPW; ++k)
                        count_nibbles(cnt[k], word[k] ^ sg);
                    if (f > 0) {
                        const uint32_t m = f >= 8 ? ~0u : (1u << (4 * f)) - 1u;
#pragma unroll
                        for (int k = 0; k < GPW; ++k)
                            count_nibbles(cnf[k], (word[k] ^ sg) & m);
                    }
                };
                auto clear = [&] {
#pragma unroll
                    for (int k = 0; k < GPW; ++k)
                        word[k] = 0;
                };
                int left = nslot;
                uint32_t at = (uint32_t)info.x;
                for (; left > 8; left -= 8) {
                    at += kBlockBytes;
                    const uint32_t sg = sign;
                    clear();
                    const SlotPair p0 = pair(q[0]), p1 = pair(q[1]);
                    sign = (uint32_t)sign_at(at);
                    q[0] = row_at(at, 0);
                    q[1] = row_at(at, 1);
                    issue_fence();
                    add(p0);
                    add(p1);
                    const SlotPair p2 = pair(q[2]), p3 = pair(q[3]);
                    q[2] = row_at(at, 2);
                    q[3] = row_at(at, 3);
                    issue_fence();
                    add(p2);
                    add(p3);
                    count(sg, nslot - left + 8 - ws);
                }
                // the last block
                clear();
                auto tail = [&](auto np) {
                    constexpr int NP = decltype(np)::value;
                    SlotPair p[NP];
#pragma unroll
                    for (int i = 0; i < NP; ++i)
                        p[i] = pair(q[i]);
                    issue_fence();
#pragma unroll
                    for (int i = 0; i < NP; ++i)
                        add(p[i]);
                };
                switch (left) {
                case 2: tail(std::integral_constant<int, 1>{}); break;
                case 4: tail(std::integral_constant<int, 2>{}); break;
                case 6: tail(std::integral_constant<int, 3>{}); break;
                default: tail(std::integral_constant<int, 4>{});
                }
                count(sign, nslot - ws);
                // on to the next chunk, while this one is decided
                info = next;
                read_block((uint32_t)info.x);
                lane_word = lane_words(next_h);
                chunk_c = next_c;
                advance();
                issue_fence();
                // the closed form: (slots that are not negated) - count per
                // replica, as four byte lanes around 128; sums and differences
                // mod 2^32, so the lanes' shares add up in any order
                uint32_t acc[GPW];
#pragma unroll
                for (int k = 0; k < GPW; ++k) {
                    uint32_t part = pack_counts(cnt[k]);
                    if (lg > 0)
                        part = lane_group_sum(part, lg);
                    else if (ws < nslot) {
                        // the odd lane's foreign slots: to the even lane
                        const uint32_t own = pack_counts(cnf[k]);
                        const uint32_t odd = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)own, 0xF5, 0xF, 0xF, false);
                        part += (lane & 1) ? 0u - odd : odd;
                    }
                    // (the lane word's share in every byte)
                    acc[k] = 0x80808080u + __builtin_amdgcn_perm(0u, (uint32_t)lw >> 20, 0u) - part;
                }
                if (v >= 0) {
                    const uint32_t xi = lds_load_u8((uint32_t)v);
                    const uint32_t *T = tl + __mul24(cl, C.stride);
                    int de[NR];
                    uint32_t flip = 0;
#pragma unroll
                    for (int k = 0; k < GPW; ++k) {
                        // byte j: 128 + dE of replica j, from acc where its x is 1,
                        // else the bytes' negatives (256 - b, 1 <= b <= 255)
                        const uint32_t ones = spread4((xi >> (4 * k)) & 0xFu), m = (ones << 8) - ones;
                        const uint32_t D = (acc[k] & m) | ((0x01010100u - acc[k]) & ~m);
                        uint32_t thr[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            de[4 * k + j] = (int)((D >> (8 * j)) & 0xFFu) - 128;
                            thr[j] = T[max(de[4 * k + j], 0)];
                        }
                        // one generator call per group gives its 4 replicas' words
                        PhiloxRounds u = {(uint32_t)v, t, (uint32_t)(g0 + k), kStreamKsatSweep, C.key0, C.key1};
#pragma unroll
                        for (int i = 0; i < 5; ++i)
                            u.round2();
                        const uint32_t w[4] = {u.c0, u.c1, u.c2, u.c3};
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            flip |= ((de[4 * k + j] <= 0) | (w[j] < thr[j])) ? 1u << (4 * k + j) : 0u;
                    }
                    flip &= amask;
                    if (flip) {
                        n_acc += __builtin_popcount(flip);
                        const uint32_t nx = xi ^ flip;
                        lds_store_u8((uint32_t)v, nx);
                        lds_store_u8((uint32_t)(n + v), ~nx & amask);
#pragma unroll
                        for (int j = 0; j < NR; ++j)
                            dsum[j] += ((flip >> j) & 1u) ? de[j] : 0;
                    }
                }
            }
        }
        chunk_c = first_c;

        // sweep end: exact energies, best, first hit, snapshot
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const int dj = wave_sum(dsum[j]);
            if (lane == 0 && dj)
                atomicAdd(&red[j], dj);
        }
        __syncthreads();
        if (tid < nact) {
            E += red[tid];
            if (E < best) {
                best = E;
                atomicOr(&red[NR], 1 << tid);
            }
            if (fh < 0 && E <= C.target)
                fh = (int)(t + 1);
        }
        __syncthreads();
        const uint32_t imp = (uint32_t)red[NR];
        if (imp) {
#pragma unroll
            for (int k = 0; k < GPW; ++k) {
                const uint32_t ik = (imp >> (4 * k)) & 0xFu;
                if (!ik)
                    continue;
                uint8_t *bg = R.best_xs + (size_t)(g0 + k) * n;
                if (wide) {
                    const uint32_t i4 = ik * 0x01010101u;
                    for (int w = tid; w < n / 16; w += nthr) {
                        uint4 o = reinterpret_cast<const uint4 *>(bg)[w];
                        uint4 c = reinterpret_cast<const uint4 *>(xt)[w];
                        if (k) {
                            c.x >>= 4;
                            c.y >>= 4;
                            c.z >>= 4;
                            c.w >>= 4;
                        }
                        o.x = (o.x & ~i4) | (c.x & i4);
                        o.y = (o.y & ~i4) | (c.y & i4);
                        o.z = (o.z & ~i4) | (c.z & i4);
                        o.w = (o.w & ~i4) | (c.w & i4);
                        reinterpret_cast<uint4 *>(bg)[w] = o;
                    }
                } else {
                    for (int v = tid; v < n; v += nthr)
                        bg[v] = (uint8_t)((bg[v] & ~ik) | ((uint32_t)(xt[v] >> (4 * k)) & ik));
                }
            }
        }
        __syncthreads();
        if (tid < 16)
            red[tid] = 0;
    }

    __syncthreads();
#pragma unroll
    for (int k = 0; k < GPW; ++k) {
        if (k == 1 && !second)
            break;
        uint8_t *xk = xg + (size_t)k * n;
        if (wide) {
            for (int w = tid; w < n / 16; w += nthr) {
                uint4 b = reinterpret_cast<const uint4 *>(xt)[w];
                if (GPW == 2) {
                    const uint32_t sh = 4 * k;
                    b = make_uint4((b.x >> sh) & 0x0F0F0F0Fu, (b.y >> sh) & 0x0F0F0F0Fu, (b.z >> sh) & 0x0F0F0F0Fu,
                                   (b.w >> sh) & 0x0F0F0F0Fu);
                }
                reinterpret_cast<uint4 *>(xk)[w] = b;
            }
        } else {
            for (int v = tid; v < n; v += nthr)
                xk[v] = GPW == 2 ? (uint8_t)((xt[v] >> (4 * k)) & 0xFu) : xt[v];
        }
    }
    if (tid < nact) {
        R.energy[r0 + tid] = E;
        R.best[r0 + tid] = best;
        R.first_hit[r0 + tid] = fh;
    }
    unsigned long long acc_w = n_acc;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        acc_w += __shfl_xor(acc_w, off, 64);
    if (lane == 0 && acc_w)
        atomicAdd(R.accepted, acc_w);
}

// ---- split sweeps -----------------------------------------------------------
//
// Instances of small colour classes.  A class of a few hundred variables is a
// few chunks of 64, one lane each, so of the 16 waves of a workgroup most
// waited at every class barrier while a few walked 40 records per lane, and
// what bounds a sweep is the latency of one class step.  Here every variable
// has 2^LG lanes (the split layout: each walks 1 / 2^LG of its records, all
// gathers in flight at once), the four lanes of its first quad decide one
// replica each, the records of a wave's next chunk are loaded while this
// one is decided, the random words are drawn by whole waves (one generator
// call per lane serves the wave's next 2^LG chunks), and thresholds, best
// states and classes stay in LDS: a sweep ends with one barrier, a second one
// if a best state was copied, and reads device memory only for threshold rows
// of more than two words per thread.
//
// Measured (us per sweep at 64 to 1024 replicas, default tuning, against one
// lane per variable with the words drawn per class, records staged in LDS at n
// = 200): 4-SAT n = 200 34.6 -> 16.3, 1000 77 -> 24, 2000 93 -> 37, 5000 104 ->
// 47, 9000 105 -> 63; 3-SAT n = 1000 23 -> 10.3, 3500 25.2 -> 18.6.  A class
// step of n = 200 takes 0.5 us: gathers, sum, threshold read, store and
// barrier in sequence.  At n = 5000 the gathers' bank conflicts counted (56 us
// before the records were placed by bank) and so did 32-bit multiplies and a
// table read under a mask in the decision.
//
// LDS: x and not-x (2 n + 2 bytes), best states (n), classes (2 n), two sweeps'
// threshold rows, the energy sums of two sweeps, and per wave its list of
// chunks, their variables (4 bytes each) and 64 generator blocks.
struct SplitLds {
    size_t best, cls, tl, red, list, list_len, vars, words, total;
};
__host__ __device__ inline SplitLds split_lds(int n, int n_colors, int n_chunks, int lg, int tab_words, int waves) {
    SplitLds L;
    L.best = align_up(2 * (size_t)n + 2, 16);
    L.cls = L.best + align_up(n, 16);
    L.tl = L.cls + align_up(2 * (size_t)n, 16);
    L.red = L.tl + align_up(2 * (size_t)tab_words * 4, 16);
    L.list = L.red + 32;
    // a wave has at most one more chunk per class than its even share
    L.list_len = (size_t)n_colors + (size_t)(n_chunks + waves - 1) / waves;
    L.vars = L.list + L.list_len * waves * 16;
    L.words = L.vars + align_up(L.list_len * waves * (kChunk >> lg) * 4, 16);
    L.total = L.words + (size_t)waves * kChunk * 16;
    return L;
}

template <int LG>
__global__ void __launch_bounds__(1024) ksat_split_kernel(KsatDev I, KsatRepDev R, SweepCall C) {
    extern __shared__ __align__(16) uint8_t smem[];
    constexpr int PER = kChunk >> LG;  // variables of a chunk
    // record pairs of the next chunk loaded ahead: 48, 64 and 96 clauses per
    // variable on 4, 8 and 16 lanes
    constexpr int PRE = LG == 2 ? kSplitAhead : LG == 3 ? 4 : 3;
    const int n = I.n, g = blockIdx.x;
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, nwaves = nthr >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tab_words = C.n_classes * C.stride;
    const SplitLds L = split_lds(n, I.n_colors, I.sp_chunks, LG, tab_words, nwaves);
    uint8_t *xt = smem, *bx = smem + L.best;
    uint16_t *cls = (uint16_t *)(smem + L.cls);  // threshold row offset of each variable's class
    uint32_t *tl = (uint32_t *)(smem + L.tl);
    int *red = (int *)(smem + L.red);
    int4 *list = (int4 *)(smem + L.list) + wave * L.list_len;
    int *vars = (int *)(smem + L.vars) + wave * L.list_len * PER;
    uint4 *words = (uint4 *)(smem + L.words) + wave * kChunk;

    const int r0 = g * kGroup, nact = min(kGroup, R.n_rep - r0);
    const uint32_t amask = (1u << nact) - 1u;
    const int j = lane & 3;  // the replica this lane decides
    uint8_t *xg = R.xs + (size_t)g * n, *bg = R.best_xs + (size_t)g * n;
    for (int v = tid; v < n; v += nthr) {
        const uint32_t b = xg[v] & amask;
        xt[v] = (uint8_t)b;
        xt[n + v] = (uint8_t)(~b & amask);
        bx[v] = bg[v];
        cls[v] = C.var_cls ? (uint16_t)(C.var_cls[v] * C.stride) : 0;
    }
    if (tid == 0) {
        xt[2 * n] = 0;
        xt[2 * n + 1] = (uint8_t)amask;
    }
    if (tid < 8)
        red[tid] = 0;
    const uint32_t *tab = C.tab + (C.reps_per_row > 0 ? (size_t)(r0 / C.reps_per_row) * tab_words : 0);
    if (C.n_sweeps > 0)
        for (int i = tid; i < tab_words; i += nthr)
            tl[i] = tab[i];
    // the wave's chunks in class order: (chunk, class, first pair-row, pairs)
    int items = 0;
    for (int c = 0; c < I.n_colors; ++c)
        for (int h = I.sp_color[c] + wave; h < I.sp_color[c + 1]; h += nwaves) {
            const int2 info = I.sp_info[h];
            list[items] = make_int4(h, c, info.x, info.y);  // (every lane the same)
            if (lane < PER)
                vars[items * PER + lane] = max(I.sp_var[(size_t)h * kChunk + (lane << LG)].x, 0);
            ++items;
        }
    int E = 0, best = 0, fh = -1;
    if (j < nact) {
        E = R.energy[r0 + j];
        best = R.best[r0 + j];
        fh = R.first_hit[r0 + j];
        if (C.check_start && fh < 0 && E <= C.target)
            fh = (int)C.t0;
    }
    const __amdgpu_buffer_rsrc_t recs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint64_t *>(I.sp_rec), 0, (int)I.sp_rec_bytes, kBufferWord3);
    uint4 q[PRE];
    int lw = -1;
    uint32_t kk = 0;
    int4 e = make_int4(0, 0, 0, 0);  // the chunk's list entry
    auto rp = [&](int row) -> uint4 {
        return __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(recs, lane * 16, row * (kChunk * 16), 0));
    };
    // loads of the chunk of entry e: lane words and the first records (rows
    // past the chunk are other chunks' or, after the last one, zeros; they are
    // not used)
    auto fetch = [&](const int4 &x) {
        e = make_int4(__builtin_amdgcn_readfirstlane(x.x), __builtin_amdgcn_readfirstlane(x.y),
                      __builtin_amdgcn_readfirstlane(x.z), __builtin_amdgcn_readfirstlane(x.w));
        const int2 w = I.sp_var[(size_t)e.x * kChunk + lane];
        lw = w.x;
        kk = (uint32_t)w.y;
#pragma unroll
        for (int i = 0; i < PRE; ++i)
            q[i] = rp(e.z + i);
    };
    __syncthreads();
    if (items)
        fetch(list[0]);
    const bool first = (lane & ((1 << LG) - 1)) < 4;  // the quad that decides
    uint32_t n_acc = 0;
    for (int s = 0; s < C.n_sweeps; ++s) {
        const uint32_t t = C.t0 + (uint32_t)s;
        const uint32_t *T = tl + (s & 1) * tab_words;
        // the next sweep's thresholds, stored at the end of this one
        uint32_t tn[2] = {0, 0};
        const uint32_t *tg = tab + (size_t)(s + 1) * C.sweep_words;
        const bool more = s + 1 < C.n_sweeps;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (more && tid + i * nthr < tab_words)
                tn[i] = tg[tid + i * nthr];
        int dsum = 0, cur = 0;
        for (int it = 0; it < items; ++it) {
            for (; cur < e.y; ++cur)
                __syncthreads();
            const int4 next = list[it + 1 < items ? it + 1 : 0];
            if ((it & ((1 << LG) - 1)) == 0) {
                // words of the wave's next 2^LG chunks, one variable per lane
                const int k = min(it * PER + lane, items * PER - 1);
                const uint32_t v = (uint32_t)vars[k];
                issue_fence();
                words[lane] = philox4x32_10(v, t, (uint32_t)g, kStreamKsatSweep, C.key0, C.key1);
                issue_fence();
            }
            const int v = max(lw, 0);
            const uint32_t xi = lds_load_u8((uint32_t)v);
            const uint32_t cl = cls[v];
            const uint32_t u =
                reinterpret_cast<const uint32_t *>(words)[((it & ((1 << LG) - 1)) * PER + (lane >> LG)) * 4 + j];
            uint32_t acc = kk;
            // straight-line code per count, every gather issued before the
            // first is used
            auto walk = [&](auto np) {
                constexpr int NP = decltype(np)::value < PRE ? decltype(np)::value : PRE;
                uint32_t x[2 * NP][3], sm[2 * NP];
#pragma unroll
                for (int i = 0; i < NP; ++i) {
                    slot_gather(make_uint2(q[i].x, q[i].y), x[2 * i], sm[2 * i]);
                    slot_gather(make_uint2(q[i].z, q[i].w), x[2 * i + 1], sm[2 * i + 1]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 2 * NP; ++i)
                    acc -= spread4(x[i][0] | x[i][1] | x[i][2]) ^ sm[i];
            };
            using std::integral_constant;
            switch (min(e.w, PRE)) {
            case 1: walk(integral_constant<int, 1>{}); break;
            case 2: walk(integral_constant<int, 2>{}); break;
            case 3: walk(integral_constant<int, 3>{}); break;
            case 4: walk(integral_constant<int, 4>{}); break;
            case 5: walk(integral_constant<int, 5>{}); break;
            default: walk(integral_constant<int, PRE>{});
            }
            for (int k = PRE; k < e.w; ++k) {
                const uint4 r = rp(e.z + k);
                acc = acc - slot_step(0u, make_uint2(r.x, r.y)) - slot_step(0u, make_uint2(r.z, r.w));
            }
            const bool live = lw >= 0 && first && j < nact;
            // the next chunk's records (the first chunk's after the last: the
            // next sweep starts with it)
            fetch(next);
            issue_fence();
            acc = lane_group_sum(acc, LG);
            const int S = (int)((acc >> (8 * j)) & 0xFFu) - 128;
            const int de = ((xi >> j) & 1u) ? S : -S;
            const uint32_t thr = T[cl + max(de, 0)];
            const bool take = live & ((de <= 0) | (u < thr));
            uint32_t flip = take ? 1u << j : 0u;
            flip |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)flip, 0xB1, 0xF, 0xF, false);
            flip |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)flip, 0x4E, 0xF, 0xF, false);
            dsum += take ? de : 0;
            n_acc += take;
            if (flip && live && j == 0) {
                const uint32_t nx = xi ^ flip;
                lds_store_u8((uint32_t)v, nx);
                lds_store_u8((uint32_t)(n + v), ~nx & amask);
            }
        }
        for (; cur < I.n_colors; ++cur)
            __syncthreads();
        // sweep end: this wave's energy changes by replica, then one barrier
        dsum += __shfl_xor(dsum, 4, 64);
        dsum += __shfl_xor(dsum, 8, 64);
        dsum += __shfl_xor(dsum, 16, 64);
        dsum += __shfl_xor(dsum, 32, 64);
        int *rs = red + 4 * (s & 1);
        if (lane < kGroup && dsum)
            atomicAdd(&rs[lane], dsum);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (more && tid + i * nthr < tab_words)
                tl[((s + 1) & 1) * tab_words + tid + i * nthr] = tn[i];
        for (int i = tid + 2 * nthr; more && i < tab_words; i += nthr)
            tl[((s + 1) & 1) * tab_words + i] = tg[i];
        __syncthreads();
        // every wave keeps the replicas' energies; the sums of the sweep
        // before last are cleared for the next one
        E += rs[j];
        if (tid < kGroup)
            red[4 * ((s + 1) & 1) + tid] = 0;
        const bool imp = j < nact && E < best;
        best = imp ? E : best;
        if (j < nact && fh < 0 && E <= C.target)
            fh = (int)(t + 1);
        const uint32_t im = (uint32_t)__ballot(imp) & 0xFu;
        if (im) {  // (the same in every wave)
            for (int v = tid; v < n; v += nthr)
                bx[v] = (uint8_t)((bx[v] & ~im) | (xt[v] & im));
            __syncthreads();
        }
    }
    __syncthreads();
    for (int v = tid; v < n; v += nthr) {
        xg[v] = xt[v];
        bg[v] = bx[v];
    }
    if (tid < nact) {
        R.energy[r0 + tid] = E;
        R.best[r0 + tid] = best;
        R.first_hit[r0 + tid] = fh;
    }
    unsigned long long acc_w = n_acc;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        acc_w += __shfl_xor(acc_w, off, 64);
    if (lane == 0 && acc_w)
        atomicAdd(R.accepted, acc_w);
}

// One item (GPW groups of 4 replicas) per workgroup (item = blockIdx.x).
template <int GPW>
__global__ void __launch_bounds__(1024) ksat_sweep_kernel(KsatDev I, KsatRepDev R, SweepCall C) {
    extern __shared__ __align__(16) uint8_t smem[];
    sweep_group<GPW>(I, R, C, blockIdx.x, smem);
}

// Batched launch: many replica sets (jobs) of different instances in one
// grid.  items[] lists (job, group) pairs in decreasing cost; workgroup b
// runs items b, b + gridDim.x, ...  The dynamic LDS block is sized for the
// largest job.
__global__ void __launch_bounds__(1024) ksat_sweep_batch_kernel(const KsatJob *jobs, const int2 *items, int n_items) {
    extern __shared__ __align__(16) uint8_t smem[];
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int2 w = items[it];
        const KsatJob &J = jobs[w.x];
        if (J.C.gpw == 2)
            sweep_group<2>(J.I, J.R, J.C, w.y, smem);
        else
            sweep_group<1>(J.I, J.R, J.C, w.y, smem);
        __syncthreads();
    }
}

// Backbone statistics for many jobs: items[] lists (job, first variable)
// blocks of 256 variables.
__global__ void ksat_magnetization_batch_kernel(const KsatJob *jobs, const int2 *items, int thr_num, int thr_den,
                                                int expand) {
    const int2 w = items[blockIdx.x];
    const KsatJob &J = jobs[w.x];
    const int v = w.y + threadIdx.x;
    if (v >= J.I.n)
        return;
    int c = 0;
    for (int g = 0; g < J.R.n_groups; ++g)
        c += __popc((uint32_t)J.R.xs[(size_t)g * J.I.n + v]);
    J.R.counts[v] = c;
    long long dev = 2ll * c - J.R.n_rep;
    if (dev < 0)
        dev = -dev;
    const uint8_t fz = (long long)thr_den * dev >= (long long)thr_num * J.R.n_rep;
    J.R.frozen[v] = fz;
    if (!expand)
        J.R.cls[v] = fz;
}

__global__ void ksat_expand_batch_kernel(const KsatJob *jobs, const int2 *items) {
    const int2 w = items[blockIdx.x];
    const KsatJob &J = jobs[w.x];
    const int v = w.y + threadIdx.x;
    if (v >= J.I.n)
        return;
    uint8_t hot = J.R.frozen[v];
    for (int q = J.I.var_ptr[v]; q < J.I.var_ptr[v + 1] && !hot; ++q) {
        const uint4 ad = reinterpret_cast<const uint4 *>(J.I.clause_addr)[J.I.var_cl[q]];
        const uint32_t a[4] = {ad.x, ad.y, ad.z, ad.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (a[j] < (uint32_t)(2 * J.I.n)) {
                const uint32_t u = a[j] < (uint32_t)J.I.n ? a[j] : a[j] - J.I.n;
                hot |= J.R.frozen[u];
            }
        }
    }
    J.R.cls[v] = hot;
}

// c_i = replicas with x_i = 1; frozen_i per the |magnetization| threshold.
__global__ void ksat_magnetization_kernel(KsatDev I, KsatRepDev R, int thr_num, int thr_den, int expand) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= I.n)
        return;
    int c = 0;
    for (int g = 0; g < R.n_groups; ++g)
        c += __popc((uint32_t)R.xs[(size_t)g * I.n + v]);
    R.counts[v] = c;
    long long dev = 2ll * c - R.n_rep;
    if (dev < 0)
        dev = -dev;
    const uint8_t fz = (long long)thr_den * dev >= (long long)thr_num * R.n_rep;
    R.frozen[v] = fz;
    if (!expand)
        R.cls[v] = fz;
}

// hot_i = frozen_i or some clause of i holds a frozen variable.
__global__ void ksat_expand_kernel(KsatDev I, KsatRepDev R) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= I.n)
        return;
    uint8_t hot = R.frozen[v];
    for (int q = I.var_ptr[v]; q < I.var_ptr[v + 1] && !hot; ++q) {
        const uint4 ad = reinterpret_cast<const uint4 *>(I.clause_addr)[I.var_cl[q]];
        const uint32_t a[4] = {ad.x, ad.y, ad.z, ad.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (a[j] < (uint32_t)(2 * I.n)) {
                const uint32_t w = a[j] < (uint32_t)I.n ? a[j] : a[j] - I.n;
                hot |= R.frozen[w];
            }
        }
    }
    R.cls[v] = hot;
}

// tally[0] = lowest best energy, tally[1] = replicas with best energy 0.
__global__ void ksat_tally_kernel(KsatRepDev R) {
    __shared__ int smin[16], scnt[16];
    int mn = INT_MAX, cnt = 0;
    for (int r = threadIdx.x; r < R.n_rep; r += blockDim.x) {
        const int b = R.best[r];
        mn = min(mn, b);
        cnt += b == 0;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        mn = min(mn, __shfl_xor(mn, off, 64));
        cnt += __shfl_xor(cnt, off, 64);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        smin[w] = mn;
        scnt[w] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < (int)(blockDim.x >> 6); ++i) {
            mn = min(mn, smin[i]);
            cnt += scnt[i];
        }
        R.tally[0] = mn;
        R.tally[1] = cnt;
    }
}

__global__ void ksat_unpack_kernel(const uint8_t *xs, int n, int n_rep, uint8_t *rows) {
    const size_t total = (size_t)n_rep * n;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (size_t)gridDim.x * blockDim.x) {
        const int r = (int)(idx / n), v = (int)(idx % n);
        rows[idx] = (xs[(size_t)(r / kGroup) * n + v] >> (r % kGroup)) & 1u;
    }
}

__global__ void ksat_pack_kernel(const uint8_t *rows, int n, int n_groups, int n_rep, uint8_t *xs) {
    const size_t total = (size_t)n_groups * n;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (size_t)gridDim.x * blockDim.x) {
        const int g = (int)(idx / n), v = (int)(idx % n);
        uint32_t b = 0;
        for (int j = 0; j < kGroup; ++j) {
            const int r = g * kGroup + j;
            if (r < n_rep)
                b |= (rows[(size_t)r * n + v] & 1u) << j;
        }
        xs[idx] = (uint8_t)b;
    }
}

__global__ void set_status_kernel(const SetStatusSrc *src, SetStatus *out) {
    __shared__ long long smin[4];
    __shared__ int scnt[4], sfh[4];
    const SetStatusSrc S = src[blockIdx.x];
    long long mn = LLONG_MAX;
    int cnt = 0, fh = INT_MAX;
    for (int r = threadIdx.x; r < S.n_rep; r += blockDim.x) {
        const long long b = S.best_is_64 ? reinterpret_cast<const long long *>(S.best)[r]
                                         : (long long)reinterpret_cast<const int32_t *>(S.best)[r];
        mn = b < mn ? b : mn;
        cnt += b == 0;
        const int f = S.first_hit[r];
        if (f >= 0 && f < fh)
            fh = f;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const long long o = __shfl_xor(mn, off, 64);
        mn = o < mn ? o : mn;
        cnt += __shfl_xor(cnt, off, 64);
        fh = min(fh, __shfl_xor(fh, off, 64));
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        smin[w] = mn;
        scnt[w] = cnt;
        sfh[w] = fh;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < (int)(blockDim.x >> 6); ++i) {
            mn = smin[i] < mn ? smin[i] : mn;
            cnt += scnt[i];
            fh = min(fh, sfh[i]);
        }
        out[blockIdx.x].best = mn;
        out[blockIdx.x].n_zero = cnt;
        out[blockIdx.x].first_hit = fh == INT_MAX ? -1 : fh;
    }
}

int grid_for(size_t total, int block) {
    size_t g = (total + block - 1) / block;
    if (g > 65536)
        g = 65536;
    return (int)(g < 1 ? 1 : g);
}

}  // namespace

size_t ksat_sweep_lds_bytes(int n, int n_classes, int stride) {
    return align_up(2 * (size_t)n + 2, 16) + align_up((size_t)n_classes * stride, 4) * 4 + 16 * sizeof(int);
}

size_t ksat_split_lds_bytes(int n, int n_colors, int n_chunks, int lg, int tab_words, int waves) {
    return split_lds(n, n_colors, n_chunks, lg, tab_words, waves).total;
}

hipError_t launch_set_status(const SetStatusSrc *src, SetStatus *out, int n_sets, hipStream_t s) {
    hipLaunchKernelGGL(set_status_kernel, dim3(n_sets), dim3(256), 0, s, src, out);
    return hipGetLastError();
}

hipError_t ksat_launch_init(const KsatDev &I, const KsatRepDev &R, uint32_t key0, uint32_t key1, hipStream_t s) {
    const size_t total = (size_t)R.n_groups * I.n;
    hipLaunchKernelGGL(ksat_init_kernel, dim3(grid_for(total, 256)), dim3(256), 0, s, I, R, key0, key1);
    return hipGetLastError();
}

hipError_t ksat_launch_recount(const KsatDev &I, const uint8_t *xs, int n_groups, int n_rep, int32_t *energy_out,
                               hipStream_t s) {
    if (I.wide)
        return hipErrorNotSupported;  // wide instances count from their packed tables
    const size_t lds = align_up(2 * (size_t)I.n + 2, 16) + 16 * sizeof(int);
    // once per process (thread-safe initialization)
    static const hipError_t attr = hipFuncSetAttribute((const void *)ksat_recount_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                       (int)kLdsBytes);
    if (attr != hipSuccess)
        return attr;
    hipLaunchKernelGGL(ksat_recount_kernel, dim3(n_groups), dim3(1024), lds, s, I, xs, n_rep, energy_out);
    return hipGetLastError();
}

hipError_t ksat_launch_reset_tallies(const KsatRepDev &R, int n, hipStream_t s) {
    hipLaunchKernelGGL(ksat_reset_tallies_kernel, dim3(grid_for((size_t)R.n_groups * kGroup, 256)), dim3(256), 0, s,
                       R);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    return hipMemcpyAsync(R.best_xs, R.xs, (size_t)R.n_groups * n, hipMemcpyDeviceToDevice, s);
}

static size_t split_lds_of(const KsatDev &I, const SweepCall &C) {
    return ksat_split_lds_bytes(I.n, I.n_colors, I.sp_chunks, I.sp_lg, C.n_classes * C.stride, I.sp_waves);
}

// At the default workgroup size, where the layout exists and its sweep fits in
// LDS.  Up to one group per CU (1024 replicas) no general workgroup of 64 to
// 1024 threads with 4 or 8 replicas is faster: 4-SAT n = 200, 1000, 5000, 9000
// 17, 24, 47, 64 us per sweep against 34, 67, 84, 90 at the best size; 3-SAT n =
// 1000, 5000 10.3, 25.6 against 19, 25.7.  Larger sets fill the CUs with small
// workgroups (4096 replicas of 4-SAT n = 1000, 2000, 9000: 58, 120, 259 against
// 70, 85, 156 at 64, 128, 512 threads); the tuner chooses those where they are
// faster, and a size set by hand is kept, but for the smallest instances: with
// kSplitAnySize clauses or fewer and up to 4096 replicas a general sweep takes
// 1.6 to 2.2 times as long at every size (4-SAT n = 60: 28 against 14 us).
// NMC_KSAT_STAGE=0, read at every launch, keeps the general sweeps, so that a
// process can compare the two.
bool ksat_takes_split(const KsatDev &I, int n_groups, const SweepCall &C, int block_threads) {
    constexpr int kSplitAnySize = 2048;
    const bool sized = block_threads == 1024 || (I.m <= kSplitAnySize && n_groups <= 1024);
    if (!I.sp_lg || C.gpw == 2 || !sized || split_lds_of(I, C) > kLdsBytes)
        return false;
    const char *e = std::getenv("NMC_KSAT_STAGE");
    return !(e && e[0] == '0');
}

hipError_t ksat_launch_sweep(const KsatDev &I, const KsatRepDev &R, const SweepCall &C, int block_threads,
                             hipStream_t s) {
    const size_t lds = ksat_sweep_lds_bytes(I.n, C.n_classes, C.stride);
    // once per process (thread-safe initialization)
    static const hipError_t attr = [] {
        hipError_t e = hipFuncSetAttribute((const void *)ksat_sweep_kernel<1>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)ksat_sweep_kernel<2>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)kLdsBytes);
        return e;
    }();
    if (attr != hipSuccess)
        return attr;
    static const hipError_t attr_split = [] {
        hipError_t e = hipSuccess;
        for (const void *f : {(const void *)ksat_split_kernel<2>, (const void *)ksat_split_kernel<3>,
                              (const void *)ksat_split_kernel<4>})
            if (e == hipSuccess)
                e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
        return e;
    }();
    if (attr_split != hipSuccess)
        return attr_split;
    if (C.gpw == 2)
        hipLaunchKernelGGL(ksat_sweep_kernel<2>, dim3((R.n_groups + 1) / 2), dim3(block_threads), lds, s, I, R, C);
    else if (ksat_takes_split(I, R.n_groups, C, block_threads))
        hipLaunchKernelGGL(I.sp_lg == 2   ? ksat_split_kernel<2>
                           : I.sp_lg == 3 ? ksat_split_kernel<3>
                                          : ksat_split_kernel<4>,
                           dim3(R.n_groups), dim3(64 * I.sp_waves), split_lds_of(I, C), s, I, R, C);
    else
        hipLaunchKernelGGL(ksat_sweep_kernel<1>, dim3(R.n_groups), dim3(block_threads), lds, s, I, R, C);
    return hipGetLastError();
}

hipError_t ksat_launch_sweep_batch(const KsatJob *jobs, const int2 *items, int n_items, size_t lds, int block_threads,
                                   int grid, hipStream_t s) {
    // once per process (thread-safe initialization)
    static const hipError_t attr = hipFuncSetAttribute((const void *)ksat_sweep_batch_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                       (int)kLdsBytes);
    if (attr != hipSuccess)
        return attr;
    hipLaunchKernelGGL(ksat_sweep_batch_kernel, dim3(grid), dim3(block_threads), lds, s, jobs, items, n_items);
    return hipGetLastError();
}

int ksat_batch_occupancy(int block_threads, size_t lds) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void *)ksat_sweep_batch_kernel, block_threads, lds) !=
        hipSuccess)
        return 1;
    return nb < 1 ? 1 : nb;
}

hipError_t ksat_launch_backbone_batch(const KsatJob *jobs, const int2 *items, int n_items, int thr_num, int thr_den,
                                      int expand, hipStream_t s) {
    hipLaunchKernelGGL(ksat_magnetization_batch_kernel, dim3(n_items), dim3(256), 0, s, jobs, items, thr_num, thr_den,
                       expand);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !expand)
        return e;
    hipLaunchKernelGGL(ksat_expand_batch_kernel, dim3(n_items), dim3(256), 0, s, jobs, items);
    return hipGetLastError();
}

hipError_t ksat_launch_backbone(const KsatDev &I, const KsatRepDev &R, int thr_num, int thr_den, int expand,
                                hipStream_t s) {
    hipLaunchKernelGGL(ksat_magnetization_kernel, dim3((I.n + 255) / 256), dim3(256), 0, s, I, R, thr_num, thr_den,
                       expand);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !expand)
        return e;
    hipLaunchKernelGGL(ksat_expand_kernel, dim3((I.n + 255) / 256), dim3(256), 0, s, I, R);
    return hipGetLastError();
}

hipError_t ksat_launch_tally(const KsatRepDev &R, hipStream_t s) {
    hipLaunchKernelGGL(ksat_tally_kernel, dim3(1), dim3(1024), 0, s, R);
    return hipGetLastError();
}

hipError_t ksat_launch_unpack(const uint8_t *xs, int n, int n_groups, int n_rep, uint8_t *rows, hipStream_t s) {
    (void)n_groups;
    hipLaunchKernelGGL(ksat_unpack_kernel, dim3(grid_for((size_t)n_rep * n, 256)), dim3(256), 0, s, xs, n, n_rep,
                       rows);
    return hipGetLastError();
}

hipError_t ksat_launch_pack(const uint8_t *rows, int n, int n_groups, int n_rep, uint8_t *xs, hipStream_t s) {
    hipLaunchKernelGGL(ksat_pack_kernel, dim3(grid_for((size_t)n_groups * n, 256)), dim3(256), 0, s, rows, n,
                       n_groups, n_rep, xs);
    return hipGetLastError();
}

}  // namespace nmc
