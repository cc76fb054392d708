// Whitening of low-energy k-SAT states for gfx950 (section "Whitening
// procedure for low energy states").
//
// A variable turns white ("star") unless some clause has the variable's
// literal as its only true literal and no other white variable; a violated
// clause pins nothing.  White sets only grow and the pin condition only
// weakens as they grow, so every inspection order that repeats until
// nothing changes reaches the same (least) fixed point: the whitening of one
// group of 4 replicas runs inside one workgroup, pass after pass, with no
// global synchronization; the 16 chunks of a round are all read before any is
// stored, so the number of passes does not depend on the waves' timing.
//
// LDS: one byte per literal at the sweep's spin-table addresses (x_v at v, its
// negation at N + v, always-false 2N, always-true 2N + 1): in the low nibble
// whether the literal is true in each of the 4 replicas, in the high one the
// variable's white bits, so the OR of a clause's other literals' bytes holds
// both "another literal is true" and "another variable is white".  The
// clause structure is the sweep's: per variable (a lane of a 64-variable
// chunk), one 8-byte record per clause slot holding the addresses of the
// clause's other literals and whether the variable's own literal is negated.
// Padding slots (always-true first address) never pin.
//
// Bound: like a sweep, the three gathers per slot and the record stream.  With
// one 16-bit word per variable, decoded by sign on every read, and records
// loaded one slot at a time, the 12 passes over N = 50,000, 1024 replicas took
// 12.5 ms; with this table and eight slots of records in flight they take 2.9
// (2.7 without the rounds' barriers), 17 passes over N = 8422, 256 replicas 0.91
// instead of 2.94.
#include <climits>

#include "nmc_internal.h"

namespace nmc {

namespace {

__global__ void __launch_bounds__(1024) ksat_whiten_kernel(KsatDev I, const uint8_t *xs, int n_rep, uint8_t *white_out,
                                                           int32_t *frozen_out, int32_t *passes_out) {
    extern __shared__ __align__(16) uint8_t tbl[];
    __shared__ int changed;
    __shared__ int cnt[4];
    const int n = I.n, g = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, nwaves = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = g * kGroup;
    const int nact = min(kGroup, n_rep - r0);
    const uint32_t amask = (1u << nact) - 1u;
    const uint8_t *xg = xs + (size_t)g * n;
    for (int v = tid; v < n; v += blockDim.x) {
        const uint32_t x = xg[v] & amask;
        tbl[v] = (uint8_t)x;
        tbl[n + v] = (uint8_t)(~x & amask);
    }
    if (tid == 0) {
        tbl[2 * n] = 0;
        tbl[2 * n + 1] = (uint8_t)amask;
    }
    if (tid < 4)
        cnt[tid] = 0;
    const __amdgpu_buffer_rsrc_t recs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint64_t *>(I.rec), 0, (int)I.rec_bytes, kBufferWord3);
    int passes = 0;
    for (;;) {
        if (tid == 0)
            changed = 0;
        __syncthreads();
        // rounds of one chunk per wave: every wave's reads, then its stores
        for (int h0 = 0; h0 < I.n_chunks; h0 += nwaves) {
            const int h = h0 + wave;
            int i = 0, lg = 0;
            uint32_t xi = 0, si = 0, ns = 0;
            bool live = false;
            if (h < I.n_chunks) {
                const int lw = I.chunk_var[(size_t)h * kChunk + lane];
                const int2 info = I.chunk_info[h];
                const int nslot = __builtin_amdgcn_readfirstlane(info.y & ((1 << kSplitShift) - 1));
                lg = __builtin_amdgcn_readfirstlane(info.y >> kSplitShift);  // 2^lg lanes per variable
                i = lw & 0xFFFFF;
                const uint32_t own = lw < 0 ? 0u : tbl[i];
                xi = own & 0xFu;
                si = own >> 4;
                // the lanes of one variable agree on skipping it
                live = lw >= 0 && si != amask;
                if (__any(live)) {
                    uint32_t pinned = 0;
                    auto step = [&](uint32_t lo, uint32_t hi) {
                        const uint32_t o = tbl[lo & kAddrMask] |
                                           tbl[__builtin_amdgcn_alignbit(hi, lo, kAddrBits) & kAddrMask] |
                                           tbl[__builtin_amdgcn_ubfe(hi, 2 * kAddrBits - 32, kAddrBits)];
                        const uint32_t sm = (uint32_t)__builtin_amdgcn_sbfe(hi, 3 * kAddrBits - 32, 1);
                        pinned |= (xi ^ sm) & ~(o | (o >> 4));
                    };
                    // 8 slots of records in flight (nslot is a multiple of 4;
                    // past the last pair it is read again, which changes nothing)
                    const int row0 = __builtin_amdgcn_readfirstlane(info.x) / 2, last = nslot / 2 - 1;
                    auto rp = [&](int row) -> uint4 {
                        return __builtin_bit_cast(
                            uint4, __builtin_amdgcn_raw_buffer_load_b128(recs, lane * 16,
                                                                         (row0 + min(row, last)) * (kChunk * 16), 0));
                    };
                    uint4 q[4] = {rp(0), rp(1), rp(2), rp(3)};
                    for (int k = 0; k < nslot / 2; k += 4) {
                        step(q[0].x, q[0].y);
                        step(q[0].z, q[0].w);
                        step(q[1].x, q[1].y);
                        step(q[1].z, q[1].w);
                        q[0] = rp(k + 4);
                        q[1] = rp(k + 5);
                        step(q[2].x, q[2].y);
                        step(q[2].z, q[2].w);
                        step(q[3].x, q[3].y);
                        step(q[3].z, q[3].w);
                        q[2] = rp(k + 6);
                        q[3] = rp(k + 7);
                    }
                    pinned &= amask;
                    for (int off = 1; off < (1 << lg); off <<= 1)
                        pinned |= (uint32_t)__shfl_xor((int)pinned, off, 64);
                    ns = si | (~pinned & amask);
                }
            }
            __syncthreads();
            if (live && (lane & ((1 << lg) - 1)) == 0 && ns != si) {
                tbl[i] = (uint8_t)((ns << 4) | xi);
                tbl[n + i] = (uint8_t)((ns << 4) | (~xi & amask));
                changed = 1;
            }
            __syncthreads();
        }
        __syncthreads();
        ++passes;
        const int c = changed;
        __syncthreads();
        if (!c)
            break;
    }
    // white bits out, frozen counts per replica
    int f0 = 0, f1 = 0, f2 = 0, f3 = 0;
    uint8_t *wg = white_out + (size_t)g * n;
    for (int v = tid; v < n; v += blockDim.x) {
        const uint32_t w = tbl[v] >> 4;
        wg[v] = (uint8_t)w;
        const uint32_t fz = ~w & amask;
        f0 += fz & 1u;
        f1 += (fz >> 1) & 1u;
        f2 += (fz >> 2) & 1u;
        f3 += (fz >> 3) & 1u;
    }
    for (int off = 32; off > 0; off >>= 1) {
        f0 += __shfl_xor(f0, off, 64);
        f1 += __shfl_xor(f1, off, 64);
        f2 += __shfl_xor(f2, off, 64);
        f3 += __shfl_xor(f3, off, 64);
    }
    if (lane == 0) {
        atomicAdd(&cnt[0], f0);
        atomicAdd(&cnt[1], f1);
        atomicAdd(&cnt[2], f2);
        atomicAdd(&cnt[3], f3);
    }
    __syncthreads();
    if (tid < nact)
        frozen_out[r0 + tid] = cnt[tid];
    if (tid == 0)
        atomicMax(passes_out, passes);
}

}  // namespace

size_t ksat_whiten_lds_bytes(int n) { return align_up((size_t)n * 2 + 2, 16); }

hipError_t ksat_launch_whiten(const KsatDev &I, const uint8_t *xs, int n_groups, int n_rep, uint8_t *white_out,
                              int32_t *frozen_out, int32_t *passes_out, hipStream_t s) {
    if (n_groups <= 0)
        return hipSuccess;
    const size_t lds = ksat_whiten_lds_bytes(I.n);
    static const hipError_t attr =
        hipFuncSetAttribute((const void *)ksat_whiten_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes - 64);
    if (attr != hipSuccess)
        return attr;
    hipLaunchKernelGGL(ksat_whiten_kernel, dim3(n_groups), dim3(1024), lds, s, I, xs, n_rep, white_out, frozen_out,
                       passes_out);
    return hipGetLastError();
}

}  // namespace nmc
