// A lane's share of a token in the scans that go in rounds of tokens
// (scan_round.hip, scan_bwd_round.hip): 32 columns per workgroup, 8 lanes per row
// of 16 bytes each, K consecutive rows per lane.  gfx950, wave64.
#pragma once

#include "sdm_common.h"

constexpr int RND_CW = 32;                    // columns per workgroup: one 128-byte line
constexpr int RND_CQ = RND_CW / 4;            // lanes per row
constexpr int RND_RG = SDM_WAVE / RND_CQ;     // row groups: rows rg K .. rg K + K - 1 per lane
constexpr uint32_t RND_OOB = 0x80000000u;     // past every table (below 2 GiB): loads give 0, stores are dropped

// EX: lists of exactly 8 K entries and whole lines of columns.
template <int K, bool EX>
struct RoundLane {
    int rg, cq;
    uint32_t dv4, lc4;      // row pitch and this lane's column offset, bytes
    bool colok;

    __device__ __forceinline__ uint32_t off(int slot, bool ok) const {
        const uint32_t o = __umul24((uint32_t)slot, dv4) + lc4;
        return EX ? o : (ok && colok ? o : RND_OOB);
    }
    // K consecutive 32-bit words of a list of n starting at row rg K (EX: n = 8 K, 16-byte aligned)
    __device__ __forceinline__ void words(const unsigned char* list, int n, int (&out)[K]) const {
        if constexpr (EX && K % 4 == 0) {
#pragma unroll
            for (int j = 0; j < K / 4; ++j) {
                const u4v x = *reinterpret_cast<const u4v*>(list + (rg * K + 4 * j) * 4);
#pragma unroll
                for (int i = 0; i < 4; ++i) out[4 * j + i] = (int)x[i];
            }
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) out[k] = reinterpret_cast<const int*>(list)[min(rg * K + k, n - 1)];
        }
    }
    __device__ __forceinline__ void floats(const unsigned char* list, int n, float (&out)[K]) const {
        int x[K];
        words(list, n, x);
#pragma unroll
        for (int k = 0; k < K; ++k) out[k] = (EX || rg * K + k < n) ? __int_as_float(x[k]) : 0.f;
    }
    __device__ __forceinline__ void links(const unsigned char* list, int n, int (&out)[K]) const {
        if constexpr (EX && K % 4 == 0) {
#pragma unroll
            for (int j = 0; j < K / 4; ++j) {
                const u2v x = *reinterpret_cast<const u2v*>(list + (rg * K + 4 * j) * 2);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    out[4 * j + 2 * i] = (int)(short)(x[i] & 0xffffu);
                    out[4 * j + 2 * i + 1] = (int)x[i] >> 16;
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int n0 = rg * K + k;
                out[k] = reinterpret_cast<const short*>(list)[min(n0, n - 1)];
                if (n0 >= n) out[k] = -1;
            }
        }
    }
};
