// Per-token records for the forward and backward scans (the read-after-write
// staging step), for gfx950.
//
// One workgroup handles pt consecutive tokens of one (b, h) stream.  Slot ids
// are clamped to [0, N) (a bad id is flagged, never dereferenced).  For every
// row a scan token reads, the record says where its current value lives when
// the token in flight that last modified it is still inside the scan's
// prefetch window: the forward's link is that token's row in the scan's ring
// (ring token times W plus entry); the backward's names the token and entry as
// (d << 8 | entry), d tokens away; -1 means the row is read from HBM.
//
// The slots of the window's lists go into a chained hash table in LDS (heads by
// a multiplicative hash, one 16-bit next index per entry), and one thread per
// (token, row) walks its slot's chain: one or two dependent LDS reads for
// almost every row, where a search of every candidate token's list took
// (window x log2 W) of them.  Chains are unordered (atomic exchange), so a walk
// visits all of a chain and keeps the nearest entry: the result does not depend
// on the order.  The lists need not be sorted.  The same walk finds the token's
// own entry of the slot.
#include <algorithm>

#include "sdm_common.h"
#include "sdm_internal.h"

namespace {

constexpr int THREADS = 256;

// Tokens per workgroup, a multiple of the round `per`.  A window of a few tokens
// (reach) costs small workgroups little, and the records of those scans are built
// beside a scan that fills the device: 8 tokens (6 KB of LDS at 32 rows a side) there
// take the least from it (1.4B-shaped forward with 64, 32, 16, 8 tokens: 6.13, 6.08,
// 6.02, 5.94 ms; training step 11.81, 11.74, 11.70, 11.57).  At 64 rows the backward's 8
// tokens take 12.5 KB, which the 64-row line kernel (154 KB) does not leave: those
// records wait for its workgroups to end, whatever the count above two tokens.  Deep
// windows, whose lists every workgroup enters again, take 32, or 16 with long lists.
int prep_tokens(int nrow, int reach, int per) {
    return std::max(per, reach <= 8 ? 8 : nrow <= 96 ? 32 : 16);
}

// Hash table size (log2) for n entries: between 2/3 and 4/3 heads per entry.
int hash_bits(int n) {
    int b = 4;
    while (3 << b < 2 * n) ++b;
    return b;
}
__device__ __forceinline__ int hash_slot(int slot, int bits) {
    return (int)(((uint32_t)slot * 2654435761u) >> (32 - bits));
}

__device__ __forceinline__ int clamp_slot(int s, int64_t N, unsigned int& bad) {
    if (s < 0 || s >= N) {
        bad |= 1u;
        return 0;
    }
    return s;
}

__device__ __forceinline__ void load_gates(const void* alpha, const void* beta, int in_dtype,
                                           size_t o, float& al, float& be) {
    if (in_dtype == SDM_DT_BF16) {
        al = to_f32(static_cast<const bf16_t*>(alpha)[o]);
        be = to_f32(static_cast<const bf16_t*>(beta)[o]);
    } else {
        al = static_cast<const float*>(alpha)[o];
        be = static_cast<const float*>(beta)[o];
    }
}

// Chain entry i of the table under its slot (heads start at -1).
__device__ __forceinline__ void hash_insert(int* head, short* nxt, int bits, int slot, int i) {
    nxt[i] = (short)atomicExch(&head[hash_slot(slot, bits)], i);
}

// i / d for 0 <= i < 2^16 and 0 < d, with inv = 1 / d rounded: (i + 1/2) / d is at
// least 1 / (2 d) away from a whole number, more than the rounding of the product.
__device__ __forceinline__ int small_div(int i, float inv) { return (int)(((float)i + 0.5f) * inv); }

// ---------------------------------------------------------------- forward
// Token t, row n of either list: the latest writer u of the same slot that the
// scan cannot yet see in HBM, as that writer's row in the scan's ring of
// written rows, (u mod ring) W + e, with e the position of the slot in its
// write list, so the scan reads the ring without index arithmetic.  The scan
// takes tokens in rounds of `per` and sees in HBM what rounds more than `depth`
// before its own wrote: writers from token (t / per - depth) per on are linked
// (per = 1, depth = PD - 1 for the scans that go token by token), and the ring
// holds (depth + 1) per tokens.  A read row whose slot token t itself writes
// (entry n) ends the token at alpha P + kappa_n e, with P the slot's value
// before the token, which is where the link points: its weight in the record is
// rho alpha, and the token's record holds yc = sum of rho kappa_n over such
// rows, so that y = sum rho' P + yc e needs nothing the token writes.  Records
// are made for tokens [ta, te) of each stream; writers before ta are not linked
// (a scan started at ta finds their rows in HBM).
__global__ __launch_bounds__(THREADS) void fwd_prep_kernel(
    const int32_t* __restrict__ w_idx, const float* __restrict__ w_val, const int32_t* __restrict__ r_idx,
    const float* __restrict__ r_val, const void* __restrict__ alpha, const void* __restrict__ beta, int in_dtype,
    int T, int ta, int te, int W, int R, int64_t N, unsigned char* __restrict__ recs,
    unsigned int* __restrict__ err, const float* __restrict__ gA, const float* __restrict__ gbdt, int H, int pt,
    int per_log2, int depth, int bits, int positive) {
    extern __shared__ __align__(16) int sm[];
    const FwdRec L = fwd_rec_layout(W, R);
    const int stream = blockIdx.y;
    const int t0 = ta + blockIdx.x * pt, per = 1 << per_log2;
    const int tw = max(ta, (t0 & -per) - depth * per);   // first token whose write list is needed
    const int lead = t0 - tw;                            // lists before t0's
    const int ntok = min(pt, te - t0);
    const int nw = (lead + ntok) * W;                    // entries held
    const int nrow = W + R;
    const int ring = (depth + 1) * per;
    const int MW = (R + 31) / 32;
    int* head = sm;                                                               // [1 << bits]
    int* wl = head + (1 << bits);                                                 // [pt + depth per][W]
    unsigned int* omask = reinterpret_cast<unsigned int*>(wl + (pt + depth * per) * W);   // [pt][MW]: read rows the token writes
    short* nxt = reinterpret_cast<short*>(omask + pt * MW);                       // [pt + depth per][W]
    const size_t sbase = (size_t)stream * T;
    unsigned int bad = 0u;

    for (int i = threadIdx.x; i < 1 << bits; i += THREADS) head[i] = -1;
    for (int i = threadIdx.x; i < pt * MW; i += THREADS) omask[i] = 0u;
    __syncthreads();
    for (int i = threadIdx.x; i < nw; i += THREADS) {
        const int s = clamp_slot(w_idx[(sbase + tw) * W + i], N, bad);
        wl[i] = s;
        hash_insert(head, nxt, bits, s, i);
    }
    __syncthreads();

    const float inv = 1.f / (float)nrow;
    for (int i = threadIdx.x; i < ntok * nrow; i += THREADS) {
        const int tl = small_div(i, inv), r = i - tl * nrow;
        const bool wrow = r < W;
        const size_t tok = sbase + t0 + tl;
        unsigned char* rec = recs + tok * L.bytes;
        const int own = (lead + tl) * W;   // the token's own first entry
        const int slot = wrow ? wl[own + r] : clamp_slot(r_idx[tok * R + r - W], N, bad);
        const float wt = wrow ? w_val[tok * W + r] : r_val[tok * R + r - W];
        const int lo = max(0, ((t0 + tl) & -per) - depth * per - tw) * W;
        int e = head[hash_slot(slot, bits)];
        int best = -1;
        bool self = false;
        while (e >= 0) {
            if (wl[e] == slot) {
                if (e < own && e >= lo) best = max(best, e);
                self |= (unsigned int)(e - own) < (unsigned int)W;
            }
            e = nxt[e];
        }
        short link = -1;
        if (best >= 0) {
            const int u = best / W;
            link = (short)(((tw + u) % ring) * W + best - u * W);
        }
        reinterpret_cast<short*>(rec + L.off_link)[r] = link;
        if (wrow) {
            reinterpret_cast<int*>(rec)[r] = slot;
            reinterpret_cast<float*>(rec + L.off_wval)[r] = wt;
        } else {
            const int m = r - W;
            float rho = wt;
            if (self) {   // rare: rho alpha
                float al, be;
                load_gates(alpha, beta, in_dtype, tok, al, be);
                sdm_gates_of(gA, gbdt, stream % H, al, be);
                if (positive) al = fmaxf(al, 1e-30f);
                rho *= al;
                atomicOr(&omask[tl * MW + m / 32], 1u << (m % 32));
            }
            reinterpret_cast<int*>(rec + L.off_rslot)[m] = slot;
            reinterpret_cast<float*>(rec + L.off_rval)[m] = rho;
        }
    }
    __syncthreads();

    for (int tl = threadIdx.x; tl < ntok; tl += THREADS) {
        const size_t tok = sbase + t0 + tl;
        unsigned char* rec = recs + tok * L.bytes;
        float al, be;
        load_gates(alpha, beta, in_dtype, tok, al, be);
        sdm_gates_of(gA, gbdt, stream % H, al, be);
        if (positive) {
            if (!(al > 0.f)) bad |= 2u;
            al = fmaxf(al, 1e-30f);
        }
        // yc: rho kappa_n summed over the (rare) read rows of slots the token writes, in row order
        const int own = (lead + tl) * W;
        float yc = 0.f;
        for (int wd = 0; wd < MW; ++wd) {
            for (unsigned int b = omask[tl * MW + wd]; b; b &= b - 1) {
                const int m = 32 * wd + __ffs((int)b) - 1;
                unsigned int dummy = 0u;
                const int slot = clamp_slot(r_idx[tok * R + m], N, dummy);
                int n = W;   // the token's (first) write entry of the slot
                for (int e = head[hash_slot(slot, bits)]; e >= 0; e = nxt[e])
                    if (wl[e] == slot && (unsigned int)(e - own) < (unsigned int)W) n = min(n, e - own);
                yc += r_val[tok * R + m] * w_val[tok * W + n];
            }
        }
        float* ab = reinterpret_cast<float*>(rec + L.off_ab);
        ab[0] = al;
        ab[1] = be;
        ab[2] = yc;
        if (nrow & 1) reinterpret_cast<short*>(rec + L.off_link)[nrow] = -1;
        for (int o = L.off_ab + 12; o < L.bytes; o += 4) *reinterpret_cast<int*>(rec + o) = 0;
    }
    if (bad) atomicOr(err, bad);
}

// ---------------------------------------------------------------- backward
// The backward visits t = T-1 .. 0.  For token t:
//  lm[m]  (M_t[j_m]): the earliest later writer t+d inside the window (d < PD;
//         in rounds, those of its own round and `depth` rounds before) whose undo
//         restored the row; entry n = its write position.
//  lgr[m] (G[j_m]) and lgw[n] (G[i_n]): the earliest later token t+d that
//         changed the adjoint row, either by its write adjoint (entry R + n,
//         which wins within one token: it runs after the read adjoint) or by
//         its read adjoint (entry m).  For lgw, d = 0 with a read entry means
//         this token's own read adjoint, which runs first.
// Entries of a token are its write rows, then its read rows, so the smallest
// entry index past the token's own is the nearest change, the write first.
__global__ __launch_bounds__(THREADS) void bwd_prep_kernel(
    const int32_t* __restrict__ w_idx, const float* __restrict__ w_val, const int32_t* __restrict__ r_idx,
    const float* __restrict__ r_val, const void* __restrict__ alpha, const void* __restrict__ beta, int in_dtype,
    int T, int tb, int te, int W, int R, int64_t N, unsigned char* __restrict__ recs,
    unsigned int* __restrict__ err, const float* __restrict__ gA, const float* __restrict__ gbdt, int H, int pt,
    int per_log2, int depth, int bits) {
    // records of tokens [tb, te); links only to tokens below te (the backward
    // of later tokens, in an earlier call, left its rows in HBM)
    extern __shared__ __align__(16) int sm[];
    const BwdRec L = bwd_rec_layout(W, R);
    const int stream = blockIdx.y;
    const int t0 = tb + blockIdx.x * pt;
    const int ntok = min(pt, te - t0);
    const int per = 1 << per_log2, reach = (depth + 1) * per - 1;   // tokens that a link can span
    const int span = min(pt + reach, te - t0);   // tokens t0 .. t0+span-1 (later ones included)
    const int nrow = W + R, nlink = 2 * R + W;
    int* head = sm;                                                    // [1 << bits]
    int* sl = head + (1 << bits);                                      // [pt + reach][W + R]
    short* nxt = reinterpret_cast<short*>(sl + (pt + reach) * nrow);   // [pt + reach][W + R]
    const size_t sbase = (size_t)stream * T;
    unsigned int bad = 0u;

    for (int i = threadIdx.x; i < 1 << bits; i += THREADS) head[i] = -1;
    __syncthreads();
    const float inv = 1.f / (float)nrow;
    for (int i = threadIdx.x; i < span * nrow; i += THREADS) {
        const int tl = small_div(i, inv), r = i - tl * nrow;
        const size_t tok = sbase + t0 + tl;
        const int s = clamp_slot(r < W ? w_idx[tok * W + r] : r_idx[tok * R + r - W], N, bad);
        sl[i] = s;
        hash_insert(head, nxt, bits, s, i);
    }
    __syncthreads();

    for (int i = threadIdx.x; i < ntok * nrow; i += THREADS) {
        const int tl = small_div(i, inv), r = i - tl * nrow;
        const bool wrow = r < W;
        const size_t tok = sbase + t0 + tl;
        unsigned char* rec = recs + tok * L.bytes;
        const int slot = sl[i];
        const float wt = wrow ? w_val[tok * W + r] : r_val[tok * R + r - W];
        const int own = tl * nrow, later = own + nrow;
        // the last token it links to: the start of the round `depth` rounds before its own
        const int end = min(span, tl + depth * per + ((te - 1 - (t0 + tl)) & (per - 1)) + 1) * nrow;
        int g = end, w = end, self = later;
        for (int e = head[hash_slot(slot, bits)]; e >= 0; e = nxt[e]) {
            if (sl[e] != slot) continue;
            if (e >= later && e < end) {
                g = min(g, e);
                if (e - small_div(e, inv) * nrow < W) w = min(w, e);
            } else if (e >= own + W && e < later) {
                self = min(self, e);   // this token's read adjoint
            }
        }
        auto src = [&](int e) -> short {   // (d << 8 | entry): R + n for a write row, m for a read row
            const int u = small_div(e, inv), x = e - u * nrow;
            return (short)(((u - tl) << 8) | (x < W ? R + x : x - W));
        };
        short* lk = reinterpret_cast<short*>(rec + L.off_lm);
        if (wrow) {
            lk[2 * R + r] = self < later ? (short)(self - own - W) : g < end ? src(g) : (short)-1;
            reinterpret_cast<int*>(rec)[r] = slot;
            reinterpret_cast<float*>(rec + L.off_wval)[r] = wt;
        } else {
            const int m = r - W;
            short lm = -1;
            if (w < end) {
                const int u = small_div(w, inv);
                lm = (short)(((u - tl) << 8) | (w - u * nrow));
            }
            lk[m] = lm;
            lk[R + m] = g < end ? src(g) : (short)-1;
            reinterpret_cast<int*>(rec + L.off_rslot)[m] = slot;
            reinterpret_cast<float*>(rec + L.off_rval)[m] = wt;
        }
    }
    for (int tl = threadIdx.x; tl < ntok; tl += THREADS) {
        const size_t tok = sbase + t0 + tl;
        unsigned char* rec = recs + tok * L.bytes;
        float al, be;
        load_gates(alpha, beta, in_dtype, tok, al, be);
        sdm_gates_of(gA, gbdt, stream % H, al, be);
        float* ab = reinterpret_cast<float*>(rec + L.off_ab);
        ab[0] = al;
        ab[1] = be;
        if (nlink & 1) reinterpret_cast<short*>(rec + L.off_lm)[nlink] = -1;
        for (int o = L.off_ab + 8; o < L.bytes; o += 4) *reinterpret_cast<int*>(rec + o) = 0;
    }
    if (bad) atomicOr(err, 1u);
}

}  // namespace

// Records of tokens [a.tb, a.te) for a scan that takes 1 << per_log2 tokens a
// round and keeps `depth` rounds in flight.
hipError_t sdm_launch_fwd_prep(const ScanFwdArgs& a, int per_log2, int depth, hipStream_t st) {
    const int S = a.B * a.H, per = 1 << per_log2;
    const int pt = prep_tokens(a.W + a.R, depth * per, per);
    const int lists = pt + depth * per;
    const int bits = hash_bits(lists * a.W);
    dim3 grid((a.te - a.tb + pt - 1) / pt, S);
    const size_t sm = sizeof(int) * (((size_t)1 << bits) + (size_t)lists * a.W + (size_t)pt * ((a.R + 31) / 32)) +
                      sizeof(short) * (size_t)lists * a.W;
    hipError_t e = hipFuncSetAttribute((const void*)fwd_prep_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fwd_prep_kernel, grid, dim3(THREADS), sm, st, a.w_idx, a.w_val, a.r_idx, a.r_val, a.alpha,
                       a.beta, a.in_dtype, a.T, a.tb, a.te, a.W, a.R, a.N, a.ws + SDM_WS_HEADER,
                       reinterpret_cast<unsigned int*>(a.ws), a.gate_A, a.gate_bdt, a.H, pt, per_log2, depth, bits,
                       (int)a.positive_gates);
    return hipGetLastError();
}

// Records of the backward's tokens [a.tb, a.te) for a scan that takes 1 << per_log2
// tokens a round, counted from te down, and keeps `depth` rounds in flight.
hipError_t sdm_launch_bwd_prep(const ScanBwdArgs& a, int per_log2, int depth, hipStream_t st) {
    const int S = a.B * a.H;
    const int pt = prep_tokens(a.W + a.R, depth << per_log2, 1 << per_log2);
    const int n = (pt + ((depth + 1) << per_log2) - 1) * (a.W + a.R);
    const int bits = hash_bits(n);
    dim3 grid((a.te - a.tb + pt - 1) / pt, S);
    const size_t sm = sizeof(int) * (((size_t)1 << bits) + n) + sizeof(short) * (size_t)n;
    hipError_t e = hipFuncSetAttribute((const void*)bwd_prep_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bwd_prep_kernel, grid, dim3(THREADS), sm, st, a.w_idx, a.w_val, a.r_idx, a.r_val, a.alpha,
                       a.beta, a.in_dtype, a.T, a.tb, a.te, a.W, a.R, a.N, a.ws + SDM_WS_HEADER,
                       reinterpret_cast<unsigned int*>(a.ws), a.gate_A, a.gate_bdt, a.H, pt, per_log2, depth, bits);
    return hipGetLastError();
}

// ---------------------------------------------------------------- debug id check
// One thread per (token, side): flags bit 0 if a slot id lies outside [0, N),
// bit 1 if an id repeats within the token's list (the backward's replace step
// G[i_n] = alpha Dbar_n needs distinct write ids).  Debug builds of a call
// only: O(K^2) compares per list.
namespace {
__global__ __launch_bounds__(256) void check_ids_kernel(const int32_t* __restrict__ w_idx, int W,
                                                        const int32_t* __restrict__ r_idx, int R,
                                                        int64_t ntok, int64_t N, unsigned int* __restrict__ flag) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * ntok) return;
    const bool wside = i < ntok;
    const int K = wside ? W : R;
    const int32_t* lst = wside ? w_idx + i * W : r_idx + (i - ntok) * R;
    unsigned int bad = 0u;
    for (int a = 0; a < K; ++a) {
        const int32_t s = lst[a];
        if (s < 0 || s >= N) bad |= 1u;
        for (int b = a + 1; b < K; ++b)
            if (lst[b] == s) bad |= 2u;
    }
    if (bad) atomicOr(flag, bad);
}
}  // namespace

hipError_t sdm_launch_check_ids(const int32_t* w_idx, int W, const int32_t* r_idx, int R, int64_t ntok,
                                int64_t N, unsigned int* flag, hipStream_t st) {
    const int64_t n = 2 * ntok;
    const unsigned int blocks = (unsigned int)((n + 255) / 256);
    hipLaunchKernelGGL(check_ids_kernel, dim3(blocks), dim3(256), 0, st, w_idx, W, r_idx, R, ntok, N, flag);
    return hipGetLastError();
}
