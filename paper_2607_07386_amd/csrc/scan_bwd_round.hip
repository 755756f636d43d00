// Backward scan in rounds of tokens (App. A.3's undo), for launches with few
// streams and for list lengths the line-cooperative backward (scan_bwd.hip) does
// not take, gfx950.  The geometry is the forward's (scan_round.hip): a workgroup
// owns 32 columns of one stream, its NWV waves take one token each, from the end
// of the sequence down, and the rows of a wave's next D tokens are in flight.
// Per token (the arithmetic of scan_bwd.hip):
//   rbar_m = <dy, M_t[j_m]>;  G[j_m] += rho_m dy;  then with g_n = G[i_n]
//   ebar = sum kappa_n g_n, dv = beta ebar, and kbar, dbeta, dalpha,
//   G[i_n] = alpha (g_n - beta kappa_n ebar), M[i_n] = P_n.
//  * A memory row that a token in flight has undone holds that token's saved row
//    (the record names token and entry): it is loaded from the undo log itself,
//    which nothing writes.
//  * An adjoint row that a token in flight has changed is taken from an LDS ring of
//    (D + 1) NWV tokens' R + W adjoint rows; a token linked to one of its own
//    round waits for that wave, on a per-wave LDS counter (waves wait on
//    lower-numbered waves only, so every wait ends).
//  * A write row whose slot the token also reads starts from its own read adjoint
//    (the ring again), and its store follows the read row's from the same wave.
// Partial scalars go out per workgroup (32 columns), as the line kernel's.
// What bounds it: as the forward, the issue of a token's operations by one wave
// (7 K row loads and stores) and a compute unit's loads in flight; with small
// tables the chain of tokens that share slots.  2048 tokens, d_v = 128, N = 65536,
// line or per-wave kernel against this one, us: 1 stream top-32 2414 / 933; 16
// streams top-8 2503 / 585, top-16 2596 / 975, top-32 2470 / 1781, top-64 4153 /
// 3625.  Taking the sums that need no adjoint row (rbar, the read-back) before the
// wait for linked rows gained nothing where tokens chain (1489 against 1467 us for
// 777 tokens, 10,000 slots, lists of 48 and 24) and lost elsewhere (top-64 3625
// against 3924), so the sums of both are taken together.
#include <algorithm>

#include "sdm_common.h"
#include "sdm_internal.h"
#include "sdm_reduce.h"
#include "sdm_round.h"
#include "sdm.h"

namespace {

constexpr int CW = RND_CW, CQ = RND_CQ, RG = RND_RG;
constexpr uint32_t OOB = RND_OOB;
constexpr int LDS_LIMIT = 160 * 1024;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int K>
constexpr int brec_chunks() {   // 16-byte record chunks per lane, for records of W, R <= 8 K
    return ((22 * RG * K + 8 + 15) / 16 + SDM_WAVE - 1) / SDM_WAVE;
}

__device__ __forceinline__ void st_buf(__amdgpu_buffer_rsrc_t rs, uint32_t o, v4f v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, (int)o, 0, 0);
}
__device__ __forceinline__ v4f ld_buf(__amdgpu_buffer_rsrc_t rs, uint32_t o) {
    return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)o, 0, 0));
}
// Sum over the 8 lanes of a row, in each of them.
__device__ __forceinline__ float quads_sum(float v) {
    v += sdm_reduce::xor_dpp<1>(v);
    v += sdm_reduce::xor_dpp<2>(v);
    return v + sdm_reduce::xor_dpp<4>(v);
}

template <typename VT, int NWV, int D, int K, bool EX>
__global__ __launch_bounds__(NWV * SDM_WAVE) void scan_bwd_round_kernel(
    const unsigned char* __restrict__ recs, const VT* __restrict__ v, float* __restrict__ mem,
    const float* __restrict__ saved, const float* __restrict__ dy, float* __restrict__ Gtab,
    float* __restrict__ dv_out, float* __restrict__ part, int T, int tb, int te, int dv, int W_, int R_, int64_t N,
    int groups, int S) {
    constexpr int NREC = D + 2, RING = (D + 1) * NWV, NC = brec_chunks<K>();
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / SDM_WAVE);
    int group, stream;
    scan_wg_coords<true>(groups, group, stream);

    RoundLane<K, EX> c;
    const int W = EX ? RG * K : W_, R = EX ? RG * K : R_, RW = R + W;
    const BwdRec L = bwd_rec_layout(W, R);
    c.rg = lane / CQ;
    c.cq = lane % CQ;
    const int col_raw = group * CW + c.cq * 4;
    c.colok = EX || col_raw < dv;
    const int col = c.colok ? col_raw : dv - 4;
    c.dv4 = (uint32_t)dv * 4;
    c.lc4 = (uint32_t)col * 4;

    extern __shared__ __align__(16) unsigned char smem[];
    int* prog = reinterpret_cast<int*>(smem);                                      // rounds done, per wave
    unsigned char* rring = smem + 64 + (size_t)w * NREC * L.bytes;                 // this wave's records
    float* gring = reinterpret_cast<float*>(smem + 64 + (size_t)NWV * NREC * L.bytes);   // [RING][R + W][CW]

    const size_t table = (size_t)stream * N * dv;
    const __amdgpu_buffer_rsrc_t mrs = __builtin_amdgcn_make_buffer_rsrc(mem + table, 0, (int)((size_t)N * dv * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t grs = __builtin_amdgcn_make_buffer_rsrc(Gtab + table, 0, (int)((size_t)N * dv * 4), 0x00020000);
    const unsigned char* srec = recs + (size_t)stream * T * L.bytes;
    const float* mcol = mem + table + col;
    const float* ss = saved + (size_t)stream * T * W * dv;
    const size_t row0 = (size_t)stream * T * dv;
    float* spart = part + ((size_t)group * S + stream) * T * (RW + 2);

    if (threadIdx.x < NWV) prog[threadIdx.x] = 0;

    // Step i = r NWV + w of the wave in round r processes token te - 1 - i.
    auto token = [&](int r) { return max(te - 1 - (r * NWV + w), tb); };
    auto rec_load = [&](u4v (&st)[NC], int r) {
        const u4v* src = reinterpret_cast<const u4v*>(srec + (size_t)token(r) * L.bytes);
#pragma unroll
        for (int j = 0; j < NC; ++j) st[j] = src[min(lane + j * SDM_WAVE, L.bytes / 16 - 1)];
    };
    auto rec_store = [&](const u4v (&st)[NC], int slot) {
        u4v* dst = reinterpret_cast<u4v*>(rring + slot * L.bytes);
#pragma unroll
        for (int j = 0; j < NC; ++j)
            if (lane + j * SDM_WAVE < L.bytes / 16) dst[lane + j * SDM_WAVE] = st[j];
    };
    v4f Mr[D][K], Gr[D][K], Gw[D][K], Ps[D][K], Dy[D];
    uint2 vb[D], vb2[D];   // v: bf16 four values, fp32 two and two
    auto issue = [&](int j, int r, int slot) {
        const unsigned char* rec = rring + slot * L.bytes;
        const int t = token(r);
        int sw[K], sr[K], lm[K];
        c.words(rec, W, sw);
        c.words(rec + L.off_rslot, R, sr);
        c.links(rec + L.off_lm, R, lm);
        const __amdgpu_buffer_rsrc_t srs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(ss) + (size_t)t * W * dv, 0, W * dv * 4, 0x00020000);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            // the row as M_t: the saved row of the token in flight that undid it, or the table's
            const size_t from = ((size_t)(t + (lm[k] >> 8)) * W + (lm[k] & 255)) * dv + col;
            Mr[j][k] = ld4(lm[k] >= 0 ? ss + from : mcol + (size_t)sr[k] * dv);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) Gr[j][k] = ld_buf(grs, c.off(sr[k], c.rg * K + k < R));
#pragma unroll
        for (int k = 0; k < K; ++k) Gw[j][k] = ld_buf(grs, c.off(sw[k], c.rg * K + k < W));
#pragma unroll
        for (int k = 0; k < K; ++k) Ps[j][k] = ld_buf(srs, c.off(c.rg * K + k, c.rg * K + k < W));
        Dy[j] = ld4(dy + row0 + (size_t)t * dv + col);
        const uint2* pv = reinterpret_cast<const uint2*>(v + row0 + (size_t)t * dv + col);
        vb[j] = pv[0];
        if constexpr (sizeof(VT) == 4) vb2[j] = pv[1];
    };

    const int rounds = (te - tb + NWV - 1) / NWV;
    u4v st[NC];
#pragma unroll
    for (int r = 0; r <= D; ++r) {
        rec_load(st, r);
        rec_store(st, r);
    }
    rec_load(st, D + 1);
#pragma unroll
    for (int j = 0; j < D; ++j) {
        __builtin_amdgcn_sched_barrier(0);   // in the order that the rounds wait for them
        issue(j, j, j);
    }
    __builtin_amdgcn_sched_barrier(0);

    // One round; as in the forward, no vector-memory operation is conditional.
    int cur = 0, nxt = D, q0 = 0;   // record slots of rounds r and r + D, ring token of the round's first step
    auto round = [&](int j, int r) {
        __syncthreads();   // stores and ring rows of rounds before r are in place
        const int t = te - 1 - (r * NWV + w);
        const bool tok = t >= tb;   // else: token tb again, nothing stored
        const unsigned char* rec = rring + cur * L.bytes;
        const float al = reinterpret_cast<const float*>(rec + L.off_ab)[0];
        const float be = reinterpret_cast<const float*>(rec + L.off_ab)[1];
        int lr[K], lw[K], sw[K], sr[K];
        float kap[K], rho[K];
        c.links(rec + L.off_lgr, R, lr);
        c.links(rec + L.off_lgw, W, lw);
        c.floats(rec + L.off_wval, W, kap);
        c.floats(rec + L.off_rval, R, rho);
        c.words(rec, W, sw);
        c.words(rec + L.off_rslot, R, sr);
        int all = -1, own = -1;   // sign clear: some link / some link to the token's own read rows
#pragma unroll
        for (int k = 0; k < K; ++k) {
            all &= lr[k] & (lw[k] >= 256 ? lw[k] : -1);
            own &= lw[k] < 256 ? lw[k] : -1;
        }
        auto ring_row = [&](int l) -> const float* {   // (d << 8 | entry): d steps back
            int q = q0 + w - (l >> 8);
            q = q < 0 ? q + RING : q;
            return gring + ((size_t)q * RW + min(l & 255, RW - 1)) * CW + c.cq * 4;
        };
        if (__builtin_amdgcn_ballot_w64(all >= 0)) {
            int top = -1;   // highest wave of this round that a row comes from
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (lr[k] >= 0) top = max(top, w - (lr[k] >> 8));
                if (lw[k] >= 256) top = max(top, w - (lw[k] >> 8));
            }
            for (int i = 0; i < w; ++i) {
                if (!__builtin_amdgcn_ballot_w64(top >= i)) break;
                while (__hip_atomic_load(&prog[i], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) <= r)
                    __builtin_amdgcn_s_sleep(1);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (lr[k] >= 0) Gr[j][k] = ld4(ring_row(lr[k]));
                if (lw[k] >= 256) Gw[j][k] = ld4(ring_row(lw[k]));
            }
        }
        const uint32_t lc = tok ? c.lc4 : OOB;
        const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc(
            spart + (size_t)max(t, tb) * (RW + 2), 0, tok ? (RW + 2) * 4 : 0, 0x00020000);
        const v4f yb = Dy[j];
        float* gr = gring + (size_t)(q0 + w) * RW * CW + c.cq * 4;
        // ---- read adjoint ----
        float out = 0.f;   // this lane's partial scalar: row rg K + cq (cq < K)
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int m = c.rg * K + k;
            const bool ok = EX || m < R;
            const float rb = quads_sum(c.colok ? v4dot(yb, Mr[j][k]) : 0.f);
            out = c.cq == k ? rb : out;
            const v4f g = v4fma(rho[k], yb, Gr[j][k]);
            if (ok) st4(gr + m * CW, g);
            st_buf(grs, ok && c.colok ? __umul24((uint32_t)sr[k], c.dv4) + lc : OOB, g);
        }
        const int prow = c.rg * K + c.cq;   // partial scalars of rows: one word per lane of the first K of a row
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(out), prs,
                                              (int)(c.cq < K && prow < R ? (uint32_t)prow * 4 : OOB), 0, 0);
        if (__builtin_amdgcn_ballot_w64(own >= 0)) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (lw[k] >= 0 && lw[k] < 256) Gw[j][k] = ld4(gr + lw[k] * CW);
        }
        // ---- write adjoint ----
        v4f Dk[K], up = v4zero(), eb = v4zero();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            Dk[k] = al * Ps[j][k];
            up = v4fma(kap[k], Dk[k], up);
            eb = v4fma(kap[k], Gw[j][k], eb);
        }
        sdm_reduce::rows_allreduce8<CQ>(up, eb);
        v4f vv;
        if constexpr (sizeof(VT) == 2)
            vv = v4f{bf16_lo(vb[j].x), bf16_hi(vb[j].x), bf16_lo(vb[j].y), bf16_hi(vb[j].y)};
        else
            vv = v4f{__uint_as_float(vb[j].x), __uint_as_float(vb[j].y), __uint_as_float(vb2[j].x),
                     __uint_as_float(vb2[j].y)};
        const v4f vmu = vv - up, e = be * vmu;
        out = 0.f;
        float ab = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int n = c.rg * K + k;
            const bool ok = EX || n < W;
            const float kb = quads_sum(c.colok ? v4dot(Gw[j][k], e) - be * v4dot(eb, Dk[k]) : 0.f);
            out = c.cq == k ? kb : out;
            const v4f Db = v4fma(-be * kap[k], eb, Gw[j][k]);
            ab += ok && c.colok ? v4dot(Db, Ps[j][k]) : 0.f;
            const v4f gn = al * Db;
            const uint32_t o = ok && c.colok ? __umul24((uint32_t)sw[k], c.dv4) + lc : OOB;
            if (ok) st4(gr + (R + n) * CW, gn);
            st_buf(grs, o, gn);
            st_buf(mrs, o, Ps[j][k]);
        }
        __hip_atomic_store(&prog[w], r + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(out), prs,
                                              (int)(c.cq < K && prow < W ? (uint32_t)(R + prow) * 4 : OOB), 0, 0);
        const float bb = quads_sum(c.colok ? v4dot(eb, vmu) : 0.f);
        ab = sdm_reduce::wave_sum(ab);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(lane ? ab : bb), prs,
                                              (int)(lane < 2 ? (uint32_t)(RW + lane) * 4 : OOB), 0, 0);
        const __amdgpu_buffer_rsrc_t drs = __builtin_amdgcn_make_buffer_rsrc(
            dv_out + row0 + (size_t)max(t, tb) * dv, 0, dv * 4, 0x00020000);
        st_buf(drs, c.rg == 0 && c.colok ? lc : OOB, be * eb);
        nxt = nxt + 1 == NREC ? 0 : nxt + 1;
        rec_store(st, nxt);
        rec_load(st, r + D + 2);
        __builtin_amdgcn_sched_barrier(0);
        issue(j, r + D, nxt == 0 ? NREC - 1 : nxt - 1);
        __builtin_amdgcn_sched_barrier(0);
        cur = cur + 1 == NREC ? 0 : cur + 1;
        q0 = q0 + NWV == RING ? 0 : q0 + NWV;
    };
    for (int r = 0; r < rounds; r += D) {   // up to D - 1 empty rounds at the end
#pragma unroll
        for (int j = 0; j < D; ++j) round(j, r + j);
    }
}

// Geometry by rows per lane: a token in flight holds 16 K + 4 registers, its
// adjoint rows (R + W) 128 bytes of ring.  Half the waves with twice the depth: 16
// streams top-32 1759 against 1781 us, top-64 (2 waves) 4155 against 3625, 128 streams
// top-8 2362 against 1927; less depth was slower throughout.
struct BRoundPlan {
    int K, nwv, depth, lds;
    bool ex;
};
template <int K>
struct BRoundCfg {
    static constexpr int NWV = K == 8 ? 4 : 8, D = K <= 2 ? 2 : 1;
};
template <int K>
bool bplan_k(const ScanBwdArgs& a, BRoundPlan* p) {
    using C = BRoundCfg<K>;
    p->K = K;
    p->nwv = C::NWV;
    p->depth = C::D;
    p->ex = a.W == RG * K && a.R == RG * K && a.dv % CW == 0;
    p->lds = 64 + C::NWV * (C::D + 2) * bwd_rec_layout(a.W, a.R).bytes + (C::D + 1) * C::NWV * (a.W + a.R) * CW * 4;
    return p->lds <= LDS_LIMIT;
}

int bround_groups(const ScanBwdArgs& a) { return (a.dv + CW - 1) / CW; }

bool bround_plan(const ScanBwdArgs& a, BRoundPlan* p) {
    if (a.dv < CW) return false;
    // the tables' 32-bit row offsets and 24-bit multiplies
    if ((size_t)a.N * a.dv * 4 >= ((size_t)1 << 31) || a.N >= (1 << 24)) return false;
    const int m = std::max(a.W, a.R);
    if (m > RG * 8) return false;
    if (m <= RG) return bplan_k<1>(a, p);
    if (m <= RG * 2) return bplan_k<2>(a, p);
    if (m <= RG * 4) return bplan_k<4>(a, p);
    return bplan_k<8>(a, p);
}

template <typename VT, int K, bool EX>
hipError_t launch_bround(const ScanBwdArgs& a, const BRoundPlan& p, float* part, hipStream_t st) {
    using C = BRoundCfg<K>;
    auto kfn = scan_bwd_round_kernel<VT, C::NWV, C::D, K, EX>;
    hipError_t e = hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, p.lds);
    if (e != hipSuccess) return e;
    const int groups = bround_groups(a), S = a.B * a.H;
    hipLaunchKernelGGL(kfn, dim3(groups * S), dim3(C::NWV * SDM_WAVE), p.lds, st, a.ws + SDM_WS_HEADER,
                       static_cast<const VT*>(a.v), a.mem, a.saved, a.dy, a.G, a.dv_out, part, a.T, a.tb, a.te, a.dv,
                       a.W, a.R, a.N, groups, S);
    return hipGetLastError();
}

template <typename VT>
hipError_t launch_bround_k(const ScanBwdArgs& a, const BRoundPlan& p, float* part, hipStream_t st) {
    switch (p.K) {
        case 1: return p.ex ? launch_bround<VT, 1, true>(a, p, part, st) : launch_bround<VT, 1, false>(a, p, part, st);
        case 2: return p.ex ? launch_bround<VT, 2, true>(a, p, part, st) : launch_bround<VT, 2, false>(a, p, part, st);
        case 4: return p.ex ? launch_bround<VT, 4, true>(a, p, part, st) : launch_bround<VT, 4, false>(a, p, part, st);
        default: return p.ex ? launch_bround<VT, 8, true>(a, p, part, st) : launch_bround<VT, 8, false>(a, p, part, st);
    }
}

}  // namespace

// Which backward launches go in rounds: as the forward's (round_faster in
// scan_round.hip), with its reasons.  The line-cooperative kernel keeps lists of 32
// or 64 rows from half the device's compute units on (128 workgroups of top-32: 2547
// us by the line kernel, 2138 here; 256: equal within the step's noise) and on tables
// whose tokens chain (256 tokens, 16 streams, top-32: N = 2048 332 / 340 us, 2925 332 /
// 310; 4 streams, top-64: N = 8192 529 / 567, 11,702 527 / 526, 16,384 529 / 479).  Other
// lists have the per-wave kernel (2048 tokens, N = 65536, 128 streams: top-8 3132 /
// 1927, top-16 5124 / 3608, top-48 13,768 / 10,716), which wins on dense tables; here
// read rows' adjoints link tokens as well, so that the slots that two tokens share go
// with (W + R)^2 / N.  Its time over this kernel's by that (d_v = 128; limits in
// brackets):
//   16 streams   top-16: 8 1.15, 1 1.50; top-24: 8 0.81, 1.4 0.96, 1 1.05 [1]
//                top-48: 2 0.76, 0.7 1.08, 0.5 1.17; write 48, read 24: 0.6 0.94, 0.5 1.00
//                [3/5] (4 streams 0.97 and 0.88 at 0.6, 60 streams 1.77 and 1.16)
//   128 streams  top-12: 2 0.72, 0.5 1.10; top-16: 8 0.72, 2 1.00, 1 1.12 [1]
//                top-24: 8 0.75, 1 1.04; top-40: 1 0.84, 0.7 1.03; top-48: 2 0.92, 1 1.11 [3/4]
//   512 streams  top-24: 8 0.75, 1 1.03; top-40: 2 0.77, 0.7 1.01, 0.5 1.09; top-48: 1 1.08
//   rows that end inside a line, 256 streams: d_v = 36 top-24 2 1.23, 1 1.55, top-48 2 1.26,
//                1.4 1.37; d_v = 68 top-24 2 1.16, top-48 2 1.24 [2, 3/2]; but 512 streams of
//                d_v = 36, whose second column group is nearly empty, top-48: 1.1 0.77
bool sdm_bwd_round(const ScanBwdArgs& a) {
    BRoundPlan p;
    if (!sdm_line_io_enabled() || sdm_scan_slice_width() || sdm_scan_prefetch()) return false;
    if (!bround_plan(a, &p)) return false;
    const int64_t cus = sdm_device_simds() / 4, wgs = (int64_t)a.B * a.H * bround_groups(a);
    const int64_t pairs = (int64_t)a.W * (a.W + a.R), links = (int64_t)(a.W + a.R) * (a.W + a.R);
    const int m = std::max(a.W, a.R);
    if (a.W == a.R && (m == 32 || m == 64) && a.dv % 32 == 0)
        return wgs <= cus / 2 && 2 * a.N >= (m == 32 ? 3 : 4) * pairs;
    if (m <= RG) return true;
    if (m <= RG * 2) return wgs <= cus || a.N >= links;
    const int ragged = a.dv % CW && wgs > cus && (a.dv > 2 * CW || wgs < 4 * cus) ? 2 : 1;
    if (m <= RG * 4) return ragged * a.N >= links;
    return 3 * ragged * a.N >= (wgs <= cus ? 5 : 4) * links;
}
int sdm_bwd_round_parts(const ScanBwdArgs& a) { return bround_groups(a); }

hipError_t sdm_launch_bwd_round_prep(const ScanBwdArgs& a, hipStream_t st) {
    BRoundPlan p;
    if (!bround_plan(a, &p)) return hipErrorInvalidConfiguration;
    return sdm_launch_bwd_prep(a, __builtin_ctz((unsigned)p.nwv), p.depth, st);
}

hipError_t sdm_launch_bwd_round(const ScanBwdArgs& a, float* part, hipStream_t st) {
    BRoundPlan p;
    if (!bround_plan(a, &p)) return hipErrorInvalidConfiguration;
    return a.in_dtype == SDM_DT_BF16 ? launch_bround_k<bf16_t>(a, p, part, st) : launch_bround_k<float>(a, p, part, st);
}
