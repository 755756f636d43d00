// Forward sparse gated-delta scan in rounds of tokens (Sec. 3.1 steps 2-3), for
// launches with few streams and for list lengths the line-cooperative kernel
// (scan_fwd.hip) does not take, gfx950.
//
// With few streams the scan is bound by how long each stream's token takes, not
// by bandwidth.  The line-cooperative kernel gives every token to all four waves
// of a workgroup and exchanges the rows' pieces through LDS, two barriers and
// about six dependent LDS round trips a token: 0.52 us.  But tokens that share no
// slot are independent, and with large tables most tokens in flight share none.
// Here a workgroup owns 32 columns (a 128-byte line of every row) of one stream,
// and its NWV waves take one token each, a round of NWV tokens at a time:
//  * a wave holds all rows of its token: 8 lanes per row (16 bytes each), K rows
//    per lane, so the sums over rows are K in-lane steps and three lane
//    exchanges, and rows go between HBM and registers as whole lines with no
//    exchange through LDS;
//  * the rows of the wave's next D tokens are in flight (D rounds);
//  * written rows also go to an LDS ring of (D + 1) NWV tokens.  A row written by
//    a token whose store the load could not see (same or the D rounds before;
//    the prep kernel links exactly those) is taken from the ring;
//  * one workgroup barrier per round orders rounds: loads issued in round r see
//    the stores of rounds before r, and a ring slot is reused D + 1 rounds later.
//    Only a token linked to one of its own round waits for that wave, on a
//    per-wave LDS counter; waves wait on lower-numbered waves only, so the wave
//    of the round's first token never waits and every wait ends;
//  * per-token records are private to the wave (it alone reads its tokens').
// Read rows are taken before the write, as in scan_fwd.hip: y = sum rho' P + yc e.
//
// What bounds it: with one stream 0.20 us a token and workgroup, the issue of
// about 250 instructions and 14 vector-memory operations by two waves per SIMD
// (0.18 with every row load and store out of bounds).  With more streams a
// compute unit's loads in flight: deeper prefetch (D = 3), other round lengths
// (4 x 4, 16 x 1), cache policies of the loads and issuing them at the round's
// start changed nothing or lost, while all rows from L2 took 0.21 us where HBM
// gave 0.37 (16 streams x 4 groups).  So where compute units are left over,
// helper workgroups touch the rows' lines a little ahead of the main workgroup,
// from the same XCD: the lines are then in its L2.  16 streams of 2048 tokens
// (top-32, d_v = 128, N = 65536): 1112 us by the line kernel, 762 here, 551 with
// two helpers per workgroup; 16 x 65,536 tokens (N = 262,144): 34.4, 24.4 and
// 16.0 ms; two heads of d_v = 1920, top-64 (4096 tokens): 3.60, 3.23, 2.74 ms.
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
constexpr int rec_chunks() {   // 16-byte record chunks per lane, for records of W, R <= 8 K
    return ((20 * RG * K + 12 + 15) / 16 + SDM_WAVE - 1) / SDM_WAVE;
}

template <int NWV, int D>
struct RoundGeom {
    static constexpr int NREC = D + 2;           // records held per wave
    static constexpr int RING = (D + 1) * NWV;   // tokens of written rows held
};

__host__ __device__ inline int round_lds(int nwv, int nrec, int ring, int rec_bytes, int W) {
    return 64 + nwv * nrec * rec_bytes + ring * W * CW * 4;
}

// A helper workgroup: touches one word of every line that its main workgroup
// will load, for tokens at most `lead` past those the main workgroup has done
// (further ahead they would leave the L2 again before they are used).  It only
// reads, and what it reads is dropped: whether it keeps up, runs late or stops
// changes no result.  `progress` (rounds done, written by the main workgroup) is
// waited for a bounded time only.
template <int NWV>
__device__ __forceinline__ void round_helper(const float* tab, int dv, int64_t N, const int32_t* wi, const int32_t* ri,
                                             int W, int R, int tb, int te, const int* progress, int h, int helpers,
                                             int lead, int w, int lane) {
    constexpr int U = 2;          // tokens per batch
    constexpr int SPINS = 4000;   // about a microsecond each
    const int step = helpers * NWV * U;
    int done = 0;
    auto slot_of = [&](int t, int i) -> int {
        const int tt = min(t, te - 1);
        const int r = min(i, W + R - 1);
        const int s = r < W ? wi[(size_t)tt * W + r] : ri[(size_t)tt * R + r - W];
        return (uint64_t)s < (uint64_t)N ? s : 0;
    };
    const bool two = W + R > SDM_WAVE;   // rows per lane (W + R <= 128)
    int sl[U][2];
    int t0 = tb + (h * NWV + w) * U;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        sl[u][0] = slot_of(t0 + u, lane);
        sl[u][1] = slot_of(t0 + u, lane + SDM_WAVE);
    }
    for (; t0 < te; t0 += step) {
        for (int spin = 0; t0 > done + lead; ++spin) {
            if (spin == SPINS) return;
            done = tb + NWV * __hip_atomic_load(progress, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (t0 > done + lead) __builtin_amdgcn_s_sleep(8);
        }
        float x[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[u][0] = tab[(size_t)sl[u][0] * dv];
            x[u][1] = two ? tab[(size_t)sl[u][1] * dv] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            sl[u][0] = slot_of(t0 + step + u, lane);
            sl[u][1] = slot_of(t0 + step + u, lane + SDM_WAVE);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) asm volatile("" ::"v"(x[u][0]), "v"(x[u][1]));
    }
}

template <typename VT, int NWV, int D, int K, bool EX, bool SAVE>
__global__ __launch_bounds__(NWV * SDM_WAVE) void scan_fwd_round_kernel(
    const unsigned char* __restrict__ recs, const VT* __restrict__ v, float* __restrict__ mem,
    float* __restrict__ y, float* __restrict__ saved, int T, int tb, int te, int dv, int W_, int R_, int64_t N,
    int groups, int S, const int32_t* __restrict__ w_idx, const int32_t* __restrict__ r_idx, int helpers, int lead,
    unsigned char* progress) {
    using Geo = RoundGeom<NWV, D>;
    constexpr int NC = rec_chunks<K>();
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / SDM_WAVE);
    // Block -> (main or helper, group, stream).  Blocks go to the 8 XCDs round-robin,
    // so a helper's block is its main's plus a multiple of 8 (and later: mains are
    // dispatched first), and the groups of a stream share an XCD where S allows.
    const int nmain = groups * S, nrnd = (nmain + 7) & ~7;
    const int main = (int)blockIdx.x % nrnd, role = (int)blockIdx.x / nrnd;
    if (main >= nmain) return;
    const bool local = S % 8 == 0;
    const int stream = local ? (main >> 3) / groups * 8 + (main & 7) : main / groups;
    const int group = local ? (main >> 3) % groups : main % groups;
    const int W = EX ? RG * K : W_, R = EX ? RG * K : R_;
    const FwdRec L = fwd_rec_layout(W, R);
    // rounds done: the spare last word of the record of token tb + group, which the prep kernel cleared
    unsigned char* const done = progress + ((size_t)stream * T + tb + group + 1) * L.bytes - 4;
    if (role) {
        round_helper<NWV>(mem + (size_t)stream * N * dv + group * CW, dv, N, w_idx + (size_t)stream * T * W,
                          r_idx + (size_t)stream * T * R, W, R, tb, te, reinterpret_cast<const int*>(done), role - 1,
                          helpers, lead, w, lane);
        return;
    }
    __builtin_amdgcn_s_setprio(3);   // latency-bound: first at each issue slot beside the addressing

    RoundLane<K, EX> c;
    c.rg = lane / CQ;
    c.cq = lane % CQ;
    const int col_raw = group * CW + c.cq * 4;
    c.colok = EX || col_raw < dv;
    const int col = c.colok ? col_raw : dv - 4;
    c.dv4 = (uint32_t)dv * 4;
    c.lc4 = (uint32_t)col * 4;

    extern __shared__ __align__(16) unsigned char smem[];
    int* prog = reinterpret_cast<int*>(smem);                                  // rounds done, per wave
    unsigned char* rring = smem + 64 + (size_t)w * Geo::NREC * L.bytes;        // this wave's records
    float* fring = reinterpret_cast<float*>(smem + 64 + (size_t)NWV * Geo::NREC * L.bytes);   // [RING][W][CW]

    const __amdgpu_buffer_rsrc_t trs = __builtin_amdgcn_make_buffer_rsrc(
        mem + (size_t)stream * N * dv, 0, (int)((size_t)N * dv * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc(
        y + (size_t)stream * T * dv, 0, (int)((size_t)T * dv * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc(done, 0, helpers ? 4 : 0, 0x00020000);
    const unsigned char* srec = recs + (size_t)stream * T * L.bytes;
    const VT* sv = v + (size_t)stream * T * dv + col;
    float* ss = SAVE ? saved + (size_t)stream * T * W * dv : nullptr;

    if (threadIdx.x < NWV) prog[threadIdx.x] = 0;

    // records of this wave's token of round r
    auto rec_load = [&](u4v (&st)[NC], int r) {
        const int t = min(tb + r * NWV + w, te - 1);
        const u4v* src = reinterpret_cast<const u4v*>(srec + (size_t)t * L.bytes);
#pragma unroll
        for (int j = 0; j < NC; ++j) st[j] = src[min(lane + j * SDM_WAVE, L.bytes / 16 - 1)];
    };
    auto rec_store = [&](const u4v (&st)[NC], int slot) {
        u4v* dst = reinterpret_cast<u4v*>(rring + slot * L.bytes);
#pragma unroll
        for (int j = 0; j < NC; ++j)
            if (lane + j * SDM_WAVE < L.bytes / 16) dst[lane + j * SDM_WAVE] = st[j];
    };
    v4f Pw[D][K], Pr[D][K];
    uint2 vb[D];     // bf16: the four values; fp32: the first two ...
    uint2 vb2[D];    // ... and the last two
    auto issue = [&](int j, int r, int slot) {
        const unsigned char* rec = rring + slot * L.bytes;
        int sw[K], sr[K];
        c.words(rec, W, sw);
        c.words(rec + L.off_rslot, R, sr);
#pragma unroll
        for (int k = 0; k < K; ++k)
            Pw[j][k] = __builtin_bit_cast(
                v4f, __builtin_amdgcn_raw_buffer_load_b128(trs, (int)c.off(sw[k], c.rg * K + k < W), 0, 0));
#pragma unroll
        for (int k = 0; k < K; ++k)
            Pr[j][k] = __builtin_bit_cast(
                v4f, __builtin_amdgcn_raw_buffer_load_b128(trs, (int)c.off(sr[k], c.rg * K + k < R), 0, 0));
        const int t = min(tb + r * NWV + w, te - 1);
        const uint2* pv = reinterpret_cast<const uint2*>(sv + (size_t)t * dv);
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

    // One round.  No vector-memory operation is conditional (tokens past te and
    // lanes with nothing to store go out of bounds instead): the compiler counts
    // them to wait for the oldest loads only, and a branch around one would make
    // it wait for the rounds in flight as well.
    int cur = 0;                                       // record slot of round r
    int nxt = D;                                       // of round r + D
    int q0 = (tb / NWV) % (D + 1) * NWV;               // ring token of the round's first token
    auto round = [&](int j, int r) {
        __syncthreads();   // stores and ring rows of rounds before r are in place
        const int t = tb + r * NWV + w;
        const bool tok = t < te;   // else: the last token's record again, nothing stored
        const unsigned char* rec = rring + cur * L.bytes;
        const float al = reinterpret_cast<const float*>(rec + L.off_ab)[0];
        const float be = reinterpret_cast<const float*>(rec + L.off_ab)[1];
        const float yc = reinterpret_cast<const float*>(rec + L.off_ab)[2];
        int lw[K], lr[K], sw[K];
        float kap[K], rho[K];
        c.links(rec + L.off_link, W, lw);
        c.links(rec + L.off_link + 2 * W, R, lr);
        c.floats(rec + L.off_wval, W, kap);
        c.floats(rec + L.off_rval, R, rho);
        c.words(rec, W, sw);
        int all = -1;
#pragma unroll
        for (int k = 0; k < K; ++k) all &= lw[k] & lr[k];
        if (__builtin_amdgcn_ballot_w64(all >= 0)) {
            // rows of tokens still in flight: wait for those of this round, then take the ring's
            int top = -1;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int a = lw[k] - q0 * W, b = lr[k] - q0 * W;
                if (lw[k] >= 0 && a < w * W) top = max(top, a);
                if (lr[k] >= 0 && b < w * W) top = max(top, b);
            }
            for (int i = 0; i < w; ++i) {
                if (!__builtin_amdgcn_ballot_w64(top >= i * W)) break;
                while (__hip_atomic_load(&prog[i], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) <= r)
                    __builtin_amdgcn_s_sleep(1);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (lw[k] >= 0) Pw[j][k] = ld4(fring + (size_t)lw[k] * CW + c.cq * 4);
                if (lr[k] >= 0) Pr[j][k] = ld4(fring + (size_t)lr[k] * CW + c.cq * 4);
            }
        }
        // the helpers' pace (device scope, so that it leaves the compute unit; no helpers: out of bounds)
        __builtin_amdgcn_raw_buffer_store_b32(r, prs, w == 0 && lane == 0 ? 0 : (int)OOB, 0, 16);
        // For the rows: a slot's offset is below 2 GiB, so OOB + offset stays out.  Not for y: a token past
        // the end may lie at 2 GiB and more, where the sum would wrap to one of y's first rows.
        const uint32_t lc = tok ? c.lc4 : OOB;
        v4f up = v4zero(), yp = v4zero();
        v4f Dk[K];
        __amdgpu_buffer_rsrc_t srs;   // the token's saved rows
        if constexpr (SAVE)
            srs = __builtin_amdgcn_make_buffer_rsrc(ss + (size_t)min(t, te - 1) * W * dv, 0, W * dv * 4, 0x00020000);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int n = c.rg * K + k;
            if constexpr (SAVE)
                __builtin_amdgcn_raw_buffer_store_b128(
                    __builtin_bit_cast(u32x4, Pw[j][k]), srs,
                    (int)(EX || (n < W && c.colok) ? (uint32_t)n * c.dv4 + lc : OOB), 0, 0);
            Dk[k] = al * Pw[j][k];
            up = v4fma(kap[k], Dk[k], up);
            yp = v4fma(rho[k], Pr[j][k], yp);
        }
        sdm_reduce::rows_allreduce8<CQ>(up, yp);
        v4f vv;
        if constexpr (sizeof(VT) == 2)
            vv = v4f{bf16_lo(vb[j].x), bf16_hi(vb[j].x), bf16_lo(vb[j].y), bf16_hi(vb[j].y)};
        else
            vv = v4f{__uint_as_float(vb[j].x), __uint_as_float(vb[j].y), __uint_as_float(vb2[j].x),
                     __uint_as_float(vb2[j].y)};
        const v4f e = be * (vv - up);
        float* fr = fring + ((size_t)(q0 + w) * W + c.rg * K) * CW + c.cq * 4;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const v4f nw = v4fma(kap[k], e, Dk[k]);
            const bool ok = c.rg * K + k < W;
            if (EX || ok) st4(fr + k * CW, nw);
            const uint32_t o = __umul24((uint32_t)sw[k], c.dv4) + lc;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, nw), trs,
                                                   (int)(EX || (ok && c.colok) ? o : OOB), 0, 0);
        }
        __hip_atomic_store(&prog[w], r + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_raw_buffer_store_b128(
            __builtin_bit_cast(u32x4, v4fma(yc, e, yp)), yrs,
            (int)(tok && c.rg == 0 && c.colok ? (uint32_t)t * c.dv4 + c.lc4 : OOB), 0, 0);
        // the record of round r + D + 1 to LDS (loaded a round ago), the next into
        // registers, then the rows of round r + D
        const int after = nxt + 1 == Geo::NREC ? 0 : nxt + 1;
        rec_store(st, after);
        rec_load(st, r + D + 2);
        __builtin_amdgcn_sched_barrier(0);
        issue(j, r + D, nxt);
        __builtin_amdgcn_sched_barrier(0);
        nxt = after;
        cur = cur + 1 == Geo::NREC ? 0 : cur + 1;
        q0 = q0 + NWV == Geo::RING ? 0 : q0 + NWV;
    };
    for (int r = 0; r < rounds; r += D) {   // up to D - 1 empty rounds at the end
#pragma unroll
        for (int j = 0; j < D; ++j) round(j, r + j);
    }
}

// Geometry by rows per lane: K = 8 (lists of up to 64) holds 64 registers and 8 KB
// of ring per token in flight, so its rounds are half as long.
struct RoundPlan {
    int K, nwv, depth, lds;
    bool ex;
};
template <int K>
struct RoundCfg {
    static constexpr int NWV = K == 8 ? 4 : 8, D = 2;
};

template <int K>
bool plan_k(const ScanFwdArgs& a, RoundPlan* p) {
    using C = RoundCfg<K>;
    p->K = K;
    p->nwv = C::NWV;
    p->depth = C::D;
    p->ex = a.W == RG * K && a.R == RG * K && a.dv % CW == 0;
    p->lds = round_lds(C::NWV, C::D + 2, (C::D + 1) * C::NWV, fwd_rec_layout(a.W, a.R).bytes, a.W);
    return p->lds <= LDS_LIMIT;
}

int round_groups(const ScanFwdArgs& a) { return (a.dv + CW - 1) / CW; }

// Whether the kernel can run these arguments, and its geometry for them.
bool round_plan(const ScanFwdArgs& a, RoundPlan* p) {
    if (a.dv < CW) return false;   // rows narrower than a line: the per-wave kernel
    // the table rows' and y's 32-bit offsets (and the slots' 24-bit multiply)
    if ((size_t)a.N * a.dv * 4 >= ((size_t)1 << 31) || a.N >= (1 << 24)) return false;
    if ((size_t)a.T * a.dv * 4 >= ((size_t)1 << 31)) return false;
    const int m = std::max(a.W, a.R);
    if (m > RG * 8) return false;
    if (m <= RG) return plan_k<1>(a, p);
    if (m <= RG * 2) return plan_k<2>(a, p);
    if (m <= RG * 4) return plan_k<4>(a, p);
    return plan_k<8>(a, p);
}

// a forced geometry is one of scan_fwd.hip's or scan_chunk.hip's
bool geometry_forced() { return !sdm_line_io_enabled() || sdm_scan_slice_width() || sdm_scan_prefetch(); }

// lists that the line-cooperative kernel takes
bool line_lists(const ScanFwdArgs& a) { return a.W == a.R && (a.W == 32 || a.W == 64) && a.dv % 32 == 0; }

// Whether it is the faster kernel for them.  Two things speak against it.
//  * Lists of exactly 32 or 64 rows have the line-cooperative kernel, which moves
//    more bytes per second once every compute unit has work (scan of 2048 tokens,
//    d_v = 128, N = 65536, line kernel against this one in us: top-32 with 16 streams
//    1112 / 551, 32: 1173 / 820, 64: 1859 / 1515, 128: 2871 / 3219; top-64 with 16
//    streams 1734 / 1243, 64: 2687 / 3103, 128: 5425 / 6746; 480 workgroups of the 1.4B
//    layer with the undo log 9.5 / 9.3 ms, without 4.9 / 4.7, no gain in its steps): so
//    one workgroup per compute unit at most with 32 rows, half of that with 64.
//  * Where tokens of a round share slots they wait for each other.  A token's rows
//    meet about (tokens of a round) W (W + R) / N slots that another writes, and the
//    limits are where that costs what the rounds gain (256 tokens of top-32, 16
//    streams, against the line kernel: N = 2048 155 / 170 us, 2925 153 / 153, 4096 152 /
//    144; top-64: 8192 223 / 253, 11,702 220 / 234, 16,384 219 / 210).
// Other lists would take the per-wave kernel, which moves 32-byte pieces of rows: it
// loses on large tables (2048 tokens, N = 65536, 16 streams top-16 1691 / 298 us, 128
// streams top-8 1720 / 794) and at up to 16 rows nearly everywhere.  On dense tables it wins
// with longer lists, and earlier where two workgroups share a compute unit; the undo
// log's stores cost it more.  Its time over this kernel's (d_v = 128, by W (W + R) / N;
// limits in brackets, without / with the log):
//   16 streams   top-24: 4 0.87, 1.4 1.00, 1 1.08, 0.25 1.49 [4/3]
//                top-48: 4 0.75, 0.7 1.00, 0.5 1.06, 0.25 1.18 [3/5]
//   128 streams  top-16: 4 1.21 / 1.21; top-24: 2 0.73 / 0.76, 0.7 0.87 / 1.11, 0.5 0.95 /
//                1.12; top-48: 2 0.62 / 1.10, 0.5 0.94 / 1.15, 0.25 1.01 / 1.24 [1/2, 5/4]
//   512 streams  top-16: 4 0.80 / 1.37, 2 0.87 / 1.52, 1.4 1.03 [3/2, 15/4]; top-24: 4 0.45 /
//                0.88, 2 0.61 / 1.11, 0.5 1.05 / 1.29; top-48: 1 0.95 / 1.17, 0.5 1.11
//   rows that end inside a line, top-48: 256 streams of d_v = 36 2 0.94 / 1.39, 1 1.10, 0.7
//                1.38; of d_v = 68 2 0.92 / 1.37, 1 1.32 [1, 5/2]
bool round_faster(const ScanFwdArgs& a) {
    const int64_t cus = sdm_device_simds() / 4, wgs = (int64_t)a.B * a.H * round_groups(a);
    const int64_t pairs = (int64_t)a.W * (a.W + a.R);
    const int m = std::max(a.W, a.R);
    if (line_lists(a)) return wgs <= (m == 32 && !a.saved ? cus : cus / 2) && 2 * a.N >= 3 * pairs;
    if (m <= RG) return true;
    if (wgs <= cus) return m <= RG * 2 || (m <= RG * 4 ? 4 * a.N >= 3 * pairs : 3 * a.N >= 5 * pairs);
    const int64_t limit = (a.saved ? 5 : 2) * (m > RG * 4 && a.dv % CW ? 2 : 1);   // quarters, of pairs / N
    return m <= RG * 2 ? wgs <= 2 * cus || 3 * limit * a.N >= 4 * pairs : limit * a.N >= 4 * pairs;
}

// Helpers per main workgroup: as many as free compute units allow, at most two
// (a third gained nothing); none for stages too short to matter or without a
// record per group to hold the progress.
int round_helpers(const ScanFwdArgs& a) {
    const FwdRec L = fwd_rec_layout(a.W, a.R);
    const int nrnd = (round_groups(a) * a.B * a.H + 7) / 8 * 8;
    if (a.te - a.tb < std::max(128, round_groups(a)) || L.off_ab + 16 > L.bytes) return 0;
    return std::max(0, std::min(2, sdm_device_simds() / 4 / nrnd - 1));
}
// Tokens a helper may run past those in flight: 1 MB of an XCD's 4 MB L2 over its
// main workgroups (16 streams top-32: 16 tokens 551 us, 32: 561, 64: 611).
int round_lead(const ScanFwdArgs& a) {
    const int per_xcd = (round_groups(a) * a.B * a.H + 7) / 8;
    return std::min(32, std::max(8, (1 << 20) / (per_xcd * (a.W + a.R) * CW * 4)));
}

template <typename VT, int K, bool EX, bool SAVE>
hipError_t launch_round(const ScanFwdArgs& a, const RoundPlan& p, hipStream_t st) {
    using C = RoundCfg<K>;
    auto kfn = scan_fwd_round_kernel<VT, C::NWV, C::D, K, EX, SAVE>;
    hipError_t e = hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, p.lds);
    if (e != hipSuccess) return e;
    const int groups = round_groups(a), nrnd = (groups * a.B * a.H + 7) / 8 * 8, helpers = round_helpers(a);
    hipLaunchKernelGGL(kfn, dim3(nrnd * (1 + helpers)), dim3(C::NWV * SDM_WAVE), p.lds, st, a.ws + SDM_WS_HEADER,
                       static_cast<const VT*>(a.v), a.mem, a.y, a.saved, a.T, a.tb, a.te, a.dv, a.W, a.R, a.N, groups,
                       a.B * a.H, a.w_idx, a.r_idx, helpers, C::D * C::NWV + round_lead(a), a.ws + SDM_WS_HEADER);
    return hipGetLastError();
}

template <typename VT, bool SAVE>
hipError_t launch_round_k(const ScanFwdArgs& a, const RoundPlan& p, hipStream_t st) {
    switch (p.K) {
        case 1: return p.ex ? launch_round<VT, 1, true, SAVE>(a, p, st) : launch_round<VT, 1, false, SAVE>(a, p, st);
        case 2: return p.ex ? launch_round<VT, 2, true, SAVE>(a, p, st) : launch_round<VT, 2, false, SAVE>(a, p, st);
        case 4: return p.ex ? launch_round<VT, 4, true, SAVE>(a, p, st) : launch_round<VT, 4, false, SAVE>(a, p, st);
        default: return p.ex ? launch_round<VT, 8, true, SAVE>(a, p, st) : launch_round<VT, 8, false, SAVE>(a, p, st);
    }
}

}  // namespace

bool sdm_round_scan(const ScanFwdArgs& a, int* per_log2, int* depth, int* lds) {
    RoundPlan p;
    if (a.rounds == 0 || !round_plan(a, &p)) return false;
    if (a.rounds < 0 && (geometry_forced() || !round_faster(a))) return false;
    *per_log2 = __builtin_ctz((unsigned)p.nwv);
    *depth = p.depth;
    *lds = p.lds;
    return true;
}

// Whether the scan in rounds of tokens is faster than the chunk form (`narrow`: its
// 8-column workgroups).  Its tokens wait for each other where they share slots, the
// chunk form's do not, so that it takes larger tables; the chunk form's workgroups of
// 32 columns move more bytes than they need, so that it loses with many streams.
// Calls of 2048 tokens, d_v = 128, chunk form / rounds in us at slots N:
//   top-32, 16 streams 8192 737 / 715, 16,384 730 / 573, 262,144 854 / 515; 8: 16,384 560 /
//     570, 32,768 547 / 474; 32 (wide): 16,384 1189 / 759.  top-16, 8 streams: 4096 371 /
//     416, 8192 398 / 346.  Write 8, read 32, 8 streams: 4096 325 / 579, 16,384 387 /
//     442, 32,768 396 / 399: with narrow workgroups the longer list counts.
//   Over 32 rows a round is a chain of long tokens: top-40, 8 streams 1024 1035 / 2701,
//     32,768 1105 / 1312, 65,536 1213 / 1170; 16: 16,384 1152 / 1524, 32,768 1314 / 1335;
//     32: 16,384 1484 / 1557; 64: 4096 2043 / 2224, 8192 2304 / 1912; 128: 4096 4065 / 3184.
//     From 49 write rows on the chunk form holds fewer workgroups: top-56, 16 streams 8192
//     1978 / 2119, 16,384 2011 / 1782; 64: 4096 2929 / 2590.  Narrow, write 8, read 64: 8
//     streams 32,768 886 / 1000, 65,536 1005 / 942; 16: 16,384 1041 / 1113, 32,768 1190 / 1017;
//     1: 262,144 789 / 857 (write 32: 65,536 1120 / 1120, 262,144 1096 / 936): its narrow
//     workgroups' time goes with the write rows.  Product keys of clustered tokens, whose
//     slots recur: 8 streams of 32 columns, 4123 tokens, write 16, read 34, 65,536 1532 / 2208.
//   Lists of exactly 64 rows (whole lines, no bounds checks): 16 streams 8192 2194 / 1825.
bool sdm_round_beats_chunk(const ScanFwdArgs& a, bool narrow) {
    RoundPlan p;
    if (geometry_forced() || !round_plan(a, &p)) return false;
    const int64_t cus = sdm_device_simds() / 4, wgs = (int64_t)a.B * a.H * round_groups(a);
    const int64_t pairs = (int64_t)a.W * (a.W + a.R);
    const int m = std::max(a.W, a.R), rows = m <= RG ? RG : m <= RG * 2 ? RG * 2 : RG * 4;
    if (line_lists(a) && wgs > (m == 32 ? cus : cus / 2)) return false;
    if (line_lists(a) && m == 64) return a.N >= pairs;
    if (a.W <= 32 && a.N < 10 * pairs) return false;
    if (m <= 32) return !narrow || a.N >= 20 * rows * rows;
    if (narrow) return a.N >= std::max<int64_t>(32768, (1 << 25) / (a.W * wgs));
    if (a.W > 48) return a.N >= std::max<int64_t>(4096, std::min<int64_t>(16384, (1 << 20) / wgs));
    return a.N >= std::max<int64_t>(4096, std::min<int64_t>(65536, (1 << 21) / wgs));
}

hipError_t sdm_launch_round_scan(const ScanFwdArgs& a, hipStream_t st) {
    RoundPlan p;
    if (!round_plan(a, &p)) return hipErrorInvalidConfiguration;
    const bool save = a.saved != nullptr;
    if (a.in_dtype == SDM_DT_BF16)
        return save ? launch_round_k<bf16_t, true>(a, p, st) : launch_round_k<bf16_t, false>(a, p, st);
    return save ? launch_round_k<float, true>(a, p, st) : launch_round_k<float, false>(a, p, st);
}
