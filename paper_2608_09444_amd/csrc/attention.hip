// Paged decode attention over the depth-indexed KV cache.
//
// One query per (row, head): the row's q (after RoPE) attends to positions
// 0..pos of its sequence in one KV plane (the row's loop plane for the core,
// the stage plane for prelude/coda).  HBM-bound: every K/V byte is read once
// and used by one query, so the kernel is built for streaming, not MFMA.
//
// Layout of one (layer, page, head): K [16 tokens][hd] then (after H*16*hd
// elements) V [16][hd], bf16; pools are layer-major (kv_offset).  A wave reads a page as four coalesced
// loads for K and four for V: lane l covers token (4*j + l/16) and dims
// [(l%16)*hd/16, +hd/16).  The 16 lanes of a DPP row reduce q.k with row DPP
// (quad_perm, half_mirror, mirror), and each DPP row keeps its own online
// softmax over the tokens it owns, so no cross-row traffic happens per page.
//
// Balance: rows of one batch have different context lengths, and all
// workgroups of a launch are resident at once, so one workgroup per row would
// leave the chip idle while the longest rows finish.  A workgroup therefore
// takes two rows -- the p-th longest and the p-th shortest, from the order
// ranked at the start of the stage call (by the first workgroup of its
// row-entry kernel, or by k_row_order for a standalone attention call) -- and
// deals the pages of both to its 4 waves.  Each wave keeps one softmax state
// per row.  With pairs, mixed and equal context lengths run at the same
// bandwidth.  More than kAttnPairs pairs (two workgroups per CU) leave some CUs
// a workgroup more than others; then every row has a workgroup of its own,
// longest first, and the short ones fill in.
//
// Order of the sums: a row's context is cut into segments (attn_segment_pages,
// by its own page count); page p belongs to class p % 4; a class's pages of one
// segment share one state, merged over the four DPP rows at the segment's end;
// a class's segments are folded in segment order, and the four classes last.
// Nothing else enters, so a row's output is bit-identical whatever shares the
// batch and however many workgroups its segments are spread over.  The output
// is written in the fragment layout the output projection reads.
//
// Measured, one layer of the Ouro shape (16 x 128 heads): 64 rows at 648
// positions 58 us (5.8 TB/s, HBM-bound; a second page in flight per wave is no
// faster, 61 us), 100 rows at 433 positions 78 -> 70 us (ids of a wave's pages
// loaded at once, fewer registers) -> 64 (rows alone), 256 rows at 3100 positions
// 1.0 ms.
#include "cdb_internal.h"

namespace cdb {


template <int DPL>
struct RawVec {
    uint32_t w[DPL / 2];
};

// DPL bf16 values (held as DPL/2 dwords) to fp32
template <int DPL>
__device__ __forceinline__ void unpack_vec(const uint32_t* w, float* out) {
#pragma unroll
    for (int e = 0; e < DPL / 2; ++e) {
        out[2 * e] = bflo(w[e]);
        out[2 * e + 1] = bfhi(w[e]);
    }
}

// K and V are read once per launch and never again by it: the loads are
// non-temporal (streamed past the caches' normal allocation), which lifts a
// plain read stream on this part from about 6.3 to 7.1 TB/s.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <int DPL>
__device__ __forceinline__ RawVec<DPL> load_raw(const uint16_t* p) {
    RawVec<DPL> r;
    if constexpr (DPL == 8) {
        const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
        r.w[0] = v[0]; r.w[1] = v[1]; r.w[2] = v[2]; r.w[3] = v[3];
    } else if constexpr (DPL == 4) {
        const u32x2 v = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p));
        r.w[0] = v[0]; r.w[1] = v[1];
    } else {
        const uint32_t* q = reinterpret_cast<const uint32_t*>(p);
        r.w[0] = __builtin_nontemporal_load(q);
        r.w[1] = __builtin_nontemporal_load(q + 1);
        r.w[2] = __builtin_nontemporal_load(q + 2);
    }
    return r;
}

#define CDB_DPP(v, ctrl) __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, (v)), (ctrl), 0xF, 0xF, true))

// Sum over the 16 lanes of a DPP row; every lane of the row gets the sum.
__device__ __forceinline__ float row_sum16(float v) {
    v += CDB_DPP(v, 0xB1);   // quad_perm [1,0,3,2]
    v += CDB_DPP(v, 0x4E);   // quad_perm [2,3,0,1]
    v += CDB_DPP(v, 0x141);  // row_half_mirror
    v += CDB_DPP(v, 0x140);  // row_mirror
    return v;
}

template <int DPL>
struct PageData {
    RawVec<DPL> k[4], v[4];
};

// One online-softmax state: running maximum (exp2 domain), sum and weighted V.
template <int DPL>
struct SoftState {
    float m, l, acc[DPL];
    __device__ __forceinline__ void clear() {
        m = -1e30f;
        l = 0.f;
#pragma unroll
        for (int e = 0; e < DPL; ++e) acc[e] = 0.f;
    }
};

// Every multiply-add of the state updates is an explicit fma, so the one- and
// many-workgroup forms of the kernel round alike.

// Online-softmax update of one row's state with one 16-token page; n_tok = how
// many of its tokens are visible (16 or more: all).
template <int DPL>
__device__ __forceinline__ void attend_page(const PageData<DPL>& pd, const float* qr, int n_tok, int g,
                                            SoftState<DPL>& st) {
    float sc[4];
    float mx = st.m;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float kf[DPL];
        unpack_vec<DPL>(pd.k[j].w, kf);
        float dot = 0.f;
#pragma unroll
        for (int e = 0; e < DPL; ++e) dot = fmaf(qr[e], kf[e], dot);
        dot = row_sum16(dot);
        sc[j] = j * 4 + g < n_tok ? dot : -1e30f;
        mx = fmaxf(mx, sc[j]);
    }
    const float corr = exp2f(st.m - mx);
    st.l *= corr;
#pragma unroll
    for (int e = 0; e < DPL; ++e) st.acc[e] *= corr;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const bool valid = j * 4 + g < n_tok;
        const float pj = valid ? exp2f(sc[j] - mx) : 0.f;
        st.l += pj;
        float vf[DPL];
        unpack_vec<DPL>(pd.v[j].w, vf);
#pragma unroll
        for (int e = 0; e < DPL; ++e) st.acc[e] = fmaf(pj, valid ? vf[e] : 0.f, st.acc[e]);
    }
    st.m = mx;
}

// t = t + s, both over the same row; scale factors of the two sums
__device__ __forceinline__ void fold_ml(float& tm, float& tl, float sm, float sl, float& a, float& b) {
    const float mx = fmaxf(tm, sm);
    a = exp2f(tm - mx);
    b = exp2f(sm - mx);
    tl = fmaf(tl, a, sl * b);
    tm = mx;
}
__device__ __forceinline__ float fold_acc(float t, float s, float a, float b) { return fmaf(t, a, s * b); }

// x + (x of the lane 16, or 32, away); every lane pair gets the same sum.  The
// swaps leave {x of the even row, x of the odd row} of each pair in both rows.
__device__ __forceinline__ void row_swap16(float x, float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void row_swap32(float x, float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ float dpp_rows_sum(float x) {
    float a, b;
    row_swap16(x, a, b);
    row_swap32(a + b, a, b);
    return a + b;
}
__device__ __forceinline__ float dpp_rows_max(float x) {
    float a, b;
    row_swap16(x, a, b);
    row_swap32(fmaxf(a, b), a, b);
    return fmaxf(a, b);
}

// Merges the states of a wave's four DPP rows (each saw its own tokens of the
// same pages); every lane of a column ends with the same merged state.
template <int DPL>
__device__ __forceinline__ void merge_dpp_rows(SoftState<DPL>& st) {
    const float mx = dpp_rows_max(st.m);
    const float f = exp2f(st.m - mx);
    st.l = dpp_rows_sum(st.l * f);
#pragma unroll
    for (int e = 0; e < DPL; ++e) st.acc[e] = dpp_rows_sum(st.acc[e] * f);
    st.m = mx;
}

constexpr int kAttnWaves = 4;

// Output of one (row, dim) from its four page-class states, in class order.
template <int HD>
__device__ __forceinline__ float merge_classes(const float (&m)[kAttnWaves], const float (&l)[kAttnWaves],
                                               const float (&acc)[kAttnWaves]) {
    float mx = -1e30f;
#pragma unroll
    for (int c = 0; c < kAttnWaves; ++c) mx = fmaxf(mx, m[c]);
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int c = 0; c < kAttnWaves; ++c) {
        const float w = exp2f(m[c] - mx);
        num = fmaf(w, acc[c], num);
        den = fmaf(w, l[c], den);
    }
    return den > 0.f ? num / den : 0.f;
}

// One row's context as the kernel sees it.
struct RowCtx {
    const int32_t* pt;  // its page ids
    int n_ctx, npg;     // visible positions, pages
    bool ok;
};
__device__ __forceinline__ RowCtx row_context(const KvTarget& kv, const int32_t* seq, const int32_t* pos, int m) {
    RowCtx r{kv.page_table, 0, 0, false};
    const int sq = seq[m];
    // a row's own loop index reads a core plane (1..r_max) only
    const int plane = kv.c_row ? kv.c_row[m] + 1 : kv.plane_fixed;
    const bool plane_ok = kv.c_row ? (plane >= 1 && plane <= kv.n_planes - 2) : (plane >= 0 && plane < kv.n_planes);
    const int nc = pos[m] + 1;
    const int np = (nc + kPage - 1) / kPage;
    if (!(sq >= 0 && sq < kv.max_seqs && plane_ok && nc >= 1 && np <= kv.max_pages)) return r;
    r.ok = true;
    r.n_ctx = nc;
    r.npg = np;
    r.pt = kv.page_table + ((size_t)sq * kv.n_planes + plane) * kv.max_pages;
    return r;
}

// K and V of one page's head into registers (V follows K after H pages' rows)
template <int HD>
__device__ __forceinline__ void fetch_page(const uint16_t* base, size_t vofs, int g, int li, PageData<HD / 16>& pd) {
    constexpr int DPL = HD / 16;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int t = j * 4 + g;
        pd.k[j] = load_raw<DPL>(base + t * HD + li * DPL);
        pd.v[j] = load_raw<DPL>(base + vofs + t * HD + li * DPL);
    }
}

// seg into sum; seg starts again
template <int DPL>
__device__ __forceinline__ void fold_segment(SoftState<DPL>& seg, SoftState<DPL>& sum) {
    merge_dpp_rows<DPL>(seg);
    float a, b;
    fold_ml(sum.m, sum.l, seg.m, seg.l, a, b);
#pragma unroll
    for (int e = 0; e < DPL; ++e) sum.acc[e] = fold_acc(sum.acc[e], seg.acc[e], a, b);
    seg.clear();
}

// a wave's folded state of row r (the same in its four DPP rows) to LDS
template <int HD>
__device__ __forceinline__ void store_state(const SoftState<HD / 16>& st, int r, int wave, int g, int li,
                                            float (&s_m)[2][kAttnWaves], float (&s_l)[2][kAttnWaves],
                                            float (&s_acc)[2][kAttnWaves][HD]) {
    if (g != 0) return;
    if (li == 0) {
        s_m[r][wave] = st.m;
        s_l[r][wave] = st.l;
    }
#pragma unroll
    for (int e = 0; e < HD / 16; ++e) s_acc[r][wave][li * (HD / 16) + e] = st.acc[e];
}

// (row pair, head) workgroups above which a row has its own.  Pairs against rows
// alone, 16 x 128 heads: 64 rows (512 pairs) at 640 positions 56 and 57 us, 66
// rows (528) 71 and 62, 80 rows 75.6 and 73, 98 rows 94 and 87, 128 rows 108 and
// 108, 160 rows 143 and 133; 55 x 96 heads at 510 positions: 18 rows (495) 33.4 and
// 34.7, 28 rows (770) 55 and 48.5, 64 rows 112 and 106.  At 40 positions rows
// alone cost up to 1.5 us (256 rows 20.7 and 22.2).  The live rows decide; the
// grid is that of the capacity, whose empty workgroups cost a call of few live
// rows 0.5 us (1 row of 128) to 1.4 us (of 256).
constexpr int kAttnPairs = 512;
__host__ __device__ __forceinline__ bool rows_alone(int n, int H) { return (n + 1) / 2 * H > kAttnPairs; }

template <int HD>
__global__ __launch_bounds__(kAttnWaves * 64) void k_attn(const float* __restrict__ q, KvTarget kv,
                                                          const int32_t* __restrict__ seq,
                                                          const int32_t* __restrict__ pos,
                                                          const int32_t* __restrict__ order, int M, int H,
                                                          uint16_t* __restrict__ out, int* err,
                                                          const int32_t* __restrict__ dn) {
    constexpr int DPL = HD / 16;
    __shared__ float s_m[2][kAttnWaves], s_l[2][kAttnWaves];
    __shared__ float s_acc[2][kAttnWaves][HD];
    const int head = blockIdx.x, pair = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, li = lane & 15;
    const int d = H * HD;
    const float qscale = 1.4426950408889634f / sqrtf((float)HD);  // log2(e) / sqrt(hd)
    const size_t vofs = (size_t)H * kPage * HD;  // V follows K within a (layer, page)

    // the pair: p-th longest and p-th shortest row (one row when they meet, or
    // with rows alone); with a device row count the grid covers the capacity M
    const int n = live_rows(dn, M);
    const bool alone = rows_alone(n, H);
    if (alone ? pair >= n : 2 * pair >= n) return;
    const int row0 = order[pair], row1 = (!alone && n - 1 - pair > pair) ? order[n - 1 - pair] : -1;
    const RowCtx rc0 = row_context(kv, seq, pos, row0);
    const RowCtx rc1 = row1 >= 0 ? row_context(kv, seq, pos, row1) : RowCtx{kv.page_table, 0, 0, false};
    if (tid == 0 && (!rc0.ok || (row1 >= 0 && !rc1.ok))) set_err(err, CDB_DEV_UNMAPPED_PAGE);
    // the concatenated page list of both rows is dealt round-robin to the
    // waves: page p of row 1 goes to wave (n0 + p) % 4.  Each wave's first 64
    // page ids of both rows and the q rows are loaded here at once, so that no
    // page waits for its id.
    const int n0 = rc0.npg;
    const int pf0 = wave, pf1 = (wave - n0 % kAttnWaves + kAttnWaves) % kAttnWaves;  // the wave's first pages
    const int step = lane * kAttnWaves;
    int ids = pf0 + step < rc0.npg ? rc0.pt[pf0 + step] : -1;
    const int ids1 = pf1 + step < rc1.npg ? rc1.pt[pf1 + step] : -1;
    float qv[DPL], q1[DPL];
    {  // an unusable row attends to no page: any row's q will do
        const float* p0 = q + (size_t)row0 * d + head * HD + li * DPL;
        const float* p1 = q + (size_t)max(row1, 0) * d + head * HD + li * DPL;
#pragma unroll
        for (int e = 0; e < DPL; ++e) {
            qv[e] = p0[e] * qscale;
            q1[e] = p1[e] * qscale;
        }
    }
    // the wave's items: its pages of row 0, then those of row 1
    const int cnt0 = rc0.npg > pf0 ? (rc0.npg - pf0 + kAttnWaves - 1) / kAttnWaves : 0;
    const int cnt1 = rc1.npg > pf1 ? (rc1.npg - pf1 + kAttnWaves - 1) / kAttnWaves : 0;
    SoftState<DPL> seg, sum;  // the current segment's state; the row's earlier segments, folded
    seg.clear();
    sum.clear();
    int row = 0, p = pf0, i = 0, n_ctx = rc0.n_ctx, sp = attn_segment_pages(rc0.npg), seg_end = sp;
    for (int t = 0; t < cnt0 + cnt1; ++t, p += kAttnWaves, ++i) {
        const bool turn = t == cnt0;  // the first page of row 1
        if (turn) {
            p = pf1;
            i = 0;
            ids = ids1;
        }
        if (i == 64) {  // past the ids loaded so far
            i = 0;
            const int pl = p + step;
            if (t < cnt0)
                ids = pl < rc0.npg ? rc0.pt[pl] : -1;
            else
                ids = pl < rc1.npg ? rc1.pt[pl] : -1;
        }
        const int pid = __builtin_amdgcn_readlane(ids, i);
        const bool mapped = pid >= 0 && pid < kv.n_pages;
        PageData<DPL> pd;
        if (mapped)
            fetch_page<HD>(kv.pool + kv_offset(kv.layer, pid, kv.n_pages, 0, head, H, 0, HD), vofs, g, li, pd);
        else if (lane == 0)
            set_err(err, CDB_DEV_UNMAPPED_PAGE);
        // a segment or row that has ended is folded while the page's loads are in flight
        if (turn || p >= seg_end) {
            fold_segment<DPL>(seg, sum);
            if (turn) {
                store_state<HD>(sum, 0, wave, g, li, s_m, s_l, s_acc);
                sum.clear();
                row = 1;
                n_ctx = rc1.n_ctx;
                sp = attn_segment_pages(rc1.npg);
#pragma unroll
                for (int e = 0; e < DPL; ++e) qv[e] = q1[e];
            }
            seg_end = (p / sp + 1) * sp;
        }
        if (mapped) attend_page<DPL>(pd, qv, n_ctx - p * kPage, g, seg);
    }
    fold_segment<DPL>(seg, sum);
    store_state<HD>(sum, row, wave, g, li, s_m, s_l, s_acc);
    if (row == 0) {  // no page of row 1 on this wave
        sum.clear();
        store_state<HD>(sum, 1, wave, g, li, s_m, s_l, s_acc);
    }
    __syncthreads();
    if (tid < 2 * HD) {
        const int r = tid / HD, dim = tid - r * HD;
        const int m = r ? row1 : row0;
        if (m >= 0 && (r ? rc1.ok : rc0.ok)) {
            // page p of row 1 ran on wave (n0 + p) % 4: classes are by p
            const int first = r == 0 ? 0 : n0 % kAttnWaves;
            float cm[kAttnWaves], cl[kAttnWaves], ca[kAttnWaves];
#pragma unroll
            for (int c = 0; c < kAttnWaves; ++c) {
                const int w = (first + c) % kAttnWaves;
                cm[c] = s_m[r][w];
                cl[c] = s_l[r][w];
                ca[c] = s_acc[r][w][dim];
            }
            out[frag_index(m, head * HD + dim, d)] = f2bf(merge_classes<HD>(cm, cl, ca));
        }
    }
}

// The same attention with each row's segments spread over several workgroups,
// for calls whose rows alone leave the chip idle: grid (head, row, nz), and
// workgroup z takes segments z, z + nz, ...  A segment's four class states go
// to `part`; the workgroup of a (row, head) that arrives last folds them in
// segment order, exactly as the one-workgroup form does in registers.
//
// Hand-over between workgroups (they run on XCDs with separate L2s): the
// states are written through to memory by agent-scope stores, waited for, then
// counted in arrive[row][head] by an agent-scope atomic; the last arriver
// reads them with agent-scope loads, which do not take stale lines.  It also
// sets the counter back to 0 for the next launch.  Nobody waits.
//
// With one workgroup per (head, pair) 6 rows at 3100 positions ran on 48 of 256
// CUs: 130 us per layer; spread over segments 38 us (4.0 TB/s).  One row at 450
// positions 13.6 -> 10.8 us.
template <int HD>
__global__ __launch_bounds__(kAttnWaves * 64) void k_attn_split(const float* __restrict__ q, KvTarget kv,
                                                                const int32_t* __restrict__ seq,
                                                                const int32_t* __restrict__ pos, int M, int H,
                                                                float* __restrict__ part, int* __restrict__ arrive,
                                                                uint16_t* __restrict__ out, int* err,
                                                                const int32_t* __restrict__ dn) {
    constexpr int DPL = HD / 16;
    constexpr int REC = kAttnWaves * (HD + 2);  // a segment's record: [4][HD] sums, [4] maxima, [4] weights
    __shared__ float s_m[kAttnWaves], s_l[kAttnWaves];
    __shared__ float s_acc[kAttnWaves][HD];
    __shared__ int s_last;
    const int head = blockIdx.x, m = blockIdx.y, z = blockIdx.z, nz = gridDim.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, li = lane & 15;
    const int d = H * HD;
    const float qscale = 1.4426950408889634f / sqrtf((float)HD);
    const size_t vofs = (size_t)H * kPage * HD;
    if (m >= live_rows(dn, M)) return;
    const RowCtx rc = row_context(kv, seq, pos, m);
    if (!rc.ok) {
        if (tid == 0 && z == 0) set_err(err, CDB_DEV_UNMAPPED_PAGE);
        return;
    }
    const int sp = attn_segment_pages(rc.npg), nseg = (rc.npg + sp - 1) / sp;
    if (z >= nseg) return;
    float qr[DPL];
#pragma unroll
    for (int e = 0; e < DPL; ++e) qr[e] = q[(size_t)m * d + head * HD + li * DPL + e] * qscale;
    float* rec0 = part + ((size_t)m * H + head) * kAttnMaxSegments * REC;

    for (int sg = z; sg < nseg; sg += nz) {
        SoftState<DPL> seg;
        seg.clear();
        const int p1 = min(rc.npg, (sg + 1) * sp);
        // two pages in flight
        auto page = [&](int p) -> const uint16_t* {
            const int pid = rc.pt[p];
            if (pid < 0 || pid >= kv.n_pages) return nullptr;
            return kv.pool + kv_offset(kv.layer, pid, kv.n_pages, 0, head, H, 0, HD);
        };
        PageData<DPL> pa, pb;
        auto attend = [&](const uint16_t* b, const PageData<DPL>& pd, int p) {
            if (b)
                attend_page<DPL>(pd, qr, rc.n_ctx - p * kPage, g, seg);
            else if (lane == 0)
                set_err(err, CDB_DEV_UNMAPPED_PAGE);
        };
        for (int p = sg * sp + wave; p < p1; p += 2 * kAttnWaves) {
            const uint16_t* ba = page(p);
            const uint16_t* bb = p + kAttnWaves < p1 ? page(p + kAttnWaves) : nullptr;
            if (ba) fetch_page<HD>(ba, vofs, g, li, pa);
            if (bb) fetch_page<HD>(bb, vofs, g, li, pb);
            attend(ba, pa, p);
            if (p + kAttnWaves < p1) attend(bb, pb, p + kAttnWaves);
        }
        merge_dpp_rows<DPL>(seg);
        float* rec = rec0 + (size_t)sg * REC;
        if (g == 0) {
#pragma unroll
            for (int e = 0; e < DPL; ++e)
                __hip_atomic_store(rec + wave * HD + li * DPL + e, seg.acc[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (li == 0) {
                __hip_atomic_store(rec + kAttnWaves * HD + wave, seg.m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(rec + kAttnWaves * (HD + 1) + wave, seg.l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // every wave's states have reached memory
    __syncthreads();
    if (tid == 0) {
        int* a = arrive + m * H + head;
        const int last = min(nz, nseg) - 1;
        s_last = __hip_atomic_fetch_add(a, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == last;
        if (s_last) __hip_atomic_store(a, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!s_last) return;
    for (int e = tid; e < kAttnWaves * HD; e += kAttnWaves * 64) {
        const int c = e / HD, dim = e - c * HD;
        float tm = -1e30f, tl = 0.f, ta = 0.f;
        float sa[kAttnMaxSegments], sm[kAttnMaxSegments], sl[kAttnMaxSegments];
#pragma unroll
        for (int sg = 0; sg < kAttnMaxSegments; ++sg)
            if (sg < nseg) {
                const float* rec = rec0 + (size_t)sg * REC;
                sa[sg] = __hip_atomic_load(rec + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                sm[sg] = __hip_atomic_load(rec + kAttnWaves * HD + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                sl[sg] = __hip_atomic_load(rec + kAttnWaves * (HD + 1) + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
        for (int sg = 0; sg < kAttnMaxSegments; ++sg)
            if (sg < nseg) {
                float a, b;
                fold_ml(tm, tl, sm[sg], sl[sg], a, b);
                ta = fold_acc(ta, sa[sg], a, b);
            }
        s_acc[c][dim] = ta;
        if (dim == 0) {
            s_m[c] = tm;
            s_l[c] = tl;
        }
    }
    __syncthreads();
    if (tid < HD) {
        float cm[kAttnWaves], cl[kAttnWaves], ca[kAttnWaves];
#pragma unroll
        for (int c = 0; c < kAttnWaves; ++c) {
            cm[c] = s_m[c];
            cl[c] = s_l[c];
            ca[c] = s_acc[c][tid];
        }
        out[frag_index(m, head * HD + tid, d)] = f2bf(merge_classes<HD>(cm, cl, ca));
    }
}

// Workgroups per (row, head) of the split form; 1: the paired form.  Enough
// workgroups for four per CU, but no more than a context the page table can hold
// has segments.
static int attn_splits(int M, int H, int max_pages) {
    if (M * H >= kAttnSplitItems) return 1;
    const int sp = attn_segment_pages(max_pages), nseg = (max_pages + sp - 1) / sp;
    // shorter rows of the same table may have up to kAttnMaxSegments segments
    const int most = max_pages >= 8 * kAttnMaxSegments ? kAttnMaxSegments : nseg;
    const int want = (4 * 256 + M * H - 1) / (M * H);
    return want < most ? want : most;
}

hipError_t launch_attention(const float* q, const KvTarget& kv, const int32_t* seq, const int32_t* pos,
                            const int32_t* order, int M, int H, int hd, uint16_t* out, int* err, hipStream_t st,
                            const int32_t* dn, const AttnScratch* scratch) {
    if (M <= 0) return hipSuccess;
    const int nz = scratch ? attn_splits(M, H, kv.max_pages) : 1;
    if (nz > 1) {
        const dim3 grid(H, M, nz);
        float* part = scratch->part;
        int* arrive = scratch->arrive;
        switch (hd) {
            case 64: k_attn_split<64><<<grid, kAttnWaves * 64, 0, st>>>(q, kv, seq, pos, M, H, part, arrive, out, err, dn); break;
            case 96: k_attn_split<96><<<grid, kAttnWaves * 64, 0, st>>>(q, kv, seq, pos, M, H, part, arrive, out, err, dn); break;
            case 128: k_attn_split<128><<<grid, kAttnWaves * 64, 0, st>>>(q, kv, seq, pos, M, H, part, arrive, out, err, dn); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    dim3 grid(H, rows_alone(M, H) ? M : (M + 1) / 2);
    switch (hd) {
        case 64: k_attn<64><<<grid, kAttnWaves * 64, 0, st>>>(q, kv, seq, pos, order, M, H, out, err, dn); break;
        case 96: k_attn<96><<<grid, kAttnWaves * 64, 0, st>>>(q, kv, seq, pos, order, M, H, out, err, dn); break;
        case 128: k_attn<128><<<grid, kAttnWaves * 64, 0, st>>>(q, kv, seq, pos, order, M, H, out, err, dn); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// order[rank] = row, ranked by descending position (ties by row index).  One
// workgroup; M <= 256.
__global__ __launch_bounds__(256) void k_row_order(const int32_t* __restrict__ pos, int M, int32_t* __restrict__ order,
                                                   const int32_t* __restrict__ dn) {
    M = live_rows(dn, M);
    for (int i = threadIdx.x; i < M; i += blockDim.x) {
        const int pi = pos[i];
        int rank = 0;
        for (int j = 0; j < M; ++j) {
            const int pj = pos[j];
            rank += (pj > pi) || (pj == pi && j < i);
        }
        order[rank] = i;
    }
}

hipError_t launch_row_order(const int32_t* pos, int M, int32_t* order, hipStream_t st, const int32_t* dn) {
    if (M <= 0) return hipSuccess;
    k_row_order<<<1, 256, 0, st>>>(pos, M, order, dn);
    return hipGetLastError();
}

}  // namespace cdb
