// Skinny bf16 GEMM for the block projections: Y[M][N] = X[M][K] . W[N][K]^T
// with M = rows of one stage call (ragged, <= 128) and the weight streamed from
// HBM exactly once per call.
//
// Design (gfx950):
//  * W is pre-packed into 32x16 operand tiles of v_mfma_f32_32x32x16_bf16 in
//    lane order (1 KiB each), so one 16-byte load per lane fetches a whole A
//    operand, coalesced; the tiles of one 32-column stripe are contiguous
//    along K.  A 32-wide stripe halves the activation (B operand) traffic per
//    weight byte compared with a 16-wide one.
//  * A workgroup owns NS (1 or 2) 32-column stripes and one K split; its KW
//    waves split that K range further.  Each wave streams its weight tiles and the matching
//    activation fragments (L2-resident), several k steps ahead in registers.
//    The KW partial tiles are summed in LDS in wave order.
//  * No reduction crosses workgroups inside the kernel.  Stripes whose K is
//    split over S workgroups write fp32 partial tiles; the row kernel that
//    runs next (residual add + RMSNorm) adds them in split order.  Every
//    reduction order depends on (N, K) only, so a row's result does not depend
//    on which other rows share the batch.
//  * Epilogues: q/k/v with RoPE and the K/V page write (a 32-column group is
//    16 first-half and the 16 matching second-half dims of one head), SwiGLU (a
//    group is 16 gate and the 16 matching up columns), plain fp32 store, and
//    the split-K partial store.
#include <algorithm>

#include "cdb_internal.h"

namespace cdb {

constexpr int kMaxKw = 8;     // waves per workgroup (2 per SIMD, so 256 registers each)

struct GemmArgs {
    const uint16_t* X;  // fragment layout, gemm_rows(M) rows (rows >= M are never read back), K columns
    const uint16_t* Wp;
    int M, N, K, S, KW;
    float* part;  // EPI_PARTIAL: [S][M][N]
    const int32_t* dn;  // optional device row count (<= M): rows at or past it are not stored
};

// Inputs of the q/k/v epilogue, staged in LDS: the RoPE factors of the
// stripe's 16 rotary pairs for every row, and each row's K/V write page and
// slot within it.
struct QkvStage {
    const float2* rope;  // [rows][16]
    const int* pid;      // [rows]
    const int* tok;      // [rows]
};

// The two halves of a rotated pair, rounded alike wherever they are computed.
__device__ __forceinline__ float rope_first(float xf, float xs, float c, float s) { return fmaf(xf, c, -(xs * s)); }
__device__ __forceinline__ float rope_second(float xf, float xs, float c, float s) { return fmaf(xs, c, xf * s); }

// Four floats of a split partial (a 16-byte aligned workspace region) or of a plain
// store: the caller's logits may start at any float, and 16-byte stores need no
// more than that alignment on this part.
typedef float floatx4_any __attribute__((ext_vector_type(4), aligned(4)));
template <int EPI>
__device__ __forceinline__ void store4(float* dst, float a, float b, float c, float d) {
    if (EPI == EPI_PARTIAL)
        *reinterpret_cast<float4*>(dst) = make_float4(a, b, c, d);
    else
        *reinterpret_cast<floatx4_any*>(dst) = floatx4_any{a, b, c, d};
}

// Epilogue of the skinny kernel from the reduced tiles fin[ns][n][m] (row
// pitch fld), with 16-byte stores: each thread takes a run of consecutive
// output columns of one row (4 fp32 values, or 8 bf16 values in the
// fragment or K/V layouts).  Same arithmetic per element as tile_epilogue.
// split: the workgroup's K split (EPI_PARTIAL writes partial tile `split`).
template <int EPI>
__device__ __forceinline__ void stripe_epilogue(const float* fin, int fld, int nt, int NS, int mcap, int split, int tid,
                                                int nthr, const GemmArgs& ga, const EpiArgs& ea, const QkvStage& qs) {
    if (EPI == EPI_PARTIAL || EPI == EPI_STORE) {
        // (ns, m, 4-column run)
        const int per = mcap * 8;
        float* base = EPI == EPI_PARTIAL ? ga.part + (size_t)split * ga.M * ga.N : ea.out;
        const int ld = EPI == EPI_PARTIAL ? ga.N : ea.ld_out;
        for (int e = tid; e < NS * per; e += nthr) {
            const int ns = e / per, r = e - ns * per;
            if (nt + ns >= (ga.N >> 5)) break;
            const int m = r >> 3, c4 = (r & 7) * 4;
            const float* f = fin + ns * 32 * fld + c4 * fld + m;
            store4<EPI>(base + (size_t)m * ld + (nt + ns) * 32 + c4, f[0], f[fld], f[2 * fld], f[3 * fld]);
        }
    } else if (EPI == EPI_SWIGLU) {
        // (ns, m, 8-feature run): gate columns c8 .. c8 + 7, up columns 16 + c8 ..
        const int per = mcap * 2;
        for (int e = tid; e < NS * per; e += nthr) {
            const int ns = e / per, r = e - ns * per;
            if (nt + ns >= (ga.N >> 5)) break;
            const int m = r >> 1, c8 = (r & 1) * 8;
            const float* f = fin + ns * 32 * fld + m;
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 8; i += 2) {
                const float g0 = f[(c8 + i) * fld], u0 = f[(16 + c8 + i) * fld];
                const float g1 = f[(c8 + i + 1) * fld], u1 = f[(16 + c8 + i + 1) * fld];
                const float s0 = g0 / (1.0f + __expf(-g0)), s1 = g1 / (1.0f + __expf(-g1));
                w[i / 2] = pack_bf16(s0 * u0, s1 * u1);
            }
            const int feat = (nt + ns) * 16 + c8;
            *reinterpret_cast<u32x4*>(ea.act + frag_index(m, feat, ea.ld_act)) = u32x4{w[0], w[1], w[2], w[3]};
        }
    } else {  // EPI_QKV: a stripe holds 16 rotary pairs (dims gi*16 + jj and + hd/2) of one head
        const int gph = ea.hd >> 5, hg = ea.H * gph;
        const int part = nt / hg, rem = nt - part * hg;
        const int head = rem / gph, gi = rem - head * gph;
        const int half_hd = ea.hd >> 1;
        if (part == 0) {
            // (m, half, 4-pair run) -> 4 consecutive fp32 q values
            for (int e = tid; e < mcap * 8; e += nthr) {
                const int m = e >> 3, half = (e >> 2) & 1, j4 = (e & 3) * 4;
                float o[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int jj = j4 + i;
                    const float val = fin[(half * 16 + jj) * fld + m], partner = fin[((half ^ 1) * 16 + jj) * fld + m];
                    const float2 cs = qs.rope[m * 16 + jj];
                    const float xf = half ? partner : val, xs = half ? val : partner;
                    o[i] = half ? rope_second(xf, xs, cs.x, cs.y) : rope_first(xf, xs, cs.x, cs.y);
                }
                float* dst = ea.q + (size_t)m * (ea.H * ea.hd) + head * ea.hd + gi * 16 + j4 + half * half_hd;
                *reinterpret_cast<float4*>(dst) = make_float4(o[0], o[1], o[2], o[3]);
            }
        } else {
            // (m, half, 8-pair run) -> 8 consecutive bf16 K or V values
            for (int e = tid; e < mcap * 4; e += nthr) {
                const int m = e >> 2, half = (e >> 1) & 1, j8 = (e & 1) * 8;
                const int pid = qs.pid[m];  // -1: unmapped (reported by the row-entry kernel)
                if (pid < 0) continue;
                const int tok = qs.tok[m];
                uint32_t w[4];
#pragma unroll
                for (int i = 0; i < 8; i += 2) {
                    float o2[2];
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const int jj = j8 + i + b;
                        const float val = fin[(half * 16 + jj) * fld + m];
                        float outv = val;
                        if (part == 1) {
                            const float partner = fin[((half ^ 1) * 16 + jj) * fld + m];
                            const float2 cs = qs.rope[m * 16 + jj];
                            const float xf = half ? partner : val, xs = half ? val : partner;
                            outv = half ? rope_second(xf, xs, cs.x, cs.y) : rope_first(xf, xs, cs.x, cs.y);
                        }
                        o2[b] = outv;
                    }
                    w[i / 2] = pack_bf16(o2[0], o2[1]);
                }
                const KvTarget& kv = ea.kv;
                uint16_t* dst = kv.pool + kv_offset(kv.layer, pid, kv.n_pages, part - 1, head, ea.H, tok, ea.hd) +
                                gi * 16 + j8 + half * half_hd;
                *reinterpret_cast<u32x4*>(dst) = u32x4{w[0], w[1], w[2], w[3]};
            }
        }
    }
}

// A buffer resource over [p, p + bytes): operand tiles are loaded with one lane
// offset register for all of them and the tile's offset in a scalar, where
// 64-bit lane addresses would take registers from the k steps in flight.  The
// arguments are wave-uniform.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void* p, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)(uint32_t)bytes, 0x00027000);
}
__device__ __forceinline__ u32x4 load_tile(__amdgpu_buffer_rsrc_t r, int lane_bytes, int tile_bytes) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, lane_bytes, tile_bytes, 0));
}

// k steps of one wave in flight in the decode kernel: as many as leave room
// for NS x MT accumulator tiles in the 256 registers of a wave
__host__ __device__ constexpr int decode_depth(int MT, int NS) {
    const int d = (224 - 16 * MT * NS) / (4 * (MT + NS));
    return d > 16 ? 16 : d;
}

// 32x32 tiles the decode kernel's wave reduction sums per round: all NS x MT
// of them when 8 waves' copies, the reduced block and the q/k/v staging fit in
// 160 KB of LDS, else one
__host__ __device__ constexpr int decode_red_tiles(bool qkv, int MT, int NS) {
    return (8 * NS * MT * 1024 + NS * 32 * (MT * 32 + 1) + (qkv ? MT * 32 * 32 + MT * 64 : 0)) * 4 <= 160 * 1024
               ? NS * MT : 1;
}

// MT = 32-row tiles of M covered by one pass (M <= 32 * MT); NS = adjacent
// 32-column stripes per workgroup (they share every activation load).
template <int EPI, int MT, int NS>
__global__ __launch_bounds__(512) void k_gemm(GemmArgs ga, EpiArgs ea) {
    extern __shared__ __align__(16) float smem[];
    // the wave index as a scalar, so each wave's K range and its batch tests
    // below are wave-uniform branches
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KW = ga.KW;
    const int KS = ga.K >> 4;  // 16-wide k steps
    const int s = blockIdx.y;
    const int a0 = (int)(((long)s * KS) / ga.S), a1 = (int)(((long)(s + 1) * KS) / ga.S);
    const int ks0 = a0 + (int)(((long)wave * (a1 - a0)) / KW);
    const int ks1 = a0 + (int)(((long)(wave + 1) * (a1 - a0)) / KW);
    const int nt = blockIdx.x * NS;  // first 32-column stripe
    const int M = ga.M;

    floatx16 acc[NS][MT];
#pragma unroll
    for (int ns = 0; ns < NS; ++ns)
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[ns][t][j] = 0.f;

    // a workgroup's last stripes may lie past the matrix (an odd stripe count
    // with NS = 2): they re-read the last stripe and their results are not stored
    const int stripes = ga.N >> 5;
    const int ns0 = min(nt, stripes - 1);
    const __amdgpu_buffer_rsrc_t wr = tile_rsrc(reinterpret_cast<const u32x4*>(ga.Wp) + (size_t)ns0 * KS * 64,
                                                (size_t)min(NS, stripes - ns0) * KS * 1024);
    int wofs[NS];
#pragma unroll
    for (int ns = 0; ns < NS; ++ns) wofs[ns] = (min(nt + ns, stripes - 1) - ns0) * KS * 1024;
    // X is in fragment layout: the operand of m-tile t at k step k is the 1 KiB tile (t, k)
    const __amdgpu_buffer_rsrc_t xr = tile_rsrc(ga.X, (size_t)MT * KS * 1024);
    const int lofs = lane * 16;
    // D k steps in flight; a slot is loaded again as soon as its MFMAs are issued
    constexpr int D = decode_depth(MT, NS);
    u32x4 w[D][NS], x[D][MT];
    auto load = [&](int i, int ks) {
#pragma unroll
        for (int ns = 0; ns < NS; ++ns) w[i][ns] = load_tile(wr, lofs, wofs[ns] + ks * 1024);
#pragma unroll
        for (int t = 0; t < MT; ++t) x[i][t] = load_tile(xr, lofs, (t * KS + ks) * 1024);
    };
    auto mma = [&](int i) {
#pragma unroll
        for (int ns = 0; ns < NS; ++ns)
#pragma unroll
            for (int t = 0; t < MT; ++t)
                acc[ns][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[i][ns]),
                                                                     __builtin_bit_cast(bf16x8, x[i][t]), acc[ns][t], 0, 0, 0);
    };
    const int n = ks1 - ks0, groups = n / D, rem = n - groups * D;
    if (groups > 0) {
#pragma unroll
        for (int i = 0; i < D; ++i) load(i, ks0 + i);
    } else {
#pragma unroll
        for (int i = 0; i < D - 1; ++i)
            if (i < rem) load(i, ks0 + i);
    }

    // q/k/v epilogue inputs, loaded while the weight stream is in flight (no
    // wait on them before the main loop ends); above 64 rows the RoPE factors
    // would cost more registers than the loop can spare and are loaded after it
    const int mcap = min(live_rows(ga.dn, M), MT * 32);
    const int nthr = KW * 64;
    constexpr int RP = MT <= 2 ? MT * 2 : 1;  // MT <= 2: >= mcap * 16 / nthr, as nthr >= 256
    float2 pf_rope[RP];
    int pf_pid = -1, pf_tok = 0;
    int q_part = 0, q_gi = 0;
    if constexpr (EPI == EPI_QKV) {
        static_assert(NS == 1, "the q/k/v epilogue takes one stripe");
        const int gph = ea.hd >> 5, hg = ea.H * gph;
        q_part = nt / hg;
        q_gi = (nt - q_part * hg) % gph;
        if (MT <= 2 && q_part < 2) {
#pragma unroll
            for (int r = 0; r < RP; ++r) {
                const int idx = tid + r * nthr;
                if (idx < mcap * 16)
                    pf_rope[r] = ea.rope[(size_t)(idx >> 4) * (ea.hd >> 1) + q_gi * 16 + (idx & 15)];
            }
        }
        if (q_part > 0 && tid < mcap) {  // a K or V stripe
            pf_pid = ea.kvpid[tid];
            pf_tok = ea.pos[tid] % kPage;
        }
    }

    if (groups > 0) {
        int ks = ks0 + D;
        for (int g = 1; g < groups; ++g, ks += D) {
#pragma unroll
            for (int i = 0; i < D; ++i) {
                mma(i);
                load(i, ks + i);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int i = 0; i < D; ++i) {
            mma(i);
            if (i < rem) load(i, ks + i);
        }
    }
#pragma unroll
    for (int i = 0; i < D - 1; ++i)
        if (i < rem) mma(i);

    // Sum the KW wave tiles in wave order: with 8 waves (a grid of one
    // workgroup per CU at most) all NS x MT 32x32 tiles in one round where they
    // fit in LDS (decode_red_tiles), else one tile at a time, which keeps the
    // LDS of wider grids small enough for several workgroups per CU.
    // acc[ns][t][j] holds D[n = (j/4)*8 + (lane/32)*4 + j%4][m = t*32 + lane%32]
    // of stripe nt + ns.
    constexpr int RT = decode_red_tiles(EPI == EPI_QKV, MT, NS);
    const bool one_round = RT > 1 && KW == 8;
    float* red = smem;                                   // [KW][RT or 1][32 n][32 m]
    float* fin = smem + KW * (one_round ? RT : 1) * 1024;  // [NS][32 n][MT*32 m + 1]
    const int fld = MT * 32 + 1;
    QkvStage qs{};
    if constexpr (EPI == EPI_QKV) {
        // a [MT*32][16] RoPE table; 32 * fld is even
        float2* s_rope = reinterpret_cast<float2*>(fin + 32 * fld);
        int* s_pid = reinterpret_cast<int*>(s_rope + MT * 32 * 16);
        int* s_tok = s_pid + MT * 32;
        if (q_part < 2) {  // V: no rotation
            if constexpr (MT <= 2) {
#pragma unroll
                for (int r = 0; r < RP; ++r) {
                    const int idx = tid + r * nthr;
                    if (idx < mcap * 16) s_rope[idx] = pf_rope[r];
                }
            } else {
                for (int idx = tid; idx < mcap * 16; idx += nthr)
                    s_rope[idx] = ea.rope[(size_t)(idx >> 4) * (ea.hd >> 1) + q_gi * 16 + (idx & 15)];
            }
        }
        if (tid < mcap) {
            s_pid[tid] = pf_pid;
            s_tok[tid] = pf_tok;
        }
        qs = QkvStage{s_rope, s_pid, s_tok};  // visible after the reduction's barriers
    }
    if (RT > 1 && one_round) {
#pragma unroll
        for (int ns = 0; ns < NS; ++ns)
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const int nn = (j >> 2) * 8 + (lane >> 5) * 4 + (j & 3);
                    red[(wave * RT + ns * MT + t) * 1024 + nn * 32 + (lane & 31)] = acc[ns][t][j];
                }
        __syncthreads();
        for (int e = tid; e < RT * 1024; e += nthr) {
            const int tile = e >> 10, r = e & 1023, ns = tile / MT, t = tile - ns * MT;
            float sum = 0.f;
            for (int w = 0; w < KW; ++w) sum += red[(w * RT + tile) * 1024 + r];
            fin[ns * 32 * fld + (r >> 5) * fld + t * 32 + (r & 31)] = sum;
        }
        __syncthreads();
    } else {
#pragma unroll
        for (int ns = 0; ns < NS; ++ns) {
#pragma unroll
            for (int t = 0; t < MT; ++t) {
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const int nn = (j >> 2) * 8 + (lane >> 5) * 4 + (j & 3);
                    red[wave * 1024 + nn * 32 + (lane & 31)] = acc[ns][t][j];
                }
                __syncthreads();
                for (int e = tid; e < 1024; e += nthr) {
                    float sum = 0.f;
                    for (int w = 0; w < KW; ++w) sum += red[w * 1024 + e];
                    fin[ns * 32 * fld + (e >> 5) * fld + t * 32 + (e & 31)] = sum;
                }
                __syncthreads();
            }
        }
    }

    stripe_epilogue<EPI>(fin, fld, nt, NS, mcap, s, tid, nthr, ga, ea, qs);
}

// Register tile GEMM: prefill chunks, and loop steps, preludes and codas of more rows
// than the skinny kernel takes (gemm_shape).
//
// A workgroup owns a (32 WM)-row x (32 WN)-column output tile and one K split;
// its 4 waves (one per SIMD, up to 512 registers each) split that K range and
// each accumulates the whole tile, so every operand tile is fetched exactly
// once per workgroup, straight into registers: no LDS staging, no barrier in
// the loop, and up to 8 k steps of WM + WN KiB per wave in flight (200 KiB per
// CU).  What bounds these shapes is the operand stream into a CU (L2 hits reach
// 130 KB per us and CU, of which WM x WN = 4 x 3 tiles need 7 KiB per 12 MFMAs)
// and the launch and epilogue around a loop of 10-15 us; a 32 KiB two-stage LDS
// ring kept too few bytes in flight.  The waves' tiles are then exchanged
// through LDS (wave w sums m-tile w, in wave order) and the epilogue runs from
// the accumulators: lane l holds row l % 32 and, for each j, column (j/4)*8 +
// (l/32)*4 + j%4, so 4 consecutive j are 4 consecutive columns, and the RoPE /
// SwiGLU partner of element j is j ^ 8.
//
// Against the kernel of 2 x 2 waves that each fetched their own operands, Ouro
// widths at 512 rows: q/k/v 35.4 -> 23.8 us, O 12.9 -> 11.5, down 24.6 -> 21.9;
// at 333 rows q/k/v 34.9 -> 22.8; Huginn widths at 300 rows: q/k/v 135 -> 95,
// O 40 -> 36, down 124 -> 104, adapter 141 -> 84.
//
// Tile order: the dispatcher hands workgroup b to XCD b % 8, so each XCD takes
// a contiguous range of tasks, row tile first: the row tiles that read one
// weight tile run together on one XCD and share its L2.
__host__ __device__ constexpr int tile_depth(int WM, int WN) { return 200 / (4 * (WM + WN)) < 8 ? 200 / (4 * (WM + WN)) : 8; }

template <int EPI, int WM, int WN>
__device__ __forceinline__ void tile_epilogue(const floatx16 (&acc)[WN], int m, int live, int nt0, int split, int lane,
                                              const GemmArgs& ga, const EpiArgs& ea) {
    const int stripes = ga.N >> 5, half = lane >> 5;
    if (EPI == EPI_QKV) {
        const int gph = ea.hd >> 5, hg = ea.H * gph, half_hd = ea.hd >> 1;
        const int mc = min(m, ga.M - 1);
        const int pid = ea.kvpid[mc], tok = ea.pos[mc] % kPage;
        // the row's RoPE factors first: the stores may alias them
        float4 cs[WN][4];
#pragma unroll
        for (int a = 0; a < WN; ++a) {
            const int gi = (min(nt0 + a, stripes - 1) % hg) % gph;
            const float2* r = ea.rope + (size_t)mc * half_hd + gi * 16 + half * 4;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                cs[a][2 * u] = *reinterpret_cast<const float4*>(r + u * 8);
                cs[a][2 * u + 1] = *reinterpret_cast<const float4*>(r + u * 8 + 2);
            }
        }
        if (m >= live) return;
#pragma unroll
        for (int a = 0; a < WN; ++a) {
            const int g = nt0 + a;
            if (g >= stripes) break;
            const int part = g / hg, rem = g - part * hg;
            const int head = rem / gph, gi = rem - head * gph;
#pragma unroll
            for (int u = 0; u < 2; ++u) {  // pairs jj = 8u + 4 half + 0..3 of the stripe's 16
                float lo[4], hi[4];
                const float c[8] = {cs[a][2 * u].x, cs[a][2 * u].y, cs[a][2 * u].z, cs[a][2 * u].w,
                                    cs[a][2 * u + 1].x, cs[a][2 * u + 1].y, cs[a][2 * u + 1].z, cs[a][2 * u + 1].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float xf = acc[a][u * 4 + i], xs = acc[a][8 + u * 4 + i];
                    lo[i] = part < 2 ? rope_first(xf, xs, c[2 * i], c[2 * i + 1]) : xf;
                    hi[i] = part < 2 ? rope_second(xf, xs, c[2 * i], c[2 * i + 1]) : xs;
                }
                const int dim = gi * 16 + u * 8 + half * 4;
                if (part == 0) {
                    float* dst = ea.q + (size_t)m * (ea.H * ea.hd) + head * ea.hd + dim;
                    *reinterpret_cast<float4*>(dst) = make_float4(lo[0], lo[1], lo[2], lo[3]);
                    *reinterpret_cast<float4*>(dst + half_hd) = make_float4(hi[0], hi[1], hi[2], hi[3]);
                } else if (pid >= 0) {  // -1: unmapped (reported by the row-entry kernel)
                    const KvTarget& kv = ea.kv;
                    uint16_t* dst = kv.pool + kv_offset(kv.layer, pid, kv.n_pages, part - 1, head, ea.H, tok, ea.hd) + dim;
                    *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]));
                    *reinterpret_cast<uint2*>(dst + half_hd) = make_uint2(pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3]));
                }
            }
        }
        return;
    }
    if (m >= live) return;
#pragma unroll
    for (int a = 0; a < WN; ++a) {
        if (nt0 + a >= stripes) break;
        if (EPI == EPI_SWIGLU) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float g = acc[a][u * 4 + i];
                    v[i] = g / (1.0f + __expf(-g)) * acc[a][8 + u * 4 + i];
                }
                const int f = (nt0 + a) * 16 + u * 8 + half * 4;
                *reinterpret_cast<uint2*>(ea.act + frag_index(m, f, ea.ld_act)) =
                    make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
            }
        } else {
            float* dst = (EPI == EPI_PARTIAL ? ga.part + ((size_t)split * ga.M + m) * ga.N : ea.out + (size_t)m * ea.ld_out) +
                         (nt0 + a) * 32 + half * 4;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                store4<EPI>(dst + u * 8, acc[a][u * 4], acc[a][u * 4 + 1], acc[a][u * 4 + 2], acc[a][u * 4 + 3]);
        }
    }
}

// Stripes per round of the exchange: all of them where the four waves' copies of WM x
// WN tiles fit in LDS, else half.
__host__ __device__ constexpr int tile_exchange_stripes(int WM, int WN) {
    return 4 * WM * WN * 1024 * 4 <= 160 * 1024 ? WN : (WN + 1) / 2;
}

template <int EPI, int WM, int WN, int PASSES>
__global__ __launch_bounds__(256) void k_gemm_tile(GemmArgs ga, EpiArgs ea, TileShape ts) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KS = ga.K >> 4, stripes = ga.N >> 5;
    const int mtiles = gemm_rows(ga.M) >> 5;  // m-tiles the activation buffer holds
    const int tasks = ts.gx * ts.gy * ts.S, per = (tasks + 7) / 8;
    const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || t >= tasks) return;
    const int by = t % ts.gy, s = (t / ts.gy) % ts.S, bx = t / (ts.gy * ts.S);
    const int a0 = (int)(((long)s * KS) / ts.S), a1 = (int)(((long)(s + 1) * KS) / ts.S);
    const int nt0 = bx * WN, mt0 = by * WM;

    floatx16 acc[WM][WN];
#pragma unroll
    for (int b = 0; b < WM; ++b)
#pragma unroll
        for (int a = 0; a < WN; ++a)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[b][a][j] = 0.f;

    // tiles past the matrix re-read the last one (their results are not stored)
    const u32x4* wsrc[WN];
    const u32x4* xsrc[WM];
#pragma unroll
    for (int a = 0; a < WN; ++a)
        wsrc[a] = reinterpret_cast<const u32x4*>(ga.Wp) + (size_t)min(nt0 + a, stripes - 1) * KS * 64;
#pragma unroll
    for (int b = 0; b < WM; ++b)
        xsrc[b] = reinterpret_cast<const u32x4*>(ga.X) + (size_t)min(mt0 + b, mtiles - 1) * KS * 64;
    constexpr int D = tile_depth(WM, WN);
    u32x4 w[D][WN], x[D][WM];
    auto load = [&](int i, int ks) {
#pragma unroll
        for (int a = 0; a < WN; ++a) w[i][a] = wsrc[a][(size_t)ks * 64 + lane];
#pragma unroll
        for (int b = 0; b < WM; ++b) x[i][b] = xsrc[b][(size_t)ks * 64 + lane];
    };
    auto mma = [&](int i) {
#pragma unroll
        for (int b = 0; b < WM; ++b)
#pragma unroll
            for (int a = 0; a < WN; ++a)
                acc[b][a] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[i][a]),
                                                                    __builtin_bit_cast(bf16x8, x[i][b]), acc[b][a], 0, 0, 0);
    };
    // The K range is cut into 4 PASSES parts, as the skinny kernel cuts it over
    // its waves: wave w takes part w and, of 8, then part w + 4; the parts are
    // summed in order.  Groups of D k steps: a slot's next load is issued as soon
    // as its MFMAs are.
    auto part_begin = [&](int part) { return a0 + (part * (a1 - a0)) / (4 * PASSES); };
    extern __shared__ __align__(16) float smem[];
    constexpr int EX = tile_exchange_stripes(WM, WN);
    floatx16 sum[WN];
#pragma unroll
    for (int a = 0; a < WN; ++a)
#pragma unroll
        for (int j = 0; j < 16; ++j) sum[a][j] = 0.f;
    int ks = part_begin(wave), groups = (part_begin(wave + 1) - ks) / D, rem = part_begin(wave + 1) - ks - groups * D;
    if (groups > 0) {
#pragma unroll
        for (int i = 0; i < D; ++i) load(i, ks + i);
    } else {
#pragma unroll
        for (int i = 0; i < D - 1; ++i)
            if (i < rem) load(i, ks + i);
    }
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
        if (pass > 0) {
#pragma unroll
            for (int b = 0; b < WM; ++b)
#pragma unroll
                for (int a = 0; a < WN; ++a)
#pragma unroll
                    for (int j = 0; j < 16; ++j) acc[b][a][j] = 0.f;
        }
        if (groups > 0) {
            for (int g = 1; g < groups; ++g, ks += D) {
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    mma(i);
                    load(i, ks + D + i);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int i = 0; i < D; ++i) {
                mma(i);
                if (i < rem) load(i, ks + D + i);
            }
        }
#pragma unroll
        for (int i = 0; i < D - 1; ++i)
            if (i < rem) mma(i);
        // exchange: wave v's copy of (m-tile b, stripe a), in lane order
#pragma unroll
        for (int r = 0; r < WN; r += EX) {
            if (r > 0 || pass > 0) __syncthreads();  // the round before has been read
            constexpr int NE = EX;
#pragma unroll
            for (int b = 0; b < WM; ++b)
#pragma unroll
                for (int a = r; a < r + NE && a < WN; ++a) {
                    float4* dst = reinterpret_cast<float4*>(smem) + (size_t)((wave * WM + b) * NE + a - r) * 256 + lane;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        dst[u * 64] = make_float4(acc[b][a][u * 4], acc[b][a][u * 4 + 1], acc[b][a][u * 4 + 2], acc[b][a][u * 4 + 3]);
                }
            __syncthreads();
            if (wave < WM) {
#pragma unroll
                for (int a = r; a < r + NE && a < WN; ++a)
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        float4 v = make_float4(sum[a][u * 4], sum[a][u * 4 + 1], sum[a][u * 4 + 2], sum[a][u * 4 + 3]);
#pragma unroll
                        for (int src = 0; src < 4; ++src) {
                            const float4 p = reinterpret_cast<const float4*>(smem)[(size_t)((src * WM + wave) * NE + a - r) * 256 + u * 64 + lane];
                            v.x += p.x;
                            v.y += p.y;
                            v.z += p.z;
                            v.w += p.w;
                        }
                        sum[a][u * 4] = v.x;
                        sum[a][u * 4 + 1] = v.y;
                        sum[a][u * 4 + 2] = v.z;
                        sum[a][u * 4 + 3] = v.w;
                    }
            }
        }
        if (pass + 1 < PASSES) {  // the second part's first loads (before the exchange they would exceed the registers)
            ks = part_begin(wave + 4);
            groups = (part_begin(wave + 5) - ks) / D;
            rem = part_begin(wave + 5) - ks - groups * D;
            if (groups > 0) {
#pragma unroll
                for (int i = 0; i < D; ++i) load(i, ks + i);
            } else {
#pragma unroll
                for (int i = 0; i < D - 1; ++i)
                    if (i < rem) load(i, ks + i);
            }
        }
    }
    if (wave < WM) tile_epilogue<EPI, WM, WN>(sum, (mt0 + wave) * 32 + (lane & 31), live_rows(ga.dn, ga.M), nt0, s, lane, ga, ea);
}

// Tile GEMM staged through LDS, for gate/up above 256 rows and full-width LM heads
// of prefill chunks: (64 WM)-row x 128-column tiles, 4 waves in 2 x 2, each 32 WM rows x 64
// columns.  Their grids take more than one round of k_gemm_tile's workgroups
// (one per CU), where two smaller ones per CU overlap one's start and epilogue
// with the other's loop: Ouro-shaped gate/up at 512 rows 36 us against 40,
// Huginn-shaped at 300 rows 183 against 217, LM heads 113 against 128 and 339
// against 365.
//
// xcd_order: the tasks of an XCD are a contiguous range, row tile first (used
// for grids of more than two workgroups per CU), else column group first.
template <int EPI, int WM>
__global__ __launch_bounds__(256) void k_gemm_lds(GemmArgs ga, EpiArgs ea, int xcd_order) {
    static_assert(WM == 1 || WM == 2, "one or two m-tiles per wave");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KS = ga.K >> 4;
    const int stripes = ga.N >> 5;
    const int mtiles = gemm_rows(ga.M) >> 5;  // m-tiles the activation buffer holds
    const int gx = (stripes + 3) / 4, gy = (ga.M + 64 * WM - 1) / (64 * WM), tasks = gx * gy;
    int bx, by;
    if (xcd_order) {
        const int per = (tasks + 7) / 8;
        const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
        if (t >= tasks) return;
        by = t % gy;
        bx = t / gy;
    } else {
        const int t = blockIdx.x;
        if (t >= tasks) return;
        bx = t % gx;
        by = t / gx;
    }
    const int nt0 = bx * 4 + (wave & 1) * 2;   // first stripe of this wave
    const int mt0 = by * 2 * WM + (wave >> 1) * WM;  // first m-tile of this wave

    floatx16 acc[WM][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < WM; ++b)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[b][a][j] = 0.f;
    // LDS ring of 2 stages of 4 k steps: a stage holds the workgroup's 4
    // weight tiles and 2 WM activation tiles of each k step (1 KiB each,
    // lane order), copied global -> LDS by the waves with direct loads (tile
    // i of a stage by wave i % 4); each wave then reads its 2 + WM operands
    // per k step
    constexpr int CH = 4, NBUF = 2;
    constexpr int TPK = 4 + 2 * WM;  // tiles per k step
    constexpr int TPS = CH * TPK;    // tiles per stage
    constexpr int LPW = TPS / 4;     // loads per wave per stage
    static_assert(TPS % 4 == 0, "a stage's tiles split evenly over the 4 waves");
    extern __shared__ __align__(16) unsigned char lds_ring[];
    const int ntb = bx * 4, mtb = by * 2 * WM;
    const u32x4* Wg = reinterpret_cast<const u32x4*>(ga.Wp);
    const u32x4* Xg = reinterpret_cast<const u32x4*>(ga.X);
    const int nst = (KS + CH - 1) / CH;
    auto issue = [&](int st) {
        unsigned char* base = lds_ring + (size_t)(st % NBUF) * TPS * 1024;
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int t = wave + 4 * i;  // tile within the stage
            const int kk = t / TPK, slot = t - kk * TPK;
            const int ks = min(st * CH + kk, KS - 1);
            const u32x4* src = slot < 4 ? Wg + ((size_t)min(ntb + slot, stripes - 1) * KS + ks) * 64
                                        : Xg + ((size_t)min(mtb + slot - 4, mtiles - 1) * KS + ks) * 64;
            __builtin_amdgcn_global_load_lds(src + lane, (__attribute__((address_space(3))) void*)(base + t * 1024),
                                             16, 0, 0);
        }
    };
    if (nst > 0) issue(0);
    const int wn = wave & 1, wm = wave >> 1;
    for (int st = 0; st < nst; ++st) {
        // this wave's loads of stage st are done; the barrier covers the
        // other waves' loads and every wave's reads of the stage refilled next
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        if (st + 1 < nst) issue(st + 1);
        const unsigned char* base = lds_ring + (size_t)(st % NBUF) * TPS * 1024 + lane * 16;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const uint32_t keep = st * CH + i < KS ? 0xffffffffu : 0u;
            u32x4 w[2], x[WM];
#pragma unroll
            for (int a = 0; a < 2; ++a)
                w[a] = *reinterpret_cast<const u32x4*>(base + (i * TPK + wn * 2 + a) * 1024);
#pragma unroll
            for (int b = 0; b < WM; ++b)
                x[b] = *reinterpret_cast<const u32x4*>(base + (i * TPK + 4 + wm * WM + b) * 1024);
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const bf16x8 wv = __builtin_bit_cast(bf16x8, w[a] & keep);
#pragma unroll
                for (int b = 0; b < WM; ++b)
                    acc[b][a] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, __builtin_bit_cast(bf16x8, x[b]),
                                                                        acc[b][a], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int b = 0; b < WM; ++b)
        tile_epilogue<EPI, WM, 2>(acc[b], (mt0 + b) * 32 + (lane & 31), ga.M, nt0, 0, lane, ga, ea);
}

// Which projections of prefill chunks take the LDS-staged kernel: gate/up above 256
// rows (figures at the kernel; up to there k_gemm_tile is ahead, LDS-staged against
// it at Ouro widths 27.6 and 19.6 us at 130 rows, 29.9 and 22.4 at 256, at Huginn
// widths 160 and 123, 181 and 139), and wide LM heads at every row count (130 rows
// 69 and 69 us, 256 rows 83 and 90).
static bool lds_tiles(int epi, int N, int M) { return (epi == EPI_SWIGLU && M > 256) || (epi == EPI_STORE && N >= 8192); }
// m-tiles per wave of that kernel: 1 where the rows span an odd number of
// 64-row tiles, which 128-row tiles would pad by 64 rows (gate/up at 300 rows:
// 36.0 -> 30.1 us; at 512 rows 64-row tiles gain nothing).
static int lds_wave_mtiles(int M) { return ((M + 63) / 64) % 2 ? 1 : 2; }

// Launch shape of the tile kernel.  Row groups of 3 or 4 m-tiles, whichever
// pads fewer; 2 (split-K epilogue only), 3 or 4 stripes and the K splits by the
// rounds that the grid takes on the 256 CUs (a workgroup fills one), each
// costing its k steps per wave and a fixed part (in KiB of operands), plus the
// split partials' trip through memory.  fixed_S: the splits are given (gemm_shape's
// may be more than the 8 that are tried here); two_parts: the kernel whose waves run
// two parts of K each.
TileShape tile_shape(int N, int K, int M, int epi, int fixed_S, bool two_parts) {
    const int mt = (M + 31) / 32, stripes = N / 32, KS = K / 16;
    // (two parts over 4 x 3 tiles spill: 192 registers with q/k/v's epilogue, 39 us against 24 with 3 m-tiles at 200
    // Ouro-shaped rows; 79 with the others, where the fewer rounds are worth it: gate/up 31 us against 40)
    const int most = two_parts && epi == EPI_QKV ? 3 : 4, gy = (mt + most - 1) / most, WM = std::max(3, (mt + gy - 1) / gy);
    TileShape best{};
    double cost = 1e30;
    for (int WN = epi == EPI_PARTIAL ? 2 : 3; WN <= (WM == 4 || two_parts ? 3 : 4); ++WN)  // (4 x 4 tiles exceed the register file)
        for (int S = fixed_S ? fixed_S : 1; S <= (fixed_S ? fixed_S : epi == EPI_PARTIAL ? 8 : 1); ++S) {
            if (!fixed_S && S > 1 && KS / S < 32) continue;
            const int gx = (stripes + WN - 1) / WN, rounds = (gx * gy * S + 255) / 256;
            const double steps = (double)((KS + S - 1) / S + 3) / 4;
            const double c = rounds * (steps * (WM + WN) + 100) + 70.0 * (S - 1) * ((double)M * N / (1 << 20));
            if (c < cost) {
                cost = c;
                best = TileShape{WM, WN, gx, gy, S};
            }
        }
    return best;
}

GemmShape gemm_shape_mn(int N, int K, int M, int epi) { return GemmShape{N, K, tile_shape(N, K, M, epi).S, 4, kTileShapes}; }

GemmShape gemm_shape(int N, int K, int epi, int M) {
    // S and KW fix every wave's K range and so the summation order of each
    // output: they depend on (N, K, epi) only, which keeps a row's result
    // independent of the rows that share its call.  NS (stripes per
    // workgroup) only regroups whole stripes, and follows the row count.
    const int stripes = N / 32;
    const int KS = K / 16;
    // K split until the grid covers the chip, keeping at least 64 k steps per
    // workgroup (a 4-way split of a 2048-long K loses more to each workgroup's
    // fixed costs than its extra workgroups gain: Ouro's O at 64 rows 6.4 ->
    // 5.8 us with 2 ways)
    int S = 1;
    if (epi == EPI_PARTIAL) {
        while (stripes * S < 256 && KS / (S * 2) >= 64) S *= 2;
    }
    // Wide projections without a K split (gate/up, LM head): two stripes per
    // workgroup share every activation load.
    const bool pair_wide = epi != EPI_QKV && epi != EPI_PARTIAL && S == 1 && stripes > 256 && stripes % 2 == 0 &&
                           KS >= 64;
    // Long K ranges (Huginn widths): 4 waves per workgroup at every row count,
    // which lets the tile kernel serve more than 64 rows with the same sums in
    // one pass (there each weight byte brings 4 activation bytes, and the skinny
    // kernel read the activations once per two stripes: at 128 rows gate/up
    // 121 -> 104 us, O 27 -> 18, down 71 -> 52, q/k/v 53 -> 55).  Split so that pairs of
    // stripes fill the chip once in the tile kernel (3 ways for 165 stripes); in
    // the skinny kernel two such workgroups share a CU (9 rows, O, down and
    // adapter together: 304 -> 246 us per step against 2 ways and 8 waves).
    // Where 8 waves fill the chip in one round, 4 cost the skinny kernel up to 2%
    // of a step and give the tile kernel more: 2 layers of d 3072 at 48 rows 304
    // and 299 us, at 160 rows 532 and 573; 1 layer of d 8192 at 64 rows 581 and
    // 572, at 65 rows 538 and 590 (4 waves against 8).
    if (KS / S >= 160) {
        int T = 1;
        if (epi == EPI_PARTIAL) {
            T = 256 / ((stripes + 1) / 2);
            T = T < 1 ? 1 : (T > 8 ? 8 : T);
            while (T > 1 && KS / T < 64) --T;
        }
        return GemmShape{N, K, T, 4, M > 64 ? kTileFixed : (pair_wide ? 2 : 1)};
    }
    const int NS = pair_wide ? 2 : 1;
    // waves per workgroup: 8 (more weight bytes in flight per CU) while the
    // grid fits the chip in one round, counted with the stripe pairs where
    // they may be used, else 4
    const int groups = pair_wide ? (stripes + 1) / 2 : stripes;
    const int KW = groups * S <= 256 && KS / S >= 32 ? 8 : 4;
    // Above 128 rows a skinny workgroup would hold 8 tiles of accumulators and
    // little in flight; the register tile kernel runs the same K parts (Ouro
    // widths at 140 rows: q/k/v 27.4 -> 23.6 us, gate/up 46.1 -> 23.3, O and down
    // 18.3 -> 13.4; at 100 rows the skinny kernel's 17.7 and 22.5 us are ahead).
    return GemmShape{N, K, S, KW, M > 128 ? kTileFixed : NS};
}

// The K splits a call's accepted size is reckoned with (see ws_layout).
int gemm_reference_splits(int N, int K) {
    int S = 1;
    while (N / 32 * S < 256 && K / 16 / (S * 2) >= 64) S *= 2;
    return S;
}

template <int EPI, int MT, int NS>
static hipError_t launch_mt(const GemmArgs& ga, const EpiArgs& ea, hipStream_t st) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm<EPI, MT, NS>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int rt = decode_red_tiles(EPI == EPI_QKV, MT, NS);
    size_t lds = ((size_t)ga.KW * (rt > 1 && ga.KW == 8 ? rt : 1) * 1024 + (size_t)NS * 32 * (MT * 32 + 1)) * 4;
    if (EPI == EPI_QKV) lds += (size_t)MT * 32 * 16 * 8 + (size_t)MT * 32 * 2 * 4;
    dim3 grid((ga.N / 32 + NS - 1) / NS, ga.S);
    k_gemm<EPI, MT, NS><<<grid, ga.KW * 64, lds, st>>>(ga, ea);
    return hipGetLastError();
}

template <int EPI, int NS>
static hipError_t launch_ns(const GemmArgs& ga, const EpiArgs& ea, hipStream_t st) {
    if (ga.M <= 32) return launch_mt<EPI, 1, NS>(ga, ea, st);
    if (ga.M <= 64) return launch_mt<EPI, 2, NS>(ga, ea, st);
    return launch_mt<EPI, 4, NS>(ga, ea, st);
}

template <int EPI>
static hipError_t launch_epi(const GemmArgs& ga, const EpiArgs& ea, int ns, hipStream_t st) {
    if (ns == 1) return launch_ns<EPI, 1>(ga, ea, st);
    if constexpr (EPI == EPI_QKV || EPI == EPI_PARTIAL)
        return hipErrorInvalidValue;  // gemm_shape pairs stripes of gate/up and LM heads only
    else
        return launch_ns<EPI, 2>(ga, ea, st);
}

template <int EPI, int WM>
static hipError_t launch_lds_wm(const GemmArgs& ga, const EpiArgs& ea, hipStream_t st) {
    const int tasks = (ga.N / 32 + 3) / 4 * ((ga.M + 64 * WM - 1) / (64 * WM));
    constexpr size_t ring = 2 * 4 * (4 + 2 * WM) * 1024;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_lds<EPI, WM>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)ring);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    k_gemm_lds<EPI, WM><<<dim3((tasks + 7) / 8 * 8), 256, ring, st>>>(ga, ea, tasks > 512 ? 1 : 0);
    return hipGetLastError();
}

template <int EPI>
static hipError_t launch_lds(const GemmArgs& ga, const EpiArgs& ea, hipStream_t st) {
    return lds_wave_mtiles(ga.M) == 1 ? launch_lds_wm<EPI, 1>(ga, ea, st) : launch_lds_wm<EPI, 2>(ga, ea, st);
}

template <int EPI, int WM, int WN, int PASSES>
static hipError_t launch_tile_passes(const GemmArgs& ga, const EpiArgs& ea, const TileShape& ts, hipStream_t st) {
    constexpr int lds = 4 * WM * tile_exchange_stripes(WM, WN) * 1024 * 4;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_tile<EPI, WM, WN, PASSES>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const dim3 grid((ts.gx * ts.gy * ts.S + 7) / 8 * 8);
    k_gemm_tile<EPI, WM, WN, PASSES><<<grid, 256, lds, st>>>(ga, ea, ts);
    return hipGetLastError();
}

template <int EPI, int WM, int WN>
static hipError_t launch_tile_shape(const GemmArgs& ga, const EpiArgs& ea, const TileShape& ts, hipStream_t st) {
    if (ga.KW != 8) return launch_tile_passes<EPI, WM, WN, 1>(ga, ea, ts, st);
    if constexpr (WN == 4 || (EPI == EPI_QKV && WM == 4))
        return hipErrorInvalidValue;  // tile_shape gives two parts no such tile
    else
        return launch_tile_passes<EPI, WM, WN, 2>(ga, ea, ts, st);
}

template <int EPI>
static hipError_t launch_tile(const GemmArgs& ga, const EpiArgs& ea, hipStream_t st) {
    const TileShape ts = tile_shape(ga.N, ga.K, ga.M, EPI, ga.S, ga.KW == 8);
    if (ts.S != ga.S) return hipErrorInvalidValue;
    if constexpr (EPI == EPI_PARTIAL) {
        if (ts.WN == 2)
            return ts.WM == 3 ? launch_tile_shape<EPI, 3, 2>(ga, ea, ts, st) : launch_tile_shape<EPI, 4, 2>(ga, ea, ts, st);
    }
    if (ts.WM == 3)
        return ts.WN == 3 ? launch_tile_shape<EPI, 3, 3>(ga, ea, ts, st) : launch_tile_shape<EPI, 3, 4>(ga, ea, ts, st);
    if (ts.WM == 4 && ts.WN == 3) return launch_tile_shape<EPI, 4, 3>(ga, ea, ts, st);
    return hipErrorInvalidValue;
}

hipError_t launch_gemm(int epi, const uint16_t* X, const uint16_t* Wp, int M, GemmShape g, float* part,
                       const EpiArgs& ea, hipStream_t st, const int32_t* dn) {
    if (M <= 0) return hipSuccess;
    if (g.K % 16 || g.N % 32 || g.S < 1 || (g.KW != 4 && g.KW != 8)) return hipErrorInvalidValue;
    GemmArgs ga{X, Wp, M, g.N, g.K, g.S, g.KW, part, dn};
    if (g.NS == kTileShapes) {  // shape from gemm_shape_mn
        if (M > kMaxPrefillRows || dn) return hipErrorInvalidValue;
        switch (epi) {
            case EPI_QKV: return launch_tile<EPI_QKV>(ga, ea, st);
            case EPI_SWIGLU:
                return lds_tiles(epi, g.N, M) ? launch_lds<EPI_SWIGLU>(ga, ea, st) : launch_tile<EPI_SWIGLU>(ga, ea, st);
            case EPI_PARTIAL: return launch_tile<EPI_PARTIAL>(ga, ea, st);
            default:
                return lds_tiles(epi, g.N, M) ? launch_lds<EPI_STORE>(ga, ea, st) : launch_tile<EPI_STORE>(ga, ea, st);
        }
    }
    if (g.NS == kTileFixed) {
        switch (epi) {
            case EPI_QKV: return launch_tile<EPI_QKV>(ga, ea, st);
            case EPI_SWIGLU: return launch_tile<EPI_SWIGLU>(ga, ea, st);
            case EPI_PARTIAL: return launch_tile<EPI_PARTIAL>(ga, ea, st);
            default: return launch_tile<EPI_STORE>(ga, ea, st);
        }
    }
    if (M > 128 || g.KW > kMaxKw || (g.NS != 1 && g.NS != 2)) return hipErrorInvalidValue;
    if (epi == EPI_QKV && g.KW < 4) return hipErrorInvalidValue;  // epilogue staging: >= 256 threads
    switch (epi) {
        case EPI_QKV: return launch_epi<EPI_QKV>(ga, ea, g.NS, st);
        case EPI_SWIGLU: return launch_epi<EPI_SWIGLU>(ga, ea, g.NS, st);
        case EPI_PARTIAL: return launch_epi<EPI_PARTIAL>(ga, ea, g.NS, st);
        default: return launch_epi<EPI_STORE>(ga, ea, g.NS, st);
    }
}

}  // namespace cdb
