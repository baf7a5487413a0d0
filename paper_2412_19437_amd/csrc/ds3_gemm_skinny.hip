// Block-scaled FP8 GEMM for few activation rows or few output tiles (decode
// batches, small layers, the weight gradient of a narrow layer): the product of
// ds3_gemm.hip, split for a different bound.
//
// Such a call is not bound by the matrix pipe but by how many bytes are in flight
// and by how long one workgroup's K-loop is.  The main kernel's 128x128 tiles
// leave most compute units without work, keep LDS for activation rows that do
// not exist, and walk all of K one step after another.  Here a workgroup takes
// BN weight rows by BM activation rows with NS stages in LDS, NS-1 of them in
// flight, and WK groups of waves take every WK-th K-step each; their partial
// sums meet in LDS in fixed order (no workspace, no second kernel, the result
// does not depend on timing).
//
// Measured against the main kernel on MI355X, kernels alone, weights from HBM
// (us, before -> now; M x N x K): 32x18432x7168 52 -> 26 (2.5 -> 5.1 TB/s of
// weights), 32x4096x7168 35 -> 13, 256x512x1024 10.2 -> 4.0, 512x2048x2048 15.8
// -> 9.1, 1024x1024x4096 27 -> 13.5; per-row scales, accumulating FP32 output:
// 512x1024x4096 35 -> 15.
// Experts' groups of few rows take the same kernel (`launch_grouped` below).
// What is left at 32 rows x 18432 is the compute units without a tile (231 of 256
// have one) and the start and end of a tile; the smallest calls are a launch and
// one latency per stage.
#include <algorithm>

#include "ds3_dev.h"
#include "ds3_internal.h"

namespace ds3 {

template <int FN_, int FM_, int WN_, int WK_, int NS_>
struct SkinnyCfg {
    static constexpr int FN = FN_, FM = FM_, WN = WN_, WK = WK_, NS = NS_;
    static constexpr int NT = 64 * WN * WK;
    static constexpr int BN = WN * FN * 16, BM = FM * 16;
    static constexpr int ROWS = BN + BM;               // rows of one K-step's codes
    static constexpr int GROUP = ROWS * 128;           // bytes of codes per K-step
    static constexpr int NSA = (BM + 63) / 64;         // activation-scale loads per wave and stage (one row a lane)
    static constexpr int SCALES = (NSA + 1) * 256;     // per wave and stage: the activation scales, then the weight block's
    static constexpr int STAGE = WK * GROUP + WN * WK * SCALES;
    static constexpr int NB = 2 * FN, NA = (BM / 8 + WN - 1) / WN;      // code loads per thread and stage: weights, activations
    static constexpr int LOADS = NB + NA + NSA + 1;         // vector-memory operations per wave and stage
    static constexpr int RLD = BN + 4;                 // floats per row of the reduction buffer
    static constexpr int RED = WK * BM * RLD * 4;
    static constexpr int LDS_BYTES = (NS * STAGE > RED ? NS * STAGE : RED);
    static_assert(FN * 16 <= 64, "one weight-scale block per wave, one weight row a lane");
    static_assert(NS >= 2 && (NS - 2) * LOADS < 64, "vmcnt immediate");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

// GROUPED: experts' groups of rows, each against its own weights; SWIQ: with SwiGLU and the 1x128 quantizer of the
// next Linear's input on the tile (gate and up rows interleaved in blocks of 128, as in ds3_gemm.hip).  Both with
// WK == 1: every output element is then the main kernel's sequence of operations, bit for bit.
template <class C, bool ROWSB, bool OUT_BF16, bool POW2, bool GROUPED = false, bool SWIQ = false>
__global__ __launch_bounds__(C::NT) void gemm_skinny_kernel(const GemmParams p) {
    static_assert(!GROUPED || (C::WK == 1 && !ROWSB), "grouped: one wave group, block scales");
    static_assert(!SWIQ || (GROUPED && C::BN == 256), "a gate and an up block per tile");
    constexpr int FN = C::FN, FM = C::FM, WN = C::WN, WK = C::WK, NS = C::NS, BN = C::BN, BM = C::BM;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[C::LDS_BYTES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, wk = wave / WN;
    const int l16 = lane & 15, g4 = lane >> 4;
    const int KB = p.K >> 7;

    // ---- which tile: the tile list is cut into one contiguous chunk per XCD (workgroups are dealt
    // round robin to them), row tiles innermost, so that those which share weights share an L2
    int tiles_m = p.tiles_m;                           // grouped: the host's upper bound
    [[maybe_unused]] auto group_row = [&](int g) { return min(p.group_offsets[min(g, p.G)], p.M); };
    [[maybe_unused]] auto tiles_before = [&](int g0, int& mine) -> int {   // row tiles of experts g0 .. g0 + lane; `mine`: of the last of them
        const int g = g0 + lane;
        mine = g < p.G ? max(0, group_row(g + 1) - group_row(g) + BM - 1) / BM : 0;
        int sum = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(sum, d);
            if (lane >= d) sum += o;
        }
        return sum;
    };
    [[maybe_unused]] int cum = 0, own = 0;             // of the first 64 experts, kept: most calls have no more
    if constexpr (GROUPED) {
        cum = tiles_before(0, own);
        tiles_m = __builtin_amdgcn_readlane(cum, 63);
        for (int g0 = 64; g0 < p.G; g0 += 64) {
            int unused;
            tiles_m += __builtin_amdgcn_readlane(tiles_before(g0, unused), 63);
        }
    }
    const int ntiles = tiles_m * p.tiles_n, per_xcd = (ntiles + 7) >> 3;
    const int local = (int)(blockIdx.x >> 3), t = (int)(blockIdx.x & 7) * per_xcd + local;
    if (local >= per_xcd || t >= ntiles) return;
    int n0, m0, m_end, grp = 0;
    if constexpr (GROUPED) {
        // the expert whose tiles [before * tiles_n, (before + its row tiles) * tiles_n) hold t
        int before = 0, g0 = 0;
        for (;;) {
            const unsigned long long past = __ballot((before + cum) * p.tiles_n > t);
            if (past != 0) {
                const int l = __builtin_ctzll(past);
                const int nt_g = __builtin_amdgcn_readlane(own, l);
                before += __builtin_amdgcn_readlane(cum, l) - nt_g;
                grp = g0 + l;
                const int r = t - before * p.tiles_n;  // its column tiles, the row tiles innermost
                n0 = r / nt_g * BN;
                m0 = __builtin_amdgcn_readfirstlane(group_row(grp)) + r % nt_g * BM;
                m_end = __builtin_amdgcn_readfirstlane(group_row(grp + 1));
                break;
            }
            before += __builtin_amdgcn_readlane(cum, 63);
            g0 += 64;
            if (g0 >= p.G) return;                     // (not reached: t is below the sum over all experts)
            cum = tiles_before(g0, own);
        }
    } else {
        n0 = t / p.tiles_m * BN; m0 = t % p.tiles_m * BM; m_end = p.M;
    }
    const int m_rows = min(m_end - m0, BM);
    const int n_rows = min(p.N - n0, BN);

    // Descriptors over the tile's valid bytes: rows beyond them move no data.
    const __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(p.a + (int64_t)m0 * p.lda), 0, (int)((int64_t)(m_rows - 1) * p.lda + p.K), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_b = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(p.b + (GROUPED ? (int64_t)grp * p.b_group_stride : 0) + (int64_t)n0 * p.ldb), 0,
        (int)((int64_t)(n_rows - 1) * p.ldb + p.K), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_sa = __builtin_amdgcn_make_buffer_rsrc((void*)p.sa, 0, 0x7ffffffc, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_sb = __builtin_amdgcn_make_buffer_rsrc((void*)p.sb, 0, 0x7ffffffc, 0x00020000);

    // Each group of WN waves moves the rows of its own K-step, 8 * WN per load; 16-byte chunks are
    // XOR-swizzled by row so that a fragment read spreads over the banks.
    const int lrow = wn * 8 + (lane >> 3);
    const int gchunk = (lane & 7) ^ swz_key(lrow);
    const unsigned voff_b = (unsigned)(lrow * (int)p.ldb + gchunk * 16), voff_a = (unsigned)(lrow * (int)p.lda + gchunk * 16);
    const unsigned step_b = (unsigned)(8 * WN * (int)p.ldb), step_a = (unsigned)(8 * WN * (int)p.lda);
    // (an odd number of waves: every other load's rows have the other key; where the activation rows are no whole loads of
    // all waves, the waves beyond the last eight rows move those once more, the same bytes to the same place)
    [[maybe_unused]] const unsigned voff_b1 = (unsigned)(lrow * (int)p.ldb + (gchunk ^ 1) * 16);
    constexpr bool kOdd = WN % 2 != 0, kAgain = (BM / 8) % WN != 0;
    static_assert(!kOdd || kAgain, "load mapping");
    [[maybe_unused]] int dst_a[C::NA];
    [[maybe_unused]] unsigned voff_ai[C::NA];
    if constexpr (kAgain) {
#pragma unroll
        for (int i = 0; i < C::NA; ++i) {
            const int g = min(i * WN + wn, BM / 8 - 1), row = g * 8 + (lane >> 3);
            dst_a[i] = (BN / 8 + g) * 1024;
            voff_ai[i] = (unsigned)(row * (int)p.lda + ((lane & 7) ^ swz_key(row)) * 16);
        }
    }
    // scales: each wave fetches for itself, an activation row's per lane, and its weight block's or (per-row
    // mode) a weight row's per lane; what lies beyond the last row repeats it
    unsigned soff_a[C::NSA];
#pragma unroll
    for (int h = 0; h < C::NSA; ++h) soff_a[h] = (unsigned)((m0 + min(h * 64 + lane, m_rows - 1)) * (int)p.sar) * 4u;
    const int sb_row = ROWSB ? n0 + min(wn * FN * 16 + lane, n_rows - 1) : min((n0 + wn * FN * 16) >> 7, ((p.N + 127) >> 7) - 1);
    unsigned soff_b = (unsigned)((GROUPED ? grp * (int)p.sb_group_stride : 0) + sb_row * (int)p.sbr) * 4u;
    unsigned sa_step = (unsigned)p.sak * 4u, sb_step = (unsigned)p.sbk * 4u;   // read once, not from the kernel arguments in the loop
    asm volatile("" : "+v"(soff_b), "+s"(sa_step), "+s"(sb_step));

    uint8_t* const codes = smem + wk * C::GROUP;                            // + stage * STAGE
    uint8_t* const scales = smem + WK * C::GROUP + wave * C::SCALES;        // + stage * STAGE
    auto issue = [&](int step, int stage) {
        const int kb = step * WK + wk;
        const unsigned koff = kb < KB ? (unsigned)kb << 7 : kOobOffset;
        const int kc = min(kb, KB - 1);
        uint8_t* dst = codes + stage * C::STAGE + wn * 1024;
#pragma unroll
        for (int i = 0; i < C::NB + C::NA; ++i) {
            const bool is_b = i < C::NB;
            unsigned voff;
            uint8_t* at = dst + i * (WN * 1024);
            if (is_b) voff = (kOdd && i % 2 ? voff_b1 : voff_b) + (koff + (unsigned)i * step_b);
            else if constexpr (kAgain) {
                voff = voff_ai[i - C::NB] + koff;
                at = codes + stage * C::STAGE + dst_a[i - C::NB];
            } else voff = voff_a + (koff + (unsigned)(i - C::NB) * step_a);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(is_b ? rs_b : rs_a, (lds_ptr_t)at, 16, (int)voff, 0, 0, 0);
        }
        uint8_t* sd = scales + stage * C::STAGE;
#pragma unroll
        for (int h = 0; h < C::NSA; ++h)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_sa, (lds_ptr_t)(sd + h * 256), 4, (int)(soff_a[h] + (unsigned)kc * sa_step), 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_sb, (lds_ptr_t)(sd + C::NSA * 256), 4, (int)(soff_b + (unsigned)kc * sb_step), 0, 0, 0);
    };
    const int key = swz_key(l16);
    const int foff0 = l16 * 128 + (((2 * g4) ^ key) << 4), foff1 = l16 * 128 + (((2 * g4 + 1) ^ key) << 4);
    auto load_frag = [&](const uint8_t* base) -> i32x8 {
        const i32x4 lo = *reinterpret_cast<const i32x4*>(base + foff0);
        const i32x4 hi = *reinterpret_cast<const i32x4*>(base + foff1);
        return i32x8{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    };

    const int steps = (KB + WK - 1) / WK;
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) issue(s, s);
    f32x4 acc[FN][FM];
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    int stage = 0;
    for (int s = 0; s < steps; ++s) {
        // This step's loads have landed (those of the NS-2 steps behind it stay in flight), in every
        // wave once the barrier is passed; and every wave is done with the stage read before it.
        asm volatile("" ::: "memory");
        constexpr int keep = (NS - 2) * C::LOADS;
        __builtin_amdgcn_s_waitcnt((keep & 15) | ((keep >> 4) << 14) | 0x70);      // vmcnt(keep) lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const uint8_t* st = codes + stage * C::STAGE;
        const float* sc = reinterpret_cast<const float*>(scales + stage * C::STAGE);
        // (everything that is read from LDS in this step is read before the next loads are issued: the
        // compiler makes an LDS read behind LDS-bound loads wait for them)
        i32x8 w[FN], x[FM];
        float sav[FM];
        const float* sbs = sc + C::NSA * 64;
        [[maybe_unused]] const float sbv = ROWSB ? 1.f : sbs[0];
        [[maybe_unused]] f32x4 un[FN];                 // per-row mode: scales of the four weight rows a lane's sums belong to
        [[maybe_unused]] float ur[FN];                 // ... and of the row whose codes it feeds (power-of-two scales)
        if constexpr (ROWSB) {
#pragma unroll
            for (int i = 0; i < FN; ++i) {
                un[i] = *reinterpret_cast<const f32x4*>(sbs + i * 16 + g4 * 4);
                ur[i] = sbs[i * 16 + l16];
            }
        }
#pragma unroll
        for (int j = 0; j < FM; ++j) sav[j] = sc[j * 16 + l16];
#pragma unroll
        for (int i = 0; i < FN; ++i) w[i] = load_frag(st + (wn * FN + i) * 2048);
#pragma unroll
        for (int j = 0; j < FM; ++j) x[j] = load_frag(st + (BN + j * 16) * 128);
        __builtin_amdgcn_sched_barrier(0);
        issue(s + NS - 1, stage == 0 ? NS - 1 : stage - 1);
        __builtin_amdgcn_sched_barrier(0);
        if (s * WK + wk < KB) {
#pragma unroll
            for (int j = 0; j < FM; ++j) {
#pragma unroll
                for (int i = 0; i < FN; ++i) {
                    if constexpr (POW2) {
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                            w[i], x[j], acc[i][j], 0, 0, 0, (int)(as_u32(ROWSB ? ur[i] : sbv) >> 23), 0, (int)(as_u32(sav[j]) >> 23));
                    } else {
                        const f32x4 pr = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w[i], x[j], f32x4{0.f, 0.f, 0.f, 0.f},
                                                                                         0, 0, 0, 0, 0, 0);
                        f32x4 t;                       // (the rescale of ds3_gemm.hip)
                        if constexpr (ROWSB) t = f32x4{sav[j] * un[i].x, sav[j] * un[i].y, sav[j] * un[i].z, sav[j] * un[i].w};
                        else t.x = t.y = t.z = t.w = sav[j] * sbv;
                        acc[i][j].x = __builtin_fmaf(pr.x, t.x, acc[i][j].x);
                        acc[i][j].y = __builtin_fmaf(pr.y, t.y, acc[i][j].y);
                        acc[i][j].z = __builtin_fmaf(pr.z, t.z, acc[i][j].z);
                        acc[i][j].w = __builtin_fmaf(pr.w, t.w, acc[i][j].w);
                    }
                }
            }
        }
        stage = stage + 1 == NS ? 0 : stage + 1;
    }

    // ---- the groups' sums meet in LDS: [wk][row][column] ----
    __builtin_amdgcn_s_waitcnt(0x70);                  // no load is on its way into the stages any more
    __syncthreads();
    float* const red = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int j = 0; j < FM; ++j)
#pragma unroll
        for (int i = 0; i < FN; ++i)
            *reinterpret_cast<f32x4*>(red + (wk * BM + j * 16 + l16) * C::RLD + (wn * FN + i) * 16 + g4 * 4) = acc[i][j];
    __syncthreads();
    auto sum4 = [&](int row, int col) -> f32x4 {
        f32x4 v = *reinterpret_cast<const f32x4*>(red + row * C::RLD + col);
#pragma unroll
        for (int g = 1; g < WK; ++g) {
            const f32x4 o = *reinterpret_cast<const f32x4*>(red + (g * BM + row) * C::RLD + col);
            v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
        }
        return v;
    };
    if constexpr (SWIQ) {
        // 16 lanes a row, eight output columns each: the main kernel's epilogue, expression for expression
        const int64_t ob = n0 >> 8;                    // 1x128 tile of the output
        for (int row = tid >> 4; row < m_rows; row += C::NT / 16) {
            const float* hr = red + row * C::RLD + l16 * 8;
            unsigned int w[4], m = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned int g = pack_bf16x2(hr[2 * e], hr[2 * e + 1]), u = pack_bf16x2(hr[128 + 2 * e], hr[128 + 2 * e + 1]);
                w[e] = pack_bf16x2(silu_mul(bf16_lo(g), bf16_lo(u)), silu_mul(bf16_hi(g), bf16_hi(u)));
                m = umax(m, umax(w[e] & 0x7fff0000u, (w[e] << 16) & 0x7fff0000u));
            }
            m = row16_max_bits(m);
            const GroupScale gs = group_scale(as_f32(m), p.q_pow2);
            const int64_t grow = m0 + row;
            *reinterpret_cast<u32x2*>(p.q_out + grow * p.ldq + ob * 128 + l16 * 8) =
                u32x2{cvt4_e4m3(bf16_lo(w[0]) * gs.r, bf16_hi(w[0]) * gs.r, bf16_lo(w[1]) * gs.r, bf16_hi(w[1]) * gs.r),
                      cvt4_e4m3(bf16_lo(w[2]) * gs.r, bf16_hi(w[2]) * gs.r, bf16_lo(w[3]) * gs.r, bf16_hi(w[3]) * gs.r)};
            if (l16 == 0) p.s_out[grow * p.sor + ob * p.sok] = gs.s;
        }
        return;
    }
    for (int idx = tid; idx < m_rows * (BN / 4); idx += C::NT) {
        const int row = idx / (BN / 4), col = idx % (BN / 4) * 4;
        if (col >= n_rows) continue;
        f32x4 v = sum4(row, col);
        const int64_t at = (int64_t)(m0 + row) * p.ldc + n0 + col;
        if constexpr (OUT_BF16) {
            uint16_t* d = static_cast<uint16_t*>(p.c) + at;
            const u32x2 o = {pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)};
            if (col + 4 <= n_rows) *reinterpret_cast<u32x2*>(d) = o;
            else for (int q = 0; col + q < n_rows; ++q) d[q] = (uint16_t)((q & 2 ? o.y : o.x) >> (16 * (q & 1)));
        } else {
            float* d = static_cast<float*>(p.c) + at;
            if (col + 4 <= n_rows) {
                if (p.accumulate) {
                    const f32x4 old = *reinterpret_cast<const f32x4*>(d);
                    v.x += old.x; v.y += old.y; v.z += old.z; v.w += old.w;
                }
                *reinterpret_cast<f32x4*>(d) = v;
            } else {
                const float o[4] = {v.x, v.y, v.z, v.w};
                for (int q = 0; col + q < n_rows; ++q) d[q] = p.accumulate ? d[q] + o[q] : o[q];
            }
        }
    }
}

// ---- host side -------------------------------------------------------------------
template <class C, bool ROWSB, bool POW2>
static ds3_status launch_one(GemmParams p, ds3_dtype ct, hipStream_t st) {
    p.tiles_m = (p.M + C::BM - 1) / C::BM;
    p.tiles_n = (p.N + C::BN - 1) / C::BN;
    const dim3 grid((unsigned)(((int64_t)p.tiles_m * p.tiles_n + 7) / 8 * 8));
    (void)hipGetLastError();                            // a stale error of earlier, unrelated work is not this launch's
    if (ct == DS3_BF16) gemm_skinny_kernel<C, ROWSB, true, POW2><<<grid, dim3(C::NT), 0, st>>>(p);
    else gemm_skinny_kernel<C, ROWSB, false, POW2><<<grid, dim3(C::NT), 0, st>>>(p);
    return hipGetLastError() == hipSuccess ? DS3_OK : DS3_ERR_LAUNCH;
}

template <class C>
static ds3_status launch_cfg(const GemmParams& p, ds3_dtype ct, bool row_scales, bool pow2, hipStream_t st) {
    if (row_scales) return pow2 ? launch_one<C, true, true>(p, ct, st) : launch_one<C, true, false>(p, ct, st);
    return pow2 ? launch_one<C, false, true>(p, ct, st) : launch_one<C, false, false>(p, ct, st);
}

// The configurations and what a call takes with each: `fixed` + one round of tiles after another, a round being
// K-steps / WK stages of `full` us when every workgroup slot has a tile and `alone` us when few have, plus the sums' way
// out.  It ranks the configurations, no more: against measured times of 146 shapes that take this kernel (M 1 .. 2048, N
// 512 .. 18432, K 512 .. 18432, weights from HBM) a configuration's own figure is 8-16% off on average and more than a
// third too low where the bytes bind (there is no term for them), but the one it picks is 0.7% slower than the best of
// the five on average, 7% at worst.  (Sizes that `one_tile_waves` takes aside, below, are not ranked.)
struct SkinnyChoice { int bn, bm, wk, per_cu; float alone, full, out, fixed; };
constexpr int kSkinnyCfgs = 5;
constexpr SkinnyChoice kSkinny[kSkinnyCfgs] = {
    {32, 32, 4, 1, 0.40f, 0.55f, 1.5f, 1.5f},
    {32, 32, 2, 2, 0.25f, 0.50f, 1.0f, 1.5f},
    {128, 32, 2, 1, 0.55f, 0.70f, 1.5f, 1.5f},
    {64, 64, 2, 1, 0.50f, 0.65f, 1.5f, 1.5f},
    {128, 64, 1, 2, 0.45f, 0.85f, 1.5f, 2.0f},
};

// Up to 64 rows and 8193 to 24576 weight rows (256 compute units): as many weight rows a tile, in 16s, as give every
// compute unit at most one of them (48, 64, 80 or 96; the number of waves side by side), and the stages that LDS then
// holds.  Tiles of 128 rows left up to half of the compute units without work, tiles of 32 some with three where others
// had two.  Weights from HBM, kernels alone, us, 128- or 32-row tiles / these: 32x18432x7168 31.3 / 26.1, 32x12288x7168
// 23.4 / 19.0, 1x18432x7168 28.9 / 25.4 (5.2 TB/s), 64x18432x7168 37 / 30; geometric mean over 11800 shapes of K 640 ..
// 18432, by width: .83 .92 .88 .94 up to 32 rows, .91 .98 .82 .91 up to 64.  128 rows in seven stages instead, 96 KiB
// in flight: 32x18432x7168 32.1.  Beyond 24576 .97 and with a shorter K a latency per stage is all there is.
// 65 to 128 rows, in one row tile: from 16385 weight rows on (80, 96 or 112 a tile), where the main kernel or 128x64 tiles
// had more than a round or read the weights twice; 7800 shapes of K 1280 .. 18432 .84 .81 .85 by width (96x18432x7168 55 /
// 44, 128x24576x1536 18.0 / 15.9); below K = 1280 .98, at 48 or 64 weight rows 1.0 and 1.08.
static int one_tile_waves(int M, int N, int K, int cus) {
    const int w = (N + 16 * cus - 1) / (16 * cus);
    if (M <= 64) return w >= 3 && w <= 6 && K >= 640 ? w : 0;
    return M <= 128 && w >= 5 && w <= 7 && K >= 1280 ? w : 0;
}

// One 128x64 tile a compute unit at most: there is room for a second group of waves, and twice the bytes in flight.  4000
// shapes of 129 to 256 tiles, time over that of one group: K 1024 .. 10112 .89, by row .87 (1.02 at worst; 768x1536x7168
// 30.8 / 24.6 us, 1024x2048x7168 31.7 / 29.4, by row 768x1536x8192 38 / 30); below .93 (1.08).  One group and six stages
// instead 1.03.
static bool two_groups(int M, int N, int K, int cus) {
    return M > 64 && K >= 1024 && (int64_t)((M + 63) / 64) * ((N + 127) / 128) <= cus;
}

// The configuration's number: the ranked ones' index, then the ones taken aside.  Up to 64 rows the one of 64 weight rows
// is number 3 itself.
enum { kOneTile32 = kSkinnyCfgs, kOneTile64 = kOneTile32 + 4, kOneTile128 = kOneTile64 + 4, kTwoGroups = kOneTile128 + 3 };
static int skinny_choice(int M, int N, int K, int cus) {
    if (const int w = one_tile_waves(M, N, K, cus)) {
        if (M <= 32) return kOneTile32 + w - 3;
        if (M <= 64) return w == 4 ? 3 : kOneTile64 + w - 3;
        return kOneTile128 + w - 5;
    }
    int best = 0;
    float best_us = 0.f;
    for (int i = 0; i < kSkinnyCfgs; ++i) {
        const SkinnyChoice& c = kSkinny[i];
        const int64_t tiles = (int64_t)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn), slots = (int64_t)cus * c.per_cu;
        const float steps = (float)((K / 128 + c.wk - 1) / c.wk);
        const int64_t rest = tiles % slots;
        float us = c.fixed + (float)(tiles / slots) * (steps * c.full + c.out);
        if (rest) us += steps * (c.alone + (c.full - c.alone) * ((float)rest / (float)slots)) + c.out;
        if (i == 0 || us < best_us) { best = i; best_us = us; }
    }
    return best == 4 && two_groups(M, N, K, cus) ? kTwoGroups : best;
}

// Up to 64 rows (nothing is gained from a second row tile: 64x32768x3072 37 -> 26 us), or fewer 128x128 tiles than
// compute units, as far as K lets them (and what `one_tile_waves` takes aside).  While every compute unit has at most
// one of this kernel's 64x128 tiles, a K-step of it is shorter than the main kernel's for a tile twice as high.  With a
// second one it is not: the two tiles move 1.5 times the bytes through LDS, and only the shorter start and end of a tile
// are left to gain, which a short K shows and a long one does not; the rescale by row costs this kernel more than the
// main one.  Weights from HBM, kernels alone, us, main kernel / this one, at the worst of the shapes measured beside each
// line (1600 shapes in four forms, M up to 16384, K 128 .. 18432; within the lines the worst is 1.003 of the main
// kernel's time, 1.03 on 900 others that the lines were not drawn from; beyond them 1.56):
//   tiles <= half the compute units   8192x128x18432 by row 103 / 68
//   tiles <= compute units            385x3392x12288 by row 69 / 68; beyond: 16384x128x18432 by row 111 / 117
//   more                              1457x2275x4096 34 / 33, by row 4933x444x3072 34 / 34, 552x4096x256 19 / 12;
//                                     beyond: by row 2560x1444x4096 46 / 47, 9612x210x18432 110 / 173; 589x3746x7168
//                                     42 / 50; one K-step: 8184x296x128 6.4 / 7.3
// From as many 128x128 tiles as compute units on calls stay with the main kernel (256 tiles: 1024x4096x7168 47 / 53; a
// short K would still gain, 2048x2048x1536 21 / 17).
bool gemm_skinny_preferred(const GemmParams& p, ds3_bscale mode, int cus) {
    if (p.M > 64) {
        const int64_t tn = (p.N + 127) / 128, tiles = (int64_t)((p.M + 63) / 64) * tn;
        if ((int64_t)((p.M + 127) / 128) * tn >= cus) return false;
        const bool rows = mode == DS3_BSCALE_PER_ROW;
        const bool too_long = tiles > cus ? p.K < 256 || p.K > (rows ? 3072 : 4096) : 2 * tiles > cus && p.K > 12288;
        if (too_long && one_tile_waves(p.M, p.N, p.K, cus) == 0) return false;
    }
    // what the kernel's 32-bit offsets and its grid do not hold stays with the main kernel; so do leading dimensions
    // that it refuses (its 128-row tiles reach further than these), for every size alike
    return (int64_t)129 * p.ldb + p.K < (1ll << 31) && (int64_t)129 * p.lda + p.K < (1ll << 31) && p.N < (1 << 26);
}

int gemm_skinny_config(const GemmParams& p, ds3_bscale mode, int cus) {
    return gemm_skinny_preferred(p, mode, cus) ? skinny_choice(p.M, p.N, p.K, cus) : -1;
}

ds3_status launch_gemm_skinny(const GemmParams& p, ds3_dtype ct, ds3_bscale mode, bool pow2, int cus, hipStream_t st) {
    const bool rows = mode == DS3_BSCALE_PER_ROW;
    switch (skinny_choice(p.M, p.N, p.K, cus)) {
        case 0: return launch_cfg<SkinnyCfg<1, 2, 2, 4, 4>>(p, ct, rows, pow2, st);
        case 1: return launch_cfg<SkinnyCfg<1, 2, 2, 2, 4>>(p, ct, rows, pow2, st);
        case 2: return launch_cfg<SkinnyCfg<2, 2, 4, 2, 3>>(p, ct, rows, pow2, st);
        case 3: return launch_cfg<SkinnyCfg<1, 4, 4, 2, 4>>(p, ct, rows, pow2, st);
        case 4: return launch_cfg<SkinnyCfg<2, 4, 4, 1, 3>>(p, ct, rows, pow2, st);
        case kOneTile32 + 0: return launch_cfg<SkinnyCfg<1, 2, 3, 2, 5>>(p, ct, rows, pow2, st);
        case kOneTile32 + 1: return launch_cfg<SkinnyCfg<1, 2, 4, 2, 5>>(p, ct, rows, pow2, st);
        case kOneTile32 + 2: return launch_cfg<SkinnyCfg<1, 2, 5, 2, 4>>(p, ct, rows, pow2, st);
        case kOneTile32 + 3: return launch_cfg<SkinnyCfg<1, 2, 6, 1, 6>>(p, ct, rows, pow2, st);
        case kOneTile64 + 0: return launch_cfg<SkinnyCfg<1, 4, 3, 2, 4>>(p, ct, rows, pow2, st);
        case kOneTile64 + 2: return launch_cfg<SkinnyCfg<1, 4, 5, 2, 3>>(p, ct, rows, pow2, st);
        case kOneTile64 + 3: return launch_cfg<SkinnyCfg<1, 4, 6, 1, 5>>(p, ct, rows, pow2, st);
        case kOneTile128 + 0: return launch_cfg<SkinnyCfg<1, 8, 5, 1, 5>>(p, ct, rows, pow2, st);
        case kOneTile128 + 1: return launch_cfg<SkinnyCfg<1, 8, 6, 1, 4>>(p, ct, rows, pow2, st);
        case kOneTile128 + 2: return launch_cfg<SkinnyCfg<1, 8, 7, 1, 4>>(p, ct, rows, pow2, st);
        case kTwoGroups: return launch_cfg<SkinnyCfg<2, 4, 4, 2, 3>>(p, ct, rows, pow2, st);
        default: return DS3_ERR_UNSUPPORTED;            // (not reached)
    }
}

// ---- grouped ----------------------------------------------------------------------
template <class C, bool SWIQ>
static ds3_status launch_grouped(GemmParams p, ds3_dtype ct, bool pow2, hipStream_t st) {
    p.tiles_m = (p.M + C::BM - 1) / C::BM + p.G;        // an upper bound; workgroups beyond the true count leave at once
    if (p.tiles_m > p.M) p.tiles_m = p.M;               // (a row tile has a row)
    p.tiles_n = (p.N + C::BN - 1) / C::BN;
    const dim3 grid((unsigned)(((int64_t)p.tiles_m * p.tiles_n + 7) / 8 * 8)), block(C::NT);
    (void)hipGetLastError();                            // a stale error of earlier, unrelated work is not this launch's
    if constexpr (SWIQ) {
        if (pow2) gemm_skinny_kernel<C, false, true, true, true, true><<<grid, block, 0, st>>>(p);
        else gemm_skinny_kernel<C, false, true, false, true, true><<<grid, block, 0, st>>>(p);
    } else if (ct == DS3_BF16) {
        if (pow2) gemm_skinny_kernel<C, false, true, true, true><<<grid, block, 0, st>>>(p);
        else gemm_skinny_kernel<C, false, true, false, true><<<grid, block, 0, st>>>(p);
    } else {
        if (pow2) gemm_skinny_kernel<C, false, false, true, true><<<grid, block, 0, st>>>(p);
        else gemm_skinny_kernel<C, false, false, false, true><<<grid, block, 0, st>>>(p);
    }
    return hipGetLastError() == hipSuccess ? DS3_OK : DS3_ERR_LAUNCH;
}

// Few rows an expert: 32-row tiles up to a mean of 16 rows, 64-row tiles up to 32, as far as uneven loads cannot make
// them the slower ones.  The host knows the rows but not whom they belong to.  Where the rows fall on few experts these
// tiles are up to four times as many as the main kernel's 128-row ones, each with the expert's whole K to walk, and
// each (expert, row tile) that does not exist is a workgroup that is launched to leave at once (2.3 ns).  So either all
// tiles that there could be are resident at once, or there are at most four times as many of them and the rows can make
// at most a quarter of a round more of them than there are experts with rows (plain, whose K is the short one: half a
// round, a third with 64-row tiles).  Beyond K = 4096 the shorter start of a tile is no longer worth its smaller size,
// but for gate|up on 32-row tiles, which keep three stages of weights in flight where the main kernel keeps two.
// Weights from HBM, kernels alone, us, main kernel / this one, gate|up + down.  Within the lines: H 7168, I 2048, 32
// experts of 4 rows 158 / 154 + 91 / 81, 8 experts of 4 58 / 54 + 29 / 24; H 2048, I 1024, 32 of 4 31 / 27 + 20 / 15, 8
// of 4 20 / 16 + 14 / 8. Over 17679 calls (1 .. 1023 experts, 1 .. 1024 rows): where the rows fall evenly, as exp(N(0,
// 0.3 .. 0.6)), or evenly on a half, an eighth or one of the experts, one of 9267 takes more than 1.02 of the main
// kernel's time (1.04, 1023 experts); with exp(N(0, 1 .. 2)) six of 3949 (1.20 at most); with loads built to need one
// tile more than a full round of them 20 of 4463 (67 / 89 at most). Beyond the lines: gate|up of 32 experts, 512 rows
// on four of them 63 / 84, 64 experts, 1024 rows on eight 71 / 126, 256 experts, 4096 rows on one 120 / 321; 1023
// experts of 16 rows each (H 2048, I 1024) 770 / 1077; plain, 24 experts of 18 rows, N 2048, K 7168 70 / 76.
static int grouped_rows(const GemmParams& p, bool swiglu_quant, int cus) {
    if ((int64_t)p.M > (int64_t)32 * p.G) return 0;
    const int rows = (int64_t)p.M <= (int64_t)16 * p.G ? 32 : 64;
    if (p.K > 4096 && !(swiglu_quant && rows == 32)) return 0;
    const int bn = swiglu_quant ? 256 : 128;           // (as launch_grouped_skinny has it)
    const int64_t cols = ((int64_t)p.N + bn - 1) / bn, slots = (int64_t)cus * (swiglu_quant ? 1 : 2);
    const int64_t most = std::min<int64_t>((p.M + rows - 1) / rows + p.G, p.M) * cols;      // workgroups launched
    const int64_t more = (int64_t)((p.M - 1) / rows) * cols;                                 // tiles beyond one an expert
    if (most > slots && (most > 4 * slots || (swiglu_quant ? 4 : rows == 32 ? 2 : 3) * more > slots)) return 0;
    return rows;
}

int grouped_skinny_rows(const GemmParams& p, bool swiglu_quant, int cus) {
    // what the kernel's 32-bit offsets do not hold stays with the main kernel
    if ((int64_t)257 * p.ldb + p.K >= (1ll << 31) || (int64_t)129 * p.lda + p.K >= (1ll << 31)) return 0;
    return grouped_rows(p, swiglu_quant, cus);
}

// Gate|up: 256 weight rows a workgroup, one per compute unit and as many stages as LDS holds; a plain product: 128
// weight rows, two workgroups per compute unit, so that one's start and end are hidden behind the other (its K is
// the short one: 256 rows and four stages take 88 us where these take 82).
ds3_status launch_grouped_skinny(const GemmParams& p, ds3_dtype ct, bool swiglu_quant, int rows, bool pow2, hipStream_t st) {
    if (rows == 32)
        return swiglu_quant ? launch_grouped<SkinnyCfg<4, 2, 4, 1, 4>, true>(p, ct, pow2, st)
                            : launch_grouped<SkinnyCfg<2, 2, 4, 1, 3>, false>(p, ct, pow2, st);
    return swiglu_quant ? launch_grouped<SkinnyCfg<2, 4, 8, 1, 3>, true>(p, ct, pow2, st)
                        : launch_grouped<SkinnyCfg<2, 4, 4, 1, 3>, false>(p, ct, pow2, st);
}

}  // namespace ds3
