// Block-scaled FP8 GEMM for a short inner dimension (K <= 512) and a large output: the latent projections' way up
// (8192 x 32768 x 512), the weight gradient over few tokens.
//
// Such a call is bound by its output.  The main kernel computes a tile in four K-steps or fewer and then writes it: all
// of its workgroups compute at the same time and write at the same time, and neither hides the other.  Here the weights
// do not move at all: a wave keeps its 64 weight rows in registers for the whole call (64 x 512 codes are 128 registers)
// and the activation rows stream past, 32 at a time, through a ring of LDS stages.  Every 32 rows a wave has 32 x 64
// finished sums, and they leave while the next rows are multiplied; two workgroups of four waves share a compute unit,
// so that one's barrier is the other's work (8192 x 32768 x 512, BF16 output: 192 -> 136 us, power-of-two scales 172 ->
// 125; the products alone take 106 us at the rate of the largest dense calls, the stores alone 94).  Per activation
// fragment read from LDS a wave issues four products (the main kernel's eight need a weight fragment each on top).
// Only FP32 output by row with K = 512 does not fit the registers (one is spilled).
//
// The workgroups that run together cover whole rows of the output: neighbouring workgroups write neighbouring
// columns (8192 x 32768 BF16, stores alone: 94 us in this order, 101-135 us with an XCD's workgroups side by side, 105-113
// us in the main kernel's tile order).
//
// Every output element is the main kernel's sequence of operations, bit for bit.
#include "ds3_dev.h"
#include "ds3_internal.h"

namespace ds3 {

constexpr int kShortRows = 32;                         // activation rows of one step
constexpr int kShortCols = 256;                        // weight rows of a workgroup, 64 of each wave
constexpr int kShortStages = 3;

// KB: K-steps (K / 128)
template <int KB, bool ROWSB, bool OUT_BF16, bool POW2>
__global__ __launch_bounds__(256, 2) void gemm_shortk_kernel(const GemmParams p, int splits) {
    constexpr int FN = 4, FM = 2, NS = kShortStages;
    constexpr int CODES = kShortRows * 128 * KB;       // one step's codes: [K-step][row][128 bytes]
    constexpr int STAGE = CODES + 4 * 256;             // behind them a slot of 64 scales for every wave
    constexpr int ESZ = OUT_BF16 ? 2 : 4;
    constexpr int ROWB = 64 * ESZ + 16;                // padded LDS row of a wave's strip
    constexpr int SROWS = OUT_BF16 ? 32 : 16;          // rows that pass through a strip at a time
    constexpr int STRIP = SROWS * ROWB;
    constexpr int UN = ROWSB ? KB * 256 : 0;           // per-row mode: a wave's weight scales, [K-step][64]
    constexpr int RING = NS * STAGE, WTMP = 4 * 2 * 8192;      // ring; on the way in, two K-steps of each wave's weights
    constexpr int LDS = (RING + 4 * STRIP > WTMP ? RING + 4 * STRIP : WTMP) + 4 * UN;
    static_assert(LDS <= 80 * 1024, "two workgroups per compute unit");
    __shared__ __attribute__((aligned(1024))) uint8_t smem[LDS];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g4 = lane >> 4;

    // this workgroup's columns and its range of 32-row steps
    // (the quotients are worked out in vector registers; said to be uniform, the descriptors live in scalar ones)
    const int s = __builtin_amdgcn_readfirstlane((int)(blockIdx.x / (unsigned)p.tiles_n)), t = (int)blockIdx.x - s * p.tiles_n;
    const int steps_all = (p.M + kShortRows - 1) / kShortRows;
    const int per = steps_all / splits, over = steps_all - per * splits;       // the first `over` ranges are a step longer
    const int step0 = __builtin_amdgcn_readfirstlane(s * per + min(s, over)), step1 = __builtin_amdgcn_readfirstlane(step0 + per + (s < over ? 1 : 0));
    if (step0 >= step1) return;
    const int n0 = t * kShortCols + wave * 64;         // this wave's first column
    const int n_cols = __builtin_amdgcn_readfirstlane(max(0, min(64, p.N - n0)));
    const int n0c = __builtin_amdgcn_readfirstlane(min(n0, p.N - 1));

    // ---- the weights: through LDS (whole lines) into registers, each wave its own 64 rows.
    // MFMA row r of fragment i is column (i / 2) * 32 + (r / 4) * 8 + (i & 1) * 4 + r % 4: a lane's sums in two
    // fragments are then eight consecutive columns.
    auto column_of = [](int i, int r) { return (i >> 1) * 32 + (r >> 2) * 8 + (i & 1) * 4 + (r & 3); };
    i32x8 w[FN][KB];
    {
        const __amdgpu_buffer_rsrc_t rs_b = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(p.b + (int64_t)n0c * p.ldb), 0, __builtin_amdgcn_readfirstlane(n_cols ? (n_cols - 1) * (int)p.ldb + p.K : 0), 0x00020000);
        const int lrow = lane >> 3;
        const unsigned voff = (unsigned)(lrow * (int)p.ldb + (((lane & 7) ^ lrow) << 4));   // chunks XOR-swizzled by row
        uint8_t* const tmp = smem + wave * 16384;
        auto fetch = [&](int kb) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_b, (lds_ptr_t)(tmp + (kb & 1) * 8192 + i * 1024), 16,
                                                         (int)(voff + (unsigned)i * 8u * (unsigned)p.ldb + ((unsigned)kb << 7)), 0, 0, 0);
        };
        fetch(0);
        if (KB > 1) fetch(1);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            asm volatile("" ::: "memory");
            if (kb + 1 < KB) __builtin_amdgcn_s_waitcnt(0x0F70 | 8);                 // the eight loads behind it may fly on
            else __builtin_amdgcn_s_waitcnt(0x0F70);
            asm volatile("" ::: "memory");
#pragma unroll
            for (int i = 0; i < FN; ++i) {
                const int row = column_of(i, l16);
                const uint8_t* base = tmp + (kb & 1) * 8192 + row * 128;
                const i32x4 lo = *reinterpret_cast<const i32x4*>(base + (((2 * g4) ^ (row & 7)) << 4));
                const i32x4 hi = *reinterpret_cast<const i32x4*>(base + (((2 * g4 + 1) ^ (row & 7)) << 4));
                w[i][kb] = i32x8{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            }
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xC07F);                                      // read before it is overwritten
            asm volatile("" ::: "memory");
            if (kb + 2 < KB) fetch(kb + 2);
        }
    }
    // weight scales: one per K-step in block mode; per row through LDS (power-of-two: the exponents of a lane's
    // rows in registers, a byte per K-step)
    [[maybe_unused]] float sb[KB];
    [[maybe_unused]] int ea[FN];
    [[maybe_unused]] float* const un_s = reinterpret_cast<float*>(smem + LDS - 4 * UN + wave * UN);
    if constexpr (!ROWSB) {
        const float* base = p.sb + (int64_t)(n0c >> 7) * p.sbr;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            sb[kb] = base[kb * p.sbk];
            asm volatile("" : "+v"(sb[kb]));           // here, not behind the first rows' loads
        }
        if constexpr (POW2) {
            unsigned e = 0;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) e |= (as_u32(sb[kb]) >> 23) << (8 * kb);
#pragma unroll
            for (int i = 0; i < FN; ++i) ea[i] = (int)e;
        }
    } else if constexpr (POW2) {
#pragma unroll
        for (int i = 0; i < FN; ++i) {
            const float* base = p.sb + (int64_t)min(n0 + column_of(i, l16), p.N - 1) * p.sbr;
            unsigned e = 0;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) e |= (as_u32(base[kb * p.sbk]) >> 23) << (8 * kb);
            ea[i] = (int)e;
        }
    } else {
        const float* base = p.sb + (int64_t)min(n0 + lane, p.N - 1) * p.sbr;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) un_s[kb * 64 + lane] = base[kb * p.sbk];
    }
    __syncthreads();                                   // the ring lies where the weights came in

    // ---- the activation rows' ring
    const int lrow = tid >> 3;
    const int gchunk = (tid & 7) ^ swz_key(lrow);
    const unsigned voff_a = (unsigned)(lrow * (int)p.lda + gchunk * 16);
    const __amdgpu_buffer_rsrc_t rs_sa = __builtin_amdgcn_make_buffer_rsrc((void*)p.sa, 0, 0x7ffffffc, 0x00020000);
    const unsigned soff = (unsigned)(min(wave, KB - 1) * (int)p.sak) * 4u;
    const unsigned sar = (unsigned)p.sar * 4u;
    auto issue = [&](int step, int stage) {            // KB + 1 loads, always
        const bool real = step < step1;
        const int m0 = min(step, step1 - 1) * kShortRows, rows = __builtin_amdgcn_readfirstlane(min(kShortRows, p.M - m0));
        const __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(p.a + (int64_t)m0 * p.lda), 0, __builtin_amdgcn_readfirstlane(real ? (rows - 1) * (int)p.lda + p.K : 0), 0x00020000);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_a, (lds_ptr_t)(smem + stage * STAGE + kb * 4096 + wave * 1024), 16,
                                                     (int)(voff_a + ((unsigned)kb << 7)), 0, 0, 0);
        // wave k fetches the rows' scales of K-step k (waves beyond the last K-step repeat it, into a slot nobody reads)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_sa, (lds_ptr_t)(smem + stage * STAGE + CODES + wave * 256), 4,
                                                 (int)(soff + (unsigned)(m0 + min(lane & 31, rows - 1)) * sar), 0, 0, 0);
    };
    const int key = swz_key(l16);
    const int foff0 = l16 * 128 + (((2 * g4) ^ key) << 4), foff1 = l16 * 128 + (((2 * g4 + 1) ^ key) << 4);
    auto load_frag = [&](const uint8_t* base) -> i32x8 {
        const i32x4 lo = *reinterpret_cast<const i32x4*>(base + foff0);
        const i32x4 hi = *reinterpret_cast<const i32x4*>(base + foff1);
        return i32x8{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    };
    uint8_t* const strip = smem + RING + wave * STRIP;
    constexpr int CPR = 64 * ESZ / 16;                 // 16-byte chunks of a wave's row
    constexpr int PASSES = SROWS * CPR / 64;           // stores per strip
    constexpr int STORES = PASSES * (32 / SROWS);      // ... and per step
    const int ch = lane % CPR, r0 = lane / CPR;
    constexpr int RPP = 64 / CPR;                      // rows a store covers
    constexpr int EPC = 16 / ESZ;                      // columns of a chunk
    const bool col_ok = ch * EPC + EPC <= n_cols;
    const int cut = n_cols % EPC;                      // columns of the last chunk where it is not a whole one
    const unsigned ldc_b = (unsigned)p.ldc * ESZ;
    const unsigned coff = (unsigned)r0 * ldc_b + (unsigned)(ch * 16);
    const bool accum = !OUT_BF16 && p.accumulate;

    for (int i = 0; i < NS - 1; ++i) issue(step0 + i, i);
    int stage = 0;
    for (int step = step0; step < step1; ++step) {
        // This step's rows have landed: what was issued behind their loads may stay in flight (NS - 2 steps' loads, NS - 1
        // steps' stores, which are issued whether or not their lanes have something to write).  The first steps have
        // fewer stores behind them.
        asm volatile("" ::: "memory");
        constexpr int keep0 = (NS - 2) * (KB + 1), keep = keep0 + (NS - 1) * STORES;
        static_assert(keep < 64, "vmcnt immediate");
        if (step - step0 < NS - 1) __builtin_amdgcn_s_waitcnt((keep0 & 15) | ((keep0 >> 4) << 14) | 0x70);
        else __builtin_amdgcn_s_waitcnt((keep & 15) | ((keep >> 4) << 14) | 0x70);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue(step + NS - 1, stage == 0 ? NS - 1 : stage - 1);
        const int m0 = step * kShortRows, rows = __builtin_amdgcn_readfirstlane(min(kShortRows, p.M - m0));
        // (a lane without a row or a column to write has an offset beyond the descriptor's bytes)
        const __amdgpu_buffer_rsrc_t rs_c = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(static_cast<uint8_t*>(p.c) + ((int64_t)m0 * p.ldc + n0) * ESZ), 0, 
            __builtin_amdgcn_readfirstlane(n_cols ? (rows - 1) * (int)ldc_b + n_cols * ESZ : 0), 0x00020000);
        auto c_off = [&](int row) -> int {             // row: of this store's first lanes
            unsigned off = col_ok && row + r0 < rows ? coff + (unsigned)row * ldc_b : kOobOffset;
            asm volatile("" : "+v"(off));              // a select: the access is issued whatever its lanes' offsets are
            return (int)off;
        };
        const uint8_t* st = smem + stage * STAGE;
        const float* sc = reinterpret_cast<const float*>(st + CODES);
        f32x4 acc[FN][FM];
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
            for (int j = 0; j < FM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        // Products in the order of the K-steps, the FMAs of one behind the products of the next two: the vector unit works
        // in the shadow of the matrix unit.  (The empty asm statements only tie values to program points.)
        constexpr int D = POW2 ? 0 : 2, PER = FN * FM, ALL = KB * PER;
        i32x8 x[2][FM];
        float sav[2][FM];
        [[maybe_unused]] f32x4 un[2][FN];
        auto fetch_x = [&](int kb) {
#pragma unroll
            for (int j = 0; j < FM; ++j) {
                x[kb & 1][j] = load_frag(st + kb * 4096 + j * 2048);
                sav[kb & 1][j] = sc[kb * 64 + j * 16 + l16];
            }
        };
        [[maybe_unused]] f32x4 part[D + 1];
        __builtin_amdgcn_sched_barrier(0);
        fetch_x(0);
#pragma unroll
        for (int q = 0; q < ALL + D; ++q) {
            const int kb = q / PER, j = q % PER / FN, i = q % FN;
            if (q < ALL) {
                if constexpr (POW2) {
                    const int eb = (int)(as_u32(sav[kb & 1][j]) >> 23);
                    f32x4& c = acc[i][j];
                    if (kb == 0) c = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w[i][0], x[0][j], c, 0, 0, 0, ea[i], 0, eb);
                    else if (kb == 1) c = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w[i][1 % KB], x[1][j], c, 0, 0, 1, ea[i], 0, eb);
                    else if (kb == 2) c = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w[i][2 % KB], x[0][j], c, 0, 0, 2, ea[i], 0, eb);
                    else c = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w[i][3 % KB], x[1][j], c, 0, 0, 3, ea[i], 0, eb);
                    asm volatile("" : "+v"(c));
                } else {
                    if constexpr (ROWSB) { if (j == 0) un[kb & 1][i] = *reinterpret_cast<const f32x4*>(un_s + kb * 64 + column_of(i, g4 * 4)); }
                    part[q % (D + 1)] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w[i][kb], x[kb & 1][j], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0, 0, 0, 0);
                }
            }
            if constexpr (!POW2) {
                if (q >= D) {
                    const int ps = q - D, pk = ps / PER, pj = ps % PER / FN, pi = ps % FN;
                    if (q < ALL) asm volatile("" : "+v"(part[q % (D + 1)]), "+v"(part[ps % (D + 1)]));
                    const f32x4 pr = part[ps % (D + 1)];
                    const float sa = sav[pk & 1][pj];
                    f32x4 tt, c = acc[pi][pj];         // (the rescale of ds3_gemm.hip)
                    if constexpr (ROWSB) { const f32x4 u = un[pk & 1][pi]; tt = f32x4{sa * u.x, sa * u.y, sa * u.z, sa * u.w}; }
                    else tt.x = tt.y = tt.z = tt.w = sa * sb[pk];
                    c.x = __builtin_fmaf(pr.x, tt.x, c.x);
                    c.y = __builtin_fmaf(pr.y, tt.y, c.y);
                    c.z = __builtin_fmaf(pr.z, tt.z, c.z);
                    c.w = __builtin_fmaf(pr.w, tt.w, c.w);
                    asm volatile("" : "+v"(c));
                    acc[pi][pj] = c;
                }
            }
            // (the scales of the K-step before are read until here)
            if (q < ALL && q % PER == D && kb + 1 < KB) fetch_x(kb + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- out: a wave's strip turns 16 rows of four columns a lane into whole row segments
        auto out_rows = [&](int h) {                   // rows [h * SROWS, + SROWS)
            [[maybe_unused]] u32x4 old[PASSES];
            if constexpr (!OUT_BF16) {
                if (accum) {
#pragma unroll
                    for (int ps = 0; ps < PASSES; ++ps)
                        old[ps] = __builtin_amdgcn_raw_buffer_load_b128(rs_c, c_off(h * SROWS + ps * RPP), 0, 2);
                }
            }
#pragma unroll
            for (int j = 0; j < SROWS / 16; ++j) {
                uint8_t* row = strip + (j * 16 + l16) * ROWB;
                if constexpr (OUT_BF16) {
#pragma unroll
                    for (int i = 0; i < FN; i += 2) {
                        const f32x4 u = acc[i][h * (SROWS / 16) + j], v = acc[i + 1][h * (SROWS / 16) + j];
                        *reinterpret_cast<u32x4*>(row + (i * 16 + g4 * 8) * 2) =
                            u32x4{pack_bf16x2(u.x, u.y), pack_bf16x2(u.z, u.w), pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)};
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < FN; ++i) *reinterpret_cast<f32x4*>(row + column_of(i, g4 * 4) * 4) = acc[i][h];
                }
            }
            __builtin_amdgcn_wave_barrier();           // same-wave LDS accesses complete in order
            u32x4 o[PASSES];
#pragma unroll
            for (int ps = 0; ps < PASSES; ++ps) o[ps] = *reinterpret_cast<const u32x4*>(strip + (ps * RPP + r0) * ROWB + ch * 16);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int ps = 0; ps < PASSES; ++ps) {
                u32x4 v = o[ps];
                if constexpr (!OUT_BF16) {
                    if (accum) {
                        v.x = as_u32(as_f32(v.x) + as_f32(old[ps].x)); v.y = as_u32(as_f32(v.y) + as_f32(old[ps].y));
                        v.z = as_u32(as_f32(v.z) + as_f32(old[ps].z)); v.w = as_u32(as_f32(v.w) + as_f32(old[ps].w));
                    }
                }
                __builtin_amdgcn_raw_buffer_store_b128(v, rs_c, c_off(h * SROWS + ps * RPP), 0, 2);
            }
            if (cut != 0 && ch == n_cols / EPC) {      // (more accesses than the counted wait knows of only make it wait longer)
#pragma unroll
                for (int ps = 0; ps < PASSES; ++ps) {
                    const int row = h * SROWS + ps * RPP + r0;
                    if (row >= rows) continue;
                    uint8_t* gp = static_cast<uint8_t*>(p.c) + ((int64_t)(m0 + row) * p.ldc + n0 + ch * EPC) * ESZ;
                    const unsigned int wd[4] = {o[ps].x, o[ps].y, o[ps].z, o[ps].w};
#pragma unroll
                    for (int e = 0; e < EPC - 1; ++e) {
                        if (e >= cut) break;
                        if constexpr (OUT_BF16) {
                            reinterpret_cast<uint16_t*>(gp)[e] = (uint16_t)(wd[e >> 1] >> (16 * (e & 1)));
                        } else {
                            float* d = reinterpret_cast<float*>(gp) + e;
                            *d = accum ? as_f32(wd[e]) + *d : as_f32(wd[e]);
                        }
                    }
                }
            }
        };
#pragma unroll
        for (int h = 0; h < 32 / SROWS; ++h) {
            out_rows(h);
            __builtin_amdgcn_sched_barrier(0);
        }
        stage = stage + 1 == NS ? 0 : stage + 1;
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);                // no load is on its way into LDS when the workgroup ends
}

// ---- host side -------------------------------------------------------------------
// Ranges of rows per column tile: the rounds of workgroups that there are, each its steps and what comes before them,
// counted as six steps.  (Measured over 9800 calls of one round, the launch and the loading of the weights take 3 us at K 128 and
// 4 to 6 at K 512, a step 1.5 to 2.2 us with BF16 output, 2.9 to 3.3 with FP32, 5.5 to 6 accumulating: two or three steps
// rather than six.  The count only matters where several rounds compete, and favours few.)
static int short_splits(int64_t tiles_n, int64_t steps, int64_t slots) {
    int best = 1;
    int64_t best_cost = 0;
    for (int64_t rounds = 1; rounds <= 4; ++rounds) {
        int64_t s = rounds * slots / tiles_n;           // as many as fit so many rounds
        s = s < 1 ? 1 : s > steps ? steps : s;
        const int64_t cost = (tiles_n * s + slots - 1) / slots * ((steps + s - 1) / s + 6);
        if (rounds == 1 || cost < best_cost) { best = (int)s; best_cost = cost; }
    }
    return best;
}

template <int KB, bool POW2>
static ds3_status launch_kb(GemmParams p, ds3_dtype ct, bool rows, int cus, hipStream_t st) {
    p.tiles_n = (p.N + kShortCols - 1) / kShortCols;
    const int splits = short_splits(p.tiles_n, (p.M + kShortRows - 1) / kShortRows, 2 * (int64_t)cus);
    const int64_t wgs = p.tiles_n * (int64_t)splits;
    if (wgs > (1 << 28)) return DS3_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)wgs), block(256);
    (void)hipGetLastError();                            // a stale error of earlier, unrelated work is not this launch's
    if (rows) {
        if (ct == DS3_BF16) gemm_shortk_kernel<KB, true, true, POW2><<<grid, block, 0, st>>>(p, splits);
        else gemm_shortk_kernel<KB, true, false, POW2><<<grid, block, 0, st>>>(p, splits);
    } else {
        if (ct == DS3_BF16) gemm_shortk_kernel<KB, false, true, POW2><<<grid, block, 0, st>>>(p, splits);
        else gemm_shortk_kernel<KB, false, false, POW2><<<grid, block, 0, st>>>(p, splits);
    }
    return hipGetLastError() == hipSuccess ? DS3_OK : DS3_ERR_LAUNCH;
}

// Beyond K = 512 the weights don't fit the registers.  Up to it the kernel is taken but for
//   * fewer than 768 rows where the main kernel needs no more than one round of its 256x256 tiles: what a workgroup takes
//     to load its weights is not made up for (453x25312x512 14.1 us main kernel / 16.6 this one, 163x30416x512 9.3 / 14.2);
//   * one round of the main kernel's tiles, and 1.5 MiB of weights or more for an XCD to fetch behind 128x128 tiles, 4 MiB
//     behind 256x256 ones.  A workgroup's ranges are then down to two to four steps.  The workgroups are dealt to the eight
//     XCDs in turn, so a column tile's lie on 8 / gcd(column tiles, 8) of them, each of which loads the weights into its
//     own L2: with 33 column tiles all XCDs load all weights (866x8320x512 10.5 us main kernel / 13.1 this one), with 32
//     an eighth each.  (Where rows end within a 16-byte piece the main kernel's epilogue is the slower one: 2048x2687x384
//     12.9 / 8.8.);
//   * accumulation with a last 16-byte piece of a row that is cut, outputs times columns of that piece from 7 * 2^24 on:
//     these columns are read and written one by one, and the workgroups that hold them end last, the later the more steps
//     they have (15489x16763x128 460 / 610; 9567x3626x512 120 / 89).
// Operands from HBM, kernels alone, us: 8192x32768x512 192 / 136, x256 147 / 93; 4096x16384x512 55 / 38; 8192x4096x128
// 21 / 15; 1320x10976x512 28 / 16; by row, accumulating FP32 18432x7168x512 258 / 193, 4096x7168x512 70 / 52.  25300
// calls of 2^19 .. 2^28 outputs, every form and alignment of the output, time over the main kernel's: .795, 1.1% of them
// above 1.03, 1.24 at worst (without the last two exceptions, 570 calls at 1.06: .796, 2.5%, 1.53).
bool gemm_shortk_preferred(const GemmParams& p, int cus) {
    if (p.K > 512) return false;
    // 32-bit byte offsets within a step's rows, and leading dimensions that the main kernel refuses stay refused
    if ((int64_t)257 * p.ldb + p.K >= (1ll << 31) || (int64_t)257 * p.lda + p.K >= (1ll << 31) ||
        (int64_t)33 * p.ldc * 4 >= (1ll << 31) || p.N > (1 << 29) || p.M > (1 << 29))
        return false;
    const int64_t tiles_n = (p.N + 255) / 256, large = (int64_t)((p.M + 255) / 256) * tiles_n;
    if (p.accumulate) {
        if ((int64_t)p.M * p.N * (p.N % 4) >= (7 << 24)) return false;
    } else if (large <= cus && p.N % 8 == 0) {
        int64_t weights = (int64_t)p.N * p.K;            // bytes an XCD fetches
        for (int f = 2; f <= 8 && tiles_n % f == 0; f *= 2) weights /= 2;
        const int64_t small = (int64_t)((p.M + 127) / 128) * ((p.N + 127) / 128);
        if (large * 8 >= 5 * (int64_t)cus ? weights >= 4 << 20 : small <= 2 * (int64_t)cus && weights >= 3 << 19) return false;
    }
    return p.M >= 768 || large > cus;
}

ds3_status launch_gemm_shortk(const GemmParams& p, ds3_dtype ct, ds3_bscale mode, bool pow2, int cus, hipStream_t st) {
    const bool rows = mode == DS3_BSCALE_PER_ROW;
    switch (p.K >> 7) {
        case 1: return pow2 ? launch_kb<1, true>(p, ct, rows, cus, st) : launch_kb<1, false>(p, ct, rows, cus, st);
        case 2: return pow2 ? launch_kb<2, true>(p, ct, rows, cus, st) : launch_kb<2, false>(p, ct, rows, cus, st);
        case 3: return pow2 ? launch_kb<3, true>(p, ct, rows, cus, st) : launch_kb<3, false>(p, ct, rows, cus, st);
        default: return pow2 ? launch_kb<4, true>(p, ct, rows, cus, st) : launch_kb<4, false>(p, ct, rows, cus, st);
    }
}

}  // namespace ds3
