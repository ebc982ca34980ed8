// Products off the recurrence (gfx950, bf16): weight gradients (Eq. 11), input
// products (Eq. 1-4) and input gradients (Eq. 10).  k_wgrad_rows and k_rows are
// matrix products over all (step, row) pairs on masked operands; k_fx_big and
// k_dx_big gather a step's kept neurons, for batches of 256 and more where
// skipping the dropped ones pays.  All stage operand chunks in LDS for a whole
// workgroup, with the loads issued two chunks ahead.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "device.h"
#include "kernels.h"
#include "../../include/lstm_sd.h"

namespace lsd {


// ---------------------------------------------------------------------------
// Forward input product for large batches (Eq. 1-4 input term; Sec. 3.2 FP
// input sparsity):
//   Gx_t = s * X_t[:, keep_t] W[keep_t, :] + bias
// grid (ceil(G/128), T, ceil(B/256)), 512 threads (8 waves).  A workgroup
// computes a 256-row x 128-column tile of Gx_t; wave w owns rows
// 64*(w/2) .. +63 and columns 64*(w%2) .. +63 (4 x 4 tiles of
// 16x16x32 MFMA).  The contraction runs over the keep list of t in chunks
// of 64 kept neurons: the gathered rows of the transposed input X_t^T
// ([K][ld], 256 batch columns) and of W (128 columns) are staged in LDS as
// K-major tiles (whole 16-byte pieces of each row, coalesced), double
// buffered so that chunk i+1 is in flight while chunk i is multiplied, and
// both operands' fragments are read with ds_read_b64_tr_b16 (lanes 4e..4e+3
// of a 16-lane group address row e of the group's four at columns 0, 4, 8,
// 12: lane i receives column i of the four rows).  Rows past the count read
// as zero (an offset past the buffer).  Rows past B and columns past G are computed and not stored.
constexpr int FB_M = 256, FB_N = 128, FB_KC = 64, FB_AP = FB_M + 16, FB_BP = FB_N + 16;
constexpr size_t FB_LDS = (size_t)2 * FB_KC * (FB_AP + FB_BP) * 2 + (size_t)(LSTM_SD_MAX_K + 2 * FB_KC) * 4;

__global__ void __launch_bounds__(512) k_fx_big(FxArgs a) {
    extern __shared__ __align__(16) char smem[];
    bf16* As = (bf16*)smem;                                  // [2][FB_KC][FB_AP]
    bf16* Bs = As + 2 * FB_KC * FB_AP;                       // [2][FB_KC][FB_BP]
    int* kidx = (int*)(Bs + 2 * FB_KC * FB_BP);              // [count]
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int t = blockIdx.y, n0 = blockIdx.x * FB_N, m0 = blockIdx.z * FB_M;
    const int K = a.K, G = a.G, B = a.B;
    const int32_t* krow = a.site.keep + (size_t)t * a.site.kmax;
    const int cnt = a.site.count[t];
    // the keep list, then -1 through two chunks past the last (rows read as
    // zero: the loop fetches two chunks ahead without a condition)
    const int cpad = ((cnt + FB_KC - 1) / FB_KC + 2) * FB_KC;
    for (int j = tid; j < cpad; j += 512) kidx[j] = j >= cnt ? -1 : krow[j];
    __syncthreads();
    const __amdgpu_buffer_rsrc_t xr = buf_rsrc((const bf16*)a.XT + (size_t)t * a.xt_tstride,
                                               (uint32_t)((size_t)K * a.xt_ld * 2));
    const __amdgpu_buffer_rsrc_t wr = buf_rsrc(a.W, (uint32_t)((size_t)K * G * 2));
    // staging: A rows (512 bytes of X^T) as 32 pieces, 4 per thread; B rows
    // (256 bytes of W) as 16 pieces, 2 per thread.  Chunk j goes through
    // register set j % 2: its loads are issued two chunks ahead, so each
    // has two chunks' products to arrive in
    u32x4_t ra[2][4], rb[2][2];
    // (every row index of a chunk is read first, then its six loads go out
    // back to back; absent rows take an offset past the buffer: no branch)
    const uint32_t aoff = (uint32_t)(m0 + 8 * (tid & 31)) * 2, boff = (uint32_t)(n0 + 8 * (tid & 15)) * 2;
    auto fetch = [&](int set, int kc) {
        int ka[4], kb[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) ka[i] = kidx[kc + (tid >> 5) + 16 * i];
#pragma unroll
        for (int i = 0; i < 2; ++i) kb[i] = kidx[kc + (tid >> 4) + 32 * i];
        uint32_t oa[4], ob[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) oa[i] = ka[i] < 0 ? OOB_OFF : (uint32_t)ka[i] * (uint32_t)(a.xt_ld * 2) + aoff;
#pragma unroll
        for (int i = 0; i < 2; ++i) ob[i] = kb[i] < 0 ? OOB_OFF : (uint32_t)kb[i] * (uint32_t)(G * 2) + boff;
#pragma unroll
        for (int i = 0; i < 4; ++i) ra[set][i] = __builtin_amdgcn_raw_buffer_load_b128(xr, oa[i], 0, 0);
#pragma unroll
        for (int i = 0; i < 2; ++i) rb[set][i] = __builtin_amdgcn_raw_buffer_load_b128(wr, ob[i], 0, 0);
    };
    auto commit = [&](int set, int buf) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int q = tid + 512 * i, r = q >> 5, c = q & 31;
            *(u32x4_t*)(As + ((size_t)buf * FB_KC + r) * FB_AP + 8 * c) = ra[set][i];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = tid + 512 * i, r = q >> 4, c = q & 15;
            *(u32x4_t*)(Bs + ((size_t)buf * FB_KC + r) * FB_BP + 8 * c) = rb[set][i];
        }
    };
    f32x4_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0, 0, 0, 0};
    const int wr0 = 64 * (w >> 1), wc0 = 64 * (w & 1);
    const int trow = 8 * (lane >> 4) + ((lane & 15) >> 2), tcol = 4 * (lane & 3);
    const int nch = (cnt + FB_KC - 1) / FB_KC;
    fetch(0, 0);
    fetch(1, FB_KC);
    commit(0, 0);
    __syncthreads();
    // chunk ch (in LDS buffer ch % 2): the loads of ch+2 go out, the
    // products of ch, then ch+1 (loaded during ch-1) into the other buffer
    // (fetch and commit run unconditionally, past the end on zero rows: a
    // conditional load leaves the compiler unsure which loads are still in
    // flight, and it then waits for all of them before the next fetch)
    auto chunk = [&](int ch, int cur) {
        fetch(cur, (ch + 2) * FB_KC);
        __builtin_amdgcn_sched_barrier(0);     // (the loads go out before anything waits)
        const int buf = cur;
        const bf16* Ab = As + (size_t)buf * FB_KC * FB_AP;
        const bf16* Bb = Bs + (size_t)buf * FB_KC * FB_BP;
#pragma unroll
        for (int ks = 0; ks < FB_KC / 32; ++ks) {
            Raw8<bf16> fa[4], fb[4];
            const bf16* a0 = Ab + (size_t)(32 * ks + trow) * FB_AP + wr0 + tcol;
            const bf16* b0 = Bb + (size_t)(32 * ks + trow) * FB_BP + wc0 + tcol;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint2 lo = lds_tr4(a0 + 16 * i), hi = lds_tr4(a0 + 4 * FB_AP + 16 * i);
                fa[i].w[0] = lo.x; fa[i].w[1] = lo.y; fa[i].w[2] = hi.x; fa[i].w[3] = hi.y;
                const uint2 lb = lds_tr4(b0 + 16 * i), hb = lds_tr4(b0 + 4 * FB_BP + 16 * i);
                fb[i].w[0] = lb.x; fb[i].w[1] = lb.y; fb[i].w[2] = hb.x; fb[i].w[3] = hb.y;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) raw_mma(fa[i], fb[j], acc[i][j]);
        }
        commit(cur ^ 1, cur ^ 1);
        __syncthreads();
    };
    // (pairs with both calls unconditional: the register sets' states agree
    // at the top of every iteration)
    int ch = 0;
    for (; ch + 1 < nch; ch += 2) {
        chunk(ch, 0);
        chunk(ch + 1, 1);
    }
    if (ch < nch) chunk(ch, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n = n0 + wc0 + 16 * j + (lane & 15);
        if (n >= G) continue;
        const float bn = a.bias[n];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + wr0 + 16 * i + acc_row(lane, r);
                if (row < B) a.Gx[((size_t)t * B + row) * G + n] = a.s * acc[i][j][r] + bn;
            }
    }
}

// ---------------------------------------------------------------------------
// Output-sparse input gradient for large batches (Eq. 10), summed over the
// directions:
//   dX_t[:, keep_t[j]] = s * sum_d DA_{d,t} W_d[keep_t[j], :]^T
// grid (8 * ceil(T/8) * ceil(K/128), 1, ceil(B/256)), 512 threads: workgroup i
// runs on XCD i % 8, which takes the steps t = i % 8 + 8j with all their
// column tiles, so DA_t is fetched into one XCD's L2 once.  A workgroup
// computes 256 rows x the 128 kept columns at keep-list positions 128*x ..
// (and, with
// scatter, writes the zeros of the dropped columns at drop-list positions
// 128*x ..); wave w owns rows 64*(w/2) and columns 64*(w%2) (4 x 4 tiles of
// 16x16x32 MFMA).  The contraction over 4H runs in chunks of 64: the DA
// chunk (fragment-major in memory: the MFMA operand layout) is copied to LDS
// as 1 KB blocks, the 128 gathered W rows' 64-column pieces are staged as
// [128][64+8] rows, double buffered, with the loads issued two chunks
// ahead; every fragment is one 16-byte LDS read.
constexpr int DB_M = 256, DB_N = 128, DB_KC = 64, DB_BP = DB_KC + 8;
constexpr size_t DB_LDS = (size_t)2 * (DB_M * DB_KC + DB_N * DB_BP) * 2 + (size_t)DB_N * 4;

__global__ void __launch_bounds__(512) k_dx_big(DxArgs a) {
    extern __shared__ __align__(16) char smem[];
    bf16* As = (bf16*)smem;                                  // [2][2 chunks][16 tiles][64 lanes][8]
    bf16* Bs = As + 2 * DB_M * DB_KC;                        // [2][DB_N][DB_BP]
    int* kcol = (int*)(Bs + 2 * DB_N * DB_BP);               // [DB_N] W rows of the tile's columns
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int ntile = (a.K + DB_N - 1) / DB_N;
    const int xcd = blockIdx.x % 8, idx = blockIdx.x / 8;
    const int t = xcd + 8 * (idx / ntile), j0 = (idx % ntile) * DB_N, m0 = blockIdx.z * DB_M;
    if (t >= a.T) return;
    const int B = a.B, G = a.G;
    const bool failed = a.status && *a.status != 0;
    const int cnt = a.site.count[t];
    const int32_t* krow = a.site.keep + (size_t)t * a.site.kmax;
    float* out = a.out + (size_t)t * B * a.ldo;
    if (a.scatter) {                           // the dropped columns of this tile's drop-list range
        const int dn = a.site.dcount[t];
        const int32_t* drow = a.site.drop + (size_t)t * a.site.kmax;
        for (int i = tid; i < DB_N * DB_M; i += 512) {
            const int jj = j0 + (i % DB_N), row = m0 + i / DB_N;
            if (jj < dn && row < B) out[(size_t)row * a.ldo + drow[jj]] = failed ? __builtin_nanf("") : 0.0f;
        }
    }
    if (j0 >= cnt) return;
    if (tid < DB_N) kcol[tid] = j0 + tid < cnt ? krow[j0 + tid] : -1;
    __syncthreads();
    const int mt0 = m0 / 16;                   // first 16-row tile of the workgroup
    const size_t das = (size_t)((G + 31) / 32) * a.mtiles * 512;
    const int wr0 = 64 * (w >> 1), wc0 = 64 * (w & 1);
    const int g8 = 8 * (lane >> 4), cl = lane & 15;
    f32x4_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0, 0, 0, 0};
    const int nch = (G + DB_KC - 1) / DB_KC;
    for (int d = 0; d < a.D; ++d) {
        const __amdgpu_buffer_rsrc_t dr = buf_rsrc((const bf16*)a.da[d] + (size_t)t * das, (uint32_t)(das * 2));
        const __amdgpu_buffer_rsrc_t wr = buf_rsrc(a.W[d], (uint32_t)((size_t)a.K * G * 2));
        // staging: A = 2 chunks x 16 tiles of 1 KB (4 pieces per thread),
        // B = 128 rows x 8 pieces of 16 bytes (2 per thread); chunk c goes
        // through register set c % 2, its loads issued two chunks ahead
        u32x4_t ra[2][4], rb[2][2];
        auto fetch = [&](int set, int c) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int q = tid + 512 * i, blk = q >> 6, l = q & 63;   // blk = chunk half * 16 + tile
                const int ck = 2 * c + (blk >> 4), mt = mt0 + (blk & 15);
                const bool ok = mt < a.mtiles && 32 * ck < G;
                ra[set][i] = __builtin_amdgcn_raw_buffer_load_b128(
                    dr, ok ? (uint32_t)(frag_lane_off(ck, mt, l, (G + 31) / 32) * 2) : OOB_OFF, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int q = tid + 512 * i, r = q >> 3, pc = q & 7;
                const int k = kcol[r], g = DB_KC * c + 8 * pc;
                rb[set][i] = __builtin_amdgcn_raw_buffer_load_b128(
                    wr, (k >= 0 && g < G) ? (uint32_t)(((size_t)k * G + g) * 2) : OOB_OFF, 0, 0);
            }
        };
        auto commit = [&](int set, int buf) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int q = tid + 512 * i;
                *(u32x4_t*)(As + (size_t)buf * DB_M * DB_KC + (size_t)q * 8) = ra[set][i];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int q = tid + 512 * i, r = q >> 3, pc = q & 7;
                *(u32x4_t*)(Bs + ((size_t)buf * DB_N + r) * DB_BP + 8 * pc) = rb[set][i];
            }
        };
        fetch(0, 0);
        fetch(1, 1);
        __syncthreads();                       // (the previous direction's last chunk is read)
        commit(0, 0);
        __syncthreads();
        auto chunk = [&](int c, int cur) {
            fetch(cur, c + 2);                 // (past the end: zeros, unconditionally)
            __builtin_amdgcn_sched_barrier(0);
            const int buf = cur;
            const bf16* Ab = As + (size_t)buf * DB_M * DB_KC;
            const bf16* Bb = Bs + (size_t)buf * DB_N * DB_BP;
#pragma unroll
            for (int ks = 0; ks < DB_KC / 32; ++ks) {
                Raw8<bf16> fa[4], fb[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    raw_lds(fa[i], Ab + ((size_t)(ks * 16 + (wr0 >> 4) + i) * 64 + lane) * 8);
                    raw_lds(fb[i], Bb + (size_t)(wc0 + 16 * i + cl) * DB_BP + 32 * ks + g8);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) raw_mma(fa[i], fb[j], acc[i][j]);
            }
            commit(cur ^ 1, cur ^ 1);
            __syncthreads();
        };
        int c = 0;
        for (; c + 1 < nch; c += 2) {
            chunk(c, 0);
            chunk(c + 1, 1);
        }
        if (c < nch) chunk(c, 0);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int jl = wc0 + 16 * j + cl, jj = j0 + jl;
        if (jj >= cnt) continue;
        const int kk = kcol[jl];                 // (a kept column: a valid row)
        const int oc = a.scatter ? kk : jj;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + wr0 + 16 * i + acc_row(lane, r);
                if (row < B) out[(size_t)row * a.ldo + oc] = failed ? __builtin_nanf("") : a.s * acc[i][j][r];
            }
    }
}

void launch_fx_big(const FxArgs& a, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    const dim3 grid((a.G + FB_N - 1) / FB_N, a.T, (a.B + FB_M - 1) / FB_M), blk(512);
    if (e0 && e1) hipExtLaunchKernelGGL(k_fx_big, grid, blk, (uint32_t)FB_LDS, st, e0, e1, 0, a);
    else k_fx_big<<<grid, blk, FB_LDS, st>>>(a);
}
void launch_dx_big(const DxArgs& a, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    const dim3 grid(8 * ((a.T + 7) / 8) * ((a.K + DB_N - 1) / DB_N), 1, (a.B + DB_M - 1) / DB_M), blk(512);
    if (e0 && e1) hipExtLaunchKernelGGL(k_dx_big, grid, blk, (uint32_t)DB_LDS, st, e0, e1, 0, a);
    else k_dx_big<<<grid, blk, DB_LDS, st>>>(a);
}

// ---------------------------------------------------------------------------
// Weight gradients (bf16), Eq. 11, every problem of a pass in one launch: a plain
// matrix product per problem over the T*B (step, batch) rows,
//   out[k][n] = s * sum_r A[r][k] da[r][n],
// with A row-major and already masked by its producer (a dropped neuron's column
// is zero at that step, so the row sparsity of Eq. 11 holds: never-kept rows are
// exact zeros) and da the published fragment-major DA blocks, read where the
// recurrence left them.  Both operands are staged with the contraction (rows)
// outermost and their fragments come from transposing LDS reads, so no transposed
// copy of either is ever written: those copies cost the backward recurrence 2.4 us
// of a 7.7 us step at batch 256, padded every step's contraction to 32 rows, and
// took a pass over the input of their own.  Rows of successive steps share a
// 32-row chunk.
// A workgroup of WM x WN waves computes a TM x TN tile (a wave MI x NI MFMA
// tiles) with its accumulators in registers over all rows.  Two LDS buffers; the
// loads of a chunk go out two chunks before it is staged, and the one barrier per
// chunk waits for LDS only.  Tiles of 256 x 256 (one workgroup per CU) read the
// fewest bytes per product; 128 x 128 and 64 x 128 fill the chip when a pass has
// few of those.  Against the kernels before (a step's rows padded to 32, transposed
// operands, 128 x 256 tiles): batch 256 x hidden 1024 826 -> 565 us, AWD 277 -> 116,
// LM-large 151 -> 83, LM-medium 38 -> 27, vocabulary head at batch 64 189 -> 105 us.
// Workgroup i runs on XCD i % 8, which takes a contiguous range of (problem,
// column block, row block): an XCD's L2 holds its columns' DA for all their row
// blocks.
template <int WM, int WN, int MI, int NI>
struct WrShape {
    static constexpr int NW = WM * WN, NTH = 64 * NW, TM = WM * MI * 16, TN = WN * NI * 16;
    static constexpr int AP = TM + 16, BP = TN + 16;                 // row pitches (32 bytes past a whole bank row)
    static constexpr size_t LDS = (size_t)2 * 32 * (AP + BP) * 2;
};

// Offsets into da are 32 bits from the step of a chunk's first row; where the steps that
// a chunk's rows lie in take 2 GiB and more (a vocabulary head whose batch x columns
// is 2^29 and more, or with a small batch a million columns), WIDE builds add up 64-bit
// addresses.
constexpr uint32_t WR_REACH = 0x7fffffffu;
static bool wr_wide(const WrBatch& b) {
    return (size_t)(b.B >= 32 ? 2 : 32 / b.B + 2) * (size_t)b.das * 2 > WR_REACH;
}

template <int WM, int WN, int MI, int NI, bool WIDE = false>
__global__ void __launch_bounds__(64 * WM * WN, 2) k_wgrad_rows(WrBatch bt) {
    using S = WrShape<WM, WN, MI, NI>;
    constexpr int NTH = S::NTH, NW = S::NW, TM = S::TM, TN = S::TN, AP = S::AP, BPITCH = S::BP;
    constexpr int PA = TM * 4 / NTH, NBLK = TN / 16, PB = NBLK / NW;  // pieces: A per thread; 16x32 blocks of da per wave
    static_assert(PA * NTH == TM * 4 && PB * NW == NBLK, "whole pieces");
    extern __shared__ __align__(16) char smem[];
    bf16* As = (bf16*)smem;                                          // [2][32][AP]
    bf16* Bs = As + 2 * 32 * AP;                                     // [2][32][BPITCH]
    int pos = (int)(blockIdx.x % 8) * bt.per + (int)(blockIdx.x / 8), pi = 0;
    if (pos >= bt.total) return;
    while (pos >= bt.p[pi].tiles) pos -= bt.p[pi++].tiles;
    const WrProblem& a = bt.p[pi];
    const int cb = pos / a.nrb, rb = pos % a.nrb;
    const int r0 = rb * TM, n0 = cb * TN, G = bt.G, B = bt.B, R = bt.R;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w / WN, wn = w % WN;
    const bool dbw = a.db && rb == a.nrb - 1;
    if (bt.status && *bt.status != 0) {        // the step's recurrence timed out: NaN in every output
        const float nan = __builtin_nanf("");
        for (int i = tid; i < TM * TN; i += NTH) {
            const int r = r0 + i / TN, n = n0 + i % TN;
            if (r < a.K && n < G) a.out[(size_t)r * G + n] = nan;
        }
        if (dbw)
            for (int n = n0 + tid; n < min(n0 + TN, G); n += NTH) a.db[n] = nan;
        return;
    }
    const int nch = (G + 31) / 32, nq = (R + 31) / 32;
    // A: piece i of this thread is row ar + i * (rows per pass), 8 columns at ac;
    // da: block w + NW*i: 16 rows (br: this lane's) x 32 columns.  Both through
    // resources that begin at the chunk's first row (first step) and end after the
    // last row (step): constant or small 32-bit offsets, rows past the last are
    // zeros.
    constexpr int APR = TM / 8;                                      // pieces per A row
    const int ar = tid / APR, ac = min(r0 + 8 * (tid % APR), a.lda - 8);
    const uint32_t aofs = (uint32_t)(ar * a.lda + ac) * 2, apass = (uint32_t)(NTH / APR * a.lda) * 2;
    const int br = lane & 15, bk = lane >> 4;
    const uint32_t dasb = (uint32_t)(bt.das * 2);
    const uint32_t msmall = 65536u / (uint32_t)B + 1u;               // (B < 32: r / B = r * msmall >> 16 for r < 64)
    typename std::conditional<WIDE, size_t, uint32_t>::type bofs[PB];   // column block, and this lane's column piece
#pragma unroll
    for (int i = 0; i < PB; ++i) {
        bofs[i] = min((n0 >> 5) + ((w + NW * i) >> 1), nch - 1);
        bofs[i] = bofs[i] * 1024u + (uint32_t)bk * 256u;
    }
    int it = 0, ib = 0;                                              // step and batch row of the next chunk's first row
    int ir = 0;                                                      // that row
    u32x4_t ra[2][PA], rbv[2][PB];
    auto issue = [&](int sl) {
        const __amdgpu_buffer_rsrc_t arc =
            buf_rsrc((const bf16*)a.A + (size_t)ir * a.lda, (uint32_t)max(min(R - ir, 32), 0) * (uint32_t)a.lda * 2u);
        const size_t left = (size_t)max(bt.T - it, 0) * dasb;
        const __amdgpu_buffer_rsrc_t brc =
            buf_rsrc((const bf16*)a.da + (size_t)it * bt.das, left < WR_REACH ? (uint32_t)left : WR_REACH);
#pragma unroll
        for (int i = 0; i < PA; ++i) ra[sl][i] = __builtin_amdgcn_raw_buffer_load_b128(arc, aofs + i * apass, 0, 0);
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const int r = ib + 16 * ((w + NW * i) & 1) + br;
            const int dt = B >= 32 ? (r >= B ? 1 : 0) : (int)(((uint32_t)r * msmall) >> 16);
            const int b = r - dt * B;
            if constexpr (WIDE) {
                const char* p = (const char*)a.da + (size_t)(it + dt) * (size_t)bt.das * 2 +
                                (size_t)(b >> 4) * nch * 1024 + (size_t)(b & 15) * 16 + bofs[i];
                rbv[sl][i] = it + dt < bt.T ? *(const u32x4_t*)p : u32x4_t{0, 0, 0, 0};
            } else {
                rbv[sl][i] = __builtin_amdgcn_raw_buffer_load_b128(
                    brc, (uint32_t)dt * dasb + (uint32_t)((b >> 4) * nch) * 1024u + (uint32_t)(b & 15) * 16u + bofs[i], 0, 0);
            }
        }
        ir += 32;
        if (B >= 32) {
            ib += 32;
            if (ib >= B) { ib -= B; ++it; }
        } else {
            ib += 32;
            const int dt = (int)(((uint32_t)ib * msmall) >> 16);
            it += dt;
            ib -= dt * B;
        }
    };
    auto stage = [&](int buf, int sl) {
        bf16* Ab = As + buf * 32 * AP;
        bf16* Bb = Bs + buf * 32 * BPITCH;
#pragma unroll
        for (int i = 0; i < PA; ++i) *(u32x4_t*)(Ab + (ar + i * (NTH / APR)) * AP + 8 * (tid % APR)) = ra[sl][i];
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const int blk = w + NW * i;
            *(u32x4_t*)(Bb + (16 * (blk & 1) + br) * BPITCH + 32 * (blk >> 1) + 8 * bk) = rbv[sl][i];
        }
    };
    f32x4_t acc[MI][NI], dbacc[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        dbacc[j] = f32x4_t{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < MI; ++i) acc[i][j] = f32x4_t{0, 0, 0, 0};
    }
    Raw8<bf16> ones;                           // the bias gradient: da fragments times ones
#pragma unroll
    for (int q = 0; q < 4; ++q) ones.w[q] = 0x3f803f80u;
    const int trow = 8 * (lane >> 4) + ((lane & 15) >> 2), tcol = 4 * (lane & 3);
    auto frag = [&](Raw8<bf16>& f, const bf16* p, int pitch) {
        const uint2 lo = lds_tr4(p), hi = lds_tr4(p + 4 * pitch);
        f.w[0] = lo.x; f.w[1] = lo.y; f.w[2] = hi.x; f.w[3] = hi.y;
    };
    auto barrier = [&]() {                     // LDS only: the loads stay in flight
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // (two builds of the loop: a branch around the bias products inside it makes
    // the compiler copy every accumulator at every chunk)
    auto run = [&](auto with_db) {
        auto multiply = [&](int buf) {
            const bf16* Ab = As + buf * 32 * AP + trow * AP + wm * MI * 16 + tcol;
            const bf16* Bb = Bs + buf * 32 * BPITCH + trow * BPITCH + wn * NI * 16 + tcol;
            Raw8<bf16> fb[NI];
#pragma unroll
            for (int j = 0; j < NI; ++j) frag(fb[j], Bb + 16 * j, BPITCH);
            if constexpr (decltype(with_db)::value)
#pragma unroll
                for (int j = 0; j < NI; ++j) raw_mma(fb[j], ones, dbacc[j]);
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                Raw8<bf16> fa;
                frag(fa, Ab + 16 * i, AP);
#pragma unroll
                for (int j = 0; j < NI; ++j) raw_mma(fb[j], fa, acc[i][j]);
            }
        };
        issue(0);
        issue(1);
        stage(0, 0);
        issue(0);
        barrier();
        // chunks in pairs (an odd last one multiplies zeros): stage q+1 (loaded two
        // chunks ago), its registers take the loads of q+3, multiply q
        for (int q = 0; q < nq; q += 2) {
            stage(1, 1);
            issue(1);
            multiply(0);
            barrier();
            stage(0, 0);
            issue(0);
            multiply(1);
            barrier();
        }
    };
    if (dbw && wm == 0) run(std::true_type());
    else run(std::false_type());
    // (transposed products) output r of this lane is gradient column
    // 4*(lane/16)+r of the column tile, in the lane's own row
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int row = r0 + (wm * MI + i) * 16 + (lane & 15);
        if (row >= a.K) continue;
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int n = n0 + (wn * NI + j) * 16 + 4 * (lane >> 4);     // (G is a multiple of 4)
            if (n < G)
                *(float4*)(a.out + (size_t)row * G + n) =
                    make_float4(a.s * acc[i][j][0], a.s * acc[i][j][1], a.s * acc[i][j][2], a.s * acc[i][j][3]);
        }
    }
    if (dbw && wm == 0 && (lane & 15) == 0) {
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int n = n0 + (wn * NI + j) * 16 + 4 * (lane >> 4) + r;
                if (n < G) a.db[n] = dbacc[j][r];
            }
    }
}

// Whether n tiles of 256 x 256, one to a compute unit at a time, fill at least `pct`
// percent of the rounds they take on 256 of them.  Such a tile does the work of four of
// 128 x 128 in two thirds to three quarters of their time, where its last round is full.
static bool rounds_fill(long n, int pct) { return n * 100 >= pct * 256 * ((n + 255) / 256); }

// The tile of a pass (us with 128 x 128 and with 256 x 256, by the share of the rounds
// that the latter fills; contraction of 640 / 2560 / 8192 rows, 2000 to 16384 columns):
//   0.56   51 /  65   147 / 182   425 / 536
//   0.75   32 /  34   111 / 117   268 / 274   (2000 to 3840 rows in the middle)
//   0.73   61 /  68   215 / 228   511 / 547   (two rounds)
//   0.87   43 /  36   126 /  96   360 / 273
//   1.00   45 /  38   131 /  98   373 / 283   (two rounds: 77 / 71, 217 / 188, 665 / 567)
// and 565 against 733 at 16384 rows, hidden 1024: the line lies at 0.8.  64 x 128 below
// one tile of 128 x 128 a compute unit: 16 against 19, 57 against 65 and 138 against 156
// us at a quarter of one; 21 / 21, 57 / 59 and 174 / 163 at one.  WIDE builds are those
// of 256 x 256 and 64 x 128, which are equal at 0.56 (532 and 536 us).
void launch_wgrad_rows(WrBatch& b, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    if (b.np == 0) return;
    auto fill = [&](int TM, int TN) {
        b.total = 0;
        for (int i = 0; i < b.np; ++i) {
            b.p[i].nrb = (b.p[i].K + TM - 1) / TM;
            b.p[i].tiles = b.p[i].nrb * ((b.G + TN - 1) / TN);
            b.total += b.p[i].tiles;
        }
        b.per = (b.total + 7) / 8;
        return b.total;
    };
    auto go = [&](auto kern, int nth, size_t lds) {
        const dim3 grid(8 * b.per), blk(nth);
        if (e0 && e1) hipExtLaunchKernelGGL(kern, grid, blk, (uint32_t)lds, st, e0, e1, 0, b);
        else kern<<<grid, blk, lds, st>>>(b);
    };
    const int mid = 256;
    if (wr_wide(b)) {
        if (rounds_fill(fill(256, 256), 50)) go(k_wgrad_rows<2, 4, 8, 4, true>, 512, WrShape<2, 4, 8, 4>::LDS);
        else {
            fill(64, 128);
            go(k_wgrad_rows<1, 4, 4, 2, true>, 256, WrShape<1, 4, 4, 2>::LDS);
        }
    } else if (rounds_fill(fill(256, 256), 80)) go(k_wgrad_rows<2, 4, 8, 4>, 512, WrShape<2, 4, 8, 4>::LDS);
    else if (fill(128, 128) >= mid) go(k_wgrad_rows<2, 2, 4, 4>, 256, WrShape<2, 2, 4, 4>::LDS);
    else {
        fill(64, 128);
        go(k_wgrad_rows<1, 4, 4, 2>, 256, WrShape<1, 4, 4, 2>::LDS);
    }
}

// ---------------------------------------------------------------------------
// Input products and input gradients (bf16) as matrix products over all T*B (step,
// row) pairs:
//   ROWS_FX: out[r][n] = s * sum_k x[r][k] W[k][n] + bias[n]   (x masked, row-major)
//   ROWS_DX: out[r][k] = s * m_t[k] * sum over directions and n of DA[r][n] W[k][n]
// At 20 to 64 rows a step, a product per step over its kept neurons reads their rows
// of W again for each step and pads its rows to the tile: that, not the
// multiplications, was its time, so one product over all steps that multiplies the
// dropped columns' zeros is 2 to 4 times as fast.
// The MFMA's row side (TM = WM*MI*16) is the output's contiguous side, so a lane
// holds four adjacent outputs of one row.  The rows' operand is staged fragment-major
// (1 KB blocks, 16 rows x 32 of the contraction); so are the rows of W for ROWS_DX,
// while W is staged contraction-major for ROWS_FX and read by transposing LDS reads.
// Two LDS buffers of KC chunks of 32 each, loads two buffers ahead of the staging, one
// LDS-only barrier per buffer: the small tiles, a few workgroups to a CU, take the time
// of a load and a barrier per buffer whatever its depth, so they run at KC 2.
// slices > 1 (ROWS_DX) splits the contraction over workgroups, each writing its
// partial product; k_rows_reduce adds them in order.
constexpr int ROWS_FX = 0, ROWS_DX = 1;
template <int MODE, int WM, int WN, int MI, int NI, int KC>
struct RowsShape {
    static constexpr int NW = WM * WN, NTH = 64 * NW, TM = WM * MI * 16, TN = WN * NI * 16;
    static constexpr int MP = TM + 16;                               // contraction-major row pitch
    static constexpr int MEL = MODE == ROWS_FX ? 32 * MP : TM * 32, NEL = TN * 32;   // elements of a chunk
    static constexpr size_t LDS = (size_t)2 * KC * (MEL + NEL) * 2;
};

template <int MODE, int WM, int WN, int MI, int NI, int KC>
__global__ void __launch_bounds__(64 * WM * WN, 2) k_rows(RowsArgs a) {
    using S = RowsShape<MODE, WM, WN, MI, NI, KC>;
    constexpr int NTH = S::NTH, NW = S::NW, TM = S::TM, TN = S::TN, MP = S::MP;
    constexpr int PM = TM * 4 / NTH, PN = TN / 16 / NW;              // row-side pieces per thread; row blocks per wave
    static_assert(PM * NTH == TM * 4 && PN * NW * 16 == TN, "whole pieces");
    extern __shared__ __align__(16) char smem[];
    bf16* Ms = (bf16*)smem;                                          // [2][KC][MEL]
    bf16* Ns = Ms + 2 * KC * S::MEL;                                 // [2][KC][NEL]
    int pos = (int)(blockIdx.x % 8) * a.per + (int)(blockIdx.x / 8);
    if (pos >= a.total) return;
    // (problem or slice, column tile, row tile): an XCD's range shares its W columns
    const int nrt = (a.R + TN - 1) / TN, nmt = (a.M + TM - 1) / TM;
    const int z = pos / (nrt * nmt), mt = pos / nrt % nmt, rt = pos % nrt;
    const int m0 = mt * TM, r0 = rt * TN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w / WN, wn = w % WN;
    const int br = lane & 15, bk = lane >> 4;
    const int G = a.G, B = a.B;
    // the steps (KC chunks of the contraction) of this workgroup: ROWS_FX all of problem
    // z; ROWS_DX slice z of the directions' steps one after the other
    const int KK = MODE == ROWS_FX ? a.K : G;
    const int nch = (KK + 31) / 32, nsd = (nch + KC - 1) / KC;
    const int nall = MODE == ROWS_FX ? nsd : a.D * nsd;
    const int c0 = MODE == ROWS_FX ? 0 : (int)((long)nall * z / a.slices);
    const int c1 = MODE == ROWS_FX ? nall : (int)((long)nall * (z + 1) / a.slices);
    const int nc = c1 - c0;
    // rows' operand: block w + NW*i holds rows r0 + 16*(w + NW*i) .. +15
    size_t nbase[PN];                                                // element offset of this lane's piece of chunk 0
#pragma unroll
    for (int i = 0; i < PN; ++i) {
        const int r = min(r0 + 16 * (w + NW * i) + br, a.R - 1);
        if constexpr (MODE == ROWS_FX) {
            nbase[i] = (size_t)r * a.lda + 8 * bk;
        } else {
            const int t = r / B, b = r % B;
            nbase[i] = (size_t)t * a.das + frag_lane_off(0, b >> 4, bk * 16 + (b & 15), nch);
        }
    }
    // W: ROWS_FX rows of the chunk (tid / (TM/8) + passes), 8 columns each; ROWS_DX
    // block (wave + NW*i): 16 rows of W, this lane's row and 8 of the contraction
    constexpr int MPR = TM / 8;
    uint32_t mofs[PM];
#pragma unroll
    for (int i = 0; i < PM; ++i) {
        if constexpr (MODE == ROWS_FX) {
            mofs[i] = (uint32_t)((tid / MPR + i * (NTH / MPR)) * G + m0 + 8 * (tid % MPR)) * 2u;
        } else {
            const int k = min(m0 + 16 * (w + NW * i) + br, a.M - 1);
            mofs[i] = ((uint32_t)k * (uint32_t)G + 8u * bk) * 2u;
        }
    }
    const uint32_t wbytes = (uint32_t)(MODE == ROWS_FX ? a.K : a.M) * (uint32_t)G * 2u;
    const void* W0 = MODE == ROWS_FX ? a.W[z] : a.W[0];
    u32x4_t rm[2][KC][PM], rn[2][KC][PN];
    int ci = c0;                                                     // next step to load
    auto issue = [&](int sl) {
        const int cc = min(ci, c1 - 1);
        const int d = MODE == ROWS_DX && cc >= nsd ? 1 : 0;
        const __amdgpu_buffer_rsrc_t wr = buf_rsrc(MODE == ROWS_FX ? W0 : a.W[d], wbytes);
        const bf16* X = (const bf16*)(MODE == ROWS_FX ? a.x : a.da[d]);
#pragma unroll
        for (int q = 0; q < KC; ++q) {
            const int c = min((cc - d * nsd) * KC + q, nch - 1);     // (chunks past the end: cleared when staged)
            const uint32_t wadd = MODE == ROWS_FX ? (uint32_t)c * 64u * (uint32_t)G : 64u * (uint32_t)c;
#pragma unroll
            for (int i = 0; i < PM; ++i) rm[sl][q][i] = __builtin_amdgcn_raw_buffer_load_b128(wr, mofs[i] + wadd, 0, 0);
#pragma unroll
            for (int i = 0; i < PN; ++i) {
                if constexpr (MODE == ROWS_FX) {
                    // (pieces past the row's end: its last one, cleared when staged)
                    const size_t o = 32 * c + 8 * bk < a.lda ? (size_t)32 * c : (size_t)(a.lda - 8 - 8 * bk);
                    rn[sl][q][i] = *(const u32x4_t*)(X + nbase[i] + o);
                } else {
                    rn[sl][q][i] = *(const u32x4_t*)(X + nbase[i] + (size_t)c * 512);
                }
            }
        }
        ++ci;
    };
    int cs = c0;                                                     // next step to stage
    auto stage = [&](int buf, int sl) {
        const int cc = MODE == ROWS_DX && cs >= nsd ? cs - nsd : cs;
#pragma unroll
        for (int q = 0; q < KC; ++q) {
            bf16* Mb = Ms + (buf * KC + q) * S::MEL;
            bf16* Nb = Ns + (buf * KC + q) * S::NEL;
            const int k0 = 32 * (cc * KC + q);
            if (k0 + 32 > KK) {                // the contraction's ragged end: zeros past it
                uint32_t m[4];
                pad_mask<bf16>(k0 + 8 * bk, KK, m);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
#pragma unroll
                    for (int i = 0; i < PN; ++i) rn[sl][q][i][e] &= m[e];
                    if constexpr (MODE == ROWS_DX)
#pragma unroll
                        for (int i = 0; i < PM; ++i) rm[sl][q][i][e] &= m[e];
                }
                if constexpr (MODE == ROWS_FX)
#pragma unroll
                    for (int i = 0; i < PM; ++i)
                        if (k0 + tid / MPR + i * (NTH / MPR) >= KK) rm[sl][q][i] = u32x4_t{0, 0, 0, 0};
            }
#pragma unroll
            for (int i = 0; i < PM; ++i) {
                if constexpr (MODE == ROWS_FX)
                    *(u32x4_t*)(Mb + (tid / MPR + i * (NTH / MPR)) * MP + 8 * (tid % MPR)) = rm[sl][q][i];
                else
                    *(u32x4_t*)(Mb + (w + NW * i) * 512 + lane * 8) = rm[sl][q][i];
            }
#pragma unroll
            for (int i = 0; i < PN; ++i) *(u32x4_t*)(Nb + (w + NW * i) * 512 + lane * 8) = rn[sl][q][i];
        }
        ++cs;
    };
    f32x4_t acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f32x4_t{0, 0, 0, 0};
    const int trow = 8 * (lane >> 4) + ((lane & 15) >> 2), tcol = 4 * (lane & 3);
    auto multiply = [&](int buf) {
#pragma unroll
        for (int q = 0; q < KC; ++q) {
            const bf16* Mb = Ms + (buf * KC + q) * S::MEL;
            const bf16* Nb = Ns + (buf * KC + q) * S::NEL + (wn * NI) * 512 + lane * 8;
            Raw8<bf16> fn[NI];
#pragma unroll
            for (int j = 0; j < NI; ++j) raw_lds(fn[j], Nb + j * 512);
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                Raw8<bf16> fm;
                if constexpr (MODE == ROWS_FX) {
                    const bf16* p = Mb + trow * MP + (wm * MI + i) * 16 + tcol;
                    const uint2 lo = lds_tr4(p), hi = lds_tr4(p + 4 * MP);
                    fm.w[0] = lo.x; fm.w[1] = lo.y; fm.w[2] = hi.x; fm.w[3] = hi.y;
                } else {
                    raw_lds(fm, Mb + (wm * MI + i) * 512 + lane * 8);
                }
#pragma unroll
                for (int j = 0; j < NI; ++j) raw_mma(fm, fn[j], acc[i][j]);
            }
        }
    };
    auto barrier = [&]() {                     // LDS only: the loads stay in flight
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    issue(0);
    issue(1);
    stage(0, 0);
    issue(0);
    barrier();
    int c = 0;
    for (; c + 1 < nc; c += 2) {
        stage(1, 1);
        issue(1);
        multiply(0);
        barrier();
        stage(0, 0);
        issue(0);
        multiply(1);
        barrier();
    }
    if (c < nc) multiply(0);
    // output r of this lane: column 4*(lane/16)+r of the tile, row lane%16
    bool nan = false;
    const bool failed = MODE == ROWS_DX && a.status && *a.status != 0;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int r = r0 + (wn * NI + j) * 16 + br;
        if (r >= a.R) continue;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int n = m0 + (wm * MI + i) * 16 + 4 * bk;
            if (n >= a.M) continue;
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = a.s * acc[i][j][e];
            if constexpr (MODE == ROWS_FX) {
                nan = nan || v[0] != v[0] || v[1] != v[1] || v[2] != v[2] || v[3] != v[3];
                const float4 bn = *(const float4*)(a.bias[z] + n);   // (M = G is a multiple of 4)
                *(float4*)(a.out[z] + (size_t)r * a.M + n) = make_float4(v[0] + bn.x, v[1] + bn.y, v[2] + bn.z, v[3] + bn.w);
            } else if (a.slices > 1) {
                float* o = a.part + ((size_t)z * a.R + r) * a.M + n;
                if ((a.M & 3) == 0) {
                    *(float4*)o = make_float4(v[0], v[1], v[2], v[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < a.M) o[e] = v[e];
                }
            } else {
                const uint8_t* mk = a.mask + (size_t)(r / B) * a.kmax + n;
                float* o = a.out[0] + (size_t)r * a.M + n;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[e] = failed ? __builtin_nanf("") : mk[min(e, a.M - 1 - n)] ? v[e] : 0.0f;
                if ((a.M & 3) == 0) {
                    *(float4*)o = make_float4(v[0], v[1], v[2], v[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < a.M) o[e] = v[e];
                }
            }
        }
    }
    // A weight row that holds Inf or NaN makes a dropped neuron's product with it NaN, where
    // the method does not read the row: outputs that are NaN are formed again, over the kept
    // neurons alone (and end at the first kept one that makes them NaN).
    if constexpr (MODE == ROWS_FX) {
        if (!nan) return;
#pragma unroll 1
        for (int x = 0; x < MI * NI * 4; ++x) {
            const int r = r0 + (wn * NI + x / (4 * MI)) * 16 + br, n = m0 + (wm * MI + x / 4 % MI) * 16 + 4 * bk + x % 4;
            if (r >= a.R || n >= a.M) continue;
            float* o = a.out[z] + (size_t)r * a.M + n;
            if (*o == *o) continue;
            const uint8_t* mk = a.mask + (size_t)(r / B) * a.kmax;
            const bf16 *xr = (const bf16*)a.x + (size_t)r * a.lda, *wc = (const bf16*)a.W[z] + n;
            float v = 0.0f;
#pragma unroll 1
            for (int k = 0; k < a.K && v == v; ++k)
                if (mk[k]) v += bf2f(xr[k]) * bf2f(wc[(size_t)k * G]);
            *o = a.s * v + a.bias[z][n];
        }
    }
}

// out[r][k] = m_t[k] * sum of the slices in order.  grid (ceil(M/256), ceil(R/4)).
__global__ void __launch_bounds__(256) k_rows_reduce(RowsArgs a) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= a.M) return;
    const bool failed = a.status && *a.status != 0;
    const size_t n = (size_t)a.R * a.M;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = blockIdx.y * 4 + i;
        if (r >= a.R) return;
        const float* p = a.part + (size_t)r * a.M + k;
        float v = 0.0f;
        for (int z = 0; z < a.slices; ++z) v += p[(size_t)z * n];
        a.out[0][(size_t)r * a.M + k] = failed ? __builtin_nanf("") : a.mask[(size_t)(r / a.B) * a.kmax + k] ? v : 0.0f;
    }
}

template <int MODE, int WM, int WN, int MI, int NI, int KC>
static void rows_go(RowsArgs& a, int z, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    using S = RowsShape<MODE, WM, WN, MI, NI, KC>;
    a.total = ((a.R + S::TN - 1) / S::TN) * ((a.M + S::TM - 1) / S::TM) * z;
    a.per = (a.total + 7) / 8;
    const dim3 grid(8 * a.per), blk(S::NTH);
    if (e0 && e1) hipExtLaunchKernelGGL((k_rows<MODE, WM, WN, MI, NI, KC>), grid, blk, (uint32_t)S::LDS, st, e0, e1, 0, a);
    else k_rows<MODE, WM, WN, MI, NI, KC><<<grid, blk, S::LDS, st>>>(a);
}
static long rows_tiles(const RowsArgs& a, int TM, int TN) {
    return (long)((a.R + TN - 1) / TN) * ((a.M + TM - 1) / TM);
}
// Tiles of the input products (us at 64 x 64, 128 x 128 and 256 x 256 tiles; contraction
// of 300, and of 1500 or 1000).
// 128 x 128 from 160 of them on, from 512 where the contraction is short (of 700 at 200
// tiles: 22 / 18 us):
//   120 tiles   9.5 / 12.7     20 / 26        320 tiles   17 / 19       33 / 30
//   140 tiles   12 / 13        26 / 26        640 tiles   28 / 26       65 / 48
//   200 tiles   13.6 / 14.0    33 / 27       1260 tiles   49 / 39      123 / 81
// 256 x 256 where they fill 0.7 of their rounds:
//   0.62 (320)  39 / 48        81 / 87        0.78 (200)  31 / 27       75 / 58
//   0.66 (170)  25 / 27        59 / 59        0.86 (440)  52 / 52       131 / 116
//   0.74 (380)  45 / 48       116 / 109       0.98 (500)  63 / 53       128 / 93
// and 349 against 462 at 16384 rows x 1024 x 4096 (four full rounds, two layers).
void launch_fx_rows(RowsArgs& a, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    a.M = a.G;
    if (rounds_fill(rows_tiles(a, 256, 256) * a.np, 70)) rows_go<ROWS_FX, 2, 4, 8, 4, 1>(a, a.np, st, e0, e1);
    else if (rows_tiles(a, 128, 128) * a.np >= (a.K >= 400 ? 160 : 512)) rows_go<ROWS_FX, 2, 2, 4, 4, 1>(a, a.np, st, e0, e1);
    else rows_go<ROWS_FX, 2, 2, 2, 2, 2>(a, a.np, st, e0, e1);
}
// Tiles of the input gradients (us; contraction D*G of 1000 / 2600 / 4600 / 6000 / 12000
// columns).
// 256 x 256 where they fill 0.55 of their rounds, against 128 x 128:
//   0.39   63 / 40    99 / 68   143 / 102   173 / 128   317 / 230
//   0.54   66 / 57   101 / 101  146 / 153   188 / 193   321 / 353
//   0.78   64 / 73   101 / 128  155 / 200   200 / 255   332 / 464
// 128 x 128 from 160 of them on, against the better of 64 x 64 and slices:
//   104    24 / 18    37 / 31    56 / 44     69 / 51    127 / 95
//   160    24 / 25    39 / 40    57 / 68     69 / 78    132 / 124
//   350    39 / 44    67 / 67   101 / 103   126 / 129   227 / 216
// below that 64 x 64 for contractions up to 5000, 128 x 128 with the contraction sliced
// to two workgroups a CU beyond (64 x 64 and slices at 20 and 80 tiles: 3000 columns 21 /
// 27 and 34 / 41, 4600 28 / 30 and 46 / 42, 5400 33 / 31 and 54 / 46, 16000 85 / 57 and
// 156 / 102).
void launch_dx_rows(RowsArgs& a, size_t part_bytes, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    const long n256 = rows_tiles(a, 256, 256), n128 = rows_tiles(a, 128, 128);
    a.slices = 1;
    if (rounds_fill(n256, 55)) return rows_go<ROWS_DX, 2, 4, 8, 4, 1>(a, 1, st, e0, e1);
    if (n128 < 160 && (long)a.D * a.G <= 5000) return rows_go<ROWS_DX, 2, 2, 2, 2, 2>(a, 1, st, e0, e1);
    const long most = (long)std::min<size_t>(part_bytes / ((size_t)a.R * a.M * 4), 16);
    const long want = std::min(std::min((512 + n128 - 1) / n128, most), (long)a.D * ((a.G + 63) / 64) / 4);
    if (n128 >= 160 || want < 2) return rows_go<ROWS_DX, 2, 4, 4, 2, 2>(a, 1, st, e0, e1);
    a.slices = (int)want;
    if (e0) (void)hipEventRecord(e0, st);
    rows_go<ROWS_DX, 2, 4, 4, 2, 2>(a, a.slices, st, nullptr, nullptr);
    k_rows_reduce<<<dim3((a.M + 255) / 256, (a.R + 3) / 4), 256, 0, st>>>(a);
    if (e1) (void)hipEventRecord(e1, st);
}

template <int MODE, int WM, int WN, int MI, int NI, int KC>
static bool rows_lds() {
    return hipFuncSetAttribute((const void*)k_rows<MODE, WM, WN, MI, NI, KC>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)RowsShape<MODE, WM, WN, MI, NI, KC>::LDS) == hipSuccess;
}
int setup_big_attributes() {
    bool ok = hipFuncSetAttribute((const void*)k_wgrad_rows<2, 4, 8, 4>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)WrShape<2, 4, 8, 4>::LDS) == hipSuccess;
    ok = hipFuncSetAttribute((const void*)k_wgrad_rows<2, 4, 8, 4, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)WrShape<2, 4, 8, 4>::LDS) == hipSuccess && ok;
    ok = hipFuncSetAttribute((const void*)k_fx_big, hipFuncAttributeMaxDynamicSharedMemorySize, (int)FB_LDS) ==
             hipSuccess && ok;
    ok = hipFuncSetAttribute((const void*)k_dx_big, hipFuncAttributeMaxDynamicSharedMemorySize, (int)DB_LDS) ==
             hipSuccess && ok;
    ok = rows_lds<ROWS_FX, 2, 4, 8, 4, 1>() && rows_lds<ROWS_DX, 2, 4, 8, 4, 1>() &&
         rows_lds<ROWS_DX, 2, 4, 4, 2, 2>() && ok;
    return ok ? 0 : -1;
}

}  // namespace lsd
