// Persistent recurrences with the weights in registers (gfx950, bf16).
//
// One launch runs every time step of its slots for a range of row groups:
// the directions of one layer, or the layers of a unidirectional stack
// together with their product workers (forward: the input product of a layer
// above the first; backward: the input gradient of a layer above the first).
// A workgroup owns (slot, tile of hidden units, group of 16 or 32 batch rows),
// has the compute unit to itself (512 threads of up to 256 registers) and
// holds its slice of the slot's weight matrix for the whole sequence as MFMA
// fragments in registers (the backward of a wide layer keeps part of it in
// LDS).
//
// What bounds a step is the chain barrier -> exchange loads -> product ->
// cross-wave sum -> pointwise -> publish, not arithmetic.  A step that writes
// 2 KB per workgroup, meets at a barrier of 32 workgroups and reads 64 / 128 /
// 256 KB of exchanged data into every compute unit measures 2.0 / 2.4 / 3.7 us
// (0.75 / 0.92 / 1.2 us of it the barrier at 8 / 32 / 82 workgroups), whatever
// the cache scope of the exchange.  Hence:
//   - rows are independent in a recurrence, so each row group has a barrier of
//     its own, over its unit tiles only;
//   - weights in registers give wide unit tiles (fewer workgroups per barrier
//     and fewer reads of the exchanged block) and fit whole stacks on the chip
//     whose slices exceed LDS: the layers then run as a pipeline, T + 2(L - 1)
//     steps (a layer and its worker are a step apart each) in place of L*T;
//   - a worker's product goes to the one workgroup of the layer that owns the
//     same tile and rows, so that hand-over is a flag, not a barrier;
//   - workgroup barriers wait for LDS only: the outputs that later kernels
//     read and the next step's inputs stay in flight over the grid barrier.
// Measured per launch, before (weights in LDS, or a large batch in two phases) and
// with this: two stacked layers of 650 at 20 rows, 35 steps: forward 172 -> 112,
// backward 200 -> 122 us; three of 1150, 70 steps: 865 -> 380, 1300 -> 570 us (5%
// between runs); one layer of 1024 at 256 rows, 64 steps: 488 -> 387, 943 -> 452 us.
// Dropped neurons are zeros in the exchanged block (the masks are known to the
// producer), in compact and dense mode alike: a step's products are a small
// part of its time, and a register slice cannot be gathered by row.
#include <hip/hip_runtime.h>

#include <stdlib.h>

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

#include "device.h"
#include "kernels.h"
#include "sync.h"
#include "../../include/lstm_sd.h"

namespace lsd {

typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));

// LDS-only workgroup barrier: this wave's LDS accesses are done, its global
// loads and stores stay in flight.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ---- grid synchronisation -----------------------------------------------------
// Group g of a launch has RB_LINES counter lines; member (tile) j adds to line
// j % RB_LINES.  A worker's group uses its lines for flags instead: member j's
// step count at word 1 + j / RB_LINES of line j % RB_LINES.
__device__ __forceinline__ unsigned* res_line(unsigned* bar, int g, int i) { return bar + (g * RB_LINES + i) * RB_PITCH; }
__device__ __forceinline__ unsigned* res_flag(unsigned* bar, int g, int tile) {
    return res_line(bar, g, tile % RB_LINES) + 1 + tile / RB_LINES;
}
// every store of the workgroup so far is complete at the coherence point
__device__ __forceinline__ void res_drain() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
}
__device__ __forceinline__ void res_arrive(unsigned* bar, int g, int tile) {
    res_drain();
    if (threadIdx.x == 0)
        __hip_atomic_fetch_add(res_line(bar, g, tile % RB_LINES), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void res_signal(unsigned* bar, int g, int tile, unsigned v) {
    res_drain();
    if (threadIdx.x == 0) __hip_atomic_store(res_flag(bar, g, tile), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Wait until group g (n members) has completed `steps` steps, and, with gf >= 0,
// member `tile` of worker group gf has signalled `fval`.  One wave polls;
// bounded by wall-clock time as grid_wait, with the same failure protocol.
__device__ __forceinline__ bool res_wait(unsigned* bar, int g, int n, unsigned steps, int gf, int tile, unsigned fval,
                                         int* err, long long timeout, int fail_bit) {
    __shared__ int ok;
    if (timeout <= 0) {
        if (threadIdx.x == 0) {
            __hip_atomic_fetch_or(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_or(sync_status(err), fail_bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        res_drain();
        return false;
    }
    if (threadIdx.x < 64) {
        const int i = threadIdx.x;
        unsigned want = 0;
        const unsigned* p = res_line(bar, g, i & (RB_LINES - 1));
        if (i < RB_LINES) want = steps * (unsigned)((n - i + RB_LINES - 1) / RB_LINES);   // (members on line i; n - i may be < 0)
        if (i < RB_LINES && i >= n) want = 0;
        if (i == RB_LINES && gf >= 0) {
            p = res_flag(bar, gf, tile);
            want = fval;
        }
        int good = 1;
        const long long t0 = wall_clock64();
        for (;;) {
            const unsigned v = want ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
            if (__builtin_amdgcn_ballot_w64(v < want) == 0) break;
            const long long el = wall_clock64() - t0;
            if (el > timeout) {
                if (i == 0) {
                    __hip_atomic_fetch_or(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_fetch_or(sync_status(err), fail_bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                }
                good = 0;
                break;
            }
            if (el > (timeout >> 12)) {
                const int e = i == 0 ? __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
                if (__builtin_amdgcn_ballot_w64(e != 0) != 0) { good = 0; break; }
            }
        }
        if (i == 0) ok = good;
    }
    lds_barrier();
    const bool r = ok != 0;
    return r;
}
// The last workgroup to leave (of `total` working ones) poisons the outputs of a failed
// pass and returns the counters, the flags and the error flag to zero for the next launch.
__device__ __forceinline__ void res_exit(unsigned* bar, int ngroups, int total, int* err, const Poison& out) {
    __shared__ int last;
    res_drain();
    if (threadIdx.x == 0)
        last = __hip_atomic_fetch_add(bar + BAR_PITCH * BAR_LINES * BAR_EXIT, 1u, __ATOMIC_ACQ_REL,
                                      __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(total - 1);
    __syncthreads();
    if (!last) return;
    poison_if_failed(out, err);
    for (int i = threadIdx.x; i < ngroups * RB_LINES * RB_PITCH; i += blockDim.x)
        __hip_atomic_store(bar + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (threadIdx.x == 0) {
        __hip_atomic_store(err, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(bar + BAR_PITCH * BAR_LINES * BAR_EXIT, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}
// Workgroup -> (group, tile); false: nothing to do.  Workgroup i runs on XCD
// i % 8.  With gpx > 0 an XCD takes whole groups (group g on XCD g % 8, gpx of
// them at most), whose exchange then stays within one L2; otherwise an XCD takes
// a contiguous range of (group, tile) positions.
__device__ __forceinline__ bool res_place(int ngroups, int ntiles, int gpx, int& g, int& tile) {
    const int x = blockIdx.x % 8, j = blockIdx.x / 8;
    if (gpx > 0) {
        g = x + 8 * (j / ntiles);
        tile = j % ntiles;
        return g < ngroups;
    }
    const int pos = x * (int)((ngroups * ntiles + 7) / 8) + j;
    g = pos / ntiles;
    tile = pos % ntiles;
    return g < ngroups;
}

__device__ __forceinline__ float4 load_coherent4(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, CPOL_SC1);
    return make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
}

// VW consecutive 16-bit elements as one load, and element v of it
template <int VW> struct LoadWords;
template <> struct LoadWords<1> { typedef uint16_t type; };
template <> struct LoadWords<2> { typedef uint32_t type; };
template <> struct LoadWords<4> { typedef uint2 type; };
__device__ __forceinline__ uint32_t half_of(uint16_t x, int) { return x; }
__device__ __forceinline__ uint32_t half_of(uint32_t x, int v) { return v ? x >> 16 : x & 0xffffu; }
__device__ __forceinline__ uint32_t half_of(uint2 x, int v) { return half_of(v & 2 ? x.y : x.x, v & 1); }

// The gate sums of unit u of row b over the kept neurons alone, from the exchanged block
// src and the weights in memory.  A weight row that holds Inf or NaN makes a dropped
// neuron's product with it NaN, where the method does not read the row: in a workgroup
// that has met one in its weights, a sum that is NaN is formed again here (and ends at
// the first kept neuron that makes all four gates NaN).
__device__ __forceinline__ float4 kept_sum(const bf16* src, const bf16* U, const uint8_t* mask, int b, int u, int H) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 1
    for (int k = 0; k < H; ++k) {
        if (!mask[k]) continue;
        const float h = bf2f(__hip_atomic_load(src + frag_off(b, k, (H + 31) / 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        const bf16* p = U + (size_t)k * (4 * H) + u;
        v.x += h * bf2f(p[0]); v.y += h * bf2f(p[H]); v.z += h * bf2f(p[2 * H]); v.w += h * bf2f(p[3 * H]);
        if (v.x != v.x && v.y != v.y && v.z != v.z && v.w != v.w) break;
    }
    return v;
}

// ---------------------------------------------------------------------------
// Forward (Eq. 1-6).  Unit tile = 4*NTL units = NTL column tiles of the four
// gates of 4 units; rows = 16*MT.  Wave w holds the 32-neuron chunks w + 8c,
// c < KC, of the contraction.  Products are taken transposed (the weight
// fragment as the left operand): a lane then holds the four gates of one unit
// of one row, so a partial sum goes through LDS as one 16-byte piece.  The
// threads of the pointwise take the pairs unit by unit (whole runs of a row in
// every global access); the piece pitches (17 per 16 rows, 68 per fragment)
// keep both the stores and these loads free of bank conflicts.
constexpr int RF_QP = 17, RF_FP = 4 * RF_QP;               // float4 pitches in red
__host__ __device__ constexpr int rf_wpitch(int NTL) { return 16 * NTL + 8; }   // staged weight row (elements)
// LDS: red (first the staged weights); then the transposed stage
template <int NTL, int MT>
constexpr size_t rf_red_bytes() {
    const size_t r = (size_t)8 * NTL * MT * RF_FP * 16, s = (size_t)8 * 32 * rf_wpitch(NTL) * 2;
    return r > s ? r : s;
}
template <int NTL, int MT>
constexpr size_t rf_lds_bytes() { return rf_red_bytes<NTL, MT>() + (size_t)2 * 4 * NTL * (16 * MT + 8) * 2; }

template <int KC, int NTL, int MT>
__global__ void __launch_bounds__(512) k_fwd_res(RFwdArgs a) {
    constexpr int UT = 4 * NTL, MG = 16 * MT, NF = NTL * MT, NP = UT * MG, NTH = 512, NW = 8;
    constexpr int PPT = (NP + NTH - 1) / NTH;
    // pairs that leave a wave over go to the upper waves: wave 0 polls the next
    // barrier as soon as it has arrived (0.3 us of a step)
    constexpr int P0 = NP <= NTH ? (NTH - NP) / 64 * 64 : 0;
    constexpr int SP = MG + 8;                             // row pitch of a transposed stage (elements)
    extern __shared__ __align__(16) char smem[];
    float4* red = (float4*)smem;                           // [8 waves][NF][RF_FP]
    bf16* sty = (bf16*)(smem + rf_red_bytes<NTL, MT>());   // [2][UT][SP] layer output of the tile, transposed
    __shared__ int len_s[MG];                              // lengths of the rows
    __shared__ int bad_s[NW];                              // Inf or NaN among a wave's weights
    const int H = a.H, G = 4 * H, B = a.B, T_ = a.T;
    const int total = a.nslots * a.mgroups * a.ntiles;
    int g, tile;
    if (!res_place(a.nslots * a.mgroups, a.ntiles, a.gpx, g, tile)) return;
    const int sl = g / a.mgroups, mgl = g % a.mgroups;
    const RFwdSlot& D = a.d[sl];
    const int u0 = tile * UT, m0 = (a.mg0 + mgl) * a.rg, m1 = min(m0 + a.rg, B);   // rows m0 .. m1-1
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g8 = 8 * (lane >> 4), cl = lane & 15;
    const bool worker = D.role == 1;
    const int gdep = D.dep >= 0 ? D.dep * a.mgroups + mgl : -1;
    const int nch = (H + 31) / 32;
    if (tid < MG) len_s[tid] = a.lengths ? a.lengths[min(m0 + tid, B - 1)] : T_;

    // The weight slice: column cl of tile j is gate cl&3 of unit u0 + 4j +
    // (cl>>2).  Each wave stages its chunks (32 rows x 16*NTL columns) through
    // its own part of LDS: runs of UT units of a gate are loaded VW units at a
    // time (as the alignment of a row's gate blocks allows), the four gates
    // side by side make whole pieces, and the fragments come back by
    // transposing reads.  (Gathering the fragments' 2-byte elements from memory
    // took 30-80 us per launch.)
    bf16x8_t ub[KC][NTL];
    u16x2_t most = {0, 0};                                 // the largest magnitudes' bits: 0x7f80 and above are Inf and NaN
    {
        const bf16* U = (const bf16*)D.U;
        constexpr int WP = rf_wpitch(NTL);
        bf16* st = (bf16*)smem + (size_t)w * 32 * WP;
        auto stage = [&](auto vw, int c) {
            constexpr int VW = decltype(vw)::value, NG = UT / VW, N = 32 * NG, IT = (N + 63) / 64;
            typedef typename LoadWords<VW>::type word;
            word x[IT][4];
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const int e = min(lane + 64 * i, N - 1), k = 32 * (w + NW * c) + e / NG, u = u0 + VW * (e % NG);
                const bf16* p = U + (size_t)min(k, H - 1) * G + min(u, H - VW);
#pragma unroll
                for (int q = 0; q < 4; ++q) x[i][q] = *(const word*)(p + q * H);
            }
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const int e = lane + 64 * i, kr = e / NG, ug = e % NG;
                const bool ok = 32 * (w + NW * c) + kr < H && u0 + VW * ug < H;
                if (e < N) {
#pragma unroll
                    for (int v = 0; v < VW; ++v) {
                        uint32_t gt[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) gt[q] = ok ? half_of(x[i][q], v) : 0u;
                        *(uint2*)(st + kr * WP + 4 * (VW * ug + v)) = make_uint2(gt[0] | (gt[1] << 16), gt[2] | (gt[3] << 16));
                    }
                }
            }
        };
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            if ((H & 3) == 0) stage(std::integral_constant<int, 4>(), c);
            else if ((H & 1) == 0) stage(std::integral_constant<int, 2>(), c);
            else stage(std::integral_constant<int, 1>(), c);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int j = 0; j < NTL; ++j) {
                const bf16* p = st + (g8 + (cl >> 2)) * WP + 16 * j + 4 * (lane & 3);
                const uint2 lo = lds_tr4(p), hi = lds_tr4(p + 4 * WP);
                ub[c][j] = __builtin_bit_cast(bf16x8_t, u32x4_t{lo.x, lo.y, hi.x, hi.y});
                for (uint32_t x : {lo.x, lo.y, hi.x, hi.y})
                    most = __builtin_elementwise_max(most, __builtin_bit_cast(u16x2_t, x & 0x7fff7fffu));
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        const bool bad = __builtin_amdgcn_ballot_w64(most[0] >= 0x7f80 || most[1] >= 0x7f80) != 0;
        if (lane == 0) bad_s[w] = bad;
        lds_barrier();                                     // (the parts overlap red of other waves)
    }
    const bool spoilt = __builtin_amdgcn_ballot_w64(bad_s[lane & (NW - 1)] != 0) != 0;
    // this thread's (row, unit) pair q.  Derived anew from the (opaque) thread
    // index where a step needs it: kept in registers it would cost the large
    // tiles their room.  A pair outside the tile or the shape reads valid
    // addresses.
    struct Pair { int b, u, i, s; bool in, ok; };          // i: its piece in red; s: its element in a transposed stage
    auto pair_of = [&](int q, int th) {
        Pair r;
        const int p = th - P0 + NTH * q;
        r.in = p >= 0 && p < NP;
        const int row = r.in ? p / UT : 0, u = r.in ? p % UT : 0;
        r.b = m0 + row;
        r.u = u0 + u;
        r.i = ((row >> 4) * NTL + (u >> 2)) * RF_FP + (u & 3) * RF_QP + (row & 15);
        r.s = u * SP + row;
        r.ok = r.in && r.b < m1 && r.u < H;
        if (!r.ok) { r.b = m0; r.u = u0; }
        return r;
    };
    auto opaque_tid = [&]() { int v = tid; asm volatile("" : "+v"(v)); return v; };
    auto step_t = [&](int s) { return D.dir == 0 ? s : T_ - 1 - s; };
    const size_t hxs = (size_t)nch * a.mtiles * 512;       // elements of one exchange slot
    // byte offset of this lane's fragment of wave w's first chunk, for its row
    auto row_ofs = [&](int row) {
        return row < m1 ? (uint32_t)(frag_lane_off(w, row >> 4, (lane & 48) + (row & 15), nch) * 2) : OOB_OFF;
    };
    uint32_t lofs[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
        lofs[mt] = row_ofs(m0 + 16 * mt + cl);
    constexpr uint32_t cstep = NW * 1024;                  // bytes from chunk c to c + 1 of a wave
    // (only a wave's last chunk can be past the last one)
    auto cofs = [&](int mt, int c) { return c + 1 < KC || w + NW * c < nch ? lofs[mt] + (uint32_t)c * cstep : OOB_OFF; };
    auto red_sum = [&](int i) {
        float4 v = red[i];
#pragma unroll
        for (int k = 1; k < NW; ++k) {
            const float4 x = red[k * NF * RF_FP + i];
            v.x += x.x; v.y += x.y; v.z += x.z; v.w += x.w;
        }
        return v;
    };
    // partial products of one exchanged block, into red: a row tile at a time
    // (its sums go to LDS under the products of the next), R loads in flight
    // (mask: the contraction's kept neurons)
    auto product = [&](const bf16* src, const uint8_t* mask) {
        // (8 in flight spill where the weights fill the registers: three layers of 1150,
        // 70 steps: 375 us with 8, 360 with 4; two of 1500, 35 steps: 213 and 195; two
        // of 1024 at 256 rows, 64 steps: 786 and 768)
        constexpr int NA = KC * MT, RM = KC * NTL >= 28 ? 4 : 8, R = NA < RM ? NA : RM;
        const __amdgpu_buffer_rsrc_t r = buf_rsrc(src, (uint32_t)(hxs * 2));
        Raw8<bf16> fa[R];
#pragma unroll
        for (int i = 0; i < R; ++i) raw_load<bf16, CPOL_SC1>(fa[i], r, cofs(i / KC, i % KC));
        __builtin_amdgcn_sched_barrier(0);                 // (before the first product)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            f32x4_t acc[NTL];
#pragma unroll
            for (int j = 0; j < NTL; ++j) acc[j] = f32x4_t{0, 0, 0, 0};
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                Raw8<bf16>& f = fa[(mt * KC + c) % R];
                if (32 * (w + NW * c) + 32 > H) {           // neurons past H were never written
                    uint32_t m[4];
                    pad_mask<bf16>(32 * (w + NW * c) + g8, H, m);
                    raw_and(f, m);
                }
                const u32x4_t av = {f.w[0], f.w[1], f.w[2], f.w[3]};
#pragma unroll
                for (int j = 0; j < NTL; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ub[c][j], __builtin_bit_cast(bf16x8_t, av), acc[j],
                                                                     0, 0, 0);
                const int n = mt * KC + c + R;
                if (n < NA) raw_load<bf16, CPOL_SC1>(f, r, cofs(n / KC < MT ? n / KC : 0, n % KC));
            }
#pragma unroll
            for (int j = 0; j < NTL; ++j)
                red[(w * NF + mt * NTL + j) * RF_FP + (lane >> 4) * RF_QP + cl] =
                    make_float4(acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
        }
        lds_barrier();
        if (__builtin_expect(spoilt, 0)) {
            const int th = opaque_tid();
#pragma unroll 1
            for (int q = 0; q < PPT; ++q) {
                const Pair r = pair_of(q, th);
                if (!r.ok) continue;
                const float4 v = red_sum(r.i);
                if (v.x == v.x && v.y == v.y && v.z == v.z && v.w == v.w) continue;
                red[r.i] = kept_sum(src, (const bf16*)D.U, mask, r.b, r.u, H);
                for (int k = 1; k < NW; ++k) red[k * NF * RF_FP + r.i] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
    };
    const uint32_t gxbytes = (uint32_t)((size_t)B * G * 4);

    if (worker) {
        // gx_t = s_nr * x~_t W + b, [T][B][H][4], as soon as the layer below
        // has published x_t; flag = steps done
        float4 bias[PPT];
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const int u = pair_of(q, tid).u;
            bias[q] = make_float4(D.bias[u], D.bias[H + u], D.bias[2 * H + u], D.bias[3 * H + u]);
        }
        for (int s = 0; s < T_; ++s) {
            const int t = step_t(s);
            if (!res_wait(a.bar, gdep, a.ntiles, (unsigned)(s + 2), -1, 0, 0, a.err, a.timeout, STATUS_FWD)) break;
            product((const bf16*)D.xin + (size_t)t * hxs, a.d[D.dep].umask + (size_t)t * a.kmax);
            const __amdgpu_buffer_rsrc_t gr = buf_rsrc(D.gxp + (size_t)t * B * G, gxbytes);
            const int th = opaque_tid();
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                const Pair r = pair_of(q, th);
                if (r.ok) {
                    const float4 v = red_sum(r.i);
                    const u32x4_t o = {__float_as_uint(D.s * v.x + bias[q].x), __float_as_uint(D.s * v.y + bias[q].y),
                                       __float_as_uint(D.s * v.z + bias[q].z), __float_as_uint(D.s * v.w + bias[q].w)};
                    __builtin_amdgcn_raw_buffer_store_b128(o, gr, (uint32_t)(r.b * H + r.u) * 16u, 0, CPOL_SC1);
                }
            }
            res_signal(a.bar, g, tile, (unsigned)(s + 1));
        }
        res_exit(a.bar, a.nslots * a.mgroups, total, a.err, a.poison);
        return;
    }

    float creg[PPT], hreg[PPT], gxr[PPT][4];
    int mnx[PPT], mup[PPT];
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        const Pair r = pair_of(q, tid);
        creg[q] = D.c0[(size_t)r.b * H + r.u];
        hreg[q] = bf2f(((const bf16*)D.h0)[(size_t)r.b * H + r.u]);
        mup[q] = 0;
    }
    const bool fed = D.dep >= 0;                           // gx comes from a worker
    // inputs of step s that do not depend on the recurrence (clamped)
    auto prefetch = [&](int s) {
        const int sc = min(s, T_ - 1), t = step_t(sc), tn = step_t(min(sc + 1, T_ - 1)), th = opaque_tid();
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const Pair r = pair_of(q, th);
            if (!fed) {
                const float* gp = D.gx + ((size_t)t * B + r.b) * G + r.u;
#pragma unroll
                for (int k = 0; k < 4; ++k) gxr[q][k] = gp[k * H];
            }
            mnx[q] = D.rmask[(size_t)tn * a.kmax + r.u];
            if (D.umask) mup[q] = D.umask[(size_t)t * a.kmax + r.u];
        }
    };
    // rows of the transposed layer output staged at step s, 4 at a time
    auto store_transposed = [&](int s) {
        const int t = step_t(s), p = tid - P0;
        if (p < 0 || p >= UT * 4 * MT) return;
        const int u = p / (4 * MT), col = 4 * (p % (4 * MT));
        if (u0 + u >= H || m0 + col >= m1) return;
        const int o = (s & 1) * UT * SP + u * SP + col;
        *(uint2*)((bf16*)D.ybufT + ((size_t)t * a.ldy + u0 + u) * a.BP + m0 + col) = *(const uint2*)(sty + o);
    };
    int done = 0;                                          // steps whose outputs are staged
    // prologue: h0 times the first step's RH mask into slot 0
    {
        const int t0 = step_t(0);
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const Pair r = pair_of(q, tid);
            if (r.ok)
                store_coherent((bf16*)D.hx, hxs, (uint32_t)frag_off(r.b, r.u, nch),
                               D.rmask[(size_t)t0 * a.kmax + r.u] ? f2bf(hreg[q]) : (bf16)0);
        }
    }
    prefetch(0);
    res_arrive(a.bar, g, tile);

    for (int s = 0; s < T_; ++s) {
        const int t = step_t(s);
        if (!res_wait(a.bar, g, a.ntiles, (unsigned)(s + 1), gdep, tile, (unsigned)(s + 1), a.err, a.timeout, STATUS_FWD))
            break;
        if (fed) {
            const __amdgpu_buffer_rsrc_t gr = buf_rsrc(D.gxp + (size_t)t * B * G, gxbytes);
            const int th = opaque_tid();
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                const Pair r = pair_of(q, th);
                const float4 v = load_coherent4(gr, (uint32_t)(r.b * H + r.u) * 16u);
                gxr[q][0] = v.x; gxr[q][1] = v.y; gxr[q][2] = v.z; gxr[q][3] = v.w;
            }
        } else {
            // (inputs loaded a step ago: waited for here.  Left to their use behind the
            // product, two directions of 256 units, 32 rows took 56 us for 20 steps and
            // 716 for 320; waited for here 52 and 657)
#pragma unroll
            for (int q = 0; q < PPT; ++q)
                asm volatile("" : "+v"(gxr[q][0]), "+v"(gxr[q][1]), "+v"(gxr[q][2]), "+v"(gxr[q][3]));
        }
        product((const bf16*)D.hx + (size_t)(s & 1) * hxs, D.rmask + (size_t)t * a.kmax);
        bf16* hxn = (bf16*)D.hx + (size_t)((s + 1) & 1) * hxs;
        float og4[PPT][4], cnv[PPT], hnv[PPT];
        const int th = opaque_tid();
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const Pair r = pair_of(q, th);
            if (!r.ok) continue;
            const float4 v = red_sum(r.i);
            og4[q][0] = sigmoid_fast(D.s * v.x + gxr[q][0]);
            og4[q][1] = sigmoid_fast(D.s * v.y + gxr[q][1]);
            og4[q][2] = tanh_fast(D.s * v.z + gxr[q][2]);
            og4[q][3] = sigmoid_fast(D.s * v.w + gxr[q][3]);
            cnv[q] = og4[q][1] * creg[q] + og4[q][0] * og4[q][2];
            hnv[q] = og4[q][3] * tanh_fast(cnv[q]);
            const bool vq = t < len_s[r.b - m0];
            const uint32_t o = (uint32_t)frag_off(r.b, r.u, nch);
            if (s + 1 < T_) store_coherent(hxn, hxs, o, mnx[q] ? f2bf(vq ? hnv[q] : hreg[q]) : (bf16)0);
            if (D.xout) store_coherent((bf16*)D.xout + (size_t)t * hxs, hxs, o, (vq && mup[q]) ? f2bf(hnv[q]) : (bf16)0);
        }
        res_arrive(a.bar, g, tile);
        // outputs only later kernels read, and the next step's inputs.  A
        // transposed copy goes through LDS: staged here, stored as pieces of a
        // unit's rows a step later (past the barriers between)
        const int tn = step_t(min(s + 1, T_ - 1));
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const Pair r = pair_of(q, th);
            if (!r.in) continue;
            const bool vq = t < len_s[r.b - m0];
            const float cn = vq ? cnv[q] : creg[q], hn = vq ? hnv[q] : hreg[q];
            creg[q] = cn;
            hreg[q] = hn;
            const bf16 hv = f2bf(hn), yv = r.ok && vq && mup[q] ? hv : (bf16)0;
            if (D.ybufT) sty[(s & 1) * UT * SP + r.s] = yv;
            if (!r.ok) continue;
            const size_t o = (size_t)t * B + r.b;
            if (s + 1 < T_) ((bf16*)D.hm)[((size_t)tn * B + r.b) * a.ldh + r.u] = mnx[q] ? hv : (bf16)0;
            *(float4*)(D.gates + o * G + 4 * r.u) = make_float4(og4[q][0], og4[q][1], og4[q][2], og4[q][3]);
            D.cres[o * H + r.u] = cn;
            if (D.y) D.y[o * a.ldy + r.u] = vq ? hn : 0.0f;
            if (D.ybuf) ((bf16*)D.ybuf)[o * a.ldyb + r.u] = yv;
        }
        if (D.ybufT && s > 0) store_transposed(s - 1);
        prefetch(s + 1);
        done = s + 1;
    }
    lds_barrier();
    if (D.ybufT && done > 0) store_transposed(done - 1);
    // final state
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        const Pair r = pair_of(q, tid);
        if (!r.ok) continue;
        D.hT[(size_t)r.b * H + r.u] = hreg[q];
        D.cT[(size_t)r.b * H + r.u] = creg[q];
    }
    res_exit(a.bar, a.nslots * a.mgroups, total, a.err, a.poison);
}

// ---------------------------------------------------------------------------
// Backward (Eq. 7-10).  Unit tile = 16*NB units, rows = 16*MT.  The recurrent
// gradient of the tile's units from DA of the step processed before, a
// contraction over 4H: wave w holds the 32-column chunks w + 8c, c < KB, of the
// tile's rows of U (chunks c < KB - KL in registers, the others in LDS), loads
// the same chunks of the published DA block R at a time, and the waves' partial
// products are summed through LDS by the threads of the pointwise.
// Pairs go to the threads unit by unit, as in the forward; pitches of red in
// words: 80 per 4 units x 16 rows, 324 per fragment (spread over the banks).
constexpr int RB_QP = 80, RB_FP = 4 * RB_QP + 4;

template <int KB, int KL, int NB, int MT, int R>
__global__ void __launch_bounds__(512) k_bwd_res(RBwdArgs a) {
    constexpr int UB = 16 * NB, MG = 16 * MT, NF = NB * MT, NP = NF * 256, NTH = 512, NW = 8, KR = KB - KL;
    constexpr int PPT = (NP + NTH - 1) / NTH, P0 = NP <= NTH ? (NTH - NP) / 64 * 64 : 0;
    constexpr int FW = RB_FP;
    extern __shared__ __align__(16) char smem[];
    float* red = (float*)smem;                             // [8 waves][NF][FW]
    __shared__ int len_s[MG];                              // lengths of the rows
    uint4* ul = (uint4*)(smem + (size_t)NW * NF * FW * 4); // [8 waves][KL][NB][64]
    const int H = a.H, G = 4 * H, B = a.B, T_ = a.T;
    const int total = a.nslots * a.mgroups * a.ntiles;
    int g, tile;
    if (!res_place(a.nslots * a.mgroups, a.ntiles, a.gpx, g, tile)) return;
    const int sl = g / a.mgroups, mgl = g % a.mgroups;
    const RBwdSlot& D = a.d[sl];
    const int u0 = tile * UB, m0 = (a.mg0 + mgl) * a.rg, m1 = min(m0 + a.rg, B);   // rows m0 .. m1-1
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g8 = 8 * (lane >> 4), cl = lane & 15;
    const bool worker = D.role == 1;
    const int gdep = D.dep >= 0 ? D.dep * a.mgroups + mgl : -1;
    const int nch = (G + 31) / 32;
    const size_t das = (size_t)nch * a.mtiles * 512;       // elements of one DA block

    if (tid < MG) len_s[tid] = a.lengths ? a.lengths[min(m0 + tid, B - 1)] : T_;

    // rows of U (a worker: of W of the layer above) for the tile's units; zero
    // past 4H (a read past the row's end would hit the next row) and past H
    u32x4_t ub[KR][NB];
    {
        const __amdgpu_buffer_rsrc_t ur = buf_rsrc(D.U, (uint32_t)((size_t)H * G * 2));
#pragma unroll
        for (int c = 0; c < KB; ++c)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int n = 32 * (w + NW * c) + g8, u = u0 + 16 * j + cl;
                u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(
                    ur, (u < H && n < G) ? (uint32_t)((size_t)u * G + n) * 2u : OOB_OFF, 0, 0);
                uint32_t m[4];
                pad_mask<bf16>(n, G, m);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] &= m[e];
                if (c < KR) ub[c < KR ? c : 0][j] = v;
                else ul[((w * KL + (c - KR)) * NB + j) * 64 + lane] = make_uint4(v[0], v[1], v[2], v[3]);
            }
    }
    lds_barrier();                                         // (the lengths)
    // pair q of this thread (derived anew per step, as in the forward)
    struct Pair { int b, u, i; bool ok; };                 // i: its word in red
    auto pair_of = [&](int q, int th) {
        Pair r;
        const int p = th - P0 + NTH * q;
        const bool in = p >= 0 && p < NP;
        const int u = in ? p % UB : 0, row = in ? p / UB : 0;
        r.b = m0 + row;
        r.u = u0 + u;
        r.i = ((row >> 4) * NB + (u >> 4)) * FW + ((u >> 2) & 3) * RB_QP + (row & 15) * 4 + (u & 3);
        r.ok = in && r.b < m1 && r.u < H;
        if (!r.ok) { r.b = m0; r.u = u0; }
        return r;
    };
    auto opaque_tid = [&]() { int v = tid; asm volatile("" : "+v"(v)); return v; };
    float dcs[PPT], dhc[PPT];
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        const Pair r = pair_of(q, tid);
        dhc[q] = D.dhT ? D.dhT[(size_t)r.b * H + r.u] : 0.f;
        dcs[q] = D.dcT ? D.dcT[(size_t)r.b * H + r.u] : 0.f;
    }
    auto step_t = [&](int s) { return D.dir == 0 ? T_ - 1 - s : s; };
    // byte offset of this lane's fragment of wave w's first chunk, for its row
    auto row_ofs = [&](int row) {
        return row < m1 ? (uint32_t)(frag_lane_off(w, row >> 4, (lane & 48) + (row & 15), nch) * 2) : OOB_OFF;
    };
    uint32_t lofs[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
        lofs[mt] = row_ofs(m0 + 16 * mt + cl);
    constexpr uint32_t cstep = NW * 1024;
    // offset of chunk c (past the last one: past the block, zeros)
    auto cofs = [&](int mt, int c) { return w + NW * c < nch ? lofs[mt] + (uint32_t)c * cstep : OOB_OFF; };
    auto product = [&](const bf16* src) {
        // (columns past 4H of the last chunk meet zero weights and were cleared
        // before the pass; chunks past the last read past the block: zeros)
        const __amdgpu_buffer_rsrc_t r = buf_rsrc(src, (uint32_t)(das * 2));
        Raw8<bf16> fa[R][MT];
        f32x4_t acc[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[f] = f32x4_t{0, 0, 0, 0};
#pragma unroll
        for (int c = 0; c < R && c < KB; ++c)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) raw_load<bf16, CPOL_SC1>(fa[c][mt], r, cofs(mt, c));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < KB; ++c) {
            u32x4_t uv[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if (c < KR) uv[j] = ub[c < KR ? c : 0][j];
                else {
                    const uint4 x = ul[((w * KL + (c - KR)) * NB + j) * 64 + lane];
                    uv[j] = u32x4_t{x.x, x.y, x.z, x.w};
                }
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                Raw8<bf16>& f = fa[c % R][mt];
                const u32x4_t av = {f.w[0], f.w[1], f.w[2], f.w[3]};
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    acc[mt * NB + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8_t, uv[j]), __builtin_bit_cast(bf16x8_t, av), acc[mt * NB + j], 0, 0, 0);
                if (c + R < KB) raw_load<bf16, CPOL_SC1>(f, r, cofs(mt, c + R));
            }
        }
        // lane: units 4*(lane>>4) .. +3 of row lane&15
#pragma unroll
        for (int f = 0; f < NF; ++f)
            *(float4*)(red + (size_t)(w * NF + f) * FW + (lane >> 4) * RB_QP + cl * 4) =
                make_float4(acc[f][0], acc[f][1], acc[f][2], acc[f][3]);
        lds_barrier();
    };
    auto red_sum = [&](int o) {
        float v = 0.f;
#pragma unroll
        for (int i = 0; i < NW; ++i) v += red[i * NF * FW + o];
        return v;
    };

    if (worker) {
        // the input gradient of the layer above restricted to this tile's
        // inputs, as soon as that layer has published DA_t; flag = steps done
        for (int s = 0; s < T_; ++s) {
            const int t = step_t(s);
            int mk[PPT];
#pragma unroll
            for (int q = 0; q < PPT; ++q) mk[q] = D.mask[(size_t)t * a.kmax + pair_of(q, tid).u];
            if (!res_wait(a.bar, gdep, a.ntiles, (unsigned)(s + 1), -1, 0, 0, a.err, a.timeout, STATUS_BWD)) break;
            product((const bf16*)D.da + (size_t)t * das);
            const int th = opaque_tid();
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                const Pair r = pair_of(q, th);
                if (r.ok) xstore(D.dxw + ((size_t)t * B + r.b) * H + r.u, mk[q] ? D.s * red_sum(r.i) : 0.0f);
            }
            res_signal(a.bar, g, tile, (unsigned)(s + 1));
        }
        res_exit(a.bar, a.nslots * a.mgroups, total, a.err, a.poison);
        return;
    }

    const bool fed = D.dep >= 0;
    // inputs of iteration s that do not depend on the recurrence (clamped)
    float4 gt[PPT];
    float ctv[PPT], cpv[PPT], dyv[PPT];
    int mkr[PPT];
    auto prefetch = [&](int s) {
        const int t = step_t(min(s, T_ - 1)), tp = D.dir == 0 ? t - 1 : t + 1, tn = step_t(max(s - 1, 0));
        const int th = opaque_tid();
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const Pair r = pair_of(q, th);
            gt[q] = *(const float4*)(D.gates + ((size_t)t * B + r.b) * G + 4 * r.u);
            ctv[q] = D.cres[((size_t)t * B + r.b) * H + r.u];
            cpv[q] = *(s >= T_ - 1 ? D.c0 + (size_t)r.b * H + r.u : D.cres + ((size_t)tp * B + r.b) * H + r.u);
            if (!fed) dyv[q] = D.dy[((size_t)t * B + r.b) * D.lddy + r.u];
            mkr[q] = D.mask[(size_t)tn * a.kmax + r.u];
        }
    };
    prefetch(0);
    for (int s = 0; s <= T_; ++s) {
        const bool final_pass = s == T_;
        const int t = final_pass ? -1 : step_t(s);
        const int tn = D.dir == 0 ? T_ - s : s - 1;         // step processed just before
        // DA of the step before from every tile of the group, and the worker's
        // dx of this step (past the last one: its last flag, already seen)
        if ((s > 0 || fed) && !res_wait(a.bar, g, a.ntiles, (unsigned)s, gdep, tile, (unsigned)min(s + 1, T_), a.err,
                                        a.timeout, STATUS_BWD))
            break;
        const int th = opaque_tid();
        if (fed && !final_pass) {
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                const Pair r = pair_of(q, th);
                dyv[q] = xload1(D.dxw + ((size_t)t * B + r.b) * H + r.u);
            }
        }
        if (s > 0) product((const bf16*)D.da + (size_t)tn * das);
        const __amdgpu_buffer_rsrc_t dw = buf_rsrc((const bf16*)D.da + (size_t)max(t, 0) * das, (uint32_t)(das * 2));
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const Pair r = pair_of(q, th);
            if (!r.ok) continue;
            float dh = dhc[q];
            // units dropped at step tn get no recurrent gradient (Eq. 10)
            if (s > 0 && mkr[q]) dh += D.s * red_sum(r.i);
            if (final_pass) {
                D.dh0[(size_t)r.b * H + r.u] = dh;
                D.dc0[(size_t)r.b * H + r.u] = dcs[q];
                continue;
            }
            float da4[4] = {0.f, 0.f, 0.f, 0.f};
            if (t < len_s[r.b - m0]) {
                dh += dyv[q];
                const float ig = gt[q].x, fg = gt[q].y, gg = gt[q].z, og = gt[q].w;
                const float tc = tanh_fast(ctv[q]);
                const float dout = dh * tc;                            // Eq. 7
                const float dc = dh * og * (1.0f - tc * tc) + dcs[q];  // Eq. 7
                da4[0] = dc * gg * ig * (1.0f - ig);                   // Eq. 9, sigmoid'
                da4[1] = dc * cpv[q] * fg * (1.0f - fg);               // Eq. 8, sigmoid'
                da4[2] = dc * ig * (1.0f - gg * gg);                   // Eq. 9, tanh'
                da4[3] = dout * og * (1.0f - og);                      // Eq. 7, sigmoid'
                dcs[q] = dc * fg;                                      // Eq. 8
                dhc[q] = 0.0f;
            } else {
                dhc[q] = dh;                                           // frozen row: pass through
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                __builtin_amdgcn_raw_buffer_store_b16(f2bf(da4[k]), dw, (uint32_t)frag_off(r.b, k * H + r.u, nch) * 2u, 0,
                                                      CPOL_SC1);
        }
        if (final_pass) break;
        res_arrive(a.bar, g, tile);                         // DA_t is published
        prefetch(s + 1);
    }
    res_exit(a.bar, a.nslots * a.mgroups, total, a.err, a.poison);
}

// ---------------------------------------------------------------------------
// Host side.

static int cu_count() {
    static std::mutex mu;
    static int n[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    std::lock_guard<std::mutex> lock(mu);
    if (!n[dev] && hipDeviceGetAttribute(&n[dev], hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) n[dev] = 0;
    return n[dev];
}

// A tiling of a launch: the unit tile and row tile classes, the rows of a group
// (a multiple of 4: a transposed copy is stored 4 rows at a time), and the
// groups that one launch takes (more rows run as further launches: rows are
// independent).
struct Tiling { int ni, mt, ntiles, rg, mg, gpl, gpx, launches; double cost; };

// Estimated ns of a time step, fitted to measured steps of single layers at hidden
// sizes 100 to 2048 and 12 to 256 rows (within 15%): a base (publish, barrier,
// pointwise), 2 per member of the barrier, the exchanged rows into a compute unit
// at 110 bytes per ns, 15 per fragment and chunk for the products (two waves per
// SIMD), `red` per fragment for the sum through LDS, 300 where every wave has
// pairs, and 450 for every further round of loads and row tile (`rounds`).
template <typename Have>
static Tiling best_tiling(int B, int H, int nslots, int ncu, int kchunks, double bytes_per_row, double base, double red,
                          const int* nis, const int* upt, int nn, Have rounds) {
    Tiling best{-1, 0, 0, 0, 0, 0, 0, 0, 0.0};
    for (int i = 0; i < nn; ++i)
        for (int mt = 1; mt <= 2; ++mt) {
            const double nr = rounds(nis[i], mt);                      // (< 0: no such build)
            if (nr < 0.0) continue;
            Tiling t;
            t.ni = nis[i]; t.mt = mt;
            t.ntiles = (H + upt[i] - 1) / upt[i];
            t.mg = (B + 16 * mt - 1) / (16 * mt);
            t.rg = ((B + t.mg - 1) / t.mg + 3) / 4 * 4;
            t.gpl = std::min(std::min(t.mg, ncu / (nslots * t.ntiles)), RB_GROUPS / nslots);
            if (t.gpl < 1 || 1 + (t.ntiles - 1) / RB_LINES >= RB_PITCH) continue;
            t.launches = (t.mg + t.gpl - 1) / t.gpl;
            t.gpl = (t.mg + t.launches - 1) / t.launches;
            const int px = (nslots * t.gpl + 7) / 8;                   // groups per XCD, if each stays on one
            t.gpx = px * t.ntiles <= ncu / 8 ? px : 0;
            const double nf = nis[i] * mt;
            t.cost = t.launches * (base + 2.0 * t.ntiles + std::min(B, t.rg) * bytes_per_row / 110.0 + 15.0 * kchunks * nf +
                                   red * nf + (upt[i] * t.rg > 448 ? 300.0 : 0.0) + 450.0 * mt * (nr - 1.0));
            if (best.ni < 0 || t.cost < best.cost) best = t;
        }
    return best;
}

hipError_t resident_limit(const void* fn, int threads, size_t lds, int nwg);

template <typename Args>
static hipError_t launch_groups(void (*fn)(Args), Args& a, const Tiling& t, size_t lds, hipStream_t st, int timer_on,
                                hipEvent_t e0, hipEvent_t e1) {
    auto grid = [&](int groups) {
        return t.gpx ? 8 * ((groups + 7) / 8) * t.ntiles : 8 * ((groups * t.ntiles + 7) / 8);
    };
    a.ntiles = t.ntiles;
    a.rg = t.rg;
    a.gpx = t.gpx;
    hipError_t e = resident_limit((const void*)fn, 512, lds, grid(a.nslots * t.gpl));
    if (e != hipSuccess) return e;
    if (timer_on) (void)hipEventRecord(e0, st);
    for (int g0 = 0; g0 < t.mg; g0 += t.gpl) {
        a.mg0 = g0;
        a.mgroups = std::min(t.gpl, t.mg - g0);
        a.timeout = launch_timeout();
        hipLaunchKernelGGL(fn, dim3(grid(a.nslots * a.mgroups)), dim3(512), lds, st, a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (timer_on) (void)hipEventRecord(e1, st);
    return hipSuccess;
}

// Forward builds: (KC, NTL, MT) with KC*NTL <= 32 fragments (128 registers), without
// those that best_tiling prefers to no other on 256 compute units (narrow tiles of a wide
// layer: their barriers have the most members)
template <int KC, int N, int MT>
constexpr bool rf_built = KC * N <= 32 && !(N == 2 && MT == 2 && KC > 2) &&
                          !(N == 3 && (KC == 7 || (MT == 2 && (KC == 5 || KC == 8))));
template <int KC, int N, int MT>
static void (*fwd_res_one(size_t* lds))(RFwdArgs) {
    if constexpr (rf_built<KC, N, MT>) {
        *lds = rf_lds_bytes<N, MT>();
        return k_fwd_res<KC, N, MT>;
    }
    return nullptr;
}
template <int KC>
static void (*fwd_res_fn(int ntl, int mt, size_t* lds))(RFwdArgs) {
#define LSD_F(N) \
    if (ntl == N) return mt == 1 ? fwd_res_one<KC, N, 1>(lds) : fwd_res_one<KC, N, 2>(lds);
    LSD_F(2) LSD_F(3) LSD_F(4) LSD_F(5) LSD_F(6) LSD_F(8)
#undef LSD_F
    return nullptr;
}
static void (*fwd_res_pick(int kc, int ntl, int mt, size_t* lds))(RFwdArgs) {
    switch (kc) {
        case 1: return fwd_res_fn<1>(ntl, mt, lds);
        case 2: return fwd_res_fn<2>(ntl, mt, lds);
        case 3: return fwd_res_fn<3>(ntl, mt, lds);
        case 4: return fwd_res_fn<4>(ntl, mt, lds);
        case 5: return fwd_res_fn<5>(ntl, mt, lds);
        case 6: return fwd_res_fn<6>(ntl, mt, lds);
        case 7: return fwd_res_fn<7>(ntl, mt, lds);
        case 8: return fwd_res_fn<8>(ntl, mt, lds);
    }
    return nullptr;
}
static Tiling fwd_res_tiling(int B, int H, int nslots) {
    const int kc = ((H + 31) / 32 + 7) / 8;
    const int nis[] = {2, 3, 4, 5, 6, 8}, upt[] = {8, 12, 16, 20, 24, 32};
    return best_tiling(B, H, nslots, cu_count(), kc, 2.0 * H, 1870.0, 75.0, nis, upt, 6, [kc](int ni, int mt) {
        size_t l;
        return fwd_res_pick(kc, ni, mt, &l) ? 1.0 : -1.0;
    });
}
// estimated ns of one time step of every slot (all launches), or < 0: does not fit
double fwd_res_cost(int B, int H, int nslots) {
    const Tiling t = fwd_res_tiling(B, H, nslots);
    return t.ni < 0 ? -1.0 : t.cost;
}
hipError_t launch_fwd_res(RFwdArgs& a, hipStream_t st, int timer_on, hipEvent_t e0, hipEvent_t e1) {
    const int kc = ((a.H + 31) / 32 + 7) / 8;
    const Tiling t = fwd_res_tiling(a.B, a.H, a.nslots);
    if (t.ni < 0) return hipErrorInvalidValue;
    size_t lds = 0;
    void (*fn)(RFwdArgs) = fwd_res_pick(kc, t.ni, t.mt, &lds);
    return launch_groups(fn, a, t, lds, st, timer_on, e0, e1);
}

// Backward builds: KB chunks per wave (KL of them in LDS for 1 / 2 unit tiles), and
// the chunks of loads in flight for (unit tiles, row tiles) = (1, 1), (1, 2), (2, 1),
// (2, 2) (0: no such build): as many as the registers hold, for an exchanged line from
// another XCD is a microsecond away.  Without those that best_tiling prefers to no other
// on 256 compute units (two unit tiles of a narrow layer, two row tiles at 20 chunks)
template <int KB, int KL1, int KL2, int R11, int R12, int R21, int R22>
static void (*bwd_res_fn(int nb, int mt, int* kl, int* r))(RBwdArgs) {
    *kl = nb == 1 ? KL1 : KL2;
    *r = nb == 1 ? (mt == 1 ? R11 : R12) : (mt == 1 ? R21 : R22);
    if (nb == 1 && mt == 1) return k_bwd_res<KB, KL1, 1, 1, R11>;
    if constexpr (R12 > 0)
        if (nb == 1) return k_bwd_res<KB, KL1, 1, 2, R12>;
    if constexpr (R21 > 0)
        if (nb == 2) return mt == 1 ? k_bwd_res<KB, KL2, 2, 1, R21> : k_bwd_res<KB, KL2, 2, 2, R22>;
    return nullptr;
}
static void (*bwd_res_pick(int kb, int nb, int mt, int* kl, int* r))(RBwdArgs) {
    if (kb <= 2) return bwd_res_fn<2, 0, 0, 2, 2, 0, 0>(nb, mt, kl, r);
    if (kb <= 4) return bwd_res_fn<4, 0, 0, 4, 4, 4, 4>(nb, mt, kl, r);
    if (kb <= 8) return bwd_res_fn<8, 0, 0, 8, 8, 8, 8>(nb, mt, kl, r);
    if (kb <= 11) return bwd_res_fn<11, 0, 0, 11, 11, 11, 8>(nb, mt, kl, r);
    if (kb <= 16) return bwd_res_fn<16, 0, 0, 16, 12, 16, 5>(nb, mt, kl, r);
    if (kb <= 20) return bwd_res_fn<20, 0, 6, 20, 0, 16, 6>(nb, mt, kl, r);
    if (kb <= 24) return bwd_res_fn<24, 0, 6, 24, 8, 8, 4>(nb, mt, kl, r);
    if (kb <= 32) return bwd_res_fn<32, 0, 0, 20, 6, 0, 0>(nb, mt, kl, r);
    return nullptr;
}
static Tiling bwd_res_tiling(int B, int H, int nslots) {
    const int kb = ((4 * H + 31) / 32 + 7) / 8;
    const int nis[] = {1, 2}, upt[] = {16, 32};
    return best_tiling(B, H, nslots, cu_count(), kb, 8.0 * H, 2200.0, 150.0, nis, upt, 2, [kb](int ni, int mt) {
        int kl, r;
        return bwd_res_pick(kb, ni, mt, &kl, &r) ? std::max(1.0, (double)kb / r) : -1.0;
    });
}
double bwd_res_cost(int B, int H, int nslots) {
    const Tiling t = bwd_res_tiling(B, H, nslots);
    return t.ni < 0 ? -1.0 : t.cost;
}
hipError_t launch_bwd_res(RBwdArgs& a, hipStream_t st, int timer_on, hipEvent_t e0, hipEvent_t e1) {
    const int kb = ((4 * a.H + 31) / 32 + 7) / 8;
    const Tiling t = bwd_res_tiling(a.B, a.H, a.nslots);
    if (t.ni < 0) return hipErrorInvalidValue;
    int kl = 0, r = 0;
    void (*fn)(RBwdArgs) = bwd_res_pick(kb, t.ni, t.mt, &kl, &r);
    const size_t lds = (size_t)8 * t.ni * t.mt * RB_FP * 4 +
                       (size_t)8 * kl * t.ni * 1024;
    return launch_groups(fn, a, t, lds, st, timer_on, e0, e1);
}

}  // namespace lsd
