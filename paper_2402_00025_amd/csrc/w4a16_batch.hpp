// Kernel for 17 to 64 activation rows (a decode batch) on gfx950, wave64; with groups of 32 and 64 also for fewer rows.
//
// The streaming kernel's row tiles (four waves on 256 columns, one wave per SIMD) split k in many parts to fill the
// chip, and the adds of 64 rows x 8 parts alone cost 6 us at the memory side; groups of 32 and 64 had no such kernel and
// streamed the weights once per 16 rows.  Here eight waves of a workgroup own one or two adjacent 64-column strips for
// all the rows and divide the workgroup's k range among them, so that most of the sum over k meets in LDS and k is
// split in a quarter as many parts.  Two waves per SIMD: while one waits, the other computes.
//
// Weights and parameters come straight into registers, 64 to 128 k ahead.  The activations come into LDS 64 k at a time,
// two stages, in the order of k (see nat_unpack: nothing is reordered).  One strip: a wave stages for itself and meets no
// other until the end.  Two strips: the two waves of a k part stage half each for both and meet at a barrier per stage
// (half the transfers; m = 64, n = k = 16384: 46.0 -> 39.7 us; four strips: 47).
//
// What bounds it: vector instructions.  A wave's chunk of 128 k and 64 rows is 64 MFMA and 260 others (16 words unpacked
// at 11 each, 64 scale products), 1.7 us for a unit's eight waves with nothing to load; the transfers into LDS cost
// 0.4 (two strips) to 0.7 us more (each occupies the unit's memory pipe for 20 cycles).  Finer interleaving of unpacking and
// products changed nothing (17.1 -> 17.7), loads of activations straight into MFMA layout cost half as much again
// (16 rows x 64 bytes each: 24.0 us), sixteen waves do not fit the registers at 32 rows (spills: 22 us).
// us per call, cold weights, before -> now (m; n x k): 64; 8192 x 8192: 22.0 -> 15.1, 64; 4096 x 4096: 14.0 -> 7.5,
// 32; 4096 x 4096: 9.1 -> 5.7, 64; 28672 x 8192: 55 -> 37, 33; 1024 x 1024: 6.7 -> 4.9; groups of 64, 29; 8192 x 8192: 21.9 -> 12.6.
// Sums of the parts through fp32 scratch and a ticket instead of the packed-fp16 adds: 17.1 instead of 15.1 us, 10.0
// instead of 7.5 (m = 64, n = k = 8192 and 4096).  One to four last rows of a call with fine groups, which the launch per 16 rows adds
// in fixed point, are added so here too: 5.7 -> 6.8 us (m = 17, n = k = 4096, groups of 64).
#pragma once
#include "w4a16_rows.hpp"

namespace w4a16 {

struct BatchArgs {
    const _Float16* A;
    const uint32_t* qweight;
    const _Float16* scales;
    const uint32_t* qzeros;
    _Float16* C;
    int m, n, k;
    int tiles;                    // of 64 strips columns
    int split_k;
    int strips;                   // 64-column strips per workgroup: 1 or 2
    int chunks_base, chunks_rem;  // k parts (slice x k part of a workgroup): chunks of 128 k each, the first chunks_rem parts one more
    int param_shift;              // log2(compute groups per quantisation group)
    // split_k > 1, the phase protocol's (see gemm_kernel)
    uint32_t* flags;
    uint32_t* counts;
    uint32_t* errors;
    uint32_t* err_host;
    uint64_t* fixed;              // not null: the rows from the last multiple of 16 on are added in fixed point, here [m % 16, n]
    int spin_limit, probe_delay;
};
// What a wave does not need before its first loads.
struct BatchRest {
    uint32_t* flags;
    uint32_t* counts;
    uint32_t* errors;
    uint32_t* err_host;
    uint64_t* fixed;
    int spin_limit, probe_delay;
};

// Launches the kernel of this field width and compute group size (32 ipg).
hipError_t launch_batch(const BatchArgs& a, int bits, int ipg, hipStream_t stream);

constexpr int kBatchWaves = 8;
// the sums of a wave's tile; its share of the stages is as large
template <int MT>
constexpr int kBatchLdsBytes = kBatchWaves * MT * 16 * 64 * 4;

constexpr int kBatchHalfK = 64;  // activations are staged 64 k at a time
template <int MT>
constexpr int kBatchStageBytes = 16 * MT * kBatchHalfK * 2;  // one stage of one wave
template <int BITS>
constexpr int kBatchWordLoads = (BITS == 8 || BITS == 3) ? 2 : 1;

// A wave's view of the matrix: what stays fixed while it walks its range.
struct BatchLane {
    uint32_t a_voff;  // this lane's 16 bytes in eight rows of a stage
    uint32_t a_voff1; // the same for every second one
    uint32_t a_piece; // bytes of A from one of its pieces to the next
    uint32_t lds;     // its first piece in the k part's two stages
    int a_read;       // this lane's operand of step 0 of row block 0 in the first stage
    uint32_t steps;   // MFMA steps (32 k) of the whole matrix
    uint32_t groups;  // compute groups of the whole matrix
    int a_slot0, a_slot1;  // its place in a row of a stage, steps 0 and 1
    int kc;           // IPG < 4: the 8 k of a half this lane stages
};

template <int BITS, int IPG>
struct BatchRegs {
    StepRegs<4, BITS> w[2][2];            // [half of a chunk][step]
    ParamRegs<4, BITS> par[4 / IPG];      // of a chunk
};

template <int BITS, int IPG>
__device__ __forceinline__ void batch_params(ParamRegs<4, BITS>& par, const LaneMap& lm, const Tensors& t, const BatchLane& bl, int gi)
{
    LaneMap at = lm;
    if constexpr (IPG < 4) {
        if (gi >= (int)bl.groups) {
            gi = (int)bl.groups - 1;
            at.off_s = 0x80000000u;
        }
    }
    issue_params<4, BITS>(par, at, t, gi);
}

template <int BITS, int IPG>
__device__ __forceinline__ void batch_weights(StepRegs<4, BITS>& w, const LaneMap& lm, const Tensors& t, const BatchLane& bl, int half, int it)
{
    uint32_t step = (uint32_t)half * 2u + it;
    if constexpr (IPG < 4) step = step < bl.steps ? step : bl.steps - 1;  // (its activations are zeros)
    issue_step_weights<4, BITS>(w, lm, t, step);
}

// This wave's share of a stage, in pieces of eight rows: all of them, or every second one.
template <int IPG, int STRIPS>
__device__ __forceinline__ void batch_stage(const Tensors& t, const BatchLane& bl, int half, uint32_t lds, int i)
{
    const bool odd = STRIPS == 1 && (i & 1);
    uint32_t voff = odd ? bl.a_voff1 : bl.a_voff;
    if constexpr (IPG < 4) voff = (uint32_t)half * 64u + 8u * (uint32_t)(odd ? bl.kc ^ 4 : bl.kc) < 32u * bl.steps ? voff : 0x80000000u;
    load_to_lds(t.A, voff + (uint32_t)i * bl.a_piece, IPG < 4 && (uint32_t)half * 2u >= bl.steps ? 0u : (uint32_t)half * 128u,
                lds + i * (STRIPS * 1024));
}

template <int BITS>
__device__ __forceinline__ void touch(StepRegs<4, BITS>& w)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(w.w.v[j]));
    if constexpr (kBatchWordLoads<BITS> == 2) {
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(w.w1.v[j]));
    }
}
template <int BITS>
__device__ __forceinline__ void touch(ParamRegs<4, BITS>& p)
{
    asm volatile("" : "+v"(p.zword), "+v"(p.s.r[0]), "+v"(p.s.r[1]));
    if constexpr (BITS == 3) asm volatile("" : "+v"(p.zword1));
}

__device__ __forceinline__ char* lds_here()
{
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    return lds_raw;
}
// The place of step `it`'s operand: k slot 4 it + lane / 16 of the lane's row.
template <int MT>
__device__ __forceinline__ const char* stage_address(const char* stage, const BatchLane& bl, int it) { return stage + (it ? bl.a_slot1 : bl.a_slot0); }

// One half (64 k) H of a chunk.  NEXT_A: there is another half behind it; NEXT_W: another two; EXPECT: weights were asked
// for behind this half's activations.  Loads complete in the order they were asked for: a half asks for the next one's
// activations first, then for the weights of the one behind that, which its first wait leaves on their way.  The wait is
// written out, and everything that it covers is touched behind it, because the compiler does not count the transfers
// into LDS and would wait for the weights too at their first use.
template <int MT, int BITS, int IPG, int STRIPS, int H, bool NEXT_A, bool NEXT_W, bool EXPECT>
__device__ __forceinline__ void batch_half(BatchRegs<BITS, IPG>& r, const LaneMap& lm, const Tensors& t, const BatchLane& bl, uint32_t magic, int chunk,
                                           NatZero<BITS> (&zc)[4], ScaleBits<4>& sc, float4_t (&tile)[MT][4], float4_t (&acc)[MT][4])
{
    constexpr uint32_t kMask = (1u << BITS) - 1u;
    constexpr int kLater = EXPECT ? 2 * kBatchWordLoads<BITS> : 0;
    const int half = 2 * chunk + H;
    uint32_t lds_next = bl.lds + (1 - H) * kBatchStageBytes<MT>;
    asm volatile("" : "+s"(lds_next));  // (worked out here: merged from several paths it would lie in a vector register)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLater) : "memory");
    if constexpr (STRIPS > 1) __builtin_amdgcn_s_barrier();
    touch<BITS>(r.w[H][0]);
    touch<BITS>(r.w[H][1]);
    if (IPG < 4 || H == 0) {
#pragma unroll
        for (int s = 0; s < 4 / IPG; ++s)
            if (IPG == 4 || s * IPG / 2 == H) touch<BITS>(r.par[s]);
    }
    __builtin_amdgcn_sched_barrier(0);
    auto take = [&](int s) {
        const ParamRegs<4, BITS>& p = r.par[s];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t z;
            if constexpr (BITS == 3) z = (__builtin_amdgcn_alignbit(p.zword1, p.zword, (uint32_t)lm.zshift) >> (3 * j)) & 7u;
            else z = (p.zword >> (lm.zshift + BITS * j)) & kMask;
            zc[j] = nat_zero<BITS>(z);
        }
        sc = p.s;
        asm volatile("" : "+v"(sc.r[0]), "+v"(sc.r[1]));
    };
    const float4_t zero4 = float4_t{0.f, 0.f, 0.f, 0.f};
    const char* stage = lds_here() + bl.a_read + H * kBatchStageBytes<MT>;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int step = 2 * H + it;
        half8_t a[MT];
#pragma unroll
        for (int rt = 0; rt < MT; ++rt) a[rt] = *(const half8_t*)(stage_address<MT>(stage, bl, it) + rt * 2048);
        if (step % IPG == 0) {
            const int s = step / IPG;
            take(s);
            if constexpr (NEXT_W) {
                __builtin_amdgcn_sched_barrier(0);
                batch_params<BITS, IPG>(r.par[s], lm, t, bl, (chunk + 1) * (4 / IPG) + s);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_s_setprio(0);
        half8_t b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t w1 = 0;
            if constexpr (kBatchWordLoads<BITS> == 2) w1 = r.w[H][it].w1.v[j];
            b[j] = nat_unpack<BITS>(r.w[H][it].w.v[j], w1, lm, zc[j], magic);
        }
        auto add = [&](int rt) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float f = scale_of<4>(sc, j);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[rt][j][e] = __builtin_fmaf(f, tile[rt][j][e], acc[rt][j][e]);
            }
        };
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int rt = 0; rt < MT; ++rt) {
            if constexpr (NEXT_A) {
                __builtin_amdgcn_sched_barrier(0);
                if (it == 0) {
#pragma unroll
                    for (int i = 0; i < 2 / STRIPS; ++i) batch_stage<IPG, STRIPS>(t, bl, half + 1, lds_next, rt * (2 / STRIPS) + i);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                tile[rt][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[rt], b[j], step % IPG == 0 ? zero4 : tile[rt][j], 0, 0, 0);
            if (step % IPG == IPG - 1 && rt > 0) add(rt - 1);
            if (IPG < 4) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (NEXT_W) {
            if (it == 1) {
                __builtin_amdgcn_sched_barrier(0);
                batch_weights<BITS, IPG>(r.w[H][0], lm, t, bl, half + 2, 0);
                batch_weights<BITS, IPG>(r.w[H][1], lm, t, bl, half + 2, 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (step % IPG == IPG - 1) add(MT - 1);
        if (IPG < 4) __builtin_amdgcn_sched_barrier(0);
    }
}

template <int MT, int BITS, int IPG, int STRIPS>
__global__ void __launch_bounds__(64 * kBatchWaves, 2) gemm_batch_kernel(const _Float16* A, const uint32_t* qweight, const _Float16* scales, const uint32_t* qzeros, _Float16* C, int packed, int n, int k,
                  int split_rem, const BatchRest rest)
{
    const int tid = threadIdx.x, lane = tid & 63;
    char* const lds_raw = lds_here();
    int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    asm volatile("" : "+s"(wave));  // (what is worked out from it stays in scalar registers)
    const int m = packed & 127, param_shift = (packed >> 7) & 3, chunks_base = (int)((unsigned)packed >> 9);
    const int split_k = split_rem & 0xFFFF, chunks_rem = (int)((unsigned)split_rem >> 16);
    __builtin_assume(m > 0 && n > 0 && k > 0);
    const int slice = blockIdx.x, tile = blockIdx.y;
    const int strip = wave % STRIPS, kpart = wave / STRIPS;
    constexpr int kParts = kBatchWaves / STRIPS;
    const int n0 = (tile * STRIPS + strip) * 64;

    const LaneMap lm = make_lane_map<4, BITS>(lane, n0, 1, n, k);
    constexpr int kFields = BITS == 3 ? 1 : 32 / BITS;
    BatchLane bl;
    bl.steps = (uint32_t)k / 32u;
    bl.groups = bl.steps / IPG;
    // A stage holds 128 bytes of a row, eight slots of 16: k slot c of row r lies at slot c ^ (r / 2 % 8), which
    // keeps the sixteen rows of a read apart.  A piece is rows 8 i + lane / 8.
    const int odd = STRIPS > 1 ? strip & 1 : 0;
    bl.kc = (lane & 7) ^ (lane >> 4) ^ (4 * odd);
    const uint32_t prow = (uint32_t)(8 * odd + (lane >> 3)) * (uint32_t)k;
    bl.a_voff = (prow + 8u * (uint32_t)bl.kc) * 2u;
    bl.a_voff1 = (prow + 8u * (uint32_t)(bl.kc ^ 4)) * 2u;
    bl.a_piece = 16u * STRIPS * (uint32_t)k;
    bl.a_read = kpart * 2 * kBatchStageBytes<MT> + (lane & 15) * 128;
    bl.lds = (uint32_t)(kpart * 2 * kBatchStageBytes<MT> + odd * 1024);
    bl.a_slot0 = ((lane >> 4) ^ ((lane & 15) >> 1)) * 16;
    bl.a_slot1 = bl.a_slot0 ^ 64;
    const uint32_t qgroups = bl.groups >> param_shift;
    Tensors t;
    t.A = make_rsrc(A, (uint32_t)m * (uint32_t)k * 2u);  // rows behind the last one lie behind its end: zeros
    t.qweight = make_rsrc(qweight, (uint32_t)(BITS == 3 ? k / 32 * 3 : k / kFields) * (uint32_t)n * 4u);
    t.scales = make_rsrc(scales, qgroups * (uint32_t)n * 2u);
    t.qzeros = make_rsrc(qzeros, qgroups * (uint32_t)(BITS == 3 ? n / 32 * 3 : n / kFields) * 4u);
    t.n = n;
    t.k = k;
    t.param_shift = param_shift;

    const rsrc_t rs_c = make_rsrc(C, (uint32_t)m * (uint32_t)n * 2u);
    constexpr uint32_t kOutside = 0x80000000u;
    // ---- split k, first part of the phase protocol: this workgroup's call count, and the zeros of slice 0, an eighth by
    // every wave.  They precede a wave's loads, so that its first wait for those covers them.
    const bool split = split_k > 1;
    // the rows that are added in fp16; those behind them are added in fixed point
    constexpr bool kFixedRows = MT > 1 && IPG < 4;
    const int half_rows = kFixedRows && split && rest.fixed ? m & ~15 : m;
    const uint32_t origin = (uint32_t)tile * (4 * STRIPS);
    uint32_t count_word = 0;
    if (split) {
        if (wave == 0) count_word = __hip_atomic_load(rest.counts + origin * (uint32_t)split_k + (uint32_t)slice, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (slice == 0) {
#pragma unroll
            for (int u = tid; u < 16 * MT * 8 * STRIPS; u += 64 * kBatchWaves) {
                const int row = u / (8 * STRIPS), col = tile * (64 * STRIPS) + 8 * (u % (8 * STRIPS));
                const uint32_t off = row < half_rows && col < n ? ((uint32_t)row * (uint32_t)n + (uint32_t)col) * 2u : kOutside;
                __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{0u, 0u, 0u, 0u}, rs_c, off, 0, kRowsDeviceScope);
            }
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }

    const int part = slice * kParts + kpart;
    const int c0 = part * chunks_base + (part < chunks_rem ? part : chunks_rem);
    uint32_t now = 0;
    const int count = chunks_base + (part < chunks_rem ? 1 : 0);
    float4_t acc[MT][4];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
    if (count > 0) {
        const uint32_t magic = unpack_magic<BITS>();
        BatchRegs<BITS, IPG> r;
        NatZero<BITS> zc[4];
        ScaleBits<4> sc;
        float4_t tile_acc[MT][4];
#pragma unroll
        for (int s = 0; s < 4 / IPG; ++s) batch_params<BITS, IPG>(r.par[s], lm, t, bl, c0 * (4 / IPG) + s);
#pragma unroll
        for (int it = 0; it < 2; ++it) batch_weights<BITS, IPG>(r.w[0][it], lm, t, bl, 2 * c0, it);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2 * MT / STRIPS; ++i) batch_stage<IPG, STRIPS>(t, bl, 2 * c0, bl.lds, i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int it = 0; it < 2; ++it) batch_weights<BITS, IPG>(r.w[1][it], lm, t, bl, 2 * c0 + 1, it);
        if (split) {
            // (the first half's own wait, put first)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kBatchWordLoads<BITS>) : "memory");
            if (slice == 0) __builtin_amdgcn_s_barrier();  // the zeros of all waves are in memory
            if (wave == 0) {
                asm volatile("" : "+v"(count_word)::"memory");
                now = __builtin_amdgcn_readfirstlane(count_word) + 1u;
                if (lane == 0) {
                    __hip_atomic_store(rest.counts + origin * (uint32_t)split_k + (uint32_t)slice, now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (slice == 0) __hip_atomic_store(rest.flags + origin, now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        const int last = c0 + count - 1;
        for (int c = c0; c < last; ++c) {
            batch_half<MT, BITS, IPG, STRIPS, 0, true, true, true>(r, lm, t, bl, magic, c, zc, sc, tile_acc, acc);
            batch_half<MT, BITS, IPG, STRIPS, 1, true, true, true>(r, lm, t, bl, magic, c, zc, sc, tile_acc, acc);
        }
        batch_half<MT, BITS, IPG, STRIPS, 0, true, false, true>(r, lm, t, bl, magic, last, zc, sc, tile_acc, acc);
        batch_half<MT, BITS, IPG, STRIPS, 1, false, false, false>(r, lm, t, bl, magic, last, zc, sc, tile_acc, acc);
    }
    if constexpr (STRIPS > 1) {  // (every wave meets the others at as many barriers)
        const int most = chunks_base + (chunks_rem > 0 ? 1 : 0);
        for (int i = count; i < most; ++i) {
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_s_barrier();
        }
    }
    uint32_t sample = 0;
    if (split && wave == 0) sample = __hip_atomic_load(rest.flags + origin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();  // (the stages give way to the sums)

    // ---- the k parts' tiles through LDS: [wave][row][64 columns]
    {
        float* mine = (float*)lds_raw + (wave * MT * 16 + 4 * (lane >> 4)) * 64 + 4 * (lane & 15);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *(float4_t*)(mine + (16 * i + r) * 64) = float4_t{acc[i][0][r], acc[i][1][r], acc[i][2][r], acc[i][3][r]};
    }
    if (split && wave == 0) {
        // wave 0 holds the barrier until this call's zeros of the tile are in memory
        bool seen = __builtin_amdgcn_readfirstlane(sample) == now;
        int polls = 0;
        while (!seen && polls < rest.spin_limit) {
            for (int i = 0; i < rest.probe_delay; ++i) __builtin_amdgcn_s_sleep(1);
            seen = __builtin_amdgcn_readfirstlane(__hip_atomic_load(rest.flags + origin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == now;
            ++polls;
        }
        if (!seen && lane == 0) phase_wait_failed(rest.errors, rest.err_host, rs_c, (uint32_t)tile * (uint32_t)(64 * STRIPS) * 2u);
    }
    __syncthreads();
    // Thread t adds up the column pairs t, t + 512, ... of the tile (strip, row, pair): consecutive lanes on consecutive
    // pairs, so that an instruction touches the fewest cache lines.
    auto sum = [&](int st, int e) {
        const float2* src = (const float2*)lds_raw + st * (MT * 512) + e;
        float2 v = src[0];
#pragma unroll
        for (int q = 1; q < kParts; ++q) {
            const float2 more = src[q * STRIPS * (MT * 512)];
            v.x += more.x;
            v.y += more.y;
        }
        v.x *= kNatScale<BITS>;
        v.y *= kNatScale<BITS>;
        return v;
    };
    auto offset = [&](int st, int e) {
        const int row = e >> 5, col = (tile * STRIPS + st) * 64 + 2 * (e & 31);
        return row < m && col < n ? ((uint32_t)row * (uint32_t)n + (uint32_t)col) * 2u : kOutside;
    };
    // The fixed-point adds first, all strips': their round trip passes beside the others.
    const bool fixed = kFixedRows && half_rows < m;
    const int last = (MT - 1) * 512 + tid;  // this thread's pair of the last row block, which the fixed rows are in
    uint64_t mine[STRIPS][2], old[STRIPS][2];
    if (fixed) {
#pragma unroll
        for (int st = 0; st < STRIPS; ++st) {
            const uint32_t off = offset(st, last);
            if (off != kOutside) {
                const float2 v = sum(st, last);
                uint64_t* const word = rest.fixed + off / 2 - (size_t)half_rows * n;
                mine[st][0] = fixed_contribution(v.x);
                mine[st][1] = fixed_contribution(v.y);
                old[st][0] = __hip_atomic_fetch_add(word, mine[st][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                old[st][1] = __hip_atomic_fetch_add(word + 1, mine[st][1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
#pragma unroll
    for (int u = tid; u < STRIPS * MT * 512; u += 64 * kBatchWaves) {
        const int st = u / (MT * 512), e = u - st * (MT * 512);
        if (kFixedRows && fixed && e >= (MT - 1) * 512) continue;
        const float2 v = sum(st, e);
        const uint32_t off = offset(st, e);
        if (split) {
            const half2_t h = {(_Float16)v.x, (_Float16)v.y};
            __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_v2f16(h, rs_c, off, 0, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b32(pack_half2(v.x, v.y), rs_c, off, 0, kRowsDeviceScope);
        }
    }
    if (fixed) {
#pragma unroll
        for (int st = 0; st < STRIPS; ++st) {
            const uint32_t off = offset(st, last);
            if (off == kOutside) continue;
            uint64_t* const word = rest.fixed + off / 2 - (size_t)half_rows * n;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float total;
                if (fixed_finish(word + i, old[st][i], mine[st][i], split_k, &total))
                    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, (_Float16)total), rs_c, off + 2u * i, 0, kRowsDeviceScope);
            }
        }
    }
}

}  // namespace w4a16
