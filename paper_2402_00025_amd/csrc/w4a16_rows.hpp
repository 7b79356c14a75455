// Kernel for many activation rows (prompts, large batches) on gfx950, wave64: the fused GEMM as a
// tiled matrix product whose weight operand is unpacked in registers.
//
// The streaming kernel's row tiles (up to 64 rows a launch) spend one unpack per 64 rows and wait for
// every chunk's products before they use them; at 64 rows they reach 410 TFLOP/s and every further 64
// rows stream the weights again.  Here a workgroup owns 128 (or 64) rows x 256 columns at a time.  Each
// of its four waves owns a 64-column strip for all the rows, so that a weight is unpacked once per tile
// and an unpacked operand serves 8 (4) row blocks.  The activations of a chunk (128 k) come straight
// from memory into LDS, one chunk ahead, as do the packed weights of each wave's own strip: neither
// passes through registers, which the sums (128), the unpacked operands (64) and the products in flight
// fill to the last ones that two waves per SIMD leave (none of them lies in memory).  Their requests are spread over the unpacking: one
// 16-byte-per-lane request occupies the unit's memory pipe for 20 cycles, and four waves that issue theirs in
// one burst stand still for it (m = 333, n = 11008, k = 4096 on whole tiles: 76 us with the burst, 59 without).
// The scale of a group is applied in fp32 to its products, as in the other kernels.
//
// What bounds it: the issue of instructions.  A 16x16x32 MFMA takes 16 cycles of the matrix unit and about
// 10 of the issue port, every other vector instruction 4; a chunk has 128 and about 340 of them per wave.
// m = 2048, n = k = 8192: 219-232 us by the run = 1185-1255 TFLOP/s (664 us with row tiles).  In a run of 232 us the
// clock is at 1.79 GHz, where the matrix units' ceiling is 1.88 PFLOP/s, and they are busy 63 % of the time.
//
// Persistent workgroups share the chunks of all tiles evenly, whatever the shape (m = 333, n = 11008, k = 4096, 129
// tiles: 40.5 us on 256 workers; 59 us with a workgroup per tile).  A tile that several workers have parts of is
// added up in fp32, in the order of k, by the worker that has its beginning.  That one waits for the other parts for
// a bounded time; where they are late (a worker that has not started, because other work holds the GPU) it leaves its
// own part in memory too, and whoever brings the last part adds the tile up, in the same order.  No result depends
// on a wait, and the words that the workers meet in are zero again when the kernel ends, however it went.
#pragma once
#include "w4a16_device.hpp"

namespace w4a16 {

struct RowsArgs {
    const _Float16* A;
    const uint32_t* qweight;
    const _Float16* scales;
    const uint32_t* qzeros;
    _Float16* C;
    // [2][workers][16 MB][256]: a worker's sums of a tile that another one began, then of the tile that it began itself
    // and has left to the others
    float* partials;
    // [2][kRowsMaxWorkers], all zero whenever no call is running: 1 while the sums that a worker handed over wait for
    // their reader; 1 while the tile that a worker began is left to the others
    uint32_t* words;
    int m, n, k;
    int tiles_m;
    int chunks;  // of a tile: 128 consecutive k each, the last one possibly shorter
    // worker w takes the chunks from start(w) to start(w + 1) of all the tiles' in a row,
    // start(i) = (i share + min(i, share_rem)) share_unit
    int share, share_rem, share_unit;
    int param_shift;  // log2(compute groups per quantisation group)
    int polls;  // how often a worker looks for the later parts of its tile before it leaves it to them
};

// Launches the kernel of these field width, compute group size (32 ipg) and tile height (16 row_blocks) on `workers` workgroups.
hipError_t launch_rows(const RowsArgs& a, int bits, int ipg, int row_blocks, int workers, hipStream_t stream);
constexpr int kRowsMaxWorkers = 512;
// Are there kernels of 128-row tiles?  (two workgroups a unit only where LDS holds both: 4- and 2-bit fields)
constexpr bool rows_tall_ok(int ipg) { return ipg == 4; }
constexpr bool rows_tall_pairs_ok(int bits) { return bits == 4 || bits == 2; }

constexpr int kRowsStrips = 4;
constexpr int kRowsTileCols = 64 * kRowsStrips;
constexpr int kRowsChunkK = 128;
constexpr int kRowsDeviceScope = 16;  // aux bits of a buffer access that other compute dies' accesses meet: sc1

// ---- Unpack in the order of k, so that the activations need no reordering on their way into LDS.
// 4-bit: a byte permute puts two neighbouring fields into the low bits of two halves, where a field v is the
// fp16 denormal v 2^-24; a packed fma by 2^15 with -z 2^-9 makes (q - z) 2^-9 of it, exactly.  The factor 2^9
// is put back when a sum is rounded (kNatScale).  The other widths' routines yield q - z itself.
template <int BITS>
struct NatZero {
    uint32_t c[BITS == 2 || BITS == 3 ? 3 : 1];
};
template <int BITS>
constexpr float kNatScale = BITS == 4 ? 512.f : 1.f;

template <int BITS>
__device__ __forceinline__ NatZero<BITS> nat_zero(uint32_t z)
{
    NatZero<BITS> r;
    const uint32_t zz = z | (z << 16);
    if constexpr (BITS == 4) {
        const half2_t f = {(_Float16)-32768.f, (_Float16)-32768.f};
        r.c[0] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, zz) * f);
    } else if constexpr (BITS == 8) {
        r.c[0] = 0xE400E400u | zz;
    } else if constexpr (BITS == 2) {
        const ZeroConst2 t = zero_const2(z);
        r.c[0] = t.c0; r.c[1] = t.c4; r.c[2] = t.c8;
    } else {
        const ZeroConst3 t = zero_const3(z);
        r.c[0] = t.c0; r.c[1] = t.c3; r.c[2] = t.c6;
    }
    return r;
}

template <int BITS>
__device__ __forceinline__ half8_t nat_unpack(uint32_t w0, uint32_t w1, const LaneMap& lm, const NatZero<BITS>& z, uint32_t magic)
{
    if constexpr (BITS == 8) {
        return unpack_shift8(w0, w1, ZeroConst8{z.c[0]}, magic);
    } else if constexpr (BITS == 2) {
        return unpack_shift2(w0, lm.half_shift, ZeroConst2{z.c[0], z.c[1], z.c[2]}, magic);
    } else if constexpr (BITS == 3) {
        const half2_t k64 = {(_Float16)0.015625f, (_Float16)0.015625f};
        const uint32_t x = __builtin_amdgcn_alignbit(w1, w0, (uint32_t)lm.half_shift);
        const uint32_t xl = x & 0xFFFu, xh = (x >> 12) & 0xFFFu;
        const uint32_t yl = xl | (xl << 13), yh = xh | (xh << 13);
        const uint32_t t0 = (yl & 0x00070007u) | magic, t1 = (yl & 0x01C001C0u) | magic;
        const uint32_t t2 = (yh & 0x00070007u) | magic, t3 = (yh & 0x01C001C0u) | magic;
        const half2_t c0 = __builtin_bit_cast(half2_t, z.c[0]), c6 = __builtin_bit_cast(half2_t, z.c[2]);
        const half2_t h0 = __builtin_bit_cast(half2_t, t0) + c0;
        const half2_t h1 = __builtin_elementwise_fma(__builtin_bit_cast(half2_t, t1), k64, c6);
        const half2_t h2 = __builtin_bit_cast(half2_t, t2) + c0;
        const half2_t h3 = __builtin_elementwise_fma(__builtin_bit_cast(half2_t, t3), k64, c6);
        const u32x4_t packed = {__builtin_bit_cast(uint32_t, h0), __builtin_bit_cast(uint32_t, h1),
                                __builtin_bit_cast(uint32_t, h2), __builtin_bit_cast(uint32_t, h3)};
        return __builtin_bit_cast(half8_t, packed);
    } else {
        const half2_t f = {(_Float16)32768.f, (_Float16)32768.f};
        const half2_t c = __builtin_bit_cast(half2_t, z.c[0]);
        const uint32_t u = w0 & 0x0F0F0F0Fu, v = (w0 >> 4) & 0x0F0F0F0Fu;
        u32x4_t packed;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t p = __builtin_amdgcn_perm(v, u, 0x0C040C00u + 0x00010001u * i);
            packed[i] = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(__builtin_bit_cast(half2_t, p), f, c));
        }
        return __builtin_bit_cast(half8_t, packed);
    }
}

// 16 bytes per lane from memory straight into LDS: lane l's go to lds + 16 l.  (A transfer into LDS reads m0, and a
// scalar write of m0 needs one wait state before it; the compiler adds none inside inline asm.  m0 is a register that
// the compiler does not allocate: it takes no note of it as a clobber but for a warning, and writes it itself right
// before an instruction that reads it, of which these kernels have none.)
__device__ __forceinline__ void load_to_lds(rsrc_t r, uint32_t voff, uint32_t soff, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(r), "s"(soff), "s"(lds)
                 : "memory");
}

// The lane's number, worked out where it is used: the compiler would hold it through the loop over chunks.
__device__ __forceinline__ int lane_here()
{
    int r;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(r));
    return r;
}

template <int BITS>
constexpr int kRowsWordLoads = (BITS == 8 || BITS == 3) ? 2 : 1;  // 16-byte loads per lane and MFMA step
template <int BITS>
constexpr int kRowsWaveWeightBytes = 4 * kRowsWordLoads<BITS> * 1024;
template <int MB, int BITS>
constexpr int kRowsLdsBytes = 2 * MB * 4096 + kRowsStrips * kRowsWaveWeightBytes<BITS>;

// MB: 16-row blocks per workgroup tile: 8 or 4, or the fewer (down to 3) that as many tiles need when they are evened
// out (m = 333, n = 11008, k = 4096: 46.5 -> 43.5 us with 7; m = 129, n = k = 4096: 18.5 -> 16.6 with 3; nothing gained where
// one workgroup a unit waits for memory: m = 150, n = 28672, k = 4096: 53).  IPG: MFMA steps (32 k) per quantisation group in a chunk (4, 2, 1).
template <int MB, int BITS, int IPG>
__global__ void __launch_bounds__(64 * kRowsStrips, 2) gemm_rows_kernel(const RowsArgs p)
{
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    constexpr int PG = 4 / IPG;  // parameter sets per chunk
    constexpr int kPartialFloats = 16 * MB * kRowsTileCols;
    const int strip = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = p.m, n = p.n, k = p.k;
    __builtin_assume(m > 0 && n > 0 && k > 0);

    // ---- this worker's range of chunks.  Workgroups go to the eight compute dies in turn; a die takes
    // neighbouring ranges, whose operands and sums its L2 then holds (neighbours on different dies: 2.5 % slower on
    // average, up to 26 %).  The later ranges first: a worker waits for ranges behind its own (see below), which
    // workgroups ahead of it in the die's order have.  Only the last worker of a die waits for another die's, and
    // that one's first range is the last to start there: with the GPU to itself all have started by then.
    const int workers = gridDim.x;
    const int die = blockIdx.x & 7, per_die = workers >> 3, dies_more = workers & 7;
    const int w = die * per_die + (die < dies_more ? die : dies_more) + per_die + (die < dies_more ? 1 : 0) - 1 -
                  (int)(blockIdx.x >> 3);
    const int U = p.chunks;
    auto range_start = [&](int i) { return (i * p.share + (i < p.share_rem ? i : p.share_rem)) * p.share_unit; };
    const int u0 = range_start(w), u1 = range_start(w + 1);
    constexpr int kFields = BITS == 3 ? 1 : 32 / BITS;
    const uint32_t cgroups = (uint32_t)k / (32 * IPG), qgroups = cgroups >> p.param_shift;
    Tensors t;
    t.qweight = make_rsrc(p.qweight, (uint32_t)(BITS == 3 ? k / 32 * 3 : k / kFields) * (uint32_t)n * 4u);
    t.scales = make_rsrc(p.scales, qgroups * (uint32_t)n * 2u);
    t.qzeros = make_rsrc(p.qzeros, qgroups * (uint32_t)(BITS == 3 ? n / 32 * 3 : n / kFields) * 4u);
    t.n = n;
    t.k = k;
    t.param_shift = p.param_shift;
    auto place = [&](int which, int* row0, int* n0) {
        const int tile_n = __builtin_amdgcn_readfirstlane(which / p.tiles_m);
        *row0 = (which - tile_n * p.tiles_m) * (16 * MB);
        *n0 = (tile_n * kRowsStrips + strip) * 64;
        return m - *row0 < 16 * MB ? m - *row0 : 16 * MB;
    };

    // ---- tiles with several parts.  The worker that has a tile's beginning, and how many workers have later parts of
    // the tile that worker i began (the ranges are never empty).
    auto first_worker = [&](int which) {
        int i = w;
        while (range_start(i) > which * U) --i;
        return i;
    };
    auto later_parts = [&](int i, int which) {
        int o = i + 1;
        while (o < workers && range_start(o) < (which + 1) * U) ++o;
        return (uint32_t)(o - i - 1);
    };
    uint32_t* const full = p.words;
    uint32_t* const left = p.words + kRowsMaxWorkers;
    auto look = [&](const uint32_t* word) {
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    };
    auto set = [&](uint32_t* word) {
        __hip_atomic_store(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto part_offset = [&](int es, int el) { return (uint32_t)(es * (MB * 4)) * 1024u + (uint32_t)el * 16u; };
    auto put_part = [&](const float4_t (&acc)[MB][4], int slot, int es, int el) {
        const rsrc_t rs = make_rsrc(p.partials + (size_t)slot * kPartialFloats, kPartialFloats * 4);
        const uint32_t off = part_offset(es, el);
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc[i][j]), rs,
                                                       off + (uint32_t)(i * 4 + j) * 1024u, 0, kRowsDeviceScope);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    };
    auto add_part = [&](float4_t (&acc)[MB][4], int slot, int es, int el) {
        const rsrc_t rs = make_rsrc(p.partials + (size_t)slot * kPartialFloats, kPartialFloats * 4);
        const uint32_t off = part_offset(es, el);
#pragma unroll
        for (int i0 = 0; i0 < MB; i0 += 4) {  // 16 loads in flight
            float4_t part[4][4];
#pragma unroll
            for (int i = 0; i < 4 && i0 + i < MB; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    part[i][j] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(
                                                                  rs, off + (uint32_t)((i0 + i) * 4 + j) * 1024u, 0, kRowsDeviceScope));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4 && i0 + i < MB; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i0 + i][j] += part[i][j];
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto taken = [&](int first, uint32_t parts, int es, int el) {
        __builtin_amdgcn_s_barrier();  // every wave has its share
        if (es == 0)
            for (uint32_t i = 1 + el; i <= parts; i += 64) __hip_atomic_store(full + first + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // The first wave's answer, for all four (through its own strip's weights, which no other wave touches and which
    // nothing is on its way to when this is called).  What follows is not moved ahead of it.
    auto tell = [&](bool answer, int es, int el) {
        uint32_t* const word = (uint32_t*)(lds_raw + 2 * MB * 4096);
        if (es == 0 && el == 0) *word = answer ? 1u : 0u;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const bool r = __builtin_amdgcn_readfirstlane(*word) != 0u;
        __builtin_amdgcn_s_barrier();  // (read by all before it is written again)
        return r;
    };
    // The first wave asks this of a tile that worker `first` has left: are all later parts there, and does nobody else
    // finish it?  Whoever looks has set its own word before (the part that it brought, or `left`), so the last one to
    // come finds all of them; the exchange lets one through.
    auto claim = [&](int first, uint32_t parts, int el) {
        for (uint32_t i = 1; i <= parts; ++i)
            if (look(full + first + i) == 0u) return false;
        uint32_t won = 0;
        if (el == 0) {
            uint32_t expected = 1u;
            won = __hip_atomic_compare_exchange_strong(left + first, &expected, 0u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT)
                      ? 1u
                      : 0u;
        }
        return __builtin_amdgcn_readfirstlane(won) != 0u;
    };
    auto store_tile = [&](const float4_t (&acc)[MB][4], int row0, int n0, int rows, int el) {
        constexpr uint32_t kOutside = 0x80000000u;
        const rsrc_t rs_c = make_rsrc(p.C + (size_t)row0 * n, (uint32_t)rows * (uint32_t)n * 2u);
        const int col = n0 + 4 * (el & 15);
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * i + 4 * (el >> 4) + r;
                const uint32_t off = col < n && row < rows ? ((uint32_t)row * (uint32_t)n + (uint32_t)col) * 2u : kOutside;
                const u32x2_t h = {pack_half2(acc[i][0][r] * kNatScale<BITS>, acc[i][1][r] * kNatScale<BITS>),
                                   pack_half2(acc[i][2][r] * kNatScale<BITS>, acc[i][3][r] * kNatScale<BITS>)};
                __builtin_amdgcn_raw_buffer_store_b64(h, rs_c, off, 0, 0);
            }
    };

    for (int at = u0; at < u1;) {
        const int tile_index = __builtin_amdgcn_readfirstlane(at / U), g0 = at - tile_index * U;
        const int g_count = u1 - at < U - g0 ? u1 - at : U - g0;
        at += g_count;
        int row0, n0;
        const int rows = place(tile_index, &row0, &n0);
        const int lane = lane_here();  // (so that nothing that is worked out from it is held in registers from piece to piece)
        const int srow = 4 * strip + (lane >> 4), skc = (lane & 15) ^ srow;
        const uint32_t a_voff = ((uint32_t)srow * (uint32_t)k + 8u * (uint32_t)skc) * 2u;
        const uint32_t lds_w = 2 * MB * 4096 + strip * kRowsWaveWeightBytes<BITS>;
        const rsrc_t rs_a = make_rsrc(p.A + (size_t)row0 * k, (uint32_t)rows * (uint32_t)k * 2u);
        const LaneMap lm = make_lane_map<4, BITS>(lane, n0, 1, n, k);
        // A chunk's activations: MB pieces of 16 rows, a quarter of each per wave.  Rows behind the last one, k behind
        // the end (a short last chunk) and whole chunks behind the last one (`voff` outside) come as zeros: their
        // offsets lie outside the buffer.  The scalar offset stays inside it always: the bound of a buffer access is its
        // size less that offset, which has no meaning below zero.
        constexpr uint32_t kOutside = 0x80000000u;  // stays outside when the pieces' rows are added
        auto stage_a = [&](int g, bool real, uint32_t voff, int i) {
            const uint32_t vo = voff + (uint32_t)i * 32u * (uint32_t)k;
            load_to_lds(rs_a, vo, real ? (uint32_t)g * 256u : 0u, (uint32_t)(g & 1) * (MB * 4096) + strip * 1024 + i * 4096);
        };
        auto stage_w = [&](int g, bool real, int it) {
            const uint32_t dst = lds_w + it * kRowsWordLoads<BITS> * 1024;
            const bool inside = real && (IPG == 4 || ((uint32_t)g * 4 + it) * 32 < (uint32_t)k);
            const uint32_t step = inside ? (uint32_t)g * 4 + it : 0u;
            const uint32_t off0 = inside ? lm.off_w : kOutside, off1 = inside ? lm.off_w1 : kOutside;
            if constexpr (BITS == 8) {
                load_to_lds(t.qweight, off0, step * 32u * (uint32_t)n, dst);
                load_to_lds(t.qweight, off0, (step * 32u + 4u) * (uint32_t)n, dst + 1024);
            } else if constexpr (BITS == 2) {
                load_to_lds(t.qweight, off0, step * 8u * (uint32_t)n, dst);
            } else if constexpr (BITS == 3) {
                load_to_lds(t.qweight, off0, step * 12u * (uint32_t)n, dst);
                load_to_lds(t.qweight, off1, step * 12u * (uint32_t)n, dst + 1024);
            } else {
                load_to_lds(t.qweight, off0, step * 16u * (uint32_t)n, dst);
            }
        };
        auto a_offset = [&](int g, bool real) { return real && (IPG == 4 || g * 128 + 8 * skc < k) ? a_voff : kOutside; };

        float4_t acc[MB][4];
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};

        uint32_t a_off[4];  // of the chunk in use
#pragma unroll
        for (int it = 0; it < 4; ++it)
            a_off[it] = (g0 & 1) * (MB * 4096) + ((lane & 15) * 16 + ((4 * it + (lane >> 4)) ^ (lane & 15))) * 16;
        const uint32_t magic = unpack_magic<BITS>();

        // The zero points' place in the lane's words of 3-bit fields is worked out again for every chunk: three registers
        // less through the loop, where 128 rows leave none (one of them kept in memory: 5 % of the time).
        auto params_map = [&]() {
            LaneMap map = lm;
            if constexpr (BITS == 3) {
                uint32_t twice = lm.off_s;  // 2 columns
                asm volatile("" : "+v"(twice));
                const uint32_t bit = twice + (twice >> 1);
                map.off_z = (bit >> 5) * 4u;
                map.zshift = (int)(bit & 31u);
                map.off_z1 = map.off_z + (map.zshift + 12 > 32 ? 4u : 0u);
            }
            return map;
        };
        ParamRegs<4, BITS> par[PG];
        auto load_params = [&](const LaneMap& map, int g, int s) {
            int gi = g * PG + s;
            // A group behind the end of k (a short last chunk) has products of zero.  The last group's parameters stand
            // for its own, with a scale of zero, since that one may be infinite: with two groups a chunk it is read
            // from outside the buffer, with four it is masked when it is used (four bits, 18432 x 1280, m = 175: 18.4
            // against 18.8 us at two; 16384 x 1024, m = 200: 17.7 against 17.4 at four).
            LaneMap at = map;
            if (gi >= (int)cgroups) {
                gi = (int)cgroups - 1;
                if (PG == 2) at.off_s = kOutside;
            }
            issue_params<4, BITS>(par[s], at, t, gi);
        };
#pragma unroll
        for (int i = 0; i < MB; ++i) stage_a(g0, true, a_offset(g0, true), i);
#pragma unroll
        for (int it = 0; it < 4; ++it) stage_w(g0, true, it);
#pragma unroll
        for (int s = 0; s < PG; ++s) load_params(params_map(), g0, s);
        for (int c = 0; c < g_count; ++c) {
            const int g = g0 + c;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            const bool more = c + 1 < g_count;
            const uint32_t a_next = a_offset(g + 1, more);
            // a chunk's zero points and scales leave the registers that the next chunk's are loaded into
            NatZero<BITS> zc[4];
            ScaleBits<4> sc[PG];
            auto take_params = [&](int s) {
                const LaneMap map = params_map();
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint32_t z;
                    if constexpr (BITS == 3)
                        z = (__builtin_amdgcn_alignbit(par[s].zword1, par[s].zword, (uint32_t)map.zshift) >> (3 * j)) & 7u;
                    else
                        z = (par[s].zword >> (map.zshift + BITS * j)) & ((1u << BITS) - 1u);
                    zc[j] = nat_zero<BITS>(z);
                }
                sc[s] = par[s].s;
                if constexpr (PG == 4) {  // (no group: see load_params)
                    const uint32_t real = g * PG + s < (int)cgroups ? 0xFFFFFFFFu : 0u;
                    sc[s].r[0] &= real;
                    sc[s].r[1] &= real;
                }
                asm volatile("" : "+v"(sc[s].r[0]), "+v"(sc[s].r[1]));
                __builtin_amdgcn_sched_barrier(0);
                load_params(map, g + 1, s);
                __builtin_amdgcn_sched_barrier(0);
            };

            half8_t a[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) a[it] = *(const half8_t*)(lds_raw + a_off[it]);
            // unpack, and the first row block's products as the operands come
            half8_t bq[4][4];
            float4_t tile[2][2];  // [pair of column sets][column set]: the products of one quantisation group
            const float4_t zero4 = float4_t{0.f, 0.f, 0.f, 0.f};
            auto mfma = [&](int it, int j, bool first) {
                float4_t& d = tile[j >> 1][j & 1];
                d = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[it], bq[it][j], first ? zero4 : d, 0, 0, 0);
            };
            auto add = [&](int i, int s, int pr, int e) {
                acc[i][2 * pr + (e >> 2)][e & 3] = __builtin_fmaf(scale_of<4>(sc[s], 2 * pr + (e >> 2)), tile[pr][e >> 2][e & 3],
                                                                  acc[i][2 * pr + (e >> 2)][e & 3]);
            };
            u32x4_t raw[2][2];
            auto read_raw = [&](int it) {
                const char* src = lds_raw + lds_w + it * kRowsWordLoads<BITS> * 1024 + lane * 16;
                raw[it & 1][0] = raw[it & 1][1] = *(const u32x4_t*)src;
                if constexpr (kRowsWordLoads<BITS> == 2) raw[it & 1][1] = *(const u32x4_t*)(src + 1024);
            };
            read_raw(0);
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int s = it / IPG;
                if (it % IPG == 0) take_params(s);
                if (it < 3) read_raw(it + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    bq[it][j] = nat_unpack<BITS>(raw[it & 1][0][j], raw[it & 1][1][j], lm, zc[j], magic);
                    mfma(it, j, it % IPG == 0);
                    if ((it * 4 + j) % (16 / MB) == 0 && (it * 4 + j) / (16 / MB) < MB) {
                        __builtin_amdgcn_sched_barrier(0);
                        stage_a(g + 1, more, a_next, (it * 4 + j) / (16 / MB));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if (PG > 1 && it % IPG == IPG - 1) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) add(0, s, e >> 3, e & 7);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // (where two workgroups share a unit, the one that has products to issue goes first)
            __builtin_amdgcn_s_setprio(2);
            if constexpr (PG == 1) {
                // The other row blocks.  Two column sets at a time: while their products run, the previous pair's
                // go into the sums, and behind the second pair's products the next block's operands are fetched.
                auto fetch = [&](int i, int it) { a[it] = *(const half8_t*)(lds_raw + a_off[it] + i * 4096); };
#pragma unroll
                for (int it = 0; it < 4; ++it) fetch(1, it);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 8; ++e) add(0, 0, 0, e);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 1; i < MB; ++i) {
#pragma unroll
                    for (int pr = 0; pr < 2; ++pr) {
                        if (i <= 2) stage_w(g + 1, more, 2 * (i - 1) + pr);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int it = 0; it < 4; ++it) {
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                mfma(it, 2 * pr + h, it == 0);
                                if (pr == 1 && h == 1 && i + 1 < MB) fetch(i + 1, it);
                                add(pr == 0 ? i - 1 : i, 0, 1 - pr, 2 * it + h);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                        }
                    }
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) add(MB - 1, 0, 1, e);
            } else {
                // The next row block's operands are fetched ahead of a block's products.  (Left to the scheduler, they come
                // late in most instantiations: 8 bits, 16384 x 1024, m = 200, groups of 32: 18.3 us without, 16.7 with.)
                half8_t ahead[4];
                auto fetch = [&](int i) {
#pragma unroll
                    for (int it = 0; it < 4; ++it) ahead[it] = *(const half8_t*)(lds_raw + a_off[it] + i * 4096);
                };
                fetch(1);
#pragma unroll
                for (int it = 0; it < 4; ++it) stage_w(g + 1, more, it);
#pragma unroll
                for (int i = 1; i < MB; ++i) {
#pragma unroll
                    for (int it = 0; it < 4; ++it) a[it] = ahead[it];
                    if (i + 1 < MB) fetch(i + 1);
#pragma unroll
                    for (int s = 0; s < PG; ++s) {
#pragma unroll
                        for (int i2 = 0; i2 < IPG; ++i2)
#pragma unroll
                            for (int j = 0; j < 4; ++j) mfma(s * IPG + i2, j, i2 == 0);
#pragma unroll
                        for (int e = 0; e < 16; ++e) add(i, s, e >> 3, e & 7);
                    }
                }
            }
            __builtin_amdgcn_s_setprio(0);
#pragma unroll
            for (int it = 0; it < 4; ++it) a_off[it] ^= MB * 4096;
        }
        // what was asked for behind the last chunk has landed (zeros): the next piece's requests go to the same places
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

        // ---- the end of a tile, or of this worker's part of one.  A tile whose chunks several workers share is
        // finished by the one that has its beginning, at the end of that one's range; the others hand their sums over
        // at the beginning of theirs, so that it hardly ever waits.
        const int el = lane_here();
        int es = strip;  // (hidden: keeps the addresses below from being held in registers through the loop)
        asm volatile("" : "+s"(es));
        if (g0 != 0) {
            put_part(acc, w, es, el);
            if (es == 0 && el == 0) set(full + w);
        } else {
            if (g_count < U) {
                const uint32_t parts = later_parts(w, tile_index);
                bool all = true;
                if (es == 0) {
                    uint32_t come = 0;
                    for (int looks = 0; looks < p.polls && come < parts; ++looks) {
                        if (looks) __builtin_amdgcn_s_sleep(4);
                        while (come < parts && look(full + w + 1 + come) != 0u) ++come;
                    }
                    all = come == parts;
                }
                if (!tell(all, es, el)) {
                    put_part(acc, workers + w, es, el);
                    if (es == 0) {
                        if (el == 0) set(left + w);
                        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                        all = claim(w, parts, el);
                    }
                    if (!tell(all, es, el)) goto range_done;  // (it was the last tile of this range)
                }
                for (uint32_t i = 1; i <= parts; ++i) add_part(acc, w + i, es, el);
                taken(w, parts, es, el);
            }
            store_tile(acc, row0, n0, rows, el);
        }
        // (every wave has read its operands before the next piece's are requested)
        __builtin_amdgcn_s_barrier();
    }
range_done:
    // ---- the tile whose sums this worker handed over: if it was left to its later parts and all of them have come,
    // one of them finishes it.  The last one to come finds it so, since it looks after it has come.
    if (u0 % U != 0 && u0 < u1) {
        const int tile_index = u0 / U, first = first_worker(tile_index);
        const uint32_t parts = later_parts(first, tile_index);
        const int el = lane_here(), es = strip;
        bool mine = false;
        if (es == 0) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            mine = look(left + first) != 0u && claim(first, parts, el);
        }
        if (tell(mine, es, el)) {
            int row0, n0;
            const int rows = place(tile_index, &row0, &n0);
            float4_t acc[MB][4];
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
            add_part(acc, workers + first, es, el);
            for (uint32_t i = 1; i <= parts; ++i) add_part(acc, first + i, es, el);
            taken(first, parts, es, el);
            store_tile(acc, row0, n0, rows, el);
        }
    }
}

}  // namespace w4a16
