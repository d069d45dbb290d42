// Base projection x W^T for large batches (prefill), where the matrix cores and the power they draw bound the kernel
// (paper Sec. 2.2: the adapter's activations are added to the backbone layer's output; Sec. 5.1.2: backbone latency
// grows linearly with the batch).
//
// What bounds it: on real values the chip lowers its clock until the power fits, so a kernel is as fast as its energy per
// flop is low.  Hence, against the kernel that stages its tiles through registers (8192 x 14336, K = 4096, normal values):
//   - four wavefronts of (BM / 2) x (BN / 2) each, one per SIMD: two thirds of the LDS reads of eight waves;
//   - tiles copied global -> LDS by the copy instruction: no registers and no LDS writes in between (781 -> 725 us);
//   - the copies spread evenly over the MFMAs, so that none waits for the CU's copy rate of 43 bytes a clock (-> 697);
//   - 16x16x32 MFMAs: an accumulator is read and written once per 32 of K, not per 16 (K = 14336: 1388 -> 1465 TFLOP/s);
//   - a workgroup keeps its CU and goes through several output tiles; the copies of its walk over K continue from one into the
//     next, and the expand is part of that walk (below), not a chain of memory latencies behind it.  The rows are stored past
//     L2 (-> 650 us; 3 % more with adapters, where the other kernel's epilogue takes 10 %).
// What is left at a change of output tile: the wave waits for the data of the tile after the next on the spot (128 x 256: first
// for its range of chunks, then for its rows), and the copies in flight land with them.  The 256 x 256 instances, whose
// accumulators take half of the 512 registers, spill 11 to 14 of the others there and read them back behind the output stores,
// which so are waited for in front of the next tile's first MFMAs; 256 x 192 spills at most one, 128 x 256 none.
// A round of 256 tiles over K = 4096: 256 x 256 112 -> 100 us (95 in a launch of several rounds), 256 x 192 90 -> 79,
// 128 x 256 67.5 -> 59.
//
// K is walked in 64-wide tiles of 128-byte rows, chunk c (16 bytes) of row r at LDS position c ^ ((r >> 1) & 7), which the
// lanes of a copy account for in the addresses they fetch from; the fragment reads (16 rows x 4 chunks) are free of bank
// conflicts.  Two stages for x and three for W: x of tile j + 1 and W of tile j + 2 are on their way while tile j is
// multiplied.  One barrier per tile, behind the first MFMAs of its second K step: every wave has its last fragments of the
// tile in registers by then, and the first fragments of the next tile are read behind the rest of that step's MFMAs.
#include "device_common.hpp"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace lora {
namespace {

template <typename F, int... Is>
__device__ __forceinline__ void direct_for_impl(F&& f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void direct_for(F&& f)
{
    direct_for_impl(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}

constexpr int kDK = 64;          // K extent of one LDS tile (bf16 elements)
constexpr int kDRow = 128;       // bytes per LDS row
constexpr int kDWaves = 4;
constexpr int kDXcdRuns = 16;    // row tiles up to which an XCD takes a contiguous run of tiles
constexpr int kDB = 16;          // rows and columns of an accumulator block

// v_mfma_f32_16x16x32_bf16: D[16x16] += A[16x32] B[32x16].  Lane l = 16 h + i supplies A[i][8h..8h+7] and B[8h..8h+7][i]; it
// receives D[4 h + e][i] in register e.
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Sixteen bytes per lane from buffer `rs` at off + k0 (bytes) to LDS address lds + 16 lane.  The register that carries the
// LDS address needs one wait state between its write and the copy.  A buffer of no bytes reads nothing from memory.
__device__ __forceinline__ void copy16(uint32_t off, u32x4 rs, uint32_t k0, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(off), "s"(rs), "s"(k0), "s"(lds) : "memory");
}

__device__ __forceinline__ u32x4 buffer_of(const void* p, uint32_t bytes)
{
    const uint64_t at = reinterpret_cast<uint64_t>(p);
    u32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((uint32_t)at);
    r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(at >> 32));
    r[2] = __builtin_amdgcn_readfirstlane(bytes);
    r[3] = 0x00020000u;
    return r;
}

template <int N>
__device__ __forceinline__ void wait_copies_then_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
}

// The launch's arguments where they lie, for reads that are repeated for every tile: what is read through a pointer the
// compiler cannot follow does not occupy scalar registers in between (it would spill them).
typedef const __attribute__((address_space(4))) LargeGemmArgs* ArgsInPlace;
__device__ __forceinline__ ArgsInPlace args_in_place()
{
    ArgsInPlace p = (ArgsInPlace)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// ---------------------------------------------------------------------------------------------------
// The expand as a continuation of the walk over K.  Per block of kDBlock grouped rows the adapters' ranks stand side by side,
// in chunks of eight: record c of a block says which adapter (location, rank) and which eight of its ranks chunk c is and
// which of the block's windows of kDB rows have it, and every row knows its own first chunk and how many it has.  Behind the
// last K tile the GEMM copies tiles of eight chunks: x part = the row's scaled shrink results where a chunk is the row's own and
// zero elsewhere, W part = rows of that adapter's B.  They are multiplied like any other K tile.  An adapter that comes back
// later in a block (RUNS) has the chunks it had before: with chunks of its own for every run, 1100 tokens of four rank-64
// adapters in turn were 256 expand tiles behind the 64 of the backbone (Llama-8B step 4032 us, now 1360; the register-staged
// kernel 1460 - 1530).
// ---------------------------------------------------------------------------------------------------
constexpr int kDBlock = 256;

// Two kinds of workgroups per block (x) and slice (y).  z < kDShares: 32 rows' shrink results, a thread per (row, eight ranks):
// sums the K chunks of the shrink, scales, rounds to bf16 once.  z = kDShares of the first slice: the block's map.  The launch
// is latency: a chain of loads per thread, so a step of a few thousand tokens wants them side by side and four chunks in
// flight.  Against one workgroup per block and slice that walks its rows: Llama-8B, 2100 tokens, q|k|v 14.5 -> 5.4 us, down (its
// shrink results in 7 chunks) 33.7 -> 7.3; 20462 tokens 5.4 - 8.9 -> 5.3.
constexpr int kDShares = kDBlock / 32;
constexpr int kDChunks = 4;                                   // shrink chunks per round of loads
__global__ __launch_bounds__(kDBlock) void expand_tiles_kernel(LargeGemmArgs a)
{
    __shared__ int s_wave[2][kDBlock / kWave], s_range[kDBlock / kWave];
    __shared__ __attribute__((aligned(16))) int s_loc[kDBlock];   // per run: its adapter's location; behind the last: -1
    __shared__ int s_same[kDBlock], s_first[kDBlock], s_windows[kDBlock];   // its adapter's first run; of such a run: first chunk, windows
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int T = a.dv.T, mr = a.dv.max_rank, m0 = (int)blockIdx.x * kDBlock, m = m0 + tid;
    if ((int)blockIdx.z == kDShares) {
        if (blockIdx.y != 0) return;
        const int mc = m < T ? m : T - 1;
        const int rl = a.dv.row_loc[mc], rr = a.dv.row_rank[mc], before = a.dv.row_loc[mc > 0 ? mc - 1 : 0];
        const int r = m < T && rl >= 0 ? rr : 0;
        const int loc = r > 0 ? rl : -1;
        const bool head = r > 0 && (tid == 0 || before != loc);
        // the row's run (rows without an adapter: any)
        const unsigned long long heads = __ballot(head);
        if (lane == 0) s_wave[0][wave] = __popcll(heads);
        s_loc[tid] = -1;
        s_windows[tid] = 0;
        __syncthreads();
        int run = __popcll(heads & ((2ull << lane) - 1ull)) - 1, runs = 0;
#pragma unroll
        for (int w = 0; w < kDBlock / kWave; ++w) {
            if (w < wave) run += s_wave[0][w];
            runs += s_wave[0][w];
        }
        if (run < 0) run = 0;
        if (head) s_loc[run] = loc;
        __syncthreads();
        int same = run;                                      // the first run of the same adapter
        if (a.ex.returns && head) {
            for (int k = 0; k < runs; k += 4) {
                const int4 o = *reinterpret_cast<const int4*>(s_loc + k);
                if (o.w == loc && k + 3 < same) same = k + 3;
                if (o.z == loc && k + 2 < same) same = k + 2;
                if (o.y == loc && k + 1 < same) same = k + 1;
                if (o.x == loc && k < same) same = k;
            }
        }
        const int chunks = head && same == run ? r / 8 : 0;
        int v = chunks;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int o = __shfl_up(v, d, kWave);
            if (lane >= d) v += o;
        }
        if (lane == kWave - 1) s_wave[1][wave] = v;
        __syncthreads();
        int end = v, all = 0;                                // chunks up to and with this row's run
#pragma unroll
        for (int w = 0; w < kDBlock / kWave; ++w) {
            if (w < wave) end += s_wave[1][w];
            all += s_wave[1][w];
        }
        if (head) s_same[run] = same;
        if (chunks > 0) s_first[run] = end - chunks;
        __syncthreads();
        const int own = r > 0 ? s_same[run] : 0;
        if (r > 0 && (head || tid % kDB == 0)) atomicOr(&s_windows[own], 1 << (tid / kDB));
        const int first = r > 0 ? s_first[own] : 0xffff;
        if (m < T) a.ex.row[m] = r > 0 ? first | (r / 8) << 16 : 0;
        int lo = first, hi = r > 0 ? first + r / 8 : 0;      // chunks of the wave's rows
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int l = __shfl_xor(lo, d, kWave), u = __shfl_xor(hi, d, kWave);
            lo = l < lo ? l : lo;
            hi = u > hi ? u : hi;
        }
        if (lane == 0) s_range[wave] = lo | hi << 16;
        __syncthreads();
        if (tid < 2) {
            const int o = s_range[2 * tid], p = s_range[2 * tid + 1];
            lo = (o & 0xffff) < (p & 0xffff) ? o & 0xffff : p & 0xffff;
            hi = o >> 16 > p >> 16 ? o >> 16 : p >> 16;
            a.ex.half[2 * blockIdx.x + tid] = hi > 0 ? (lo & ~7) | hi << 16 : 0;
        }
        const size_t at = (size_t)blockIdx.x * kDBlock * (mr / 8);
        for (int c = 0; c < chunks; ++c) a.ex.record[at + end - chunks + c] = int2{loc, r | (c * 8) << 8 | s_windows[run] << 16};
        if (tid == 0) a.ex.count[blockIdx.x] = all;
        if (tid < 4 && blockIdx.x == 0) a.ex.zero[tid] = 0;
        return;
    }
    const int si = (int)blockIdx.y, segs = mr / 8;
    const int row = m0 + (int)blockIdx.z * 32 + tid / segs, seg = tid % segs;
    if (tid >= 32 * segs || row >= T) return;
    const int loc = a.dv.row_loc[row], rank = a.dv.row_rank[row];
    const float sc = a.dv.row_scale[row];
    if (loc < 0 || seg * 8 >= rank) return;
    const size_t chunk = (size_t)T * mr;
    const float* const vp = pick_slice(a.g, si).vpart + (size_t)row * mr + seg * 8;
    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < a.n_kc; c0 += kDChunks) {
        f32x4 l[kDChunks], u[kDChunks];
#pragma unroll
        for (int d = 0; d < kDChunks; ++d) {
            const float* const p = vp + (c0 + d < a.n_kc ? c0 + d : c0) * chunk;
            l[d] = *reinterpret_cast<const f32x4*>(p);
            u[d] = *reinterpret_cast<const f32x4*>(p + 4);
        }
#pragma unroll
        for (int d = 0; d < kDChunks; ++d)
            if (c0 + d < a.n_kc) {
                lo += l[d];
                hi += u[d];
            }
    }
    bf16x8 vb;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        vb[e] = (__bf16)(lo[e] * sc);
        vb[4 + e] = (__bf16)(hi[e] * sc);
    }
    *reinterpret_cast<u32x4*>(a.ex.v + (size_t)si * T * mr + (size_t)row * mr + seg * 8) = __builtin_bit_cast(u32x4, vb);
}

// Sixteen bytes per lane from an address of its own to LDS address lds + 16 lane (see copy16).
__device__ __forceinline__ void copy16_from(const void* p, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p), "s"(lds) : "memory");
}

constexpr uint32_t kNowhere = 0xffffff00u;                   // an offset behind the end of every buffer: reads zeros, writes nothing

// BIAS: some slice of the launch has a bias (an instance of its own, so that the others carry nothing for it).
template <int BM, int BN, bool GLU, bool BIAS>
__global__ __launch_bounds__(kDWaves* kWave, 1) void gemm_direct_kernel(LargeGemmArgs a)
{
    constexpr int WTM = BM / 2, WTN = BN / 2;               // wave tile: 2 x 2 waves
    constexpr int MB = WTM / kDB, NB = WTN / kDB;           // accumulator blocks per wave
    constexpr int NSX = 2, NSW = 3;
    constexpr int XST = BM * kDRow, WST = BN * kDRow;       // bytes per stage
    constexpr int XQ = BM / 8 / kDWaves, WQ = BN / 8 / kDWaves;   // copy instructions (8 rows) per wave and tile
    constexpr int RING = NSX * XST + NSW * WST;
    constexpr int MW = WTM / kWave;                         // registers that hold one value per row of the wave
    static_assert(WTM % kWave == 0 && WTN % 32 == 0 && RING <= 160 * 1024, "tile");
    static_assert(WQ % 2 == 0, "even and odd copies");
    static_assert(!GLU || WQ == 8, "blocks of 32 rows change the matrix every fourth copy");
    __shared__ __attribute__((aligned(1024))) uint8_t ring[RING];
    uint8_t* const x_ring = ring;
    uint8_t* const w_ring = ring + NSX * XST;

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int i = lane & 15, h = lane >> 4;
    const int wm = wave & 1, wn = wave >> 1;
    const int T = a.m_end, K = a.K;                         // rows past m_end are computed, never stored
    const int nk = K / kDK;                                 // at least 3 (host): K tile 0 and the last two are not the same ones
    if (a.ex.long_chunks > 0 && expand_is_long(a)) return;  // uniform over the launch: the other kernel's

    // ---- the tiles of this workgroup ----
    // Consecutive workgroups go to different XCDs.  Row tile fastest; with up to kDXcdRuns row tiles every XCD takes a
    // contiguous run of the tiles.  Every round deals the next t_deal tiles (of the XCD's run, or of all) to as many
    // workgroups, `turn` places further on than the round before: see tile_turn().
    struct Tile {
        int m0, n0, si;
        int on;
    };
    const int t_all = a.tiles_m * a.tiles_n;
    int t_deal = (int)gridDim.x, t_place = (int)blockIdx.x, t_number = t_place, t_end = t_all;
    if (a.tiles_m <= kDXcdRuns) {
        const int xcd = (int)blockIdx.x & 7, per = t_all >> 3, more = t_all & 7;
        const int start = xcd * per + (xcd < more ? xcd : more);
        t_place = (int)blockIdx.x >> 3;
        t_number = start + t_place;
        t_deal = ((int)gridDim.x - xcd + 7) >> 3;
        t_end = start + per + (xcd < more ? 1 : 0);
    }
    int tile_m = t_number % a.tiles_m, tile_n = t_number / a.tiles_m;
    const int step_m = (t_deal + a.turn) % a.tiles_m, step_n = (t_deal + a.turn) / a.tiles_m;
    auto tile_here = [&]() {
        Tile t{0, 0, 0, t_number < t_end ? 1 : 0};
        if (!t.on) return t;
        const ArgsInPlace ka = args_in_place();
        if (!GLU)
            for (int k = 1; k < ka->g.n; ++k)
                if (tile_n >= ka->g.s[k].tile0) t.si = k;
        t.m0 = ka->m_begin + tile_m * BM;
        t.n0 = (tile_n - ka->g.s[t.si].tile0) * (GLU ? BN / 2 : BN);
        return t;
    };
    auto next_tile = [&]() {
        const bool wrap = t_place + a.turn >= t_deal;        // behind the round's last place comes its first
        t_place += wrap ? a.turn - t_deal : a.turn;
        t_number += wrap ? a.turn : t_deal + a.turn;
        tile_m += wrap ? a.turn : step_m;                    // below 2 tiles_m
        tile_n += wrap ? 0 : step_n;
        if (tile_m >= a.tiles_m) {
            tile_m -= a.tiles_m;
            ++tile_n;
        }
        return tile_here();
    };

    // ---- copies ----
    // Instruction q of wave w fills stage rows 8 (w XQ + q) .. + 7 of the x part (same for the W part with WQ); lane l owns
    // row l / 8 of those and the chunk that belongs at position l % 8.  W rows are counted from the tile's first one, which
    // the buffer starts at; rows behind the matrix read zeros.
    auto x_row = [&](int q, int lane) { return (wave * XQ + q) * 8 + (lane >> 3); };
    auto w_row = [&](int q, int lane) { return (wave * WQ + q) * 8 + (lane >> 3); };
    auto chunk_of = [](int r, int lane) { return (lane & 7) ^ ((r >> 1) & 7); };
    auto w_column = [](int r) { return GLU ? (r >> 6) * 32 + (r & 31) : r; };
    // W offsets of copy 0 and copy 1; the even and the odd ones have the same chunks and lie whole rows further on
    uint32_t woff[2];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const int r = w_row(o, lane) - o * 8;
        woff[o] = (uint32_t)w_column(r) * (uint32_t)K * 2u + (uint32_t)(chunk_of(r + o * 8, lane) * 16);
    }
    // What the copies and the epilogue of one output tile need; asked for two tiles ahead, and waited for there.  Per lane: of row l of the rows the
    // wave copies (8 XQ of them) the token and the chunks (ExpandTiles::row), the tokens of rows l and 64 + l of the wave's part of
    // the tile, record l % 8 of the tile's chunks.
    struct Info {
        int xtok, xrow, tok[MW];
        int2 rec;
    };
    auto load_info = [&](const Tile& t, Info& f, int lane, int first_chunk) {
        const ArgsInPlace ka = args_in_place();
        const int32_t* const perm = ka->dv.perm;
        const bool ex = ka->ex.on != 0;                      // uniform over the launch; otherwise nothing looks at these two
        const int32_t* const row = ex ? ka->ex.row : perm;
        const int2* const rec = ex ? ka->ex.record + (size_t)(t.m0 / kDBlock) * kDBlock * (ka->dv.max_rank / 8) : reinterpret_cast<const int2*>(perm);
        int m = t.m0 + wave * (8 * XQ) + (lane & (8 * XQ - 1));
        if (m > T - 1) m = T - 1;
        f.xtok = perm[m];
        f.xrow = row[m];
        f.rec = rec[ex ? first_chunk + (lane & 7) : 0];
#pragma unroll
        for (int k = 0; k < MW; ++k) {
            int mk = t.m0 + wm * WTM + k * kWave + lane;
            if (mk > T - 1) mk = T - 1;
            f.tok[k] = perm[mk];
        }
    };
    // The chunks that the rows of the tile use: the first (a multiple of eight) | the end << 16, and the K tiles of the expand
    // that they take behind the backbone's.  128 rows go through those between their first and their last adapter's only: with
    // all of the block's, a launch of one round whose last rows are a hundred one-token requests ends with them (1300 tokens, 128
    // adapters of 8 to 64 ranks, Llama-8B o: 112 -> 91 us; down 238 -> 206).
    auto expand_chunks = [&](const Tile& t) {
        const ArgsInPlace ka = args_in_place();
        if (!t.on || !ka->ex.on) return 0;
        return BM == kDBlock ? __builtin_amdgcn_readfirstlane(ka->ex.count[t.m0 / kDBlock]) << 16 : __builtin_amdgcn_readfirstlane(ka->ex.half[t.m0 / (kDBlock / 2)]);
    };
    static_assert(BM == kDBlock || BM == kDBlock / 2, "a block or half of one");
    auto expand_tiles = [](int chunks) { return ((chunks >> 16) - (chunks & 0xffff) + 7) / 8 * (GLU ? 2 : 1); };
    // Both.  A block's first chunk is its chunk 0, which saves the wait for the one in front of the other (q|k|v and o of
    // Qwen2.5-7B at 4099 tokens 98 -> 96 us, 94 -> 92).
    auto load_tile = [&](const Tile& t, const Tile& in_place, Info& f, int lane) {
        const Tile of = t.on ? t : in_place;
        if constexpr (BM == kDBlock) {
            load_info(of, f, lane, 0);
            return expand_chunks(t);
        } else {
            const int c = expand_chunks(t);
            load_info(of, f, lane, c & 0xffff);
            return c;
        }
    };
    auto x_buffer = [&](const Tile& t) {
        const ArgsInPlace ka = args_in_place();
        return buffer_of(ka->g.s[t.si].x, t.on ? (uint32_t)ka->dv.T * (uint32_t)K * 2u : 0u);
    };
    auto w_buffer = [&](const Tile& t, bool up) {
        const ArgsInPlace ka = args_in_place();
        const int si = GLU && up ? 1 : t.si;
        return buffer_of(ka->g.s[si].W + (size_t)t.n0 * K, t.on ? (uint32_t)(ka->g.s[si].N - t.n0) * (uint32_t)K * 2u : 0u);
    };
    const uint32_t x_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)x_ring + wave * XQ * 1024;
    const uint32_t w_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)w_ring + wave * WQ * 1024;

    // ---- fragments and MFMAs ----
    const int sw_i = (i >> 1) & 7;
    int rd[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) rd[kk] = i * kDRow + (((4 * kk + h) ^ sw_i) << 4);
    const uint8_t* const x_mine = x_ring + wm * WTM * kDRow;
    const uint8_t* const w_mine = w_ring + wn * WTN * kDRow;
    f32x4 acc[MB][NB];
    bf16x8 Fw[2][NB], Fx[2][MB];
    constexpr int NM = MB * NB;                              // MFMAs per K step (32 of K; two steps per tile)
    constexpr int NR = MB + NB;                              // LDS reads per K step
    constexpr int HEAD = 8;                                  // MFMAs of the second K step in front of the barrier
    constexpr int TAIL = NM - HEAD;                          // and behind it
    static_assert(NR <= TAIL, "reads are spread one per MFMA");
    auto read_one = [&](int f, uint32_t xs, uint32_t ws, int kk, int r) {
        if (r < NB) Fw[f][r] = as_bf16x8(*reinterpret_cast<const u32x4*>(w_mine + ws + rd[kk] + r * kDB * kDRow));
        else Fx[f][r - NB] = as_bf16x8(*reinterpret_cast<const u32x4*>(x_mine + xs + rd[kk] + (r - NB) * kDB * kDRow));
    };
    auto mma_one = [&](int f, int t) {
        const int mb = t / NB, nb = t % NB;
        acc[mb][nb] = mfma16(Fw[f][nb], Fx[f][mb], acc[mb][nb]);
    };
    // x copies are spread over the TAIL MFMAs, W copies over the K step behind them
    constexpr int SX = TAIL / XQ, SW = NM / WQ;
    static_assert(SX >= 1 && SW >= 1, "copies fit");

    Tile cur = tile_here();
    if (!cur.on) return;                                     // uniform over the workgroup (no such workgroup is launched)
    Info info, info_next;
    uint32_t xoff[XQ];
    auto x_offsets = [&](const Info& f, int lane) {
#pragma unroll
        for (int q = 0; q < XQ; ++q) {
            xoff[q] = (uint32_t)__shfl(f.xtok, q * 8 + (lane >> 3), kWave) * (uint32_t)K * 2u + (uint32_t)(chunk_of(x_row(q, lane), lane) * 16);
            asm volatile("" : "+v"(xoff[q]));
        }
    };
    int chunks = load_tile(cur, cur, info, lane);
    u32x4 xrs = x_buffer(cur), wrs = w_buffer(cur, false), urs = GLU ? w_buffer(cur, true) : wrs;
    u32x4 xrs_next, wrs_next, urs_next;
    x_offsets(info, lane);
    // a vector memory instruction may read a scalar register that a vector instruction wrote five wait states later at the
    // earliest, and the compiler does not look into the copy statement
    asm volatile("s_nop 4" ::: "memory");
    uint32_t xk = 0, wk = 0;                                 // byte offset of the tile to copy inside a row
    // q: compile-time at every call site; stage: byte offset of the stage in its ring
    auto copy_x = [&](auto qc, uint32_t stage) {
        constexpr int q = decltype(qc)::value;
        copy16(xoff[q], xrs, xk, x_lds + stage + q * 1024);
    };
    auto copy_w = [&](auto qc, uint32_t stage) {
        constexpr int q = decltype(qc)::value;
        // the product stays out of the registers between copies
        uint32_t row_bytes = (uint32_t)K * 2u;
        asm volatile("" : "+s"(row_bytes));
        copy16(woff[q & 1] + (uint32_t)((GLU ? q & 3 : q) * 8) * row_bytes, GLU && (q >> 2) ? urs : wrs, wk, w_lds + stage + q * 1024);
    };
    direct_for<WQ>([&](auto q) { copy_w(q, 0); });
    direct_for<XQ>([&](auto q) { copy_x(q, 0); });
    wk = xk = kDK * 2;
    direct_for<WQ>([&](auto q) { copy_w(q, WST); });
    direct_for<XQ>([&](auto q) { copy_x(q, XST); });
    Tile nxt = next_tile();
    int chunks_next = load_tile(nxt, cur, info_next, lane);
    xrs_next = x_buffer(nxt);
    wrs_next = w_buffer(nxt, false);
    urs_next = GLU ? w_buffer(nxt, true) : wrs_next;
    // Stages (byte offsets): of the tile being multiplied, of the next one, and the W stage to fill.
    uint32_t xs = 0, xn = XST, ws = 0, wnx = WST, wf = 2 * WST;
    auto rotate = [&]() {
        const uint32_t s = xs;
        xs = xn;
        xn = s;
        const uint32_t o = ws;
        ws = wnx;
        wnx = wf;
        wf = o;
    };
    __builtin_amdgcn_s_waitcnt(0x0f70);                      // vmcnt(0): the first tiles and the row data are there
    wait_copies_then_barrier<0>();
    direct_for<NR>([&](auto r) { read_one(0, xs, ws, 0, r.value); });

    constexpr int OC = GLU ? WTN / 2 : WTN;                  // output columns of the wave
    constexpr int CHP = OC > 64 ? 16 : 8;                    // 16-byte chunk positions per LDS row of the epilogue
    constexpr int ORow = CHP * 16, RPI = kWave / CHP;        // bytes per LDS row, rows per store instruction
    constexpr int IT = kDB / RPI;
    constexpr int kStores = MB * IT;                         // of a whole output tile, per wave
    // pieces per wave: with one, a window's reads are issued before the next one's writes, and LDS serves a wave in order
    constexpr int PIECES = kDWaves * 2 * kDB * ORow <= WST ? 2 : 1;
    static_assert(kDWaves * PIECES * kDB * ORow <= WST, "the pieces fit the stage");
    static_assert(kStores + WQ <= 63, "vmcnt range");
    bool stored = false;                                     // kStores stores stand behind the copies of K tile 1

    for (;;) {
        const int nl = expand_tiles(chunks), nkt = nk + nl;  // K tiles of this output tile
        // K tile j.  While it is multiplied, W of tile j + 2 is copied into the third W stage and, behind the barrier that
        // says every wave has its last fragments, x of tile j + 2 into the stage of tile j.  The walk over K goes on into the
        // expand's tiles and into the workgroup's next output tile.
        auto k_tile = [&](auto first_c, auto&& mma, auto&& w_copy, auto&& x_copy) __attribute__((always_inline)) {
            constexpr bool FIRST = decltype(first_c)::value;
            direct_for<NM>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                if constexpr (FIRST) acc[t / NB][t % NB] = mfma16(Fw[0][t % NB], Fx[0][t / NB], f32x4{0.f, 0.f, 0.f, 0.f});
                else mma(0, t);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (t < NR) read_one(1, xs, ws, 1, t);
                if constexpr (t % SW == 0 && t / SW < WQ) w_copy(std::integral_constant<int, t / SW>{}, wf);
                __builtin_amdgcn_sched_barrier(0);
            });
            direct_for<HEAD>([&](auto tc) {
                mma(1, decltype(tc)::value);
                __builtin_amdgcn_sched_barrier(0);
            });
            // this wave's last fragments of tile j are in registers; tile j + 1 has landed (W of tile j + 2 stays in flight,
            // and so do the stores of the output tile before, where no spilled register was read back behind them)
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (FIRST && stored) wait_copies_then_barrier<WQ + kStores>();
            else wait_copies_then_barrier<WQ>();
            __builtin_amdgcn_sched_barrier(0);
            direct_for<TAIL>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                mma(1, HEAD + t);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (t < NR) read_one(0, xn, wnx, 0, t);
                if constexpr (t % SX == 0 && t / SX < XQ) x_copy(std::integral_constant<int, t / SX>{}, xs);
                __builtin_amdgcn_sched_barrier(0);
            });
            rotate();
        };
        wk = xk = 2 * kDK * 2;
        k_tile(std::true_type{}, mma_one, copy_w, copy_x);
        for (int j = 1; j < nk - 2; ++j) {
            wk = xk = (uint32_t)(j + 2) * (kDK * 2);
            k_tile(std::false_type{}, mma_one, copy_w, copy_x);
        }
        // The last tiles: what is copied are the expand's tiles or the next output tile's first two.
        Tile after = nxt;
        Info info_after;
        if (nxt.on) after = next_tile();
        int lr = lane;
        asm volatile("" : "+v"(lr));
        const int chunks_after = load_tile(after, cur, info_after, lr);
        const u32x4 xrs_after = x_buffer(after), wrs_after = w_buffer(after, false), urs_after = GLU ? w_buffer(after, true) : wrs_after;
        int users = 0, users_next = 0;                       // per lane: windows that have chunk l % 8 of K tile j and of the next one
        auto last_tile = [&](int j, auto expand_c) __attribute__((always_inline)) {
            constexpr bool EXPAND = decltype(expand_c)::value;   // K tile j is one of the expand's
            const int l = j + 2 - nk;                        // the tile to copy: of the expand, while below nl
            const bool ex = l < nl;                          // uniform over the workgroup
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const ArgsInPlace ka = args_in_place();
            const int mr = ka->dv.max_rank, p = GLU ? l & 1 : 0, c8 = (chunks & 0xffff) + (GLU ? l >> 1 : l) * 8;
            // W copies of either kind have a first row, a distance between rows and a place in the row per lane, for even and
            // for odd copies (whose chunk positions differ by four); [1]: of the matrix `up`
            const Tile of = ex || !nxt.on ? cur : nxt;
            const int n_first = of.n0, n_last = ka->g.s[of.si].N - 1;
            const uint8_t* from[2][2];
            uint32_t pitch[2][2];
            if (ex) {
                // x: the row's own chunks among the eight of this tile
                xrs = buffer_of(ka->ex.v + (size_t)(GLU ? p : cur.si) * ka->dv.T * mr, (uint32_t)ka->dv.T * (uint32_t)mr * 2u);
                xk = 0;
#pragma unroll
                for (int q = 0; q < XQ; ++q) {
                    const int own_chunks = __shfl(info.xrow, q * 8 + (ln >> 3), kWave);
                    const int r = x_row(q, ln), d = c8 + chunk_of(r, ln) - (own_chunks & 0xffff);
                    const bool own = (unsigned)d < (unsigned)(own_chunks >> 16) && cur.m0 + r < T;
                    xoff[q] = own ? (uint32_t)((cur.m0 + r) * mr + d * 8) * 2u : kNowhere;
                    asm volatile("" : "+v"(xoff[q]));
                }
                if (l > 0 && p == 0) info.rec = ka->ex.record[(size_t)(cur.m0 / kDBlock) * kDBlock * (mr / 8) + c8 + (ln & 7)];
                const int end = chunks >> 16;
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const int c = chunk_of(o * 8 + (ln >> 3), ln);
                    const int loc = __shfl(info.rec.x, c, kWave), rr = __shfl(info.rec.y, c, kWave);
                    const uint32_t rank = (uint32_t)(rr & 0xff), from_rank = (uint32_t)(rr >> 8) & 0xffu;
                    const uint8_t* const at = reinterpret_cast<const uint8_t*>(ka->dv.slots + (size_t)(uint32_t)loc * kLocUnit + (size_t)rank * ka->g.s[GLU ? p : cur.si].b_unit + from_rank);
#pragma unroll
                    for (int up = 0; up < 2; ++up) {
                        const bool on = c8 + c < end && (!GLU || up == p);
                        from[up][o] = on ? at : reinterpret_cast<const uint8_t*>(ka->ex.zero);
                        pitch[up][o] = on ? rank * 2u : 0u;
                    }
                }
            } else {
                if (l == nl) x_offsets(info_next, ln);
                xrs = xrs_next;
                wrs = wrs_next;
                urs = urs_next;
                const uint32_t k0 = (uint32_t)(l - nl) * (kDK * 2);
                xk = xrs[2] == 0u ? 0u : k0;
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int up = 0; up < 2; ++up) {
                        from[up][o] = reinterpret_cast<const uint8_t*>(ka->g.s[GLU ? up : of.si].W) + k0 + chunk_of(o * 8 + (ln >> 3), ln) * 16;
                        pitch[up][o] = (uint32_t)K * 2u;
                    }
            }
            xk = __builtin_amdgcn_readfirstlane(xk);
            asm volatile("s_nop 4" ::: "memory");
            auto w_copy = [&](auto qc, uint32_t stage) {
                constexpr int q = decltype(qc)::value, up = GLU ? q >> 2 : 0;
                int n = n_first + w_column(w_row(q, ln));
                if (n > n_last) n = n_last;
                copy16_from(from[up][q & 1] + (size_t)(uint32_t)n * pitch[up][q & 1], w_lds + stage + q * 1024);
            };
            if constexpr (!EXPAND) {
                k_tile(std::false_type{}, mma_one, w_copy, copy_x);
            } else {
                // The same steps without an order of their own.  A window of 16 rows takes the chunks its own rows use and no
                // others, whatever these hold (their x part is zero, but zero times infinity is not).
                const int window0 = (cur.m0 % kDBlock + wm * WTM) / kDB;
                auto multiply = [&](auto fc) __attribute__((always_inline)) {
                    constexpr int f = decltype(fc)::value;
                    const uint32_t mine = (uint32_t)__shfl(users, f * 4 + (ln >> 4), kWave) >> (16 + window0);
                    direct_for<MB>([&](auto wc) {
                        constexpr int w = decltype(wc)::value;
                        const bool own = (mine >> w & 1u) != 0u;
                        if (__builtin_amdgcn_ballot_w64(own) != 0) {
#pragma unroll
                            for (int nb = 0; nb < NB; ++nb) {
                                const u32x4 v = own ? __builtin_bit_cast(u32x4, Fw[f][nb]) : u32x4{0u, 0u, 0u, 0u};
                                acc[w][nb] = mfma16(as_bf16x8(v), Fx[f][w], acc[w][nb]);
                            }
                        }
                    });
                };
                direct_for<WQ>([&](auto q) { w_copy(q, wf); });
                direct_for<NR>([&](auto r) { read_one(1, xs, ws, 1, r.value); });
                multiply(std::integral_constant<int, 0>{});
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                wait_copies_then_barrier<WQ>();
                direct_for<XQ>([&](auto q) { copy_x(q, xs); });
                direct_for<NR>([&](auto r) { read_one(0, xn, wnx, 0, r.value); });
                multiply(std::integral_constant<int, 1>{});
                rotate();
            }
            users = users_next;
            users_next = info.rec.y;
        };
#pragma clang loop unroll(disable)
        for (int j = nk - 2; j < nk; ++j) last_tile(j, std::false_type{});
#pragma clang loop unroll(disable)
        for (int j = nk; j < nkt; ++j) last_tile(j, std::true_type{});

        // ---------------- epilogue ----------------
        // The fragments of the next output tile's first K step are on their way; xs, ws: its K tile 0, wf: free.
        // What depends on the lane only is computed again for every tile (hidden from the compiler, which would otherwise
        // keep some hundred such values in registers across the main loop, and spill).
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int i = ln & 15, h = ln >> 4;
        const ArgsInPlace ka = args_in_place();
        const int N = ka->g.s[cur.si].N;
        const int mw0 = cur.m0 + wm * WTM, nw0 = cur.n0 + wn * OC;
        // The rows leave through the free W stage (a piece or two per wave): window after window they are rounded to bf16, turned,
        // and stored in sixteen-byte pieces of which consecutive lanes cover a whole run of an output row.
        uint8_t* const piece = w_ring + wf + wave * (PIECES * kDB * ORow);
        u32x2 bias[BIAS ? NB : 1];
        if constexpr (BIAS) {
            const uint16_t* const bias_at = ka->g.s[cur.si].bias;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                int n = nw0 + nb * kDB + h * 4;               // N is a multiple of 8: all four or none
                if (n > N - 4) n = N - 4;
                bias[nb] = u32x2{0u, 0u};
                if (bias_at != nullptr) bias[nb] = *reinterpret_cast<const u32x2*>(bias_at + n);
            }
        }
        // Stores go through a buffer too: lanes whose row or column does not exist are given an offset behind its end and
        // write nothing, so that there are no branches.
        const __amdgpu_buffer_rsrc_t obuf = __builtin_amdgcn_make_buffer_rsrc(ka->g.s[cur.si].out, 0, (int)((uint32_t)ka->dv.T * (uint32_t)N * 2u), 0x00020000);
        uint32_t row_off[MW];                                 // where the lane's rows start; behind the end: no such row
#pragma unroll
        for (int k = 0; k < MW; ++k)
            row_off[k] = mw0 + k * kWave + ln < T ? (uint32_t)info.tok[k] * (uint32_t)N * 2u : kNowhere;
        cur = nxt;
        nxt = after;
        chunks = chunks_next;
        chunks_next = chunks_after;
        __builtin_amdgcn_s_waitcnt(0x0f70);                  // vmcnt(0): the data of the tile after the next
        info = info_next;
        info_next = info_after;
        xrs_next = xrs_after;
        wrs_next = wrs_after;
        urs_next = urs_after;
        __builtin_amdgcn_sched_barrier(0);
        const int orow = ln / CHP, opos = ln % CHP;
        auto turn = [&](auto wc) {
            constexpr int w = decltype(wc)::value;
            uint8_t* const to = piece + (w % PIECES) * (kDB * ORow);
            f32x4 y[OC / kDB];
#pragma unroll
            for (int c = 0; c < OC / kDB; ++c) {
                if (GLU) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        y[c][e] = silu_f32(acc[w][(c >> 1) * 4 + (c & 1)][e]) * acc[w][((c >> 1) * 4 + 2 + (c & 1)) % NB][e];
                } else {
                    y[c] = acc[w][c];
                }
            }
            if constexpr (BIAS) {
#pragma unroll
                for (int c = 0; c < OC / kDB; ++c) {
                    const bf16x4 b = __builtin_bit_cast(bf16x4, bias[c]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[c][e] += (float)b[e];
                }
            }
#pragma unroll
            for (int c = 0; c < OC / kDB; ++c) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (__bf16)y[c][e];
                const int pos = (c * 2 + (h >> 1)) ^ (CHP == 16 ? i : (i >> 1));
                *reinterpret_cast<u32x2*>(to + i * ORow + pos * 16 + (h & 1) * 8) = __builtin_bit_cast(u32x2, o);
            }
        };
        turn(std::integral_constant<int, 0>{});
        __builtin_amdgcn_sched_barrier(0);
        direct_for<MB>([&](auto wc) {
            constexpr int w = decltype(wc)::value;
            const uint8_t* const from = piece + (w % PIECES) * (kDB * ORow);
            u32x4 v[IT];
            uint32_t off[IT];
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int row = it * RPI + orow;
                v[it] = *reinterpret_cast<const u32x4*>(from + row * ORow + opos * 16);
                off[it] = __shfl(row_off[w / 4], (w % 4) * kDB + row, kWave);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (w + 1 < MB) turn(std::integral_constant<int, (w + 1) % MB>{});
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int row = it * RPI + orow;
                const int chunk = opos ^ (CHP == 16 ? row : (row >> 1));
                const int n = nw0 + chunk * 8;
                const bool on = chunk * 8 < OC && n < N && off[it] != kNowhere;
                __builtin_amdgcn_raw_buffer_store_b128(v[it], obuf, on ? (int)(off[it] + (uint32_t)n * 2u) : (int)kNowhere, 0, 2);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        stored = true;
        if (!cur.on) break;                                   // uniform over the workgroup
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
}

// By how many places the deal of the tiles turns from round to round.  Unturned, the row tile of a workgroup steps by the
// workgroups of a round (32 on an XCD); where that is a multiple of the row tiles, it never changes, and the workgroups whose
// rows are the one-token requests of a mixed step, with many times the expand tiles of the others, have them in every
// round and hold up the launch.  There, and only there, it turns by an odd number near half the row tiles: the row tiles with
// many adapters are neighbours, and a workgroup shall not go from one of them to the next.  (With more than kDXcdRuns row
// tiles by a multiple of eight, so that it stays with its XCD's row tiles.)  Other counts are dealt out well as they are: turned
// too, so that a workgroup goes through all row tiles in order, 6 and 12 row tiles lost what 8 and 16 gained (gated, Llama-8B,
// 128 adapters, 3000 tokens 1627 -> 1806 us).  Gated steps with nearly half their tokens from 128 adapters, staged kernel /
// unturned / turned: Llama-8B 1800 tokens 1248 / 1458 / 1236 us, 4000 tokens 2157 / 2325 / 1806; Qwen2.5-7B 4000 tokens
// 2321 / 2951 / 2111.
int tile_turn(int tiles_m, int grid)
{
    const bool runs = tiles_m <= kDXcdRuns;
    const int deal = runs ? grid / 8 : grid, unit = runs ? 1 : 8;
    if (tiles_m < 2 || deal < tiles_m || deal % tiles_m != 0) return 0;
    const int turn = unit * std::max(1, tiles_m / unit / 2 - 1);
    return turn < tiles_m ? turn : 0;                     // below tiles_m and so below every XCD's deal
}

template <int BM, int BN, bool GLU, bool BIAS>
hipError_t launch_direct(LargeGemmArgs a, int n_cus, hipStream_t stream)
{
    a.tiles_m = (a.m_end - a.m_begin + BM - 1) / BM;
    a.tiles_n = 0;
    if (GLU) {                                            // gate and up together: BN / 2 output columns per tile
        a.g.s[0].tile0 = a.g.s[1].tile0 = 0;
        a.tiles_n = (a.g.s[0].N + BN / 2 - 1) / (BN / 2);
    } else {
        for (int k = 0; k < a.g.n; ++k) {
            a.g.s[k].tile0 = a.tiles_n;
            a.tiles_n += (a.g.s[k].N + BN - 1) / BN;
        }
    }
    const int tiles = a.tiles_m * a.tiles_n, grid = tiles < n_cus ? tiles : n_cus;
    a.turn = tile_turn(a.tiles_m, grid);
    hipLaunchKernelGGL((gemm_direct_kernel<BM, BN, GLU, BIAS>), dim3(grid), dim3(kDWaves * kWave), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_expand_tiles(const LargeGemmArgs& a, hipStream_t stream)
{
    hipLaunchKernelGGL(expand_tiles_kernel, dim3((a.dv.T + kDBlock - 1) / kDBlock, a.g.n, kDShares + 1), dim3(kDBlock), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_gemm_direct_glu(const LargeGemmArgs& a, int n_cus, hipStream_t stream)
{
    return launch_direct<256, 256, true, false>(a, n_cus, stream);
}

hipError_t launch_gemm_direct_fused(const LargeGemmArgs& a, int tile, int n_cus, hipStream_t stream)
{
    bool bias = false;
    for (int k = 0; k < a.g.n; ++k) bias = bias || a.g.s[k].bias != nullptr;
    switch (tile) {
        case 1: return bias ? launch_direct<256, 192, false, true>(a, n_cus, stream) : launch_direct<256, 192, false, false>(a, n_cus, stream);
        case 2: return bias ? launch_direct<128, 256, false, true>(a, n_cus, stream) : launch_direct<128, 256, false, false>(a, n_cus, stream);
    }
    return bias ? launch_direct<256, 256, false, true>(a, n_cus, stream) : launch_direct<256, 256, false, false>(a, n_cus, stream);
}

}  // namespace lora
