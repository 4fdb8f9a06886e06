// The convolution's ScMult/Add step on the matrix cores.
//
// For one coefficient index i the step is a dense product  S_i[m][c] = sum_k W_i[m][k] * X_i[k][c]  of 60-bit
// residues (m: output block x kernel order, k: input ciphertext x tap, c: input x polynomial), accumulated
// exactly and reduced mod q once at the end.  It is mapped on the int8 MFMA units by writing every residue in
// eight balanced base-256 digits d_0..d_7 in [-128,127] (x = sum d_u 256^u): then
//     S = sum_{s=0..14} 256^s * D_s,   D_s[m][c] = sum_{u+v=s} sum_k W_u[m][k] * X_v[k][c]
// and every D_s is an int8 x int8 -> int32 matrix product (|D_s| <= 8 * 192 * 2^14 < 2^31 and S < 192 * 2^120 < 2^128
// for the at most 192 terms summed between two reductions mod q, given q < 2^60: exact).
// One v_mfma_i32_16x16x64_i8 multiplies a 16x64 by a 64x16 digit tile; the 64 (u,v) digit pairs of a tile feed
// 15 accumulators of four registers each.  The recombination of the 15 diagonals, the reduction mod q and the
// transposition back to coefficient-major order run on the vector ALU in the same kernel.
//
// Operand images ("digit planes") are made of 16-byte chunks: lane l of the MFMA holds row/column l%16 of a
// tile and the 16 terms k = 64*kblock + 16*(l/16) + j of one digit.
//   row operand (encoded kernels):     [i][tile][kblock][digit][lane]   one digit plane of a tile is 1 KiB
//   column operand (rotated inputs):   [tile][kblock][lane][i][digit]   the 8 digits of a coefficient are 128 B
// The column layout lets the kernel that produces the rotated inputs write it with the coefficient index
// running across the lanes.  Chunks whose 16 terms all lie beyond the last term are never read.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "gala_internal.h"

namespace gala {
namespace {

typedef digit_chunk_t v4i;

// term blocks of 64 between two reductions of the running sums (conv_mfma_kernel); q < 2^60 is required
constexpr int kFoldBlocks = 3;

// balanced base-256 digits of x < 2^61, one per byte: the bytes of x + 0x80..80 are the digits plus 128
__device__ __forceinline__ u64 balanced_digits(u64 x) {
    const u64 k = 0x8080808080808080ull;
    return (x + k) ^ k;
}

// Builds the digit-plane image of 16 rows x 16 terms x 16 coefficients per workgroup; one that holds no term has nothing to do.
// COLUMNS: the source is the tap-rotated inputs [input][e][polynomial][i] with row = 2*input + polynomial, otherwise the encoded
// kernels [row][e][i].  Both are read with the coefficient index fastest (128-byte segments).
// Bound by memory: the columns of 16x16x128 to 128 channels at batch 16 are 75 MB in and 75 MB out, 30.9 us (4.9 TB/s).  It took 40.0 when
// the columns' residues went through LDS too, though a thread got back what it had put there, their chunks were stored to an
// eighth of the banks, and the quarter of the image beyond the last term was written; that layer with special-prime keys 433.9 -> 422.6 us.
template <bool COLUMNS>
__global__ __launch_bounds__(256) void limb_pack_kernel(const u64 *src, int rows, int nterm, int n, int tiles, int kblocks, v4i *dst) {
    // rows: the residues [row][term][coefficient], coefficient dimension padded; columns: chunks [row][coefficient][digit]
    __shared__ __attribute__((aligned(16))) u64 stage[COLUMNS ? 16 * 16 * 16 : 16 * 16 * 17];
    const int i0 = blockIdx.x * 16, tile = blockIdx.y, kb = blockIdx.z >> 2, g = blockIdx.z & 3;
    if (kb * 64 + g * 16 >= nterm) return;
    const int il = threadIdx.x & 15, rl = threadIdx.x >> 4, row = tile * 16 + rl;
    const size_t row_off = COLUMNS ? ((size_t)(row >> 1) * nterm * 2 + (row & 1)) * n : (size_t)row * nterm * n;
    const size_t e_stride = COLUMNS ? 2 * (size_t)n : (size_t)n;
    u64 d[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int e = kb * 64 + g * 16 + j;
        d[j] = (row < rows && e < nterm && i0 + il < n) ? src[row_off + (size_t)e * e_stride + i0 + il] : 0;
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) d[j] = balanced_digits(d[j]);
    v4i chunk[8];
    if constexpr (!COLUMNS) {
        // written with the row across the threads: 16 of them (the rows of a tile) write 256 contiguous bytes per digit
#pragma unroll
        for (int j = 0; j < 16; ++j) stage[(rl * 16 + j) * 17 + il] = d[j];
        __syncthreads();
        const int to_row = threadIdx.x & 15, to_i = threadIdx.x >> 4;
        if (i0 + to_i >= n) return;
#pragma unroll
        for (int j = 0; j < 16; ++j) d[j] = stage[(to_row * 16 + j) * 17 + to_i];
        digit_chunks(d, chunk);
        const size_t base = ((((size_t)(i0 + to_i) * tiles + tile) * kblocks + kb) * 8) * 64 + (size_t)(g * 16 + to_row);
#pragma unroll
        for (int limb = 0; limb < 8; ++limb) dst[base + (size_t)limb * 64] = chunk[limb];
    } else {
        // a row's 16 coefficients x 8 digits are 2 KiB contiguous in the image, but a thread owns the 128
        // bytes of one coefficient: the chunks change owner in LDS so that the 16 threads of a row write 256
        // contiguous bytes per instruction instead of 16 bytes in each of 16 lines.  Within a coefficient the digits are xored
        // with its number halved: the 16 threads that store a digit then use all banks instead of an eighth of them.
        digit_chunks(d, chunk);
        v4i *tr = reinterpret_cast<v4i *>(stage);
#pragma unroll
        for (int limb = 0; limb < 8; ++limb) tr[(rl * 16 + il) * 8 + (limb ^ (il >> 1))] = chunk[limb];
        __syncthreads();
        const size_t base = ((((size_t)tile * kblocks + kb) * 64 + (size_t)(g * 16 + rl)) * n + i0) * 8;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int c = k * 16 + il, from = c >> 3;      // chunk c of the row: digit c % 8 of coefficient c / 8
            if (i0 + from < n) dst[base + c] = tr[rl * 128 + (c ^ (from >> 1))];
        }
    }
}

// sum_s 256^s * c[s] for 15 signed 32-bit diagonals, as an unsigned 128-bit value (the true sum is non-negative).
// Four diagonals at a time fit a signed 64-bit word (|e| < 2^56); the four words, 32 bits apart, are then added
// with 32-bit carries.
__device__ __forceinline__ u128 recombine(const int (&c)[15]) {
    // the multipliers are hidden from the optimiser so that each term is one 32x32+64 multiply-add instead of a
    // sign extension, a 64-bit shift and a 64-bit addition
    int m8 = 256, m16 = 65536, m24 = 16777216;
    asm volatile("" : "+s"(m8), "+s"(m16), "+s"(m24));
    i64 e[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        e[j] = (i64)c[4 * j] + (i64)c[4 * j + 1] * m8 + (i64)c[4 * j + 2] * m16;
        if (j < 3) e[j] += (i64)c[4 * j + 3] * m24;
    }
    i64 t = e[0];
    const u64 w0 = (uint32_t)t;
    t = (t >> 32) + e[1];
    const u64 w1 = (uint32_t)t;
    t = (t >> 32) + e[2];
    const u64 w2 = (uint32_t)t;
    t = (t >> 32) + e[3];
    const u64 w3 = (uint32_t)t;
    return ((u128)(w2 | (w3 << 32)) << 64) | (w0 | (w1 << 32));
}

// f(integral_constant k) for k = FROM .. TO - 1
template <int FROM, int TO, class F>
__device__ __forceinline__ void for_each(F f) {
    if constexpr (FROM < TO) {
        f(std::integral_constant<int, FROM>{});
        for_each<FROM + 1, TO>(f);
    }
}
// Moves 16 bytes a lane from base + offset (a byte offset of each lane) + AT to LDS, 1 KiB in the order of the lanes from
// to + AT on.  Nothing comes back to a register: what is in flight costs LDS only.  The caller waits with vmcnt, and reads
// what it waited for behind a barrier that also orders memory; the load itself may move among reads of other parts of LDS.
// m0 is the compiler's register too: it is named as overwritten (the product takes as long as without, 243.4 and 243.8 us).
template <bool ONCE, int AT>
__device__ __forceinline__ void load_to_lds(const v4i *base, u32 offset, u32 to) {
    if (ONCE)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3 nt" : : "s"(to), "v"(offset), "s"(base), "n"(AT) : "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3" : : "s"(to), "v"(offset), "s"(base), "n"(AT) : "m0");
}

// A task of the product: one coefficient, RT row tiles and CT column tiles.  groups = row groups x column groups.
// A workgroup's next task is `step` = coefficients groups + part further on its XCD.
struct MfmaTasks {
    u32 row_groups, groups, count, step_coefs, step_part;         // count = groups n
};

// A workgroup of RT x CT wavefronts, one 16x16 tile each, takes every gridDim.x-th task.  Its work is one sequence of stages, a
// stage being one term block of one coefficient: 8 KiB of digit planes for each row and column tile, moved straight into
// LDS STAGES - 1 stages ahead, through the ends of coefficients.
// No single part bounds it.  16x16x128 to 128 channels at batch 16, the launch alone 100 us: 91 without the loads, 90 without the
// products, 91 without the stores, as long without the recombination, 70 without loads and products, 86 without loads and stores.  Its
// 445 MB, at 4.4 TB/s of the 6.2 that a read reaches, mostly hide behind the rest; every stage ends with its slowest wavefront.  Sums of
// one term block are bound by their eight-byte stores: 256 to 256 channels 1x1 at 7x7, batch 16, 97 us, 71 without them.
// One workgroup for each coefficient, its loads in registers one block ahead and two workgroups a CU, spent half of its time on
// the first trip to memory and the last block's recombination: 16x16x128 to 128 channels at batch 16 254 us from wire to wire, 238 in
// stages (246 with one stage ahead instead of two; 257 with five stages of half a block ahead), 230 with the loads among the products
// and the next task found by two additions; at batch 3 162 -> 131, 13x11x24 to 40 channels at batch 5 73.5 -> 66.3, 22x29x154 to
// 21 at batch 6 276 -> 219.  Eight consecutive coefficients a workgroup lost the gain: the eight-byte pieces of an output
// line (BLK8) left the L2 one by one (285 us).
// Output: tmp[i][row][column] (rows and columns padded to tiles), transposed afterwards; or, BLK8, in blocks of
// eight coefficients tmp[i/8][row][column][i%8], which the Perm kernels read as they are (a thread's eight
// consecutive coefficients of c0 and of c1 are the two halves of one 128-byte line).
// ONCE: the row operand is past what the last-level cache holds and is loaded without being kept, which leaves the caches
// to the column operand and the sums: 16x16x128 to 128 channels at batch 16 291.5 -> 275.4 us, with a special prime 523.7 -> 515.6 us.
template <int RT, int CT, bool BLK8, bool FOLD, bool ONCE>
__global__ __launch_bounds__(64 * RT * CT, 2) void conv_mfma_kernel(const v4i *wl, const v4i *xl, u64 *tmp, int mtiles, int ntiles,
                                                                int kblocks, int nblk16, int n, MfmaTasks tasks, Modulus mod) {
    constexpr int STAGES = RT * CT == 8 ? 3 : 2, TILE = 8192, STAGE = (RT + CT) * TILE;
    constexpr int A_LOADS = 8 / CT, B_LOADS = 8 / RT, LOADS = A_LOADS + B_LOADS;       // of a wavefront and stage
    __shared__ __attribute__((aligned(16))) unsigned char lds[STAGES * STAGE];
    const u32 lds_at = (u32)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
    // the wavefront's number is the same in all its lanes: kept in a scalar register, with everything derived from it
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row_tile = wave / CT, col_tile = wave % CT;
    const int rem = nblk16 - 4 * (kblocks - 1);       // groups of 16 terms in the last term block

    // Consecutive workgroups go to the eight XCDs in turn.  An XCD takes every eighth block of eight coefficients, one after the
    // other with all of their groups: those read the same operands at the same time, and the coefficients of a
    // block fill the same lines of the output (BLK8) while its L2 holds them.
    const u32 spread = ((n >> 3) & 7) == 0 ? 8 : 1, xcd = blockIdx.x & (spread - 1);
    struct Task {
        u32 coef, group;        // number of the coefficient on the XCD, and group
    };
    auto coefficient = [&](const Task &t) { return (int)(((t.coef >> 3) * spread + xcd) * 8 + (t.coef & 7)); };
    auto step = [&](Task &t) {
        t.coef += tasks.step_coefs;
        t.group += tasks.step_part;
        if (t.group >= tasks.groups) {
            t.group -= tasks.groups;
            ++t.coef;
        }
    };
    // what a wavefront loads: digits of its row tile, and eighths of a column tile
    const int load_row = wave / CT, load_digit = wave % CT * A_LOADS, load_col = wave / RT, load_eighth = wave % RT * B_LOADS;
    // Lanes beyond the last term read the last group's chunks again: every stage is the same number of loads, and nothing
    // beyond the last term is read.
    const u32 a_lane = (u32)lane * 16u, a_last = (u32)((min(lane >> 4, rem - 1) << 4) + (lane & 15)) * 16u;
    // A column tile's chunks lie [lane][digit] in LDS, the digit xored with the lane's low bits: the eight digits of a
    // coefficient are one line of memory, and 8 lanes that read the same digit find it in all of the banks.
    u32 b_lane[B_LOADS], b_last[B_LOADS];
#pragma unroll
    for (int r = 0; r < B_LOADS; ++r) {
        const int eighth = load_eighth + r, from = min(eighth >> 1, rem - 1) * 2 + (eighth & 1);
        const u32 chunk = (u32)(lane >> 3) * (u32)n * 8u + (u32)((lane & 7) ^ (lane >> 3));
        b_lane[r] = (chunk + (u32)(eighth * 64 * n)) * 16u;
        b_last[r] = (chunk + (u32)(from * 64 * n)) * 16u;
    }
    const v4i zero = v4i{0, 0, 0, 0};
    v4i s[15];
    // D_(u+v) += W_u X_v for all digit pairs.  A last block of at most 32 terms puts two digit pairs of the same sum into the
    // 64 terms of an instruction, one of at most 16 terms four: 36 and 22 instructions instead of 64.
    // load(r), r < LOADS: the next stage's loads.  With eight wavefronts they are asked for between the products (SPREAD): all at the
    // start of a stage they held every wavefront up for 1070 clocks, 51 000 of a launch's 238 000.
    constexpr bool SPREAD = RT * CT == 8;
    auto multiply = [&](const unsigned char *A, const unsigned char *B, auto groups, bool partial, auto load) {
        constexpr int G = decltype(groups)::value, STEPS = 7 + G;
        const int g = lane / (64 / G), ln = lane % (64 / G);
        auto column = [&](int v) {
            const int digit = v - g;
            v4i bv = *reinterpret_cast<const v4i *>(B + ln * 128 + ((digit ^ ln) & 7) * 16);
            if (G > 1 && (v < G - 1 || v > 7) && (digit < 0 || digit > 7)) bv = zero;
            return bv;
        };
        if constexpr (!SPREAD) for_each<0, LOADS>(load);
        v4i av[8 / G], bv = column(0);
#pragma unroll
        for (int u = 0; u < 8 / G; ++u) {
            av[u] = *reinterpret_cast<const v4i *>(A + (u * G + g) * 1024 + ln * 16);
            if (G == 1 && partial && lane >= 48) av[u] = zero;
        }
        for_each<0, STEPS>([&](auto number) {
            constexpr int v = decltype(number)::value;
            const v4i next = column(v + 1 < STEPS ? v + 1 : v);
            if constexpr (SPREAD) for_each<v * LOADS / STEPS, (v + 1) * LOADS / STEPS>(load);
#pragma unroll
            for (int u = 0; u < 8 / G; ++u) s[u * G + v] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[u], bv, s[u * G + v], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            bv = next;
        });
    };

    const int mine = ((int)tasks.count - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x, total = mine * kblocks;
    const u32 place = blockIdx.x / spread;
    // the stage to load next and the stage at hand
    Task ahead{place / tasks.groups, place % tasks.groups}, now = ahead;
    int ahead_kb = 0, loaded = 0, kb = 0, i = 0, mt = 0, nt = 0;
    u32 to = lds_at, from = 0;
    const v4i *a_next, *b_next;        // this wavefront's chunks of the stage to load next
    auto start = [&] {
        const u32 ng = tasks.groups == tasks.row_groups ? 0 : ahead.group / tasks.row_groups, mg = ahead.group - ng * tasks.row_groups;
        const size_t row = (size_t)coefficient(ahead) * mtiles + min((int)mg * RT + load_row, mtiles - 1);
        a_next = wl + (row * kblocks * 8 + load_digit) * 64;
        b_next = xl + ((size_t)min((int)ng * CT + load_col, ntiles - 1) * kblocks * 64 * n + coefficient(ahead)) * 8;
    };
    start();
    // load r of this wavefront's of the next stage
    auto load_one = [&](auto number) {
        constexpr int r = decltype(number)::value;
        if (loaded >= total) return;
        const bool last = ahead_kb == kblocks - 1;
        if constexpr (r < A_LOADS)
            load_to_lds<ONCE, r % 4 * 1024>(a_next + r / 4 * 256, last ? a_last : a_lane,
                                            to + (u32)(load_row * TILE + (load_digit + r / 4 * 4) * 1024));
        else
            load_to_lds<false, 0>(b_next, last ? b_last[r - A_LOADS] : b_lane[r - A_LOADS],
                                  to + (u32)((RT + load_col) * TILE + (load_eighth + r - A_LOADS) * 1024));
    };
    auto loaded_all = [&] {
        if (loaded >= total) return;
        ++loaded;
        to = to + STAGE == lds_at + STAGES * STAGE ? lds_at : to + STAGE;
        if (++ahead_kb < kblocks) {
            a_next += 512;
            b_next += 512 * (size_t)n;
        } else {
            ahead_kb = 0;
            step(ahead);
            start();
        }
    };
#pragma unroll
    for (int k = 0; k < STAGES - 1; ++k) {
        for_each<0, LOADS>(load_one);
        loaded_all();
    }
    for (int stage = 0; stage < total; ++stage) {
        // this stage's loads are done, and everybody's products of the stage before: its buffer is the next one's
        if (STAGES == 3 && stage + 1 < total) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(LOADS) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : : : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" : : : "memory");
        if (kb == 0) {
            const u32 ng = tasks.groups == tasks.row_groups ? 0 : now.group / tasks.row_groups;
            i = coefficient(now);
            mt = (int)(now.group - ng * tasks.row_groups) * RT + row_tile;
            nt = (int)ng * CT + col_tile;
            step(now);
#pragma unroll
            for (int k = 0; k < 15; ++k) s[k] = zero;
        }
        const bool live = mt < mtiles && nt < ntiles;
        if (live) {
            const unsigned char *A = lds + from + row_tile * TILE, *B = lds + from + (RT + col_tile) * TILE;
            if (kb < kblocks - 1 || rem == 4) multiply(A, B, std::integral_constant<int, 1>{}, false, load_one);
            else if (rem == 3) multiply(A, B, std::integral_constant<int, 1>{}, true, load_one);
            else if (rem == 2) multiply(A, B, std::integral_constant<int, 2>{}, false, load_one);
            else multiply(A, B, std::integral_constant<int, 4>{}, false, load_one);
        } else {
            for_each<0, LOADS>(load_one);
        }
        loaded_all();
        from = from + STAGE == STAGES * STAGE ? 0 : from + STAGE;
        // The exact sum of K products of residues below 2^60 needs K * 2^120 < 2^128, and an int32 diagonal
        // 8 * K * 2^14 < 2^31: after every kFoldBlocks term blocks (192 terms) the sums so far are reduced mod q
        // and put back as three small non-negative diagonals (24 + 24 + 12 bits at 256^0, 256^3, 256^6), so sums
        // of any length stay exact.  Layers of at most 192 terms run the instantiation without this branch.
        if (FOLD && live && kb % kFoldBlocks == kFoldBlocks - 1 && kb + 1 < kblocks) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                int c[15];
#pragma unroll
                for (int k = 0; k < 15; ++k) c[k] = s[k][r];
                const u64 val = reduce128(recombine(c), mod);
#pragma unroll
                for (int k = 0; k < 15; ++k) s[k][r] = 0;
                s[0][r] = (int)(val & 0xffffff);
                s[3][r] = (int)((val >> 24) & 0xffffff);
                s[6][r] = (int)(val >> 48);
            }
        }
        if (++kb < kblocks) continue;
        kb = 0;
        if (!live) continue;
        // lane holds rows 4*(lane/16) + r, column lane%16 of the 16x16 output tile
        const size_t rowsP = (size_t)mtiles * 16, colsP = (size_t)ntiles * 16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int c[15];
#pragma unroll
            for (int k = 0; k < 15; ++k) c[k] = s[k][r];
            const u64 val = reduce128(recombine(c), mod);
            const int m = mt * 16 + 4 * (lane >> 4) + r, col = nt * 16 + (lane & 15);
            if (BLK8) tmp[(((size_t)(i >> 3) * rowsP + m) * colsP + col) * 8 + (i & 7)] = val;
            else tmp[((size_t)i * rowsP + m) * colsP + col] = val;
        }
    }
}

// acc[input][row][polynomial][i] = tmp[i][row][2*input + polynomial]: a tiled transpose through LDS
__global__ __launch_bounds__(256) void conv_untranspose_kernel(const u64 *tmp, u64 *acc, int rowsP, int colsP, int groups,
                                                               int cols, int n) {
    __shared__ u64 tile[32][33];
    const int i0 = blockIdx.x * 32, r0 = blockIdx.y * 32;       // r = row * colsP + column, flattened
    const size_t flat = (size_t)rowsP * colsP;
    for (int k = threadIdx.x; k < 32 * 32; k += 256) {
        const int di = k >> 5, dr = k & 31;
        if (i0 + di < n && (size_t)(r0 + dr) < flat) tile[di][dr] = tmp[(size_t)(i0 + di) * flat + r0 + dr];
    }
    __syncthreads();
    for (int k = threadIdx.x; k < 32 * 32; k += 256) {
        const int dr = k >> 5, di = k & 31;
        const int r = r0 + dr, row = r / colsP, col = r % colsP;
        if (i0 + di < n && row < groups && col < cols)
            acc[(((size_t)(col >> 1) * groups + row) * 2 + (col & 1)) * n + i0 + di] = tile[di][dr];
    }
}

}  // namespace

void conv_mfma_geometry(int groups, int cols, int nterm, int *mtiles, int *ntiles, int *kblocks) {
    *mtiles = (groups + 15) / 16;
    *ntiles = (cols + 15) / 16;
    *kblocks = (nterm + 63) / 64;
}
size_t conv_mfma_image_bytes(int n, int tiles, int kblocks) {
    return (size_t)n * tiles * kblocks * 8 * 64 * 16;
}
size_t conv_mfma_tmp_bytes(int n, int mtiles, int ntiles) { return (size_t)n * mtiles * 16 * ntiles * 16 * sizeof(u64); }
// mode 0: encoded kernels (rows = groups), mode 1: rotated inputs (rows = 2*batch columns)
int launch_limb_pack(const gala_ctx *c, void *stream, const u64 *src, int mode, int rows, int nterm, u64 *dst) {
    int tiles, unused, kblocks;
    conv_mfma_geometry(rows, rows, nterm, &tiles, &unused, &kblocks);
    const dim3 grid((unsigned)((c->n + 15) / 16), (unsigned)tiles, (unsigned)(kblocks * 4));
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, (hipStream_t)stream, src, rows, nterm, c->n, tiles, kblocks,
                           reinterpret_cast<v4i *>(dst));
    };
    if (mode) go(limb_pack_kernel<true>);
    else go(limb_pack_kernel<false>);
    return (int)hipGetLastError();
}
int launch_conv_mfma(const gala_ctx *c, void *stream, const u64 *wl, const u64 *xl, int batch, int groups, int nterm,
                     u64 *tmp, bool blocks_of_eight) {
    int mtiles, ntiles, kblocks;
    conv_mfma_geometry(groups, 2 * batch, nterm, &mtiles, &ntiles, &kblocks);
    const bool fold = kblocks > kFoldBlocks;
    auto go = [&](auto kernel, int row_tiles, int col_tiles, int slots) {
        const int row_groups = (mtiles + row_tiles - 1) / row_tiles, groups = row_groups * ((ntiles + col_tiles - 1) / col_tiles);
        const long count = (long)groups * c->n, grid = count < slots ? count : slots;
        const int step = (int)grid / (((c->n >> 3) & 7) == 0 ? 8 : 1);
        const MfmaTasks tasks{(u32)row_groups, (u32)groups, (u32)count, (u32)(step / groups), (u32)(step % groups)};
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * row_tiles * col_tiles), 0,
                           (hipStream_t)stream, reinterpret_cast<const v4i *>(wl), reinterpret_cast<const v4i *>(xl), tmp, mtiles, ntiles,
                           kblocks, (nterm + 15) / 16, c->n, tasks, c->dev_q.mod);
    };
    auto pick = [&](auto once, auto rows, auto cols) {
        constexpr bool ONCE = decltype(once)::value;
        constexpr int RT = decltype(rows)::value, CT = decltype(cols)::value;
        // as many workgroups as a CU's LDS holds: 144 KiB each, 64 to 80, or 48
        auto run = [&](auto kernel) { go(kernel, RT, CT, RT * CT == 8 ? 256 : RT * CT == 2 ? 768 : 512); };
        if (blocks_of_eight) fold ? run(conv_mfma_kernel<RT, CT, true, true, ONCE>) : run(conv_mfma_kernel<RT, CT, true, false, ONCE>);
        else fold ? run(conv_mfma_kernel<RT, CT, false, true, ONCE>) : run(conv_mfma_kernel<RT, CT, false, false, ONCE>);
    };
    // the chunks of the row operand that are read: none beyond the last term
    const size_t row_bytes = (size_t)c->n * mtiles * 16 * ((nterm + 15) / 16) * 16 * sizeof(u64);
    const bool once = streams_past_cache(row_bytes);
    std::integral_constant<int, 1> one;
    std::integral_constant<int, 2> two;
    std::integral_constant<int, 4> four;
    // Two row tiles a workgroup where there are no more of them: 40 channels 3x3 at 22x7 to 5, batch 16, 77.7 -> 71.5 us from wire to
    // wire, 16x16x128 to 32 at batch 16 119.1 -> 112.3, to 16 at batch 8 78.8 -> 75.9.  With four and eight row tiles four are
    // faster: 64 to 64 channels 1x1 at batch 16 94.7 us against 96.2, 128 to 128 3x3 237.7 against 254.8.
    if (mtiles <= 2 && ntiles == 1) once ? pick(std::true_type{}, two, one) : pick(std::false_type{}, two, one);
    else if (mtiles <= 2) once ? pick(std::true_type{}, two, two) : pick(std::false_type{}, two, two);
    else if (ntiles == 1) once ? pick(std::true_type{}, four, one) : pick(std::false_type{}, four, one);
    else once ? pick(std::true_type{}, four, two) : pick(std::false_type{}, four, two);
    return (int)hipGetLastError();
}
int launch_conv_untranspose(const gala_ctx *c, void *stream, const u64 *tmp, int batch, int groups, u64 *acc) {
    int mtiles, ntiles, kblocks;
    const int cols = 2 * batch;
    conv_mfma_geometry(groups, cols, 1, &mtiles, &ntiles, &kblocks);
    const int rowsP = mtiles * 16, colsP = ntiles * 16;
    const dim3 tgrid((unsigned)((c->n + 31) / 32), (unsigned)((rowsP * colsP + 31) / 32));
    hipLaunchKernelGGL(conv_untranspose_kernel, tgrid, dim3(256), 0, (hipStream_t)stream, tmp, acc, rowsP, colsP, groups,
                       cols, c->n);
    return (int)hipGetLastError();
}

}  // namespace gala
