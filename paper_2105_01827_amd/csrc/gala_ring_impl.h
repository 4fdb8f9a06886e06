// Kernels on the transforms of one ring size, n = 2^GALA_LOGN (1024 to 8192), for q < 2^60: Perm and its hoisted halves,
// share masks, import and export, the client's steps.  Included once per ring by gala_ring1024.hip ... gala_ring8192.hip,
// which define GALA_LOGN; the launchers leave through the RingOps table at the end.
//
// One workgroup of n / 8 threads (four wavefronts at n = 2048) owns one polynomial; every thread
// keeps 8 coefficients in registers and runs radix-8 passes (three butterfly
// stages each) on them, so a 2048-point transform is 3 + 3 + 3 + 2 stages with
// only three exchanges through LDS.  The LDS image is padded against bank conflicts (pad below), and two buffers
// alternate so that each exchange needs a single barrier.
//
// Index ownership of register k of thread t in a pass on bits B .. B+2 of the coefficient index: those three bits are
// k, the bits below are t's low B bits, the bits above the rest of t.
//   forward:  from the top bits down in threes; the last pass (what is left of the bits, one or two stages, none at
//             n = 4096) owns 8t + k          n = 2048: 8-10 | 5-7 | 2-4 | 0-1
//   inverse:  from bit 0 up in threes, the last pass owns t + (n/8) k      n = 2048: 0-2 | 3-5 | 6-8 | 9-10
// so the inverse transform of c1 ends exactly where the forward transforms of
// its digits begin, and the digits never leave registers.
//
// Butterflies are lazy: residues are signed 64-bit words (below), and a transform brings only a few values near the
// modulus on its way.
//
// Rings of 4096 slots on these kernels instead of the any-n ones: he_fc 500x1024 at batch 8 706 -> 130 us from wire to
// wire (there a lone workgroup per item also added the 256 partial sums one after the other).
#ifndef GALA_LOGN
#error "define GALA_LOGN before including this file"
#endif
#include <hip/hip_runtime.h>

#include <type_traits>

#include "gala_internal.h"

namespace gala {
namespace {

constexpr int LOGN = GALA_LOGN, N = 1 << LOGN, PER = 8, NT = N / PER;
// a wavefront's 64 threads own the same 512 consecutive indices in every pass on bits at or below this one
constexpr int LOCAL_BITS = 6;
// ... and an exchange between the passes on bits b_out and b_in up hands words from one wavefront to another
constexpr bool crosses(int b_out, int b_in) { return b_out > LOCAL_BITS || b_in > LOCAL_BITS; }

// Images of a polynomial in LDS.  A wavefront's range of 512 words has a stride of its own, 512 + 512 / 2^S words, and
// inside it an exchange pads by one word every 2^SHIFT, SHIFT >= S: ranges do not move with the padding, so wavefronts
// that are one exchange apart stay out of each other's way.  Measured clocks of a wavefront's eight-byte instruction on
// the gfx950 LDS (a free read takes 2.2, a write 6): SHIFT 5 write 6 and read 2.2 between passes on bits 5 and up, but 7.8
// and 15.6 write, 7.8 read in the patterns of bits 0, 2 and 3, where SHIFT 4 takes 6 to 7.9 and 4, SHIFT 3 6 and 2.2.  S is the
// best that a kernel's LDS has room for.
constexpr int stride_of(int S) { return 512 + (512 >> S); }
constexpr int lds_words(int S) { return N / 512 * stride_of(S); }
template <int S, int SHIFT = 5>
__device__ __forceinline__ constexpr int pad(int i) {
    // (i >> 9) stride + (i & 511) + ((i & 511) >> SHIFT)
    return i + (i >> SHIFT) + (SHIFT == S ? 0 : (i >> 9) * ((512 >> S) - (512 >> SHIFT)));
}
// images of 32-bit words
__device__ __forceinline__ int pad32(int i) { return i + (i >> 5); }
__device__ __forceinline__ int bitrev(int v) { return (int)(__brev((unsigned)v) >> (32 - LOGN)); }
__device__ __forceinline__ int galois_index(int i, int gal) {
    const int e = ((2 * bitrev(i) + 1) * gal) & (2 * N - 1);
    return bitrev((e - 1) >> 1);
}
// index of register 0 of thread t in the pass on bits B .. B+2
template <int B>
__device__ __forceinline__ int owner(int t) {
    return ((t >> B) << (B + 3)) | (t & ((1 << B) - 1));
}

// ---- 64-bit modular primitives shaped for the gfx950 VALU ---------------------------------------
// Residues are signed 64-bit words v, |v| < 2^63, that stand for v mod m; a bound of c below means |v| <= c 2^60.
// 32x32+64-bit multiply-adds issue at the full rate of the vector ALU, so the cost of a product is their number.  A
// product by a constant w is a Montgomery product: with y = y1 2^32 + y0, both words signed, and the MontPair
// (A, B) = (w 2^32, w 2^64) mod m, also in signed words,
//     L = y0 A0 + y1 B0,   H = y0 A1 + y1 B1,   k = L m^-1 mod 2^32 (signed),   w y = H + (L - k m0) / 2^32 - k m1   (mod m)
// Nothing needs a quotient of its own: seven multiply-adds and one 32-bit product, against thirteen instructions with a
// precomputed quotient, and the constants take the same 16 bytes.  x + w y costs no more: x is the addend of H.
// |w y| <= (y0 A + y1 B - k m) / 2^32 in absolute values <= (0.75 + c/32) m for |y| <= c 2^60: tight enough that a
// transform corrects a few values once.
// The words of y have to be signed: y1 is the high word of y + 2^31.  Transforms therefore run on biased values,
// v + 2^31 in place of v: the high word is then y1 and the low one, its top bit flipped, y0.  A butterfly hands the bias of
// its x on to both results.
// L - k m0 must fit 64 bits: |y0 A0| + |k m0| + |y1 B0| <= 2^62 + 2^31 |m0| + 2^31 |y1|.  With |m0| <= 2^28 that holds up
// to |y| <= 7 2^60 (WIDE = false).  Otherwise the high words of L and k m0 are added one by one, for one multiply-add
// more, and |y| only has to stay below 2^63 - 2^31 (WIDE = true).
// Measured alone (registers only, three wavefronts per SIMD): 1.27 times the butterflies of the form with precomputed
// quotients a second, 1.18 times with WIDE.  From wire to wire: he_fc 128x1024 at batch 64 159 -> 150 us, 500x1024 at n = 4096
// (WIDE), batch 8, 128 -> 114 us, 100x784 at batch 7 with the special prime 74 -> 67 us, the 16x16x128 convolution at batch 16
// 288 -> 269 us.
constexpr u64 BIAS = 0x80000000ull;
struct MontQ {
    u32 inv;              // m^-1 mod 2^32
    int nlo, nhi, lo;     // the signed words of -m, and the low one of m
};
struct Words { u32 lo, hi; };     // y0, y1
__device__ __forceinline__ Words biased_words(u64 y) { return {(u32)y ^ (u32)BIAS, (u32)(y >> 32)}; }
__device__ __forceinline__ Words plain_words(u64 y) { return {(u32)y, (u32)((y + BIAS) >> 32)}; }
// The instructions of a product are written in blocks: the compiler keeps a wait state between an inline-asm statement and
// the next one that reads its result, inside a block there is none.  A block ends where the next step needs one half
// of a 64-bit result (halves cannot be named inside a block).
template <bool WIDE>
__device__ __forceinline__ u64 mont_reduce(u64 L, u64 H, const MontQ &q) {
    int k;
    if (WIDE) {
        asm("v_mul_lo_u32 %1, %2, %3\n\t"
            "v_mad_i64_i32 %0, vcc, %1, %4, %0\n\t"
            "v_mul_hi_i32 %1, %1, %5\n\t"
            "v_mad_i64_i32 %0, vcc, %6, 1, %0\n\t"
            "v_mad_i64_i32 %0, vcc, %1, -1, %0"
            : "+v"(H), "=&v"(k)
            : "v"((u32)L), "s"(q.inv), "s"(q.nhi), "s"(q.lo), "v"((u32)(L >> 32))
            : "vcc");
    } else {
        asm("v_mul_lo_u32 %2, %3, %4\n\t"
            "v_mad_i64_i32 %0, vcc, %2, %5, %0\n\t"
            "v_mad_i64_i32 %1, vcc, %2, %6, %1"
            : "+v"(L), "+v"(H), "=&v"(k)
            : "v"((u32)L), "s"(q.inv), "s"(q.nlo), "s"(q.nhi)
            : "vcc");
        asm("v_mad_i64_i32 %0, vcc, %1, 1, %0" : "+v"(H) : "v"((u32)(L >> 32)) : "vcc");
    }
    return H;
}
template <bool WIDE>
__device__ __forceinline__ void mont_reduce2(u64 &L, u64 &H, u64 &M, u64 &I, const MontQ &q) {
    int k, l;
    if (WIDE) {
        asm("v_mul_lo_u32 %2, %4, %8\n\t"
            "v_mul_lo_u32 %3, %5, %8\n\t"
            "v_mad_i64_i32 %0, vcc, %2, %9, %0\n\t"
            "v_mad_i64_i32 %1, vcc, %3, %9, %1\n\t"
            "v_mul_hi_i32 %2, %2, %10\n\t"
            "v_mul_hi_i32 %3, %3, %10\n\t"
            "v_mad_i64_i32 %0, vcc, %6, 1, %0\n\t"
            "v_mad_i64_i32 %1, vcc, %7, 1, %1\n\t"
            "v_mad_i64_i32 %0, vcc, %2, -1, %0\n\t"
            "v_mad_i64_i32 %1, vcc, %3, -1, %1"
            : "+v"(H), "+v"(I), "=&v"(k), "=&v"(l)
            : "v"((u32)L), "v"((u32)M), "v"((u32)(L >> 32)), "v"((u32)(M >> 32)), "s"(q.inv), "s"(q.nhi), "s"(q.lo)
            : "vcc");
    } else {
        asm("v_mul_lo_u32 %4, %6, %8\n\t"
            "v_mul_lo_u32 %5, %7, %8\n\t"
            "v_mad_i64_i32 %0, vcc, %4, %9, %0\n\t"
            "v_mad_i64_i32 %2, vcc, %5, %9, %2\n\t"
            "v_mad_i64_i32 %1, vcc, %4, %10, %1\n\t"
            "v_mad_i64_i32 %3, vcc, %5, %10, %3"
            : "+v"(L), "+v"(H), "+v"(M), "+v"(I), "=&v"(k), "=&v"(l)
            : "v"((u32)L), "v"((u32)M), "s"(q.inv), "s"(q.nlo), "s"(q.nhi)
            : "vcc");
        asm("v_mad_i64_i32 %0, vcc, %2, 1, %0\n\t"
            "v_mad_i64_i32 %1, vcc, %3, 1, %1"
            : "+v"(H), "+v"(I)
            : "v"((u32)(L >> 32)), "v"((u32)(M >> 32))
            : "vcc");
    }
}
// w y, or x + w y.  UNIFORM: the constant is the same for all lanes and sits in scalar registers.
template <bool WIDE, bool ADD = false, bool UNIFORM = false>
__device__ __forceinline__ u64 mont(Words y, const ulonglong2 w, const MontQ &q, u64 x = 0) {
    const u32 a0 = (u32)w.x, a1 = (u32)(w.x >> 32), b0 = (u32)w.y, b1 = (u32)(w.y >> 32);
    u64 L, H;
#define GALA_MONT(X, WHERE, ...)                                                                                       \
    asm("v_mad_i64_i32 %0, vcc, %2, %4, 0\n\t"                                                                       \
        "v_mad_i64_i32 %1, vcc, %2, %5, " X "\n\t"                                                                    \
        "v_mad_i64_i32 %0, vcc, %3, %6, %0\n\t"                                                                       \
        "v_mad_i64_i32 %1, vcc, %3, %7, %1"                                                                           \
        : "=&v"(L), "=&v"(H)                                                                                          \
        : "v"(y.lo), "v"(y.hi), WHERE(a0), WHERE(a1), WHERE(b0), WHERE(b1) __VA_ARGS__                                \
        : "vcc")
    if (UNIFORM) {
        if (ADD) GALA_MONT("%8", "s", , "v"(x));
        else GALA_MONT("0", "s");
    } else {
        if (ADD) GALA_MONT("%8", "v", , "v"(x));
        else GALA_MONT("0", "v");
    }
#undef GALA_MONT
    return mont_reduce<WIDE>(L, H, q);
}
// Two products at once, xa + wa ya and xb + wb yb, their instructions in turn: a wavefront alone on its SIMD issues a
// multiply-add every other slot only and waits for each result, so what it finds to do in between counts.  Butterflies of
// one wavefront per SIMD 1.15 times as fast as one by one, of two 1.03 times, of three the same.
// KIND: products alone, added to xa and xb, or added to what ra and rb hold (running sums, nobody needs them afterwards).
enum Addend { NONE, ADD, IN_PLACE };
template <bool WIDE, bool UNIFORM = false, Addend KIND = ADD>
__device__ __forceinline__ void mont2(u64 &ra, u64 &rb, Words ya, const ulonglong2 wa, Words yb, const ulonglong2 wb, const MontQ &q,
                                      u64 xa = 0, u64 xb = 0) {
    u64 L, H, M, I;
#define GALA_MONT2(WHERE, OUT, XA, XB, ...)                                                                           \
    asm("v_mad_i64_i32 %0, vcc, %4, %8, 0\n\t"                                                                       \
        "v_mad_i64_i32 %2, vcc, %6, %12, 0\n\t"                                                                      \
        "v_mad_i64_i32 %1, vcc, %4, %9, " XA "\n\t"                                                                  \
        "v_mad_i64_i32 %3, vcc, %6, %13, " XB "\n\t"                                                                 \
        "v_mad_i64_i32 %0, vcc, %5, %10, %0\n\t"                                                                     \
        "v_mad_i64_i32 %2, vcc, %7, %14, %2\n\t"                                                                     \
        "v_mad_i64_i32 %1, vcc, %5, %11, %1\n\t"                                                                     \
        "v_mad_i64_i32 %3, vcc, %7, %15, %3"                                                                          \
        : "=&v"(L), OUT(H), "=&v"(M), OUT(I)                                                                          \
        : "v"(ya.lo), "v"(ya.hi), "v"(yb.lo), "v"(yb.hi), WHERE((u32)wa.x), WHERE((u32)(wa.x >> 32)), WHERE((u32)wa.y), \
          WHERE((u32)(wa.y >> 32)), WHERE((u32)wb.x), WHERE((u32)(wb.x >> 32)), WHERE((u32)wb.y),                     \
          WHERE((u32)(wb.y >> 32)) __VA_ARGS__                                                                        \
        : "vcc")
    if (KIND == IN_PLACE) {        // the first operands are tied to their outputs: %4 to %15 are still the inputs
        H = ra;
        I = rb;
        GALA_MONT2("v", "+&v", "%1", "%3");
    } else if (UNIFORM) {
        if (KIND == ADD) GALA_MONT2("s", "=&v", "%16", "%17", , "v"(xa), "v"(xb));
        else GALA_MONT2("s", "=&v", "0", "0");
    } else {
        if (KIND == ADD) GALA_MONT2("v", "=&v", "%16", "%17", , "v"(xa), "v"(xb));
        else GALA_MONT2("v", "=&v", "0", "0");
    }
#undef GALA_MONT2
    mont_reduce2<WIDE>(L, H, M, I, q);
    ra = H;
    rb = I;
}
// x + w y for 0 <= y < 2^31 (a gadget digit, not biased), w in scalar registers: half of the products have nothing to do
template <bool WIDE>
__device__ __forceinline__ u64 mont_small(u32 y, const ulonglong2 w, const MontQ &q, u64 x) {
    u64 L, H;
    asm("v_mad_i64_i32 %0, vcc, %2, %3, 0\n\t"
        "v_mad_i64_i32 %1, vcc, %2, %4, %5"
        : "=&v"(L), "=&v"(H)
        : "v"(y), "s"((u32)w.x), "s"((u32)(w.x >> 32)), "v"(x)
        : "vcc");
    return mont_reduce<WIDE>(L, H, q);
}
// x - h m with h = floor(x / 2^60), biased or not: at most 1 + h (1 - m / 2^60), so never above 3 for |x| <= 8 m and close
// to 1 when m is close to 2^60
__device__ __forceinline__ u64 shrink(u64 x, const MontQ &q) {
    const int h = (int)(x >> 32) >> 28;
    u64 r;
    asm("v_mad_i64_i32 %0, vcc, %1, %2, %3" : "=v"(r) : "v"(h), "s"(q.nlo), "v"(x) : "vcc");
    return r + ((u64)((u32)h * (u32)q.nhi) << 32);
}
// a product, in (-m, m), to [0, m)
__device__ __forceinline__ u64 unsign(u64 r, u64 m) { return r + ((u64)((i64)r >> 63) & m); }
// x - c if x >= c else x, in 4 instructions (the borrow of the subtraction selects);
// needs x - c < 2^63 when x >= c, which holds for every use here (x < 2c, c < 2^61).
__device__ __forceinline__ u64 csub_dev(u64 x, u64 c) {
    u32 r0, r1;
    asm("v_sub_co_u32 %0, vcc, %2, %4\n\tv_subb_co_u32 %1, vcc, %3, %5, vcc\n\t"
        "v_cndmask_b32 %0, %0, %2, vcc\n\tv_cndmask_b32 %1, %1, %3, vcc"
        : "=&v"(r0), "=&v"(r1)
        : "v"((u32)x), "v"((u32)(x >> 32)), "v"((u32)c), "v"((u32)(c >> 32))
        : "vcc");
    return ((u64)r1 << 32) | r0;
}

// x, y -> x + w y, x - w y without any correction; the bound grows by 0.75 + c/32, c the bound of y.  Both biased.
template <bool WIDE, bool UNIFORM = false>
__device__ __forceinline__ void bf2(u64 &xa, u64 &ya, const ulonglong2 wa, u64 &xb, u64 &yb, const ulonglong2 wb, const MontQ &q) {
    u64 sa, sb;
    mont2<WIDE, UNIFORM>(sa, sb, biased_words(ya), wa, biased_words(yb), wb, q, xa, xb);
    ya = (xa << 1) - sa;
    xa = sa;
    yb = (xb << 1) - sb;
    xb = sb;
}
// y not biased, the constant in scalar registers
template <bool WIDE>
__device__ __forceinline__ void bf_plain(u64 &x, u64 &y, const ulonglong2 w, const MontQ &q) {
    const u64 s = mont<WIDE, true, true>(plain_words(y), w, q, x);
    y = (x << 1) - s;
    x = s;
}
// the butterfly whose constant is one; y not biased
__device__ __forceinline__ void bf_one(u64 &x, u64 &y) {
    const u64 s = x + y;
    y = x - y;
    x = s;
}

// The seven constants one thread needs for a radix-8 pass on index bits B..B+2 are tw[T], tw[2T], tw[2T+1],
// tw[4T..4T+3] of the natural table order, with T = (n >> (B+3)) + (index >> (B+3)): "block" T.  A pass uses the
// blocks c .. 2c-1 of one level c = n >> (B+3) (1, 8, 64, 256 at n = 2048).  The table is stored level by
// level with the constant's number before the block's: level c is [e][j] = constant e of block c + j.  Constant e
// of the 64 lanes of a wavefront is then 16 to 1024 contiguous bytes; stored block by block (128 bytes per block)
// the same load touched up to 64 different lines, and the twiddles were two thirds of all the lines the Perm
// kernel asked its vector cache for.
//
// Radix-8 forward pass on the three index bits held in the register number (bit 2 of k first).
// STAGE > 0 skips the first stage or two (the last pass of a transform has what is left of the bits).
// The seven constants of a pass are fetched with tw_level() BEFORE the exchange that precedes the pass: a load
// cannot move across the exchange's barrier, and issued after it its latency is fully exposed, pass after pass.
struct Tw7 {
    ulonglong2 t[7];
};
// offset, in pairs, of level c inside the forward table (levels 1, 8, 64, (512,) n/8 in this order, each once)
__host__ __device__ constexpr int level_offset(int c) {
    int at = 0;
    for (int l = 1; l < c; l *= 8) at += 7 * l;
    return at;
}
constexpr int FWD_PAIRS = level_offset(N / 8) + 7 * (N / 8);
// The first pass has one block: its constants are the same for all lanes and come through the scalar cache.  The vector
// cache hands a CU 64 bytes a clock, 16 clocks for a wavefront's load of a constant whether its lanes differ or not, and that
// is what the Perm kernel runs into next to the vector ALU; scalar loads and LDS reads (4 clocks) do not count there.
__device__ __forceinline__ Tw7 tw_first(const ulonglong2 *table) {
    typedef __attribute__((address_space(4))) const u64 scalar_u64;
    asm volatile("" : "+s"(table));        // loaded where it is used, not once for the whole kernel
    scalar_u64 *p = (scalar_u64 *)reinterpret_cast<uintptr_t>(table);
    Tw7 w;
#pragma unroll
    for (int e = 0; e < 7; ++e) w.t[e] = make_ulonglong2(p[2 * e], p[2 * e + 1]);
    return w;
}
// Loads above this line stay above it: constants are requested a whole pass before their use, from the L2 as a rule, and
// the compiler would sink the requests to where they are needed.
__device__ __forceinline__ void pin_loads() { __builtin_amdgcn_sched_barrier(0x387); }
// constants of block COUNT + j: the level's start is uniform, j*16 a 32-bit offset
template <int COUNT>
__device__ __forceinline__ Tw7 tw_level(const ulonglong2 *__restrict__ table, unsigned j) {
    const char *level = reinterpret_cast<const char *>(table + level_offset(COUNT));
    const unsigned off = j * 16u;
    Tw7 w;
#pragma unroll
    for (int e = 0; e < 7; ++e) w.t[e] = *reinterpret_cast<const ulonglong2 *>(level + (size_t)(e * COUNT * 16) + off);
    return w;
}
// STAGE: the first of the three stages to run.  CORRECT: the values that the first stage does not multiply are shrunk.
template <bool WIDE, int STAGE, bool CORRECT = false, bool UNIFORM = false>
__device__ __forceinline__ void fwd_pass(u64 (&a)[8], const Tw7 &w, const MontQ &q) {
    if (CORRECT) {
#pragma unroll
        for (int k = 0; k < 4; ++k) a[k] = shrink(a[k], q);
    }
    if (STAGE == 0) {
        bf2<WIDE, UNIFORM>(a[0], a[4], w.t[0], a[1], a[5], w.t[0], q);
        bf2<WIDE, UNIFORM>(a[2], a[6], w.t[0], a[3], a[7], w.t[0], q);
    }
    if (STAGE <= 1) {
        bf2<WIDE, UNIFORM>(a[0], a[2], w.t[1], a[1], a[3], w.t[1], q);
        bf2<WIDE, UNIFORM>(a[4], a[6], w.t[2], a[5], a[7], w.t[2], q);
    }
    bf2<WIDE, UNIFORM>(a[0], a[1], w.t[3], a[2], a[3], w.t[4], q);
    bf2<WIDE, UNIFORM>(a[4], a[5], w.t[5], a[6], a[7], w.t[6], q);
}
// The first pass on eight gadget digits x_0 .. x_7, not biased; a biased.  Digits are short, so products of several of them by
// constants add up in the words of one product and are reduced together: three of stages 1 and 2 for x_0, x_2, x_4, x_6, and what stage 3
// adds to and takes from those, sums of four products of x_1, x_3, x_5, x_7 each.  91 instructions instead of 144, or 132 with
// a first stage of small factors.  Constants (see digit_pass_constants): words w 2^32 mod m alone, the other half of a pair has nothing to
// multiply.  Bounds with digits of 30 bits: 0.63 | 1.4 | 2.4; of 31, taken where the low words leave room: 0.75 | 1.75 | 3.25.
// A launch of the Perm kernel has 3.5 % fewer instructions, the byte offsets of its gathers included.  From wire to wire he_fc 1000x2048 at batch 64
// 1711 -> 1676 us, 128x1024 135.2 -> 133.1, the 16x16x128 convolution at batch 16 245.0 -> 241.9: 1 to 2 %, within what runs timed
// in turn differ by.  The byte offsets alone 1670 -> 1664, 131.9 -> 131.3 and 235.7 -> 235.0, 500x1024 at n = 4096 90.0 -> 90.6: nothing.
template <bool WIDE>
__device__ __forceinline__ void digit_pass(u64 (&a)[8], const u32 (&x)[8], const u64 *constants, const MontQ &q) {
    typedef __attribute__((address_space(4))) const u64 scalar_u64;
    asm volatile("" : "+s"(constants));        // loaded where it is used, as in tw_first
    scalar_u64 *c = (scalar_u64 *)reinterpret_cast<uintptr_t>(constants);
#define GALA_WORDS(C) "s"((u32)(C)), "s"((u32)((C) >> 32))
    const u64 x0 = (u64)x[0] + BIAS;
    u64 e0 = mont_small<WIDE>(x[4], make_ulonglong2(c[0], 0), q, x0), e1 = (x0 << 1) - e0;
    u64 L, H, M, I;
    asm("v_mad_i64_i32 %0, vcc, %4, %6, 0\n\t"
        "v_mad_i64_i32 %2, vcc, %4, %8, 0\n\t"
        "v_mad_i64_i32 %1, vcc, %4, %7, 0\n\t"
        "v_mad_i64_i32 %3, vcc, %4, %9, 0\n\t"
        "v_mad_i64_i32 %0, vcc, %5, %10, %0\n\t"
        "v_mad_i64_i32 %2, vcc, %5, %12, %2\n\t"
        "v_mad_i64_i32 %1, vcc, %5, %11, %1\n\t"
        "v_mad_i64_i32 %3, vcc, %5, %13, %3"
        : "=&v"(L), "=&v"(H), "=&v"(M), "=&v"(I)
        : "v"(x[2]), "v"(x[6]), GALA_WORDS(c[1]), GALA_WORDS(c[2]), GALA_WORDS(c[3]), GALA_WORDS(c[4])
        : "vcc");
    mont_reduce2<WIDE>(L, H, M, I, q);
    const u64 p[4] = {e0 + H, e0 - H, e1 + I, e1 - I};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        scalar_u64 *d = c + 6 + 8 * h;
        asm("v_mad_i64_i32 %0, vcc, %4, %8, 0\n\t"
            "v_mad_i64_i32 %2, vcc, %4, %10, 0\n\t"
            "v_mad_i64_i32 %1, vcc, %4, %9, 0\n\t"
            "v_mad_i64_i32 %3, vcc, %4, %11, 0\n\t"
            "v_mad_i64_i32 %0, vcc, %5, %12, %0\n\t"
            "v_mad_i64_i32 %2, vcc, %5, %14, %2\n\t"
            "v_mad_i64_i32 %1, vcc, %5, %13, %1\n\t"
            "v_mad_i64_i32 %3, vcc, %5, %15, %3\n\t"
            "v_mad_i64_i32 %0, vcc, %6, %16, %0\n\t"
            "v_mad_i64_i32 %2, vcc, %6, %18, %2\n\t"
            "v_mad_i64_i32 %1, vcc, %6, %17, %1\n\t"
            "v_mad_i64_i32 %3, vcc, %6, %19, %3\n\t"
            "v_mad_i64_i32 %0, vcc, %7, %20, %0\n\t"
            "v_mad_i64_i32 %2, vcc, %7, %22, %2\n\t"
            "v_mad_i64_i32 %1, vcc, %7, %21, %1\n\t"
            "v_mad_i64_i32 %3, vcc, %7, %23, %3"
            : "=&v"(L), "=&v"(H), "=&v"(M), "=&v"(I)
            : "v"(x[1]), "v"(x[5]), "v"(x[3]), "v"(x[7]), GALA_WORDS(d[0]), GALA_WORDS(d[1]), GALA_WORDS(d[2]), GALA_WORDS(d[3]),
              GALA_WORDS(d[4]), GALA_WORDS(d[5]), GALA_WORDS(d[6]), GALA_WORDS(d[7])
            : "vcc");
        mont_reduce2<WIDE>(L, H, M, I, q);
        a[4 * h] = p[2 * h] + H;
        a[4 * h + 1] = p[2 * h] - H;
        a[4 * h + 2] = p[2 * h + 1] + I;
        a[4 * h + 3] = p[2 * h + 1] - I;
    }
#undef GALA_WORDS
}
// Inverse transform.  The values sit in bit-reversed order, which is what a decimation-in-time transform starts from:
// it evaluates the plain cyclic sum over the powers of psi^-2, and a multiplication of coefficient j by psi^-j / n at
// the end makes it negacyclic (the separate scaling by 1/n costs as many products).  Against the usual inverse, whose
// butterflies (x + y, (x - y) w) carry psi inside: the sum rides on the product, seven of the first pass's twelve
// constants are one, and only four values need shrinking after the first pass and four before the third.
//
// First pass, bits 0-2: the constants are 1, i, w8 and w8^3 with w8 = psi^(-2n/8), i = w8^2.  Not biased on entry, |a| < m
// (eight of them add up to less than 2^63, with no room for a bias), biased on return.
template <bool WIDE>
__device__ __forceinline__ void inv_first_pass(u64 (&a)[8], const ulonglong2 (&w8)[3], const MontQ &q) {
    bf_one(a[0], a[1]);
    bf_one(a[2], a[3]);
    bf_one(a[4], a[5]);
    bf_one(a[6], a[7]);                              // 2
    bf_one(a[0], a[2]);
    bf_one(a[4], a[6]);                              // 4
    a[1] += BIAS;
    a[2] += BIAS;
    bf_plain<WIDE>(a[1], a[3], w8[1], q);
    bf_plain<WIDE>(a[5], a[7], w8[1], q);            // 2.9
    bf_one(a[0], a[4]);                              // 8
    bf_plain<WIDE>(a[1], a[5], w8[0], q);            // 3.7
    bf_plain<WIDE>(a[2], a[6], w8[1], q);            // 4.9
    bf_plain<WIDE>(a[3], a[7], w8[2], q);            // 3.7
#pragma unroll
    for (int k = 0; k < 8; k += 2) a[k] = shrink(a[k], q);
    a[0] += BIAS;
    a[4] += BIAS;
}
// Radix-8 pass on bits B .. B+2 held in the register number (bit 0 first).  A stage of half-length t multiplies by
// psi^(-2j n / 2t), j the index modulo t: one constant for bit B, two for B+1, four for B+2, of the thread's low bits.
// CORRECT: the values that the first stage only adds are shrunk.
template <bool WIDE, bool CORRECT>
__device__ __forceinline__ void inv_pass(u64 (&a)[8], const Tw7 &w, const MontQ &q) {
    if (CORRECT) {
#pragma unroll
        for (int k = 0; k < 8; k += 2) a[k] = shrink(a[k], q);
    }
    bf2<WIDE>(a[0], a[1], w.t[0], a[2], a[3], w.t[0], q);
    bf2<WIDE>(a[4], a[5], w.t[0], a[6], a[7], w.t[0], q);
    bf2<WIDE>(a[0], a[2], w.t[1], a[1], a[3], w.t[2], q);
    bf2<WIDE>(a[4], a[6], w.t[1], a[5], a[7], w.t[2], q);
    bf2<WIDE>(a[0], a[4], w.t[3], a[1], a[5], w.t[4], q);
    bf2<WIDE>(a[2], a[6], w.t[5], a[3], a[7], w.t[6], q);
}
// The inverse table: bits 3-5 as [7][8], bits 6-8 as [7][64], from n = 4096 on bits 9-11 as [7][512], the last pass's one
// or two stages as [4] or [6][n/8] (constant, low bits of the index), then psi^-j / n for j = 0 .. n-1.
constexpr int TOP_STAGES = LOGN % 3, TOP_CONSTS = TOP_STAGES == 2 ? 6 : 4;
constexpr int INV_MID = 7 * 8, INV_HIGH = INV_MID + 7 * 64, INV_TOP = INV_HIGH + (LOGN >= 12 ? 7 * 512 : 0),
              INV_TWIST = INV_TOP + (TOP_STAGES ? TOP_CONSTS * NT : 0);
template <int CONSTANTS, int COUNT>
__device__ __forceinline__ void inv_level(ulonglong2 (&t)[CONSTANTS], const ulonglong2 *__restrict__ level, unsigned j) {
    const char *base = reinterpret_cast<const char *>(level);
    const unsigned off = j * 16u;
#pragma unroll
    for (int e = 0; e < CONSTANTS; ++e) t[e] = *reinterpret_cast<const ulonglong2 *>(base + (size_t)(e * COUNT * 16) + off);
}

// Exchange between the pass on bits B_OUT .. B_OUT+2 and the one on B_IN .. B_IN+2: store, barrier, load.  The owned
// indices have zeros in the three bits the register number fills, so the padded address of
// register k is pad(owner) plus a compile-time offset.
template <int S, int SHIFT, int B>
__device__ __forceinline__ constexpr int reg_offset(int k) { return pad<S, SHIFT>(k << B); }
// Where every word a thread loads was stored by a thread of its own wavefront (both index sets lie in the
// wavefront's 512-word range of the buffer), a wavefront's LDS instructions execute in order, so its loads see
// its stores without a workgroup barrier; the fences only keep the compiler from moving the loads up.  At n = 2048
// four of the seven exchanges of an inverse + forward transform pair are of this kind; <8,5>, <6,8> and the final
// store of the forward transform cross wavefronts and keep the barrier.  BARRIER: one for the sake of what came before.
template <int S, int B_OUT, int B_IN, bool BARRIER = false>
__device__ __forceinline__ void exchange(u64 (&a)[8], u64 *buf, int tid) {
    constexpr int SHIFT = B_OUT < 5 || B_IN < 5 ? S : 5;
    u64 *po = buf + pad<S, SHIFT>(owner<B_OUT>(tid));
#pragma unroll
    for (int k = 0; k < 8; ++k) po[reg_offset<S, SHIFT, B_OUT>(k)] = a[k];
    if (!crosses(B_OUT, B_IN) && !BARRIER) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
    const u64 *pi = buf + pad<S, SHIFT>(owner<B_IN>(tid));
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] = pi[reg_offset<S, SHIFT, B_IN>(k)];
}

struct RingTables {
    const ulonglong2 *tw, *itw;   // MontPairs, forward (see tw_level) and inverse (see inv_level)
    const u64 *digits;            // constants of digit_pass; null: its sums might not fit their words
    ulonglong2 w8[3];             // w8, w8^2, w8^3 of the inverse transform's first pass
    ulonglong2 one;               // the constant 1
    Modulus mod;
    MontQ mont;
};
// |y| < 8 m (7 unless WIDE) -> [0, m)
template <bool WIDE>
__device__ __forceinline__ u64 canonical(Words y, const RingTables &T) {
    return unsign(mont<WIDE, false, true>(y, T.one, T.mont), T.mod.q);
}
template <bool WIDE>
__device__ __forceinline__ void canonical2(u64 &ra, u64 &rb, Words ya, Words yb, const RingTables &T) {
    mont2<WIDE, true, NONE>(ra, rb, ya, T.one, yb, T.one, T.mont);
    ra = unsign(ra, T.mod.q);
    rb = unsign(rb, T.mod.q);
}

// The thread id goes through an empty asm so that the address arithmetic of a transform is redone
// where it is used instead of being hoisted out of the rotation loop into long-lived registers.
__device__ __forceinline__ int fresh(int tid) {
    asm volatile("" : "+v"(tid));
    return tid;
}

// The twiddle levels that few lanes tell apart, copied to LDS by kernels that run many transforms: the forward transform's
// level of 8 blocks and the inverse's bits 3-5 (896 bytes each), LEVELS = 2 also the level of 64 and bits 6-8 (7 KiB each).
struct NoCopy {
    static constexpr int LEVELS = 0;
    const ulonglong2 *f8 = nullptr, *i8 = nullptr, *f64 = nullptr, *i64 = nullptr;
    template <int COUNT>
    __device__ __forceinline__ Tw7 get(const ulonglong2 *, unsigned) const { return Tw7{}; }
};
template <int L>
struct TableCopy {
    static constexpr int LEVELS = L, PAIRS = L == 2 ? 14 * 72 : 14 * 8;
    ulonglong2 *f8, *i8, *f64, *i64;
    __device__ __forceinline__ TableCopy(ulonglong2 *at) : f8(at), i8(at + 56), f64(at + 112), i64(at + 112 + 7 * 64) {}
    // a barrier has to follow
    __device__ __forceinline__ void fill(const RingTables &T, int tid) {
        for (int k = tid; k < 56; k += NT) {
            f8[k] = T.tw[level_offset(8) + k];
            i8[k] = T.itw[k];
        }
        if (L < 2) return;
        for (int k = tid; k < 7 * 64; k += NT) {
            f64[k] = T.tw[level_offset(64) + k];
            i64[k] = T.itw[INV_MID + k];
        }
    }
    template <int COUNT>
    __device__ __forceinline__ Tw7 get(const ulonglong2 *level, unsigned j) const {
        Tw7 w;
#pragma unroll
        for (int e = 0; e < 7; ++e) w.t[e] = level[e * COUNT + j];
        return w;
    }
};

// Forward transform of the 8 registers (ownership t + (n/8) k); the result is left in LDS buffer `res` (natural index,
// padded), biased, below 7.3 (5.4 at n = 2048).  LDS phases: other, res, other, res; at n = 8192, where a
// fifth phase would start and end on the same buffer, res, other, res, other, res behind a barrier.
// IN: what the registers hold on entry.  digit: the transform of the gadget digits digit(0) .. digit(7) instead, whatever the registers hold.
// Bounds from |a| < m: 1.8, 2.6, 3.5 | 4.3, 5.2, 6.1 |
// shrunk, 2.0, 2.8, 3.6 | 4.5, 5.4, 6.3 | 7.2.
// `ahead` runs before the last pass: loads of what is multiplied with the result can be issued there.
struct NothingAhead {
    __device__ __forceinline__ void operator()() const {}
};
enum Entry { PLAIN, BIASED };
// S: the padding of the images.  copy: the kernel's copy of the small levels in LDS (TableCopy), or nothing.
// ALONE: the launch leaves registers idle and a workgroup's chain of steps is what it takes: all constants are requested at
// the start, one trip to the L2 for a transform instead of one a pass.
// FORWARD_BARRIERS: those of this transform and of forward_small_to_lds, for wavefronts of the workgroup that take no part: the one at
// the start, the exchanges' in their order, the one at the end.
constexpr int FORWARD_BARRIERS = (LOGN == 13) + crosses(LOGN - 3, LOGN - 6) + crosses(LOGN - 6, LOGN - 9) +
                                 crosses(LOGN - 9, LOGN < 12 ? 0 : LOGN - 12) + (LOGN == 13 && crosses(LOGN - 12, 0)) + 1;
struct WholeWords {};
template <bool WIDE, int S, Entry IN = PLAIN, bool ALONE = false, class Digit = WholeWords, class Copy = NoCopy, class Ahead = NothingAhead>
__device__ __forceinline__ void forward_to_lds(u64 (&a)[8], u64 *res, u64 *other, const RingTables &T, int tid_,
                                               Digit digit = Digit{}, Copy copy = Copy{}, Ahead ahead = Ahead{}) {
    const int tid = fresh(tid_);
    const MontQ q = T.mont;
    constexpr int B1 = LOGN - 3, B2 = LOGN - 6, B3 = LOGN - 9, B4 = LOGN >= 12 ? LOGN - 12 : 0;
    u64 *first = LOGN == 13 ? res : other, *second = LOGN == 13 ? other : res;
    if (LOGN == 13) __syncthreads();
    Tw7 w8, w64, w512, last;        // levels 8, 64, 512 (from n = 4096 on) and n/8 (but at n = 4096, where it is level 512)
    auto get8 = [&] {
        if (Copy::LEVELS >= 1) w8 = copy.template get<8>(copy.f8, (unsigned)tid >> B2);
        else w8 = tw_level<8>(T.tw, (unsigned)tid >> B2);
    };
    auto get64 = [&] {
        if (Copy::LEVELS >= 2) w64 = copy.template get<64>(copy.f64, (unsigned)tid >> B3);
        else w64 = tw_level<64>(T.tw, (unsigned)tid >> B3);
    };
    auto get512 = [&] { w512 = tw_level<LOGN >= 12 ? 512 : NT>(T.tw, (unsigned)tid >> B4); };
    auto get_last = [&] { last = tw_level<NT>(T.tw, (unsigned)tid); };
    if (ALONE) {
        get8();
        get64();
        if (LOGN >= 12) get512();
        if (LOGN != 12) get_last();
        pin_loads();
    }
    // stages 1-3
    auto whole = [&] {
        if (IN == PLAIN) {
#pragma unroll
            for (int k = 0; k < 8; ++k) a[k] += BIAS;
        }
        fwd_pass<WIDE, 0, false, true>(a, tw_first(T.tw), q);
    };
    if constexpr (std::is_same_v<Digit, WholeWords>) {
        whole();
    } else if (T.digits) {
        u32 x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = (u32)digit(k);
        digit_pass<WIDE>(a, x, T.digits, q);
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] = digit(k);
        whole();
    }
    if (!ALONE) get8();
    exchange<S, B1, B2>(a, first, tid);
    if (!ALONE && Copy::LEVELS < 2) {
        get64();
        pin_loads();
    }
    fwd_pass<WIDE, 0>(a, w8, q);                                                         // stages 4-6
    if (!ALONE && Copy::LEVELS >= 2) get64();
    exchange<S, B2, B3>(a, second, tid);
    if (!ALONE) {
        if (LOGN < 12) get_last();
        else get512();
        pin_loads();
    }
    fwd_pass<WIDE, 0, true>(a, w64, q);                                                  // stages 7-9
    if (LOGN < 12) {
        exchange<S, B3, 0>(a, first, tid);
        ahead();
        fwd_pass<WIDE, 3 - LOGN % 3>(a, last, q);                                        // stages 10, 11
    } else {
        exchange<S, B3, B4>(a, first, tid);
        if (LOGN == 12) {
            ahead();
        } else if (!ALONE) {
            get_last();
            pin_loads();
        }
        fwd_pass<WIDE, 0>(a, w512, q);                                                   // stages 10-12
        if (LOGN == 13) {
            exchange<S, B4, 0>(a, second, tid);
            ahead();
            fwd_pass<WIDE, 2>(a, last, q);                                               // stage 13
        }
    }
    u64 *po = res + pad<S>(tid << 3);
#pragma unroll
    for (int k = 0; k < 8; ++k) po[k] = a[k];
    __syncthreads();
}

// Inverse transform: registers hold index 8t + k (not biased, |a| < m) on entry and index t + (n/8) k, canonical, on
// return.  LDS phases A B A, one more on B at n = 8192.
// FENCE: a barrier in the first exchange, for the sake of reads of bufB before the call.  ALONE: as above.
// INVERSE_BARRIERS: without FENCE, those of this transform and of inverse_small_in_regs: the exchanges' in their order.
constexpr int INVERSE_BARRIERS = crosses(0, 3) + crosses(3, 6) + (LOGN >= 12 && crosses(6, 9)) +
                                 (TOP_STAGES && crosses(LOGN >= 12 ? 9 : 6, LOGN - 3));
template <bool WIDE, int S, bool FENCE = false, bool ALONE = false, class Copy = NoCopy>
__device__ __forceinline__ void inverse_in_regs(u64 (&a)[8], u64 *bufA, u64 *bufB, const RingTables &T, int tid_, Copy copy = Copy{}) {
    const int tid = fresh(tid_);
    const MontQ q = T.mont;
    constexpr int TOP = LOGN - 3;
    Tw7 w8, w64, w512;        // of bits 3-5, 6-8 and, from n = 4096 on, 9-11
    ulonglong2 t[TOP_CONSTS], c[8];
    auto get64 = [&] {
        if (Copy::LEVELS >= 2) w64 = copy.template get<64>(copy.i64, (unsigned)tid & 63);
        else inv_level<7, 64>(w64.t, T.itw + INV_MID, (unsigned)tid & 63);
    };
    auto get512 = [&] { inv_level<7, 512>(w512.t, T.itw + INV_HIGH, (unsigned)tid & 511); };
    auto top = [&] { inv_level<TOP_CONSTS, NT>(t, T.itw + INV_TOP, (unsigned)tid); };
    auto twist = [&] { inv_level<8, NT>(c, T.itw + INV_TWIST, (unsigned)tid); };
    if (Copy::LEVELS >= 1) w8 = copy.template get<8>(copy.i8, (unsigned)tid & 7);
    else inv_level<7, 8>(w8.t, T.itw, (unsigned)tid & 7);
    if (ALONE || Copy::LEVELS < 2) get64();
    if (ALONE) {
        if (LOGN >= 12) get512();
        if (TOP_STAGES) top();
        twist();
    }
    pin_loads();
    inv_first_pass<WIDE>(a, T.w8, q);                                                    // bits 0-2: 3.7
    exchange<S, 0, 3, FENCE>(a, bufA, tid);
    inv_pass<WIDE, false>(a, w8, q);                                                     // bits 3-5: 6.4
    if (!ALONE && Copy::LEVELS >= 2) get64();
    exchange<S, 3, 6>(a, bufB, tid);
    if (!ALONE) {
        if (LOGN >= 12) get512();
        else top();
        pin_loads();
    }
    inv_pass<WIDE, true>(a, w64, q);                                                     // bits 6-8: 3.6
    if (LOGN >= 12) {
        exchange<S, 6, 9>(a, bufA, tid);
        if (!ALONE) {
            if (TOP_STAGES) top();
            else twist();
            pin_loads();
        }
        inv_pass<WIDE, false>(a, w512, q);                                               // bits 9-11: 6.3
    }
    if (TOP_STAGES) {
        // the last pass (register bit 2 is the top bit): 5.4, 7.2 at n = 8192
        if (LOGN >= 12) exchange<S, 9, TOP>(a, bufB, tid);
        else exchange<S, 6, TOP>(a, bufA, tid);
        if (!ALONE) {
            twist();
            pin_loads();
        }
        if (TOP_STAGES == 2) {
            bf2<WIDE>(a[0], a[2], t[0], a[1], a[3], t[1], q);
            bf2<WIDE>(a[4], a[6], t[0], a[5], a[7], t[1], q);
        }
#pragma unroll
        for (int k = 0; k < 4; k += 2)
            bf2<WIDE>(a[k], a[k + 4], t[TOP_CONSTS - 4 + k], a[k + 1], a[k + 5], t[TOP_CONSTS - 3 + k], q);
    }
#pragma unroll
    for (int k = 0; k < PER; k += 2) mont2<WIDE, false, NONE>(a[k], a[k + 1], biased_words(a[k]), c[k], biased_words(a[k + 1]), c[k + 1], q);
#pragma unroll
    for (int k = 0; k < PER; ++k) a[k] = unsign(a[k], T.mod.q);
}

// ---- transforms modulo a small plaintext prime -------------------------------------------------------------------
// Below 2^26 the plaintext modulus leaves 32-bit words room for every stage without corrections (at most 36p after 13
// stages), and a product by a constant is three 32-bit multiplies instead of eight: the slots of masks and messages are
// transformed this way, half the LDS words included.  Same passes, ownership and tables as above, with (constant,
// floor(constant 2^32 / p)) pairs of eight bytes; larger plaintext primes keep the 64-bit transforms.
// From wire to wire: 16x128 on one input 24.1 -> 22.4 us, 1000x512 39.6 -> 37.2 us; 1024 encryptions 67.5 -> 62.4 us, 256
// decryptions 28.2 -> 26.0 us.
struct SmallTables {
    const uint2 *tw, *itw;        // null: the plaintext modulus is not below 2^26
    uint2 w8[3];
    u32 p, one_s;                 // the modulus and floor(2^32 / p)
};
__device__ __forceinline__ u32 mul_small(u32 y, uint2 w, u32 p) { return y * w.x - __umulhi(y, w.y) * p; }     // below 2p
__device__ __forceinline__ void bf_small(u32 &x, u32 &y, uint2 w, u32 p) {
    const u32 t = mul_small(y, w, p);
    y = x - t + 2 * p;
    x += t;
}
__device__ __forceinline__ void bf_small_one(u32 &x, u32 &y, u32 off) {
    const u32 s = x + y;
    y = x - y + off;
    x = s;
}
template <int CONSTANTS, int COUNT>
__device__ __forceinline__ void small_level(uint2 (&t)[CONSTANTS], const uint2 *__restrict__ level, unsigned j) {
#pragma unroll
    for (int e = 0; e < CONSTANTS; ++e) t[e] = level[e * COUNT + j];
}
template <int B_OUT, int B_IN>
__device__ __forceinline__ void exchange_small(u32 (&a)[8], u32 *buf, int tid) {
    u32 *po = buf + pad32(owner<B_OUT>(tid));
#pragma unroll
    for (int k = 0; k < 8; ++k) po[pad32(k << B_OUT)] = a[k];
    if (!crosses(B_OUT, B_IN)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
    const u32 *pi = buf + pad32(owner<B_IN>(tid));
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] = pi[pad32(k << B_IN)];
}
template <int STAGE>
__device__ __forceinline__ void fwd_pass_small(u32 (&a)[8], const uint2 (&w)[7], u32 p) {
    if (STAGE == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) bf_small(a[k], a[k + 4], w[0], p);
    }
    if (STAGE <= 1) {
        bf_small(a[0], a[2], w[1], p);
        bf_small(a[1], a[3], w[1], p);
        bf_small(a[4], a[6], w[2], p);
        bf_small(a[5], a[7], w[2], p);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) bf_small(a[2 * k], a[2 * k + 1], w[3 + k], p);
}
__device__ __forceinline__ void inv_pass_small(u32 (&a)[8], const uint2 (&w)[7], u32 p) {
#pragma unroll
    for (int k = 0; k < 4; ++k) bf_small(a[2 * k], a[2 * k + 1], w[0], p);
    bf_small(a[0], a[2], w[1], p);
    bf_small(a[1], a[3], w[2], p);
    bf_small(a[4], a[6], w[1], p);
    bf_small(a[5], a[7], w[2], p);
#pragma unroll
    for (int k = 0; k < 4; ++k) bf_small(a[k], a[k + 4], w[3 + k], p);
}
// as forward_to_lds; inputs canonical, the result in `res` canonical up to reduce_small()
__device__ __forceinline__ u32 reduce_small(u32 x, const SmallTables &T) {
    const u32 r = x - __umulhi(x, T.one_s) * T.p;      // below 2p
    return r >= T.p ? r - T.p : r;
}
__device__ __forceinline__ void forward_small_to_lds(u32 (&a)[8], u32 *res, u32 *other, const SmallTables &T, int tid) {
    constexpr int B1 = LOGN - 3, B2 = LOGN - 6, B3 = LOGN - 9, B4 = LOGN >= 12 ? LOGN - 12 : 0;
    u32 *first = LOGN == 13 ? res : other, *second = LOGN == 13 ? other : res;
    if (LOGN == 13) __syncthreads();
    uint2 w[7];
    small_level<7, 1>(w, T.tw, 0);
    fwd_pass_small<0>(a, w, T.p);
    small_level<7, 8>(w, T.tw + level_offset(8), (unsigned)tid >> B2);
    exchange_small<B1, B2>(a, first, tid);
    fwd_pass_small<0>(a, w, T.p);
    small_level<7, 64>(w, T.tw + level_offset(64), (unsigned)tid >> B3);
    exchange_small<B2, B3>(a, second, tid);
    fwd_pass_small<0>(a, w, T.p);
    if (LOGN < 12) {
        small_level<7, NT>(w, T.tw + level_offset(NT), (unsigned)tid);
        exchange_small<B3, 0>(a, first, tid);
        fwd_pass_small<3 - LOGN % 3>(a, w, T.p);
    } else {
        small_level<7, 512>(w, T.tw + level_offset(512), (unsigned)tid >> B4);
        exchange_small<B3, B4>(a, first, tid);
        fwd_pass_small<0>(a, w, T.p);
        if (LOGN == 13) {
            small_level<7, NT>(w, T.tw + level_offset(NT), (unsigned)tid);
            exchange_small<B4, 0>(a, second, tid);
            fwd_pass_small<2>(a, w, T.p);
        }
    }
    u32 *po = res + pad32(tid << 3);
#pragma unroll
    for (int k = 0; k < 8; ++k) po[k] = a[k];
    __syncthreads();
}
// The constants of the inverse transform, 28 to 36 pairs of eight bytes: requested all at once, before what precedes the
// transform is done (a mask of a lone workgroup's launch: he_fc 1000x512 on one input 34.3 -> 32.5 us).  At n = 8192, where a lane
// has 128 registers whatever the launch, each pass requests its own behind the pass before it: an encryption 50.5 us, 53.2 with
// all at once, 16x512 on one input 46.1 and 47.4.
struct SmallInverse {
    static constexpr bool AT_ONCE = LOGN < 13;
    uint2 w8[7], w64[7], w512[7], t[TOP_CONSTS], c[8];
    __device__ __forceinline__ void low(const SmallTables &T, int tid) { small_level<7, 8>(w8, T.itw, (unsigned)tid & 7); }
    __device__ __forceinline__ void mid(const SmallTables &T, int tid) { small_level<7, 64>(w64, T.itw + INV_MID, (unsigned)tid & 63); }
    __device__ __forceinline__ void high(const SmallTables &T, int tid) {
        if (LOGN >= 12) small_level<7, 512>(w512, T.itw + INV_HIGH, (unsigned)tid & 511);
    }
    __device__ __forceinline__ void top(const SmallTables &T, int tid) {
        if (TOP_STAGES) small_level<TOP_CONSTS, NT>(t, T.itw + INV_TOP, (unsigned)tid);
    }
    __device__ __forceinline__ void twist(const SmallTables &T, int tid) { small_level<8, NT>(c, T.itw + INV_TWIST, (unsigned)tid); }
    __device__ __forceinline__ void request(const SmallTables &T, int tid) {
        if (!AT_ONCE) return;
        low(T, tid);
        mid(T, tid);
        high(T, tid);
        top(T, tid);
        twist(T, tid);
    }
};
// as inverse_in_regs: canonical in, canonical out
__device__ __forceinline__ void inverse_small_in_regs(u32 (&a)[8], u32 *bufA, u32 *bufB, const SmallTables &T, SmallInverse &I, int tid) {
    constexpr int TOP = LOGN - 3;
    constexpr bool LATE = !SmallInverse::AT_ONCE;
    const u32 p = T.p;
    if (LATE) I.low(T, tid);
#pragma unroll
    for (int k = 0; k < 4; ++k) bf_small_one(a[2 * k], a[2 * k + 1], p);                 // below 2p
    bf_small_one(a[0], a[2], 2 * p);
    bf_small_one(a[4], a[6], 2 * p);                                                     // below 4p
    bf_small(a[1], a[3], T.w8[1], p);
    bf_small(a[5], a[7], T.w8[1], p);
    bf_small_one(a[0], a[4], 4 * p);                                                     // below 8p
    bf_small(a[1], a[5], T.w8[0], p);
    bf_small(a[2], a[6], T.w8[1], p);
    bf_small(a[3], a[7], T.w8[2], p);
    exchange_small<0, 3>(a, bufA, tid);
    inv_pass_small(a, I.w8, p);
    if (LATE) I.mid(T, tid);
    exchange_small<3, 6>(a, bufB, tid);
    inv_pass_small(a, I.w64, p);
    if (LOGN >= 12) {
        if (LATE) I.high(T, tid);
        exchange_small<6, 9>(a, bufA, tid);
        inv_pass_small(a, I.w512, p);
    }
    if (TOP_STAGES) {
        if (LATE) I.top(T, tid);
        if (LOGN >= 12) exchange_small<9, TOP>(a, bufB, tid);
        else exchange_small<6, TOP>(a, bufA, tid);
        if (LATE) I.twist(T, tid);
        if (TOP_STAGES == 2) {
            bf_small(a[0], a[2], I.t[0], p);
            bf_small(a[1], a[3], I.t[1], p);
            bf_small(a[4], a[6], I.t[0], p);
            bf_small(a[5], a[7], I.t[1], p);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) bf_small(a[k], a[k + 4], I.t[TOP_CONSTS - 4 + k], p);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const u32 r = mul_small(a[k], I.c[k], p);
        a[k] = r >= p ? r - p : r;
    }
}

// The plaintext polynomial of a slot image: slot values sit at the padded position of bufB, as 32-bit words when the plaintext
// modulus is small (put_slot); coefficients t + (n/8) k come back in registers.  The image is padded like an exchange's,
// because a wavefront reads the words it then writes in the second exchange, and no barrier separates those writes from
// the other wavefronts' reads.
template <int S>
__device__ __forceinline__ void put_slot(u64 *bufB, int position, u64 v, bool small) {
    if (small) reinterpret_cast<u32 *>(bufB)[pad32(position)] = (u32)v;
    else bufB[pad<S>(position)] = v;
}
template <bool WIDE, int S>
__device__ __forceinline__ void slots_to_coefficients(u64 (&a)[8], u64 *bufA, u64 *bufB, const RingTables &Tp,
                                                      const SmallTables &small, SmallInverse &consts, int tid) {
    if (small.tw) {
        u32 *A = reinterpret_cast<u32 *>(bufA), *B = reinterpret_cast<u32 *>(bufB), v[8];
#pragma unroll
        for (int k = 0; k < PER; ++k) v[k] = B[pad32(8 * tid) + k];
        inverse_small_in_regs(v, A, B, small, consts, tid);
#pragma unroll
        for (int k = 0; k < PER; ++k) a[k] = v[k];
    } else {
#pragma unroll
        for (int k = 0; k < PER; ++k) a[k] = bufB[pad<S>(8 * tid) + k];
        inverse_in_regs<WIDE, S>(a, bufA, bufB, Tp, tid);
    }
}

// the padding of kernels that have nothing but two images in LDS: four workgroups of them per CU at n = 2048
constexpr int ALONE_S = 3;

// Share generation inside the same launch: the workgroups after the last (item, chunk) pair build the
// negated mask of one output ciphertext each and store it as one more partial ciphertext.
struct MaskJob {
    int enabled;
    int first_chunk;            // the first chunk's workgroup builds the mask of its item behind its rotations; no workgroups for masks alone
    int nout;                   // output ciphertexts per batch element
    const u64 *r;               // batch x r_stride server shares mod p
    size_t r_stride;
    u64 mask_seed;
    MaskLayoutDev layout;
    int pbits;
    ulonglong2 delta;           // delta = floor(q/p), a MontPair mod q
    RingTables Tp;              // inverse-transform tables of the plaintext modulus
    SmallTables small;
};

// The state of the generator behind rand64(seed, stream, idx, attempt) that all draws of a stream share.
__device__ __forceinline__ u64 stream_state(u64 seed, u64 stream) { return mix64(mix64(seed + 0x9E3779B97F4A7C15ull) + stream); }
// draw_uniform of the indices first + k STEP.  The first attempts are made together: one by one, each with its own chance of
// another attempt, the draws of a lone wavefront are one chain of multiplications.
template <int STEP, int COUNT>
__device__ __forceinline__ void draw_uniforms(u64 (&v)[COUNT], u64 m, int bits, u64 state, u64 first) {
    u64 h[COUNT];
#pragma unroll
    for (int k = 0; k < COUNT; ++k) {
        h[k] = mix64(state + (first + (u64)(k * STEP)));
        v[k] = mix64(h[k]) >> (64 - bits);
    }
#pragma unroll
    for (int k = 0; k < COUNT; ++k) {
        u64 attempt = 0;
        while (v[k] >= m) v[k] = mix64(h[k] + ++attempt) >> (64 - bits);
    }
}

// store(k, i, m): mask word i = threadIdx.x + k NT GROUPS of the evaluation domain, canonical.  before() runs once ahead of them.
// ALONE: as in the transforms.  GROUPS: the workgroup's threads in units of NT; the first group runs the transforms.
// Bound by its own chain of steps: at n = 2048 with 1000 rows, in a launch of one workgroup a CU, 34 400 clocks when each thread
// drew its slots one after the other (10 100) and then walked the rows, each with its row pointers, indices and share behind
// each other and two divisions (12 900); 29 200 by slots, with 7 600 and 3 800.  Rotations hide it where there are any.
// SOLE: the launch is its masks; others hide what the rows take behind their rotations.
// BY_ROWS: thread t forms the first slots of rows t, t + NT, ...  Where a thread does that for its own slots and there are many rows, every
// wavefront does it OWN times for a few lanes each, and the loads of their shares wait for one another.  The layer alone on one input,
// n = 4096: 256x16 16.5 -> 14.3 us, 512x8 16.7 -> 14.5, 16x128 14.4 both; n = 8192: 512x16 25.5 -> 22.7.  Two groups of threads have half as
// many slots each: 256x8 10.2 by slots, as fast as by rows.
template <bool WIDE, int S, bool ALONE = false, int GROUPS = 1, bool SOLE = false, class Store, class Before = NothingAhead>
__device__ __forceinline__ void mask_role(const RingTables &T, const MaskJob &mj, int item, u64 *bufA, u64 *bufB, Store store,
                                          Before before = Before{}) {
    constexpr int ALL = NT * GROUPS, OWN = PER / GROUPS;
    const int tid = threadIdx.x;
    const bool transforms = GROUPS == 1 || __builtin_amdgcn_readfirstlane(tid) < NT;
    const int b = item / mj.nout, O = item % mj.nout;
    const u64 p = mj.Tp.mod.q;
    const bool small = mj.small.tw != nullptr, sums = mj.layout.sums;
    // everything read from memory is requested before the draws
    const int2 *meta = reinterpret_cast<const int2 *>(mj.layout.slot_mask) + (size_t)O * N;
    const u64 *r = mj.r + (size_t)b * mj.r_stride;
    int slot[OWN], rindex[OWN];
    u64 share[OWN];
#pragma unroll
    for (int k = 0; k < OWN; ++k) {
        const int2 m = meta[tid + k * ALL];
        slot[k] = m.x;
        rindex[k] = m.y;
    }
    constexpr bool BY_ROWS = SOLE && GROUPS == 1;
    const int2 *row_first = reinterpret_cast<const int2 *>(mj.layout.row_first) + (size_t)O * N;
    const int nrows = BY_ROWS ? mj.layout.nrows[O] : 0;
    int2 first = make_int2(-1, 0);
    if (BY_ROWS) {
        if (tid < nrows) first = row_first[tid];
    } else {
#pragma unroll
        for (int k = 0; k < OWN; ++k) share[k] = slot[k] & MaskSlot::kFirst ? r[rindex[k]] : 0;
    }
    SmallInverse consts;
    if (small && transforms) consts.request(mj.small, tid);
    unsigned long long *rowsum = reinterpret_cast<unsigned long long *>(bufA);
    if (sums) {
#pragma unroll
        for (int k = 0; k < OWN; ++k) rowsum[tid + k * ALL] = 0;
    }
    // every slot but the first of each real output is a draw from the mask stream; values go to the position the mod-p
    // transform expects them at
    u64 v[OWN];
    draw_uniforms<ALL>(v, p, mj.pbits, stream_state(mj.mask_seed, kStreamMask), ((u64)b << 32) + ((u64)O << 16) + (u64)tid);
    u64 row_share = 0;
    if (BY_ROWS && first.x >= 0) row_share = r[first.y];
    if (sums) __syncthreads();
    // plain integer sums of a row's values below p: at most n of them, far from 64 bits
    auto add = [&](int row, u64 x) { atomicAdd(&rowsum[row], (unsigned long long)x); };
    if (SOLE && __builtin_expect(mj.layout.strided, 0)) {
        // A thread adds up what it has in a row before it goes to the row's cell, which all lanes are after where there is a single
        // row.  The layer alone, 1x4096 on one input at n = 4096 17.2 -> 14.7 us, at n = 8192 25.9 -> 23.3, 1x2048 on one 10.0 -> 9.0.
        int row = -1;
        u64 part = 0;
#pragma unroll
        for (int k = 0; k < OWN; ++k) {
            if (slot[k] & MaskSlot::kFirst) continue;
            put_slot<S>(bufB, slot[k] & (N - 1), v[k], small);
            if (!(slot[k] & MaskSlot::kInRow)) continue;
            const int t = slot[k] >> MaskSlot::kBits & (N - 1);
            if (t != row) {
                if (row >= 0) add(row, part);
                row = t;
                part = 0;
            }
            part += v[k];
        }
        if (row >= 0) add(row, part);
    } else {
#pragma unroll
        for (int k = 0; k < OWN; ++k) {
            if (slot[k] & MaskSlot::kFirst) continue;
            put_slot<S>(bufB, slot[k] & (N - 1), v[k], small);
            if (sums && (slot[k] & MaskSlot::kInRow)) add(slot[k] >> MaskSlot::kBits & (N - 1), v[k]);
        }
    }
    if (sums) __syncthreads();
    // the first slot of every real row absorbs r minus the row's other slots
    auto first_slot = [&](int position, u64 x, int row) {
        if (x >= p) x %= p;
        if (sums) {
            const u64 sum = rowsum[row];
            x = sub_mod(x, csub(sum - mulhi64(sum, mj.Tp.mod.one_s) * p, p), p);
        }
        put_slot<S>(bufB, position, x, small);
    };
    if (BY_ROWS) {
        if (first.x >= 0) first_slot(first.x, row_share, tid);
        for (int t = tid + ALL; t < nrows; t += ALL) {
            const int2 f = row_first[t];
            if (f.x >= 0) first_slot(f.x, r[f.y], t);
        }
    } else {
#pragma unroll
        for (int k = 0; k < OWN; ++k)
            if (slot[k] & MaskSlot::kFirst) first_slot(slot[k] & (N - 1), share[k], slot[k] >> MaskSlot::kBits & (N - 1));
    }
    __syncthreads();
    // slots -> plaintext polynomial (inverse transform mod p) -> delta * m mod q -> evaluation domain mod q
    if (transforms) {
        u64 a[PER];
        slots_to_coefficients<WIDE, S>(a, bufA, bufB, mj.Tp, mj.small, consts, tid);        // LDS phases A B A
#pragma unroll
        for (int k = 0; k < PER; ++k) a[k] = mont<WIDE, true, true>(plain_words(a[k]), mj.delta, T.mont, BIAS);
        forward_to_lds<WIDE, S, BIASED, ALONE>(a, bufA, bufB, T, tid);      // LDS phases B A B A, result in bufA
    } else {
#pragma unroll
        for (int k = 0; k < INVERSE_BARRIERS + FORWARD_BARRIERS; ++k) __syncthreads();
    }
    before();
#pragma unroll
    for (int k = 0; k < OWN; ++k) {
        const int i = tid + k * ALL;
        store(k, i, canonical<WIDE>(biased_words(bufA[pad<S>(i)]), T));
    }
}
// ... as one more partial ciphertext of the item: minus the mask on c0
template <bool WIDE, int S, bool ALONE = false, int GROUPS = 1>
__device__ __forceinline__ void mask_partial(const PermJob &job, const RingTables &T, const MaskJob &mj, int item, u64 *bufA,
                                             u64 *bufB) {
    u64 *out = job.partial + ((size_t)item * job.slots + job.nchunks) * 2 * N;
    const u64 q = T.mod.q;
    mask_role<WIDE, S, ALONE, GROUPS>(T, mj, item, bufA, bufB, [&](int, int i, u64 m) {
        out[i] = m ? q - m : 0;
        out[N + i] = 0;
    });
}
// ... or taken off the c0 of a partial ciphertext that the same threads have written.
template <bool WIDE, int S, bool ALONE>
__device__ __forceinline__ void mask_behind(const RingTables &T, const MaskJob &mj, int item, u64 *bufA, u64 *bufB, u64 *out) {
    const u64 q = T.mod.q;
    __syncthreads();        // the images may still be read
    mask_role<WIDE, S, ALONE>(T, mj, item, bufA, bufB, [&](int, int i, u64 m) { out[i] = sub_mod(out[i], m, q); });
}
// The kernel's arguments, read again where this is called; Args lists them as the kernel does (the segment holds them in order, each
// at its natural alignment, as a struct does).  What a mask behind the rotations takes from them was otherwise loaded at the kernel's
// start and kept through the rotations, in scalar registers that spilled to lanes of vector registers: 84 instead of 20 with weights, 23
// now, and rotations up to a tenth slower: he_fc 1000x4096 at batch 8 (32 rotations a chunk) 611 us, 574 with
// masks in workgroups of their own, 570 now; 500x1024 at batch 8 (four) 78.5, 84.8 and 73.9.
template <class Args>
__device__ __forceinline__ const Args &arguments_again() {
    typedef __attribute__((address_space(4))) const char kernarg;
    kernarg *p = (kernarg *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const Args *)(const char *)p;
}
struct PermArgs {
    PermJob job;
    RingTables T;
    MaskJob mj;
};
// At n = 4096 a workgroup has a CU to itself and sums are cut into whole rounds of the 256 CUs.  In a launch of one round the masks
// wait for the first workgroups to end, and then start from the beginning.  Where the G - 1 rotations do not divide by the number of
// chunks the first chunk is one of the shorter ones, and a mask takes less than a rotation: there its workgroup builds the mask.
// The layer alone: he_fc 500x1024 at batch 8 84.8 -> 73.9 us, 16x2048 at batch 64 54.4 -> 42.4, with the special prime 101.2 -> 90.0, 100x1000
// at batch 23 (253 chunks) 69.2 -> 58.1; a convolution of 64 channels of 16x16 to 64, 3x3, at batch 16 181 -> 170, with the special
// prime 338 -> 324.  What it saves is one mask, so it fades with the rotations of a chunk: of the longest chunk's 8 rotations
// 147 -> 135 us (500x1024 at batch 16), of 32 518 -> 507 (120x4000 at batch 64), of 64 1017 -> 1006 (250x4000 at
// batch 64) and with the special prime 2301 -> 2293; of 103 (1000x4096 at batch 25) 1734 -> 1739 and with it 4086 -> 4098, of 256 (batch 64)
// 4241 -> 4264.  So up to 64.
// Not where CUs are left for a good part of the masks (9x600 at batch 100, 200 chunks), nor in launches of several rounds, whose
// tail the masks fill: measured before the arguments were read again, 43.6 and 46.9 us, 16x2048 at batch 300 209 and 220.
// Since then 42.7 and 42.1, 205 and 191, with the special prime 87.7 and 87.3, 424 and 424: no longer a loss, and not taken up here.
static bool mask_in_first_chunk(const PermJob &job) {
    const long chunks = (long)job.items * job.nchunks, idle = 256 - chunks;
    const int longest = (job.G - 2) / job.nchunks + 1;
    return LOGN == 12 && (job.G - 1) % job.nchunks != 0 && longest <= 64 && idle >= 0 && 4 * idle <= job.items;
}
// A layer without rotations (he_fc with G = 1: a matrix that fits one ciphertext; a convolution always has two kernel
// orders at least) is one product and the mask: the workgroup that builds an item's mask forms its output at once, in one
// launch and without partial ciphertexts.
// From wire to wire (with the layout's loads requested ahead of the draws): 16x128 on one input 27.5 -> 24.1 us; that
// and he_fc 1000x512 on one input, where a mask is the longest workgroup, 40.9 -> 39.6 us.
// GROUPS = 2: as in mask_role, for launches that leave a CU two wavefronts per SIMD at most; larger ones are bound by the
// vector ALU.  16x128 on one input 20.9 us, 19.6 with the slots' draws together and 18.2 with two groups.
// EARLY: launches that leave registers idle (few) request the operands ahead of the mask and all constants of the forward
// transform at its start.  Elsewhere that takes 181 to 191 registers, so that two wavefronts are left on a SIMD; behind the mask and
// within 128 there are four.  The layer alone, operands early and late: 16x128 on 513 inputs 21.0 and 16.8 us, 768 23.1 and 18.6, 3000 70.8
// and 55.0; n = 1024, 16x64 on 1025 18.9 and 15.9, 4000 47.9 and 38.8; n = 4096, 16x128 on 257 28.7 and 22.4, 1000 65.9 and 43.2.
// Late operands all at once where workgroups are small, one index after the other from n = 4096 on (with all at once n = 4096 on
// 1000 inputs 45.7, n = 8192, 16x512 on 256, 30.7 and 28.4; one by one 16x128 on 3000 56.5, n = 1024 on 1025 17.6).
template <bool WIDE, int GROUPS, bool EARLY>
__global__ __launch_bounds__(NT * GROUPS, EARLY ? 2 : 4) void scmult_masked_ring(PermJob job, RingTables T, MaskJob mj, u64 *ct_out) {
    __shared__ u64 bufA[lds_words(ALONE_S)], bufB[lds_words(ALONE_S)];
    const int item = blockIdx.x;
    const u64 *c0 = job.ct_in + (size_t)item * job.in_item_stride, *c1 = c0 + N;
    const ulonglong2 *w = reinterpret_cast<const ulonglong2 *>(job.w2);
    constexpr int OWN = PER / GROUPS, AT_ONCE = EARLY || LOGN < 12 ? OWN : 1;
    u64 x0[AT_ONCE], x1[AT_ONCE];
    ulonglong2 ww[AT_ONCE];
    auto request = [&](int first) {
#pragma unroll
        for (int k = 0; k < AT_ONCE; ++k) {
            const int i = threadIdx.x + (first + k) * NT * GROUPS;
            ww[k] = w[i];
            x0[k] = c0[i];
            x1[k] = c1[i];
        }
    };
    if (EARLY) request(0);
    u64 *out = ct_out + (size_t)item * 2 * N;
    mask_role<WIDE, ALONE_S, EARLY, GROUPS, true>(
        T, mj, item, bufA, bufB,
        [&](int k, int i, u64 m) {
            if (AT_ONCE == 1) request(k);
            const int h = AT_ONCE == 1 ? 0 : k;
            u64 a, b;
            mont2<WIDE, false, NONE>(a, b, plain_words(x0[h]), ww[h], plain_words(x1[h]), ww[h], T.mont);
            out[i] = sub_mod(unsign(a, T.mod.q), m, T.mod.q);
            out[N + i] = unsign(b, T.mod.q);
        },
        [&] {
            if (!EARLY && AT_ONCE > 1) request(0);
        });
}

// Workgroup -> (item, chunk).  Consecutive workgroup ids go to the eight XCDs in turn, each with an L2 of its own.  Long sums
// are handed out so that an XCD has consecutive chunks for all items, and starts the workgroups that read the same keys and
// weights one after the other: a chunk count that is a multiple of eight gives every XCD its eighth of the chunks, eight chunks
// at a time, item by item; other counts are split anywhere, chunk by chunk.  Eighths in order rather than every eighth
// chunk, because the longer chunks recur: 63 rotations in 24 chunks left three XCDs with two thirds of the others' work (145 us
// instead of 133).  Eight at a time, because item by item through all of an XCD's chunks the keys of many chunks do not
// stay in its L2, and one at a time its workgroups ask for the same keys in step (he_fc 128x1024 at batch 64 134 us, 132 with
// eight; 100x784 at batch 7 38.2 us with four, 37.6 with eight).  From wire to wire, against item by item and every eighth
// chunk: he_fc 1000x1024 at batch 5 109 -> 92 us, at batch 16 242 -> 232, 1000x1024 at n = 4096, batch 13, 264 -> 243; against
// item by item where the count is no multiple of eight: 100x784 at batch 7 with the special prime 64.7 -> 60.6 us, 1000x512 at batch 5 with
// it 131 -> 123, 100x2048 at n = 4096, batch 9, 142 -> 137.
// Short sums (a convolution's kernel orders) of other counts have keys that fit an L2: the chunks of an item in turn.  With an odd count
// every XCD gets chunks of each length.  With an even one it does not: of two chunks an item the even XCDs have all of the shorter
// ones and the odd XCDs all of the longer.
__device__ __forceinline__ void item_and_chunk(const PermJob &job, int &item, int &chunk) {
    const u32 w = blockIdx.x, xcd = w & 7, s = w >> 3, items = (u32)job.items, nchunks = (u32)job.nchunks;
    if ((nchunks & 7) == 0) {
        const u32 per = nchunks >> 3, first = s / (8 * items) * 8, width = min(8u, per - first), r = s - first * items;
        item = (int)(r / width);
        chunk = (int)(xcd * per + first + r - (u32)item * width);
    } else if (job.G >= 32) {
        const u32 total = items * nchunks, at = xcd * (total >> 3) + min(xcd, total & 7) + s;
        chunk = (int)(at / items);
        item = (int)(at - (u32)chunk * items);
    } else {
        item = (int)(w / nchunks);
        chunk = (int)(w - (u32)item * nchunks);
    }
}

// Folded keys.  The digits of a coefficient x add up to it, x = sum_j B^j d_j, and the transform is linear, so the last
// digit's transform is B^(1-L) (X - sum_(j<L-1) B^j D_j) with X = the transform of x, i.e. the very polynomial the
// inverse transform started from.  The inner product sum_j K_j D_j is then sum_(j<L-1) (K_j - B^(j-L+1) K_(L-1)) D_j +
// B^(1-L) K_(L-1) X modulo q: the pair image of the keys holds those combinations (key_pack_kernel), and a rotation
// takes L-1 forward transforms instead of L, for one more product (c1 (.) w at the rotated index).
// From wire to wire, three digits: he_fc 128x1024 at batch 64 209 -> 162 us, 1000x2048 2669 -> 2195 us (the share of the
// import and export transforms in that is 12 us); two digits and a special prime, 100x784 at batch 7: 92 -> 80 us.

// the word at a byte offset of an image
__device__ __forceinline__ u64 word_at(const u64 *image, u32 offset) {
    return *reinterpret_cast<const u64 *>(reinterpret_cast<const char *>(image) + offset);
}
// Brings the constants of digit_pass into the scalar cache while something else is waited for: its own three loads, one after the other,
// each wait for memory otherwise.  he_fc 1000x512 on one input 32.3 -> 31.7 us from wire to wire.  Not for a second entry of a sum (32.0
// with the first two), nor where registers are short: with the special prime 58.9 -> 59.8 (100x784 at batch 7), on blocks of eight four
// spilled at n = 4096 (a convolution of 7x7x17 to 48 channels at batch 6 111.9 -> 114.1 us, 112.2 before the digit pass) and nothing was gained
// at 2048 (13x11x24 to 40 at batch 5 64.3 and 64.2, 32x32x23 to 13, 1x1, at batch 2 39.9 -> 41.8).
struct DigitLines {
    u64 w[4];
    __device__ __forceinline__ void request(const u64 *digits) {
        typedef __attribute__((address_space(4))) const u64 scalar_u64;
        scalar_u64 *c = (scalar_u64 *)reinterpret_cast<uintptr_t>(digits);
#pragma unroll
        for (int l = 0; l < 4; ++l) w[l] = c[7 * l];        // a word of every line
    }
    __device__ __forceinline__ void wait() const {
#pragma unroll
        for (int l = 0; l < 4; ++l) asm volatile("" : : "s"(w[l]));
    }
};
// a pair of a polynomial of which the start is uniform: a scalar base and 32 bits of offset, no address arithmetic
__device__ __forceinline__ ulonglong2 pair_at(const ulonglong2 *base, int tid) {
    typedef __attribute__((address_space(1))) const char global_char;
    typedef __attribute__((address_space(1))) const u64 global_u64;
    global_char *p = (global_char *)reinterpret_cast<uintptr_t>(base);
    asm("" : "+s"(p));
    global_u64 *at = (global_u64 *)(p + (unsigned)tid * 16u);
    return make_ulonglong2(at[0], at[1]);
}
// What bounds the Perm kernel, in clocks of a CU per wavefront and rotation at n = 2048 with weights: the vector ALU, some 2625
// instructions at one a clock, and behind it the vector cache, 113 loads at 16 clocks (178 before the first pass's
// constants came through the scalar cache, the small levels through LDS, and c0 and c1 were read once, by the threads that own
// them, instead of being gathered from memory), and the LDS, about 1250.  Most of what it waited for was the L2, where constants of 94 KiB a workgroup
// come from (the vector cache has 32): requested a pass earlier than needed and pinned there, a wavefront's time in waits
// fell from two fifths to one fifth.  From wire to wire, all of that: he_fc 1000x2048 at batch 64 2073 -> 1722 us, 128x1024 150 -> 135
// us, 500x1024 at n = 4096, batch 8, 114 -> 103 us.
//
// Wavefronts per SIMD: what its LDS (two images and the stash) leaves room for, which
// bounds the registers: three at n = 1024 and 2048 (168 registers), two at 4096 (one workgroup), the workgroup's own four at 8192.
constexpr int PERM_WAVES = LOGN <= 11 ? 3 : LOGN == 12 ? 2 : 4;
// What else fits: the padding of the images and the twiddle levels copied to LDS (TableCopy).  Three workgroups of n = 2048
// take 53 504 bytes each of a CU's 160 KiB.
constexpr int PERM_S = LOGN == 10 ? 5 : LOGN == 12 ? 3 : 4, PERM_LEVELS = LOGN == 10 ? 0 : LOGN == 11 ? 1 : 2;
template <int L = PERM_LEVELS>
__device__ __forceinline__ auto make_copy(ulonglong2 *at, const RingTables &T, int tid) {
    if constexpr (L == 0) {
        return NoCopy{};
    } else {
        TableCopy<L> copy(at);
        copy.fill(T, tid);
        return copy;
    }
}

// Every product on this path is a multiplication by a constant (twiddles, encoded weights, key polynomials), so sums of
// products stay in 64-bit registers: each product is below 0.99, a running sum is shrunk to 5 at most (1.1 when m is close to
// 2^60) and may take four more products before it is shrunk again.
// IN8: the inputs lie in blocks of eight coefficients (PermJob::in8_S), as the matrix-core product leaves them.
// FEW: the launch leaves a CU at most two workgroups, so what counts is one workgroup's chain of dependent steps, not the
// chip's issue rate: it takes up to 256 registers, requests all key pairs of a digit before its transform's last
// pass and a transform's constants at its start.  A convolution of 13x11x24 to 40 channels at batch 5 (175 workgroups) 86.7 -> 82.8 us, he_fc 1000x512 on one
// input (257) 40.7 -> 40.2 us; the constants at the start and products two at a time 78.2 -> 72.9 and 33.8 -> 32.5 us.  Sharing a rotation's two digits out to two workgroups as well lost: 45.8 us, the inverse
// transforms and the partial ciphertexts double.
template <bool WIDE, bool HAS_W, bool IN8 = false, bool FEW = false, bool MASK_BEHIND = false>
__global__ __launch_bounds__(NT, FEW ? 2 : PERM_WAVES) void perm_accumulate_ring(PermJob job, RingTables T, MaskJob mj,
                                                                                 int gadget_bits, int ndigits) {
    __shared__ u64 bufA[lds_words(PERM_S)], bufB[lds_words(PERM_S)];
    __shared__ ulonglong2 tables[PERM_LEVELS ? TableCopy<PERM_LEVELS>::PAIRS : 1];
    // each thread parks its 8 coefficients here between digits (private slots, no barrier); at n = 8192 there is no LDS
    // left for them and they are variables: the workgroup's four wavefronts per SIMD leave 128 registers, and the
    // compiler spills 62 with weights, 74 on blocks of eight and 54 on whole ciphertexts (188, 260 and 212 bytes of
    // scratch a lane).  Against the any-n kernel he_fc 200x8192 at batch 40 takes 2345 us instead of 5562 all the same.
    // Before that a rotation's c0 (.) w waits here, and c1 (.) w in bufB, for the threads that gather them.
    constexpr bool PARK = LOGN < 13;
    __shared__ u64 stash[PARK ? lds_words(5) : 1];
    u64 coef[PARK ? 1 : PER];
    // Key pairs of a digit requested before its transform's last pass, and of the last digit's products before their
    // barrier: as many as the registers hold.  At three wavefronts per SIMD four and all eight instead of none: he_fc 1000x2048 at
    // batch 64 1734 -> 1722 us, the 16x16x128 convolution at batch 16 279 -> 271 us; eight and eight spill, 2085 and 279 us.  At n = 4096,
    // two wavefronts per SIMD, six: 103.2 us instead of 104.5 with three or eight.
    constexpr int AHEAD = FEW ? PER : LOGN == 12 ? 6 : LOGN == 13 ? 0 : 4, EARLY = LOGN == 13 ? 0 : PER;
    const int tid = threadIdx.x;
    if (!MASK_BEHIND && (int)blockIdx.x >= job.items * job.nchunks) {   // only launched when mj.enabled
        mask_partial<WIDE, PERM_S, FEW>(job, T, mj, (int)blockIdx.x - job.items * job.nchunks, bufA, bufB);
        return;
    }
    int item, chunk;
    item_and_chunk(job, item, chunk);
    int g0, g1;
    chunk_range(chunk, job.nchunks, job.G, g0, g1);
    const auto copy = make_copy(tables, T, tid);
    const MontQ q = T.mont;
    const u64 digit_mask = (1ull << gadget_bits) - 1;
    const size_t key_pairs = (size_t)ndigits * 2 * N;

    u64 sum0[PER], sum1[PER];   // running sums over the rotations of this chunk, at most 5 between rotations
#pragma unroll
    for (int k = 0; k < PER; ++k) sum0[k] = sum1[k] = 0;

    for (int g = g0; g < g1; ++g) {
        const u64 *c0 = IN8 ? job.ct_in + (size_t)(item % job.in8_nout) * job.in8_o_stride + (size_t)(item / job.in8_nout) * 16 +
                                  (size_t)g * job.in_g_stride
                            : job.ct_in + (size_t)item * job.in_item_stride + (size_t)g * job.in_g_stride;
        const u64 *c1 = IN8 ? c0 + 8 : c0 + N;
        const size_t S = IN8 ? job.in8_S : 0;
        auto at = [&](const u64 *poly, int i) -> u64 { return IN8 ? poly[(size_t)(i >> 3) * S + (i & 7)] : poly[i]; };
        const ulonglong2 *w = HAS_W ? reinterpret_cast<const ulonglong2 *>(job.w2) + (size_t)g * N : nullptr;
        // middle of this wavefront's 8 KiB in the ownership-order copy: all eight loads are immediate offsets of it
        const char *wo = HAS_W ? reinterpret_cast<const char *>(w + (size_t)job.G * N) : nullptr;
        const unsigned wmid = ((unsigned)(fresh(tid) >> 6) * 512u + 256u + (unsigned)(tid & 63)) * 16u;
        const int gal = job.gal[g];
        if (gal == 1) {   // rotation by zero: ScMult and Add only
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int i = tid + k * NT;
                if (HAS_W) {
                    const ulonglong2 ww = w[i];
                    sum0[k] = shrink(mont<WIDE, true>(plain_words(c0[i]), ww, q, sum0[k]), q);
                    sum1[k] = shrink(mont<WIDE, true>(plain_words(c1[i]), ww, q, sum1[k]), q);
                } else {
                    sum0[k] = shrink(sum0[k] + at(c0, i), q);
                    sum1[k] = shrink(sum1[k] + at(c1, i), q);
                }
            }
            continue;
        }
        DigitLines lines;
        const bool lone = FEW && !IN8 && T.digits && g == g0;
        if (lone) lines.request(T.digits);
        // LDS phases of one rotation: the stash and B (gathers), A B A (inverse), then B A B A per digit.  Consecutive phases
        // use different buffers, which is what lets each exchange do with one barrier.
        const ulonglong2 *key = reinterpret_cast<const ulonglong2 *>(job.keys2) + (size_t)job.key_idx[g] * key_pairs;
        // where the automorphism takes output index tid + (n/8) k from: with i = bitrev(tid) + bitrev3(k) the index is
        // bitrev(((2i + 1) gal - 1) / 2)
        auto turn_of = [&](int t) { return (unsigned)((2 * bitrev(t) + 1) * gal) >> 1; };
        auto source = [&](unsigned turn, int k) {
            const int k3 = ((k & 1) << 2) | (k & 2) | (k >> 2);
            return (int)(__brev(turn + (unsigned)(k3 * gal)) >> (32 - LOGN));
        };
        const unsigned turn = turn_of(tid);
        // ScMult of the thread's own eight coefficients.  c1 (.) w stays in registers for the inverse transform.
        u64 a[PER];
        // Where the automorphism takes the eight outputs from: byte offsets into an image, two to a register.  At n = 8192 they
        // are worked out again for each digit: kept, they were spilled with what they displaced (700 rotations 173 us, 151 now;
        // he_fc 100x784 at batch 64 250 us, 217 now).
        u32 from[PARK ? 4 : 1];
        static_assert(!PARK || 8 * lds_words(PERM_S) <= 1 << 16);
        {
            const ulonglong2 *c0v = reinterpret_cast<const ulonglong2 *>(IN8 ? c0 + (size_t)tid * S : c0 + 8 * tid),
                             *c1v = reinterpret_cast<const ulonglong2 *>(IN8 ? c1 + (size_t)tid * S : c1 + 8 * tid);
            u64 *x0 = stash + pad<5>(8 * fresh(tid)), *x1 = bufB + pad<PERM_S>(8 * fresh(tid));
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const ulonglong2 cv = c1v[k];
                a[2 * k] = cv.x;
                a[2 * k + 1] = cv.y;
                ulonglong2 c = make_ulonglong2(0, 0);
                if (PARK) c = c0v[k];
                if (HAS_W) {     // the copy in ownership order: 64 lanes read 1 KiB of whole lines
                    const ulonglong2 wa = *reinterpret_cast<const ulonglong2 *>(wo + (wmid + (unsigned)((2 * k - 4) * 1024))),
                                     wb = *reinterpret_cast<const ulonglong2 *>(wo + (wmid + (unsigned)((2 * k - 3) * 1024)));
                    u64 va, vb;
                    mont2<WIDE, false, NONE>(a[2 * k], a[2 * k + 1], plain_words(cv.x), wa, plain_words(cv.y), wb, q);
                    if (PARK) {
                        mont2<WIDE, false, NONE>(va, vb, plain_words(c.x), wa, plain_words(c.y), wb, q);
                        c = make_ulonglong2(va, vb);
                    }
                }
                if (PARK) {
                    x0[2 * k] = c.x;
                    x0[2 * k + 1] = c.y;
                    x1[2 * k] = a[2 * k];
                    x1[2 * k + 1] = a[2 * k + 1];
                }
            }
        }
        const ulonglong2 *kb_last = key + (size_t)(2 * (ndigits - 1)) * N, *ka_last = kb_last + N;
        ulonglong2 kbl[EARLY ? EARLY : 1], kal[EARLY ? EARLY : 1];
#pragma unroll
        for (int k = 0; k < EARLY; ++k) {
            kbl[k] = pair_at(kb_last + k * NT, tid);
            kal[k] = pair_at(ka_last + k * NT, tid);
        }
        if (EARLY) pin_loads();
        if (lone) lines.wait();
        __syncthreads();
        // the c0 part, permuted c0 (.) w, and the last digit's products: with the folded keys
        // (key_pack_kernel) they are products of the rotated c1 (.) w itself
        {
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int src = source(turn, k);
                u64 d;
                if (PARK) {
                    const u32 at = (u32)pad<PERM_S>(src) * 8;
                    from[PARK ? k & 3 : 0] = k < 4 ? at : from[PARK ? k & 3 : 0] | at << 16;
                    sum0[k] += stash[pad<5>(src)];
                    d = word_at(bufB, at);
                } else if (HAS_W) {
                    const ulonglong2 ww = w[src];
                    sum0[k] = mont<WIDE, true>(plain_words(c0[src]), ww, q, sum0[k]);
                    d = mont<WIDE>(plain_words(c1[src]), ww, q);
                } else {
                    sum0[k] += at(c0, src);
                    d = at(c1, src);
                }
                const ulonglong2 b = k < EARLY ? kbl[k < EARLY ? k : 0] : pair_at(kb_last + k * NT, tid),
                                 aa = k < EARLY ? kal[k < EARLY ? k : 0] : pair_at(ka_last + k * NT, tid);
                const Words y = plain_words(d);
                mont2<WIDE, false, IN_PLACE>(sum0[k], sum1[k], y, b, y, aa, q);
            }
        }
        inverse_in_regs<WIDE, PERM_S, PARK, FEW>(a, bufA, bufB, T, tid, copy);
        // Parked only where a digit reads it back.  With one digit no transform follows, so no barrier would lie between these
        // stores and those of the next rotation's c0 (.) w by other wavefronts; the gathers of the stash end at the barrier of
        // the inverse transform's first exchange.  Variables need no such care.
        if (!PARK || ndigits > 1) {
#pragma unroll
            for (int k = 0; k < PER; ++k) (PARK ? stash[tid + k * NT] : coef[PARK ? 0 : k]) = a[k];
        }

        int pending = 2;   // products added to sum0 since it was last shrunk
        for (int j = 0; j < ndigits - 1; ++j) {
            auto digit = [&](int k) { return ((PARK ? stash[tid + k * NT] : coef[PARK ? 0 : k]) >> (j * gadget_bits)) & digit_mask; };
            const ulonglong2 *kb = key + (size_t)(2 * j) * N, *ka = kb + N;
            ulonglong2 kbv[AHEAD ? AHEAD : 1], kav[AHEAD ? AHEAD : 1];
            forward_to_lds<WIDE, PERM_S, PLAIN, FEW>(a, bufA, bufB, T, tid, digit, copy, [&] {
#pragma unroll
                for (int k = 0; k < AHEAD; ++k) {
                    kbv[k] = pair_at(kb + k * NT, tid);
                    kav[k] = pair_at(ka + k * NT, tid);
                }
                if (AHEAD) pin_loads();
            });
            if (pending == 4) {       // from four digits on
                asm volatile("");     // not worth doing in advance
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    sum0[k] = shrink(sum0[k], q);
                    sum1[k] = shrink(sum1[k], q);
                }
                pending = 0;
            }
            const unsigned turn_j = PARK ? 0 : turn_of(fresh(tid));
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const u32 at = !PARK ? (u32)pad<PERM_S>(source(turn_j, k)) * 8 : from[PARK ? k & 3 : 0] >> (k < 4 ? 0 : 16) & 0xffff;
                const Words d = biased_words(word_at(bufA, at));
                const ulonglong2 b = k < AHEAD ? kbv[k < AHEAD ? k : 0] : pair_at(kb + k * NT, tid),
                                 aa = k < AHEAD ? kav[k < AHEAD ? k : 0] : pair_at(ka + k * NT, tid);
                mont2<WIDE, false, IN_PLACE>(sum0[k], sum1[k], d, b, d, aa, q);       // the sums ride on the products
            }
            ++pending;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            sum0[k] = shrink(sum0[k], q);
            sum1[k] = shrink(sum1[k], q);
        }
    }
    u64 *out = job.partial + ((size_t)item * job.slots + chunk) * 2 * N;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = tid + k * NT;
        out[i] = canonical<WIDE>(plain_words(sum0[k]), T);
        out[N + i] = canonical<WIDE>(plain_words(sum1[k]), T);
    }
    if (MASK_BEHIND && chunk == 0) {
        const PermArgs &again = arguments_again<PermArgs>();
        mask_behind<WIDE, PERM_S, FEW>(again.T, again.mj, item, bufA, bufB, out);
    }
}

// Hoisted rotations of the input ciphertexts (Sec. III-B: one DecPerm shared by all the taps of a kernel,
// then one HstPerm per tap), as two launches so that both fill the chip at small batches.
//
// DecPerm: one workgroup per (ciphertext, digit but the last); each repeats the inverse transform of c1 and runs the
// forward transform of its digit.  digits[ct][j][i] holds the transform's biased values, which is
// what the products of the inner product take.  In the place of the last digit the inner products
// take c1 itself (folded keys).  stored: L-1 digits.
template <bool WIDE, bool FEW>
__global__ __launch_bounds__(NT) void decperm_ring(const u64 *ct_in, u64 *digits, RingTables T, int gadget_bits,
                                                   int stored) {
    __shared__ u64 bufA[lds_words(ALONE_S)], bufB[lds_words(ALONE_S)];
    const int tid = threadIdx.x;
    const int ct = blockIdx.x / stored, j = blockIdx.x % stored;
    const u64 *c1 = ct_in + (size_t)ct * 2 * N + N;
    u64 a[PER];
    const ulonglong2 *c1v = reinterpret_cast<const ulonglong2 *>(c1 + 8 * tid);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const ulonglong2 cv = c1v[k];
        a[2 * k] = cv.x;
        a[2 * k + 1] = cv.y;
    }
    inverse_in_regs<WIDE, ALONE_S, false, FEW>(a, bufA, bufB, T, tid);      // LDS phases A B A
    const u64 digit_mask = (1ull << gadget_bits) - 1;
    auto digit = [&](int k) { return (a[k] >> (j * gadget_bits)) & digit_mask; };
    forward_to_lds<WIDE, ALONE_S, PLAIN, FEW>(a, bufA, bufB, T, tid, digit);       // LDS phases B A B A, ends on a barrier
    u64 *out = digits + ((size_t)ct * stored + j) * N;
#pragma unroll
    for (int k = 0; k < PER; ++k) out[tid + k * NT] = bufA[pad<ALONE_S>(tid + k * NT)];
}

// HstPerm: one workgroup per (ciphertext, tap).  c0 and the digits are read through the automorphism's index
// map straight from memory: the map sends every aligned block of 64 indices onto another such block, so a
// wavefront's gather still touches whole cache lines.  Output: xrot[ct][tap][c0|c1][i], canonical.
template <bool WIDE>
__global__ __launch_bounds__(NT) void hstperm_taps_ring(const u64 *ct_in, const u64 *digits, TermList terms,
                                                        const u64 *keys2, u64 *xrot, RingTables T, int ndigits) {
    const int tid = threadIdx.x;
    const int b = blockIdx.x / terms.nterm, e = blockIdx.x % terms.nterm;
    const size_t ct = (size_t)b * terms.nin + terms.ct[e];
    const u64 *c0 = ct_in + ct * 2 * N, *c1 = c0 + N;
    u64 *out = xrot + (size_t)blockIdx.x * 2 * N;
    const int gal = terms.gal[e];
    if (gal == 1) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = tid + k * NT;
            out[i] = c0[i];
            out[N + i] = c1[i];
        }
        return;
    }
    const MontQ q = T.mont;
    const u64 *dsrc = digits + ct * (ndigits - 1) * N;
    const ulonglong2 *key = reinterpret_cast<const ulonglong2 *>(keys2) + (size_t)terms.key[e] * ndigits * 2 * N;
    // two batches of four coefficients keep the loads of a batch in flight together at a modest register count
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
        constexpr int H = PER / 2;
        int idx[H], src[H];
        u64 s0[H], s1[H];
#pragma unroll
        for (int k = 0; k < H; ++k) {
            idx[k] = tid + (half * H + k) * NT;
            src[k] = galois_index(idx[k], gal);
            s0[k] = c0[src[k]];
            s1[k] = 0;
        }
        for (int j = 0; j < ndigits; ++j) {
            const ulonglong2 *kb = key + (size_t)(2 * j) * N, *ka = kb + N;
            const u64 *dj = j == ndigits - 1 ? c1 : dsrc + (size_t)j * N;      // folded keys: c1 for the last digit
            const u64 bias = j == ndigits - 1 ? BIAS : 0;
            ulonglong2 b[H], aa[H];
            u64 d[H];
#pragma unroll
            for (int k = 0; k < H; ++k) {
                d[k] = dj[src[k]];
                b[k] = kb[idx[k]];
                aa[k] = ka[idx[k]];
            }
#pragma unroll
            for (int k = 0; k < H; ++k) {
                const Words y = biased_words(d[k] + bias);
                mont2<WIDE, false, IN_PLACE>(s0[k], s1[k], y, b[k], y, aa[k], q);    // each product is below 1: at most 4 in all
            }
        }
#pragma unroll
        for (int k = 0; k < H; ++k) {
            out[idx[k]] = canonical<WIDE>(plain_words(s0[k]), T);
            out[N + idx[k]] = canonical<WIDE>(plain_words(s1[k]), T);
        }
    }
}

// HstPerm of all taps written straight into the column-operand image of the matrix-core multiply-accumulate
// (16-byte chunks [tile][kblock][lane][i][digit], lane = 16*(term block % 4) + column % 16, one balanced
// base-256 digit of 16 consecutive terms per chunk).  One thread owns one coefficient of one input and 16
// consecutive terms (input ciphertext, tap), so a chunk is assembled in registers and the eight digit
// chunks of a coefficient leave as 128 contiguous bytes.
constexpr int PACK_THREADS = 256;      // whatever the ring: a workgroup is 64 coefficients of 4 inputs
typedef digit_chunk_t v4i_t;
// ND: the number of digits when it is 3 (unrolled), else 0 (run-time loop).  ANY_ROT false: no term rotates, there
// are no keys and no digits to read.
template <bool WIDE, int ND, bool ANY_ROT>
__global__ __launch_bounds__(PACK_THREADS) void hstperm_pack_ring(const u64 *ct_in, const u64 *digits, TermList terms, int kblocks,
                                                        const u64 *keys2, v4i_t *xl, RingTables T, int ndigits_rt, int batch) {
    // a workgroup is 64 coefficients x 4 inputs: its wavefronts read the same key words, which then come out of
    // the vector cache for three of them
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane, eb = blockIdx.y;
    const bool b_live = (int)blockIdx.z * 4 + wave < batch;
    const int b = min((int)blockIdx.z * 4 + wave, batch - 1);
    const int nterm = terms.nterm, ndigits = ND ? ND : ndigits_rt;
    const MontQ q = T.mont;
    const size_t key_pairs = (size_t)ndigits * 2 * N;
    // Terms come in (tap, input ciphertext) order, so the sixteen terms of a thread share their rotation in runs: the
    // automorphism's source index and the key pairs of the tap are fetched when the rotation changes (a decision all
    // lanes share), not per term; what differs from term to term is the input ciphertext, i.e. c0 and the digits at
    // the source index.  Terms of the central tap (no rotation) are copies.  A term past the end repeats the last
    // one and is zeroed.
    u64 D0[16], D1[16];     // balanced digits of the 16 terms' c0 and c1 values
    constexpr int KD = ND ? ND : 1;
    ulonglong2 kwb[KD], kwa[KD];
    const ulonglong2 *key = nullptr;
    int cur_gal = 0, src = i;
    bool ident = true;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        const int e = min(eb * 16 + t, nterm - 1);
        const bool live = eb * 16 + t < nterm;
        const int gal = terms.gal[e];
        if (gal != cur_gal) {          // the same for every lane
            cur_gal = gal;
            ident = gal == 1;
            src = ident ? i : galois_index(i, gal);
            if (ANY_ROT && !ident) {
                key = reinterpret_cast<const ulonglong2 *>(keys2) + (size_t)terms.key[e] * key_pairs;
                if (ND) {
#pragma unroll
                    for (int j = 0; j < KD; ++j) {
                        kwb[j] = key[(size_t)(2 * j) * N + i];
                        kwa[j] = key[(size_t)(2 * j + 1) * N + i];
                    }
                }
            }
        }
        const size_t ct = (size_t)b * terms.nin + terms.ct[e];
        const u64 *c0 = ct_in + ct * 2 * N;
        u64 v0, v1;
        if (!ANY_ROT || ident) {
            v0 = c0[i];
            v1 = c0[N + i];
        } else {
            const u64 *dsrc = digits + ct * (ndigits - 1) * N;
            const u64 last = c0[N + src];         // folded keys: c1 in the place of the last digit
            u64 s0 = c0[src], s1 = 0;
            if (ND) {
#pragma unroll
                for (int j = 0; j < KD; ++j) {
                    const Words d = j == KD - 1 ? plain_words(last) : biased_words(dsrc[(size_t)j * N + src]);
                    mont2<WIDE, false, IN_PLACE>(s0, s1, d, kwb[j], d, kwa[j], q);       // each product is below 1: at most 4 in all
                }
            } else {
                for (int j = 0; j < ndigits; ++j) {
                    const Words d = biased_words(j == ndigits - 1 ? last + BIAS : dsrc[(size_t)j * N + src]);
                    const ulonglong2 wb = key[(size_t)(2 * j) * N + i], wa = key[(size_t)(2 * j + 1) * N + i];
                    mont2<WIDE, false, IN_PLACE>(s0, s1, d, wb, d, wa, q);
                }
            }
            canonical2<WIDE>(v0, v1, plain_words(s0), plain_words(s1), T);
        }
        if (!live) v0 = v1 = 0;
        const u64 k80 = 0x8080808080808080ull;   // bytes of x + 0x80..80 are the balanced digits plus 128
        D0[t] = (v0 + k80) ^ k80;
        D1[t] = (v1 + k80) ^ k80;
    }
    // A thread holds the eight 16-byte chunks of its coefficient (128 contiguous bytes); stored straight from
    // the registers, every store instruction would touch 64 different lines with 16 bytes each.  The chunks go
    // through LDS instead (row = lane, padded to 144 bytes), so that instruction k of a wavefront writes the
    // 1 KiB of coefficients 8k..8k+7.
    __shared__ v4i_t tr[PACK_THREADS / 64][64][9];
    const int kb = eb >> 2, g = eb & 3;
    const int i_wave = blockIdx.x * 64;
#pragma unroll
    for (int poly = 0; poly < 2; ++poly) {
        const int col = 2 * b + poly, row = g * 16 + (col & 15);
        v4i_t c[8];
        digit_chunks(poly ? D1 : D0, c);
#pragma unroll
        for (int limb = 0; limb < 8; ++limb) tr[wave][lane][limb] = c[limb];
        __syncthreads();
        v4i_t *dst = xl + ((((size_t)(col >> 4) * kblocks + kb) * 64 + row) * N + i_wave) * 8;
        if (b_live)
#pragma unroll
            for (int k = 0; k < 8; ++k) dst[64 * k + lane] = tr[wave][8 * k + (lane >> 3)][lane & 7];
        __syncthreads();
    }
}


// ---- plain transforms (import, export, key upload) ------------------------------------------------------------
// One workgroup per polynomial, forward or inverse, canonical results, in place or not (a polynomial is read whole
// before its first word is written).  Few polynomials: bound by one workgroup's chain of passes, so three exchanges
// instead of the any-n kernel's eleven barriers; many: by the butterflies.  Against that kernel: encrypting and
// exporting 1024 ciphertexts 83.7 -> 68.2 us, a 16x128 FC layer with one ciphertext imported and one exported
// 41.7 -> 28.8 us.
// Inputs as the any-n kernel takes them: below 4q forward, below 2q inverse.
template <bool WIDE, bool INVERSE>
__global__ __launch_bounds__(NT) void ntt_ring(const u64 *src, u64 *dst, RingTables T) {
    __shared__ u64 bufA[lds_words(ALONE_S)], bufB[lds_words(ALONE_S)];
    const int tid = threadIdx.x;
    src += (size_t)blockIdx.x * N;
    dst += (size_t)blockIdx.x * N;
    u64 a[PER];
    if (INVERSE) {
        // coalesced reads, then through LDS to the eight consecutive coefficients a thread starts from
#pragma unroll
        for (int k = 0; k < PER; ++k) bufB[pad<ALONE_S>(tid + k * NT)] = csub_dev(src[tid + k * NT], T.mod.q);
        __syncthreads();
        const u64 *pi = bufB + pad<ALONE_S>(tid << 3);
#pragma unroll
        for (int k = 0; k < PER; ++k) a[k] = pi[k];
        inverse_in_regs<WIDE, ALONE_S>(a, bufA, bufB, T, tid);       // LDS phases A B A; the reads of bufB above precede its barriers
#pragma unroll
        for (int k = 0; k < PER; ++k) dst[tid + k * NT] = a[k];
    } else {
#pragma unroll
        for (int k = 0; k < PER; ++k) a[k] = shrink(src[tid + k * NT], T.mont);
        forward_to_lds<WIDE, ALONE_S>(a, bufA, bufB, T, tid);
#pragma unroll
        for (int k = 0; k < PER; ++k) dst[tid + k * NT] = canonical<WIDE>(biased_words(bufA[pad<ALONE_S>(tid + k * NT)]), T);
    }
}

// ---- the client's two steps with the radix-8 transforms (one workgroup per ciphertext) ------------------------
// ct = (-a s + e + delta m, a) (Sec. II-C(1)), bit for bit the any-n kernel: m = the plaintext polynomial of the
// slots, a uniform, e Gaussian, all drawn from the ciphertext's seed by coefficient index.
//
// The Gaussian draws by buckets: a draw compared with all 38 thresholds takes as long as three butterfly passes for each of a
// thread's coefficients.  The products by the secret as those by any constant.  Bound by the vector ALU: the generator's draws and five
// transforms at four wavefronts per SIMD.  1024 encryptions from wire to wire 59.4 -> 52.0 us; on another box 50 at n = 8192 53.9 -> 47.4.
template <bool WIDE>
__global__ __launch_bounds__(NT, 4) void encrypt_ring(const u64 *slots, const u64 *seeds, const ulonglong2 *s_hat, u64 *ct_out,
                                                   RingTables T, RingTables Tp, SmallTables small, const int *slot_to_idx, GaussBuckets gauss,
                                                   int qbits, ulonglong2 delta) {
    __shared__ u64 bufA[lds_words(ALONE_S)], bufB[lds_words(ALONE_S)];
    __shared__ u64 thresholds[2 * kGaussBound];
    __shared__ unsigned char passed[256];
    const int tid = threadIdx.x;
    const u64 q = T.mod.q, p = Tp.mod.q, seed = seeds[blockIdx.x];
    const u64 *sl = slots + (size_t)blockIdx.x * N;
    u64 *c0 = ct_out + (size_t)blockIdx.x * 2 * N, *c1 = c0 + N;
    {
        u64 v[PER];
        int to[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            v[k] = sl[tid + k * NT];
            to[k] = slot_to_idx[tid + k * NT];
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) put_slot<ALONE_S>(bufB, to[k], v[k] >= p ? v[k] % p : v[k], small.tw != nullptr);
    }
    for (int b = tid; b < 256; b += NT) passed[b] = gauss.passed[b];
    if (tid < 2 * kGaussBound) thresholds[tid] = gauss.t[tid];
    SmallInverse consts;
    if (small.tw) consts.request(small, tid);
    __syncthreads();
    u64 a[PER];
    slots_to_coefficients<WIDE, ALONE_S>(a, bufA, bufB, Tp, small, consts, tid);      // m, coefficient tid + (n/8) k, canonical mod p
    {
        const u64 state = stream_state(seed, kStreamCtE);
        u64 u[PER];
        int e[PER], several = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            u[k] = mix64(mix64(state + (u64)(tid + k * NT)));
            e[k] = passed[u[k] >> 56];
            several |= e[k];
            e[k] &= GaussBuckets::kSeveral - 1;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) e[k] += e[k] < 2 * kGaussBound && u[k] >= thresholds[e[k]] ? 1 : 0;
        if (several & GaussBuckets::kSeveral) {
#pragma unroll
            for (int k = 0; k < PER; ++k)
                while (e[k] < 2 * kGaussBound && u[k] >= thresholds[e[k]]) ++e[k];
        }
#pragma unroll
        for (int k = 0; k < PER; ++k)
            a[k] = mont<WIDE, true, true>(plain_words(a[k]), delta, T.mont, BIAS + (u64)(i64)(e[k] - kGaussBound));
    }
    forward_to_lds<WIDE, ALONE_S, BIASED>(a, bufA, bufB, T, tid);            // (e + delta m) in the evaluation domain, in bufA
    // biased; with the product by the secret on top it has to stay below 8, which the transform's 7.3 at n = 8192 would not
    u64 t0[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        t0[k] = bufA[pad<ALONE_S>(tid + k * NT)];
        if (LOGN == 13) t0[k] = shrink(t0[k], T.mont);
    }
    draw_uniforms<NT>(a, q, qbits, stream_state(seed, kStreamCtA), (u64)tid);
    forward_to_lds<WIDE, ALONE_S>(a, bufA, bufB, T, tid);            // its first barrier comes after every read of bufA above
#pragma unroll
    for (int k = 0; k < PER; k += 2) {
        u64 ah[2], as[2], c[2];
        canonical2<WIDE>(ah[0], ah[1], biased_words(bufA[pad<ALONE_S>(tid + k * NT)]), biased_words(bufA[pad<ALONE_S>(tid + (k + 1) * NT)]), T);
        mont2<WIDE, false, NONE>(as[0], as[1], plain_words(ah[0]), pair_at(s_hat + k * NT, tid), plain_words(ah[1]),
                                 pair_at(s_hat + (k + 1) * NT, tid), T.mont);
        canonical2<WIDE>(c[0], c[1], biased_words(t0[k] - as[0]), biased_words(t0[k + 1] - as[1]), T);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int i = tid + (k + h) * NT;
            c1[i] = ah[h];
            c0[i] = c[h];
        }
    }
}
// slots = decode(round(p (c0 + c1 s) / q) mod p).  per_q = floor(p 2^64 / q): the high word of a per_q is the quotient of
// p a by q or one less, and what is left of p a + floor(q/2) is below 3q.  One round of workgroups, a chain of two transforms: 256
// decryptions from wire to wire 25.8 -> 24.8 us against a 128-bit remainder and eight consecutive words a thread; on another box 1000
// 50.3 -> 48.0.  The slots' positions are requested at the start, not slot by slot behind the transforms: 21.1 -> 18.8 us.
template <bool WIDE>
__global__ __launch_bounds__(NT) void decrypt_ring(const u64 *ct_in, const ulonglong2 *s_hat, u64 *slots, RingTables T,
                                                   RingTables Tp, SmallTables small, const int *slot_to_idx, u64 per_q) {
    __shared__ u64 bufA[lds_words(ALONE_S)], bufB[lds_words(ALONE_S)];
    const int tid = threadIdx.x;
    const u64 q = T.mod.q, p = Tp.mod.q;
    const u64 *c0 = ct_in + (size_t)blockIdx.x * 2 * N, *c1 = c0 + N;
    int from[PER];        // the slots' positions in the transform modulo p
#pragma unroll
    for (int k = 0; k < PER; ++k) from[k] = slot_to_idx[tid + k * NT];
    u64 a[PER];
    // coalesced, then through LDS to the eight consecutive coefficients a thread starts from
#pragma unroll
    for (int k = 0; k < PER; k += 2) {
        u64 x, y;
        mont2<WIDE, false, NONE>(x, y, plain_words(c1[tid + k * NT]), pair_at(s_hat + k * NT, tid), plain_words(c1[tid + (k + 1) * NT]),
                                 pair_at(s_hat + (k + 1) * NT, tid), T.mont);
        bufB[pad<ALONE_S>(tid + k * NT)] = add_mod(c0[tid + k * NT], unsign(x, q), q);
        bufB[pad<ALONE_S>(tid + (k + 1) * NT)] = add_mod(c0[tid + (k + 1) * NT], unsign(y, q), q);
    }
    __syncthreads();
    const u64 *own = bufB + pad<ALONE_S>(tid << 3);
#pragma unroll
    for (int k = 0; k < PER; ++k) a[k] = own[k];
    inverse_in_regs<WIDE, ALONE_S>(a, bufA, bufB, T, tid);           // c0 + c1 s, coefficient tid + (n/8) k, canonical
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        u64 quot = mulhi64(a[k], per_q);
        const u64 left = p * a[k] + (q >> 1) - quot * q;
        quot += left >= q ? 1 : 0;
        quot += left >= 2 * q ? 1 : 0;
        a[k] = quot >= p ? quot - p : quot;
    }
    u64 *out = slots + (size_t)blockIdx.x * N;
    // the slots' values at their transform positions, in bufA
    if (small.tw) {
        u32 v[PER], *A = reinterpret_cast<u32 *>(bufA);
#pragma unroll
        for (int k = 0; k < PER; ++k) v[k] = (u32)a[k];
        forward_small_to_lds(v, A, reinterpret_cast<u32 *>(bufB), small, tid);
#pragma unroll
        for (int k = 0; k < PER; ++k) out[tid + k * NT] = reduce_small(A[pad32(from[k])], small);
    } else {
        forward_to_lds<WIDE, ALONE_S>(a, bufA, bufB, Tp, tid);
#pragma unroll
        for (int k = 0; k < PER; ++k) out[tid + k * NT] = canonical<WIDE>(biased_words(bufA[pad<ALONE_S>(from[k])]), Tp);
    }
}

#if GALA_LOGN < 13   // at n = 8192 the remainder sums do not fit beside the images: the any-n kernels serve it
// ---- key switching with a special prime P -------------------------------------------------------------
// Keys hold four polynomials per digit ((b, a) modulo q, then modulo P).  Per rotation the digits are
// transformed in both moduli and multiplied into sums modulo q and modulo P; the sums modulo P go back to
// coefficients r in [0,P), and the rotation contributes (t_q - r) / P.  After the lift r -> r mod q everything is
// linear modulo q, so the lifted remainders of a workgroup's rotations are added in the coefficient domain
// (R0, R1) and transformed once at the end; terms that are not divided by P (the c0 part, rotations by zero)
// enter the sums multiplied by P.  Needs P < 2^60 and P < 2q.
struct SpecialJob {
    RingTables TP;          // transform tables of P
    ulonglong2 Pq, minus_Pinv;    // P and -P^-1 mod q, MontPairs
};
struct SpecialArgs {        // as PermArgs
    PermJob job;
    RingTables T;
    SpecialJob S;
    MaskJob mj;
};

// IN8: the inputs lie in blocks of eight coefficients (PermJob::in8_S), as the matrix-core product leaves them.
template <bool WIDE, bool HAS_W, bool IN8 = false, bool MASK_BEHIND = false>
__global__ __launch_bounds__(NT, 2) void perm_accumulate_special_ring(PermJob job, RingTables T, SpecialJob S, MaskJob mj,
                                                                      int gadget_bits, int ndigits) {
    constexpr int PS = 5;
    __shared__ u64 bufA[lds_words(PS)], bufB[lds_words(PS)];
    __shared__ u64 stash[lds_words(PS)];      // a rotation's c0 (.) w for the threads that gather it, then the parked coefficients
    // Sums of the lifted remainders (coefficient domain modulo q, canonical, index tid + (n/8) k): 15 of a thread's 16
    // words live in LDS slots of its own (no barrier), which is what two workgroups per CU leave room for.
    __shared__ u64 Rl[15 * NT];
    const int tid = threadIdx.x;
    if (!MASK_BEHIND && (int)blockIdx.x >= job.items * job.nchunks) {   // only launched when mj.enabled
        mask_partial<WIDE, PS>(job, T, mj, (int)blockIdx.x - job.items * job.nchunks, bufA, bufB);
        return;
    }
    int item, chunk;
    item_and_chunk(job, item, chunk);
    int g0, g1;
    chunk_range(chunk, job.nchunks, job.G, g0, g1);
    const MontQ q = T.mont, qP = S.TP.mont;
    const u64 digit_mask = (1ull << gadget_bits) - 1;
    // key pairs of a digit and modulus requested before the transform's last pass: three of eight, what 256 registers hold.
    // With them pinned there, c0 and c1 gathered in LDS and the weights read in the threads' order: he_fc 100x784 at batch 7 66.9 -> 64.8
    // us.
    constexpr int AHEAD = 3;
    const size_t key_pairs = (size_t)ndigits * 4 * N;

    u64 sum0[PER], sum1[PER];   // evaluation domain modulo q, at most 5 between rotations
    u64 Rlast = 0;              // the sixteenth word of the remainder sums
#pragma unroll
    for (int k = 0; k < PER; ++k) sum0[k] = sum1[k] = 0;
#pragma unroll
    for (int s = 0; s < 15; ++s) Rl[s * NT + tid] = 0;

    for (int g = g0; g < g1; ++g) {
        const u64 *c0 = IN8 ? job.ct_in + (size_t)(item % job.in8_nout) * job.in8_o_stride + (size_t)(item / job.in8_nout) * 16 +
                                  (size_t)g * job.in_g_stride
                            : job.ct_in + (size_t)item * job.in_item_stride + (size_t)g * job.in_g_stride;
        const u64 *c1 = IN8 ? c0 + 8 : c0 + N;
        const size_t S8 = IN8 ? job.in8_S : 0;
        auto at = [&](const u64 *poly, int i) -> u64 { return IN8 ? poly[(size_t)(i >> 3) * S8 + (i & 7)] : poly[i]; };
        const ulonglong2 *w = HAS_W ? reinterpret_cast<const ulonglong2 *>(job.w2) + (size_t)g * N : nullptr;
        const int gal = job.gal[g];
        if (gal == 1) {   // rotation by zero: ScMult and Add only, times P
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int i = tid + k * NT;
                u64 x0 = at(c0, i), x1 = at(c1, i);
                if (HAS_W) {
                    const ulonglong2 ww = w[i];
                    x0 = mont<WIDE>(plain_words(x0), ww, q);
                    x1 = mont<WIDE>(plain_words(x1), ww, q);
                }
                sum0[k] = shrink(mont<WIDE, true, true>(plain_words(x0), S.Pq, q, sum0[k]), q);
                sum1[k] = shrink(mont<WIDE, true, true>(plain_words(x1), S.Pq, q, sum1[k]), q);
            }
            continue;
        }
        // as in the one-prime kernel: what the automorphism moves goes through LDS
        const ulonglong2 *key = reinterpret_cast<const ulonglong2 *>(job.keys2) + (size_t)job.key_idx[g] * key_pairs;
        const unsigned turn = (unsigned)((2 * bitrev(tid) + 1) * gal) >> 1;
        u64 a[PER];
        u32 from[4];      // byte offsets into an image, two to a register
        static_assert(8 * lds_words(PS) <= 1 << 16);
        {
            const ulonglong2 *c0v = reinterpret_cast<const ulonglong2 *>(IN8 ? c0 + (size_t)tid * S8 : c0 + 8 * tid),
                             *c1v = reinterpret_cast<const ulonglong2 *>(IN8 ? c1 + (size_t)tid * S8 : c1 + 8 * tid);
            const int own = pad<PS>(8 * fresh(tid));
            const char *wo = HAS_W ? reinterpret_cast<const char *>(w + (size_t)job.G * N) : nullptr;
            const unsigned wmid = ((unsigned)(fresh(tid) >> 6) * 512u + 256u + (unsigned)(tid & 63)) * 16u;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const ulonglong2 cv = c1v[k], c = c0v[k];
                a[2 * k] = cv.x;
                a[2 * k + 1] = cv.y;
                u64 xa = c.x, xb = c.y;
                if (HAS_W) {
                    const ulonglong2 wa = *reinterpret_cast<const ulonglong2 *>(wo + (wmid + (unsigned)((2 * k - 4) * 1024))),
                                     wb = *reinterpret_cast<const ulonglong2 *>(wo + (wmid + (unsigned)((2 * k - 3) * 1024)));
                    mont2<WIDE, false, NONE>(a[2 * k], a[2 * k + 1], plain_words(cv.x), wa, plain_words(cv.y), wb, q);
                    mont2<WIDE, false, NONE>(xa, xb, plain_words(c.x), wa, plain_words(c.y), wb, q);
                }
                stash[own + 2 * k] = xa;
                stash[own + 2 * k + 1] = xb;
                bufB[own + 2 * k] = a[2 * k];
                bufB[own + 2 * k + 1] = a[2 * k + 1];
            }
        }
        __syncthreads();
        // the c0 part, times P, and the last digit's products modulo q (folded keys: the rotated c1 (.) w itself)
        {
            const ulonglong2 *kb = key + (size_t)(4 * (ndigits - 1)) * N, *ka = kb + N;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int k3 = ((k & 1) << 2) | (k & 2) | (k >> 2);
                const u32 at = (u32)pad<PS>((int)(__brev(turn + (unsigned)(k3 * gal)) >> (32 - LOGN))) * 8;
                from[k & 3] = k < 4 ? at : from[k & 3] | at << 16;
                const u64 x = word_at(stash, at);
                const Words y = plain_words(word_at(bufB, at));
                const ulonglong2 b = pair_at(kb + k * NT, tid), aa = pair_at(ka + k * NT, tid);
                sum0[k] = mont<WIDE, true, true>(plain_words(x), S.Pq, q, sum0[k]);
                mont2<WIDE, false, IN_PLACE>(sum0[k], sum1[k], y, b, y, aa, q);
            }
        }
        inverse_in_regs<WIDE, PS, true>(a, bufA, bufB, T, tid);
#pragma unroll
        for (int k = 0; k < PER; ++k) stash[tid + k * NT] = a[k];
        int pending = 2, pendingP = 0;
        u64 tp0[PER], tp1[PER];   // this rotation's sums modulo P
#pragma unroll
        for (int k = 0; k < PER; ++k) tp0[k] = tp1[k] = 0;
        for (int j = 0; j < ndigits; ++j) {
            const ulonglong2 *kb = key + (size_t)(4 * j) * N, *ka = kb + N;
            auto digit = [&](int k) { return (stash[tid + k * NT] >> (j * gadget_bits)) & digit_mask; };
            if (j + 1 < ndigits) {
                ulonglong2 kbv[AHEAD], kav[AHEAD];
                auto ahead = [&] {
#pragma unroll
                    for (int k = 0; k < AHEAD; ++k) {
                        kbv[k] = pair_at(kb + k * NT, tid);
                        kav[k] = pair_at(ka + k * NT, tid);
                    }
                    pin_loads();
                };
                forward_to_lds<WIDE, PS>(a, bufA, bufB, T, tid, digit, NoCopy{}, ahead);
                if (pending == 4) {
                    asm volatile("");
#pragma unroll
                    for (int k = 0; k < PER; ++k) {
                        sum0[k] = shrink(sum0[k], q);
                        sum1[k] = shrink(sum1[k], q);
                    }
                    pending = 0;
                }
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    const Words d = biased_words(word_at(bufA, k < 4 ? from[k] & 0xffff : from[k & 3] >> 16));
                    const ulonglong2 b = k < AHEAD ? kbv[k < AHEAD ? k : 0] : pair_at(kb + k * NT, tid),
                                     aa = k < AHEAD ? kav[k < AHEAD ? k : 0] : pair_at(ka + k * NT, tid);
                    mont2<WIDE, false, IN_PLACE>(sum0[k], sum1[k], d, b, d, aa, q);
                }
                ++pending;
            }
            // the same digit modulo P
            const ulonglong2 *kbP = kb + 2 * (size_t)N, *kaP = kbP + N;
            ulonglong2 kbv[AHEAD], kav[AHEAD];
            auto ahead = [&] {
#pragma unroll
                for (int k = 0; k < AHEAD; ++k) {
                    kbv[k] = pair_at(kbP + k * NT, tid);
                    kav[k] = pair_at(kaP + k * NT, tid);
                }
                pin_loads();
            };
            forward_to_lds<WIDE, PS>(a, bufA, bufB, S.TP, tid, digit, NoCopy{}, ahead);
            if (pendingP == 4) {
                asm volatile("");
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    tp0[k] = shrink(tp0[k], qP);
                    tp1[k] = shrink(tp1[k], qP);
                }
                pendingP = 0;
            }
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const Words d = biased_words(word_at(bufA, k < 4 ? from[k] & 0xffff : from[k & 3] >> 16));
                const ulonglong2 b = k < AHEAD ? kbv[k < AHEAD ? k : 0] : pair_at(kbP + k * NT, tid),
                                 aa = k < AHEAD ? kav[k < AHEAD ? k : 0] : pair_at(kaP + k * NT, tid);
                mont2<WIDE, false, IN_PLACE>(tp0[k], tp1[k], d, b, d, aa, qP);
            }
            ++pendingP;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            sum0[k] = shrink(sum0[k], q);
            sum1[k] = shrink(sum1[k], q);
        }
        // remainders modulo P: below P, to the ownership the inverse transform starts from (through bufB, which
        // nobody reads any more), back to coefficients in [0,P), reduced modulo q and added up
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int k = 0; k < PER; k += 2) {
                u64 ra, rb;
                mont2<WIDE, true, NONE>(ra, rb, plain_words(h ? tp1[k] : tp0[k]), S.TP.one, plain_words(h ? tp1[k + 1] : tp0[k + 1]), S.TP.one, qP);
                bufB[pad<PS>(tid + k * NT)] = ra;
                bufB[pad<PS>(tid + (k + 1) * NT)] = rb;
            }
            __syncthreads();
            {
                const u64 *pi = bufB + pad<PS>(tid << 3);
#pragma unroll
                for (int k = 0; k < PER; ++k) a[k] = pi[k];
            }
            inverse_in_regs<WIDE, PS>(a, bufA, bufB, S.TP, tid);
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const u64 r = csub_dev(a[k], T.mod.q);
                if (h && k == PER - 1) {
                    Rlast = csub_dev(Rlast + r, T.mod.q);
                } else {
                    u64 *slot = Rl + (h * PER + k) * NT + tid;
                    *slot = csub_dev(*slot + r, T.mod.q);
                }
            }
        }
    }
    // partial = (sum - transform(R)) / P
    u64 *out = job.partial + ((size_t)item * job.slots + chunk) * 2 * N;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        u64 a[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) a[k] = (h && k == PER - 1) ? Rlast : Rl[(h * PER + k) * NT + tid];
        forward_to_lds<WIDE, PS>(a, bufA, bufB, T, tid);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = tid + k * NT;
            const u64 minus = shrink(bufA[pad<PS>(i)], q) - (h ? sum1[k] : sum0[k]);
            out[h * N + i] = unsign(mont<WIDE, false, true>(biased_words(minus), S.minus_Pinv, q), T.mod.q);
        }
    }
    if (MASK_BEHIND && chunk == 0) {
        const SpecialArgs &again = arguments_again<SpecialArgs>();
        mask_behind<WIDE, PS, false>(again.T, again.mj, item, bufA, bufB, out);
    }
}

// ---- hoisted input rotations with a special prime ----------------------------------------------------------
// DecPerm: one workgroup per (ciphertext, digit, modulus); digits[ct][j][modulus][i], biased values of that modulus.
// The last digit modulo q is not needed (folded keys), its place stays empty.
template <bool WIDE>
__global__ __launch_bounds__(NT) void decperm_special_ring(const u64 *ct_in, u64 *digits, RingTables T, RingTables TP,
                                                           int gadget_bits, int ndigits) {
    __shared__ u64 bufA[lds_words(ALONE_S)], bufB[lds_words(ALONE_S)];
    const int tid = threadIdx.x;
    const int per_ct = 2 * ndigits - 1, ct = blockIdx.x / per_ct, v = blockIdx.x % per_ct;
    const int m = v == per_ct - 1 ? 1 : v & 1, j = v >> 1;
    const u64 *c1 = ct_in + (size_t)ct * 2 * N + N;
    u64 a[PER];
    const ulonglong2 *c1v = reinterpret_cast<const ulonglong2 *>(c1 + 8 * tid);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const ulonglong2 cv = c1v[k];
        a[2 * k] = cv.x;
        a[2 * k + 1] = cv.y;
    }
    inverse_in_regs<WIDE, ALONE_S>(a, bufA, bufB, T, tid);
    const u64 digit_mask = (1ull << gadget_bits) - 1;
    auto digit = [&](int k) { return (a[k] >> (j * gadget_bits)) & digit_mask; };
    if (m) forward_to_lds<WIDE, ALONE_S>(a, bufA, bufB, TP, tid, digit);
    else forward_to_lds<WIDE, ALONE_S>(a, bufA, bufB, T, tid, digit);
    u64 *out = digits + (((size_t)ct * ndigits + j) * 2 + m) * N;
#pragma unroll
    for (int k = 0; k < PER; ++k) out[tid + k * NT] = bufA[pad<ALONE_S>(tid + k * NT)];
}

// HstPerm: one workgroup per (ciphertext, tap, output polynomial h): inner products in both moduli from the stored digits, the
// sum modulo P back to coefficients, lifted, reduced modulo q and transformed forward again, then
// out = (P c0(X^g) + t_b - NTT(r_b)) / P or (t_a - NTT(r_a)) / P.  Output: xrot[ct][tap][c0|c1][i], canonical.
// A polynomial a workgroup instead of both, one after the other: 118 registers instead of 146, so four wavefronts per SIMD instead
// of three, and half the chain of steps: the 16x16x128 convolution at batch 16 (2048 rotations) 421 -> 413 us,
// which is within what runs timed in turn differ by.  The vector ALU
// (1700 instructions a wavefront) and the vector cache (some 100 loads at 16 clocks) are busy for about 50 of its 90 us each.
template <bool WIDE>
__global__ __launch_bounds__(NT, 4) void hstperm_special_ring(const u64 *ct_in, const u64 *digits, TermList terms,
                                                           const u64 *keys2, u64 *xrot, RingTables T, SpecialJob S,
                                                           int ndigits) {
    __shared__ u64 bufA[lds_words(ALONE_S)], bufB[lds_words(ALONE_S)];
    const int tid = threadIdx.x, h = blockIdx.y;
    const int b = blockIdx.x / terms.nterm, e = blockIdx.x % terms.nterm;
    const size_t ct = (size_t)b * terms.nin + terms.ct[e];
    const u64 *c0 = ct_in + ct * 2 * N, *c1 = c0 + N;
    u64 *out = xrot + ((size_t)blockIdx.x * 2 + h) * N;
    const int gal = terms.gal[e];
    if (gal == 1) {
        const u64 *c = h ? c1 : c0;
#pragma unroll
        for (int k = 0; k < PER; ++k) out[tid + k * NT] = c[tid + k * NT];
        return;
    }
    const MontQ q = T.mont, qP = S.TP.mont;
    const u64 *dsrc = digits + ct * ndigits * 2 * N;
    const ulonglong2 *key = reinterpret_cast<const ulonglong2 *>(keys2) + (size_t)terms.key[e] * ndigits * 4 * N;
    u64 sum[PER], tp[PER];      // modulo q and modulo P, at most 4 (at most three digits)
    {
        int src[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) src[k] = galois_index(tid + k * NT, gal);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            sum[k] = h ? 0 : mont<WIDE, false, true>(plain_words(c0[src[k]]), S.Pq, q);
            tp[k] = 0;
        }
        for (int j = 0; j < ndigits; ++j) {
            const ulonglong2 *kq = key + (size_t)(4 * j + h) * N, *kP = key + (size_t)(4 * j + 2 + h) * N;
            const u64 *djq = j == ndigits - 1 ? c1 : dsrc + (size_t)(2 * j) * N;       // folded keys modulo q
            const u64 bias = j == ndigits - 1 ? BIAS : 0;
            const u64 *djP = dsrc + (size_t)(2 * j + 1) * N;
#pragma unroll
            for (int k = 0; k < PER; k += 2) {
                const u64 qa = djq[src[k]], qb = djq[src[k + 1]], Pa = djP[src[k]], Pb = djP[src[k + 1]];
                const ulonglong2 wqa = pair_at(kq + k * NT, tid), wqb = pair_at(kq + (k + 1) * NT, tid),
                                 wPa = pair_at(kP + k * NT, tid), wPb = pair_at(kP + (k + 1) * NT, tid);
                mont2<WIDE, false, IN_PLACE>(sum[k], sum[k + 1], biased_words(qa + bias), wqa, biased_words(qb + bias), wqb, q);
                mont2<WIDE, false, IN_PLACE>(tp[k], tp[k + 1], biased_words(Pa), wPa, biased_words(Pb), wPb, qP);
                if (k == 2) __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    u64 a[PER];
    // LDS phases: B (ownership change), A B A (inverse), B A B A (forward), then reads of A
#pragma unroll
    for (int k = 0; k < PER; ++k) bufB[pad<ALONE_S>(tid + k * NT)] = mont<WIDE, false, true>(plain_words(tp[k]), S.TP.one, qP);
    __syncthreads();
    {
        const u64 *pi = bufB + pad<ALONE_S>(tid << 3);
#pragma unroll
        for (int k = 0; k < PER; ++k) a[k] = pi[k];
    }
    inverse_in_regs<WIDE, ALONE_S>(a, bufA, bufB, S.TP, tid);
#pragma unroll
    for (int k = 0; k < PER; ++k) a[k] = csub_dev(a[k], T.mod.q);
    forward_to_lds<WIDE, ALONE_S>(a, bufA, bufB, T, tid);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = tid + k * NT;
        const u64 minus = shrink(bufA[pad<ALONE_S>(i)], q) - sum[k];
        out[i] = unsign(mont<WIDE, false, true>(biased_words(minus), S.minus_Pinv, q), T.mod.q);
    }
}

#endif

// out[item] = sum over the first `used` partial ciphertexts of the item (mod q).  A workgroup owns 64 consecutive
// words; its SG wavefronts each add every SG-th partial (independent loads, several in flight) and the SG sums
// meet in LDS: with one input and a few hundred partials a single thread per word would wait for them one by one.
template <int SG>
__global__ __launch_bounds__(64 * SG) void sum_partials_kernel(const u64 *partial, int slots, int used, u64 *out, size_t words,
                                                               u64 q) {
    __shared__ u64 red[SG][64];
    const int lane = threadIdx.x & 63, sg = threadIdx.x >> 6;
    const size_t id = (size_t)blockIdx.x * 64 + lane;          // words is a multiple of 2N, so of 64
    const size_t item = id / (2 * N), e = id % (2 * N);
    const u64 *src = partial + item * slots * 2 * N + e;
    u64 acc = 0;
#pragma unroll 4
    for (int s = sg; s < used; s += SG) acc = add_mod(acc, src[(size_t)s * 2 * N], q);
    red[sg][lane] = acc;
    __syncthreads();
    if (sg) return;
#pragma unroll
    for (int g = 1; g < SG; ++g) acc = add_mod(acc, red[g][lane], q);
    out[id] = acc;
}

// the same with one thread per word, for a handful of partials, MOST at most, all of them requested together (one after the other a
// convolution of 13x11x24 to 40 channels at batch 5 took 66.1 us from wire to wire, 64.8 now)
template <int MOST>
__global__ void sum_few_partials_kernel(const u64 *partial, int slots, int used, u64 *out, size_t words, u64 q) {
    const size_t id = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= words) return;
    const size_t item = id / (2 * N), e = id % (2 * N);
    const u64 *src = partial + item * slots * 2 * N + e;
    u64 v[MOST], acc = 0;
#pragma unroll
    for (int s = 0; s < MOST; ++s) v[s] = src[(size_t)min(s, used - 1) * 2 * N];
#pragma unroll
    for (int s = 0; s < MOST; ++s) acc = add_mod(acc, s < used ? v[s] : 0, q);
    out[id] = acc;
}

}  // namespace

static ulonglong2 as_words(const MontPair &w) { return make_ulonglong2(w.a, w.b); }
static RingTables make_tables(const MontPair *pairs, const NttHost &h) {
    RingTables T;
    T.tw = reinterpret_cast<const ulonglong2 *>(pairs);
    T.itw = T.tw + FWD_PAIRS;
    T.digits = h.digit_sums ? reinterpret_cast<const u64 *>(T.itw + INV_TWIST + N) : nullptr;
    for (int e = 0; e < 3; ++e) T.w8[e] = as_words(h.w8m[e]);
    T.one = as_words(h.one_m);
    T.mod = h.mod;
    u32 inv = (u32)h.mod.q;                           // Newton's iteration for m^-1 mod 2^32 (m is odd)
    for (int i = 0; i < 5; ++i) inv *= 2 - (u32)h.mod.q * inv;
    T.mont.inv = inv;
    T.mont.lo = (int)(u32)h.mod.q;
    T.mont.nlo = -T.mont.lo;
    T.mont.nhi = -(int)((h.mod.q + BIAS) >> 32);
    return T;
}
// Runs go(std::integral_constant<bool, WIDE>).  WIDE = false needs |y| <= 7 2^60, which the bounds of the passes keep up to n = 2048 for
// moduli close to 2^60, and low words up to 2^28 (with a special prime both moduli).  Primes searched from 2^60 down are
// close to it; the low word is a matter of luck unless 2n is all that the prime has to fit.
// The same variant also transforms modulo the plaintext prime, 2^26 <= p < 2^31, whose low word is p itself: |m0| <= 2^31, but
// the constants are at most p / 2 < 2^30 and a value stays below 20 p < 2^36 (shrink adds p to a negative one), so |y0 A0| + |k m0| +
// |y1 B0| <= 2^61 + 2^62 + 2^35.  A plaintext prime of 2^31 or more is refused by gala_ctx_create.
template <class Go>
static auto by_width(const gala_ctx *c, Go go) {
#if GALA_LOGN < 12
    auto narrow = [](u64 m) {
        const int lo = (int)(u32)m;
        return m >= (1ull << 60) - (1ull << 56) && lo <= 1 << 28 && lo >= -(1 << 28);
    };
    if (narrow(c->q) && (!c->special || narrow(c->special))) return go(std::false_type{});
#endif
    return go(std::true_type{});
}
#if GALA_LOGN < 13
static SpecialJob make_special(const gala_ctx *c) {
    SpecialJob S;
    S.TP = make_tables(c->d_tw2P, c->ntt_P);
    S.Pq = as_words(c->Pq_m);
    S.minus_Pinv = as_words(c->minus_Pinv_m);
    return S;
}
#endif

static SmallTables make_small(const gala_ctx *c) {
    SmallTables S{};
    if (!c->d_tw32p) return S;
    S.tw = reinterpret_cast<const uint2 *>(c->d_tw32p);
    S.itw = S.tw + FWD_PAIRS;
    S.p = (u32)c->p;
    S.one_s = (u32)((1ull << 32) / c->p);
    for (int e = 0; e < 3; ++e) S.w8[e] = make_uint2((u32)c->ntt_p.w8[e], (u32)((c->ntt_p.w8[e] << 32) / c->p));
    return S;
}

// whether a launch of so many workgroups leaves a CU at most two wavefronts per SIMD: two workgroups at n = 2048.  A workgroup of
// n = 8192 has four per SIMD by itself, 128 registers each, whatever the launch.
static bool few(size_t workgroups) { return workgroups * NT <= (size_t)256 * 4 * 2 * 64; }
static int launch_perm(const gala_ctx *c, void *stream, const PermJob &job, const MaskJob &mj) {
    hipStream_t st = (hipStream_t)stream;
    const RingTables T = make_tables(c->d_tw2, c->ntt_q);
    const dim3 grid((unsigned)(job.items * job.nchunks + (mj.enabled && !mj.first_chunk ? job.items : 0)));
    if (job.in8_S && job.w) return (int)hipErrorInvalidValue;
    return by_width(c, [&](auto width) {
        constexpr bool WIDE = decltype(width)::value;
#if GALA_LOGN < 13
        if (c->special) {
            const SpecialJob S = make_special(c);
            auto go = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, grid, dim3(NT), 0, st, job, T, S, mj, c->gadget_bits, c->ndigits);
            };
#if GALA_LOGN == 12
            if (mj.first_chunk) {
                if (job.w) go(perm_accumulate_special_ring<WIDE, true, false, true>);
                else if (job.in8_S) go(perm_accumulate_special_ring<WIDE, false, true, true>);
                else go(perm_accumulate_special_ring<WIDE, false, false, true>);
                return (int)hipGetLastError();
            }
#endif
            if (job.w) go(perm_accumulate_special_ring<WIDE, true>);
            else if (job.in8_S) go(perm_accumulate_special_ring<WIDE, false, true>);
            else go(perm_accumulate_special_ring<WIDE, false>);
            return (int)hipGetLastError();
        }
#endif
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(NT), 0, st, job, T, mj, c->gadget_bits, c->ndigits);
        };
#if GALA_LOGN == 12
        if (mj.first_chunk) {        // with all constants at the start the layer 500x1024 at batch 8 takes 76.7 us, 74.4 without
            if (job.w) go(perm_accumulate_ring<WIDE, true, false, false, true>);
            else if (job.in8_S) go(perm_accumulate_ring<WIDE, false, true, false, true>);
            else go(perm_accumulate_ring<WIDE, false, false, false, true>);
            return (int)hipGetLastError();
        }
#endif
#if GALA_LOGN < 13
        if (few(grid.x)) {
            if (job.w) go(perm_accumulate_ring<WIDE, true, false, true>);
            else if (job.in8_S) go(perm_accumulate_ring<WIDE, false, true, true>);
            else go(perm_accumulate_ring<WIDE, false, false, true>);
            return (int)hipGetLastError();
        }
#endif
        if (job.w) go(perm_accumulate_ring<WIDE, true>);
        else if (job.in8_S) go(perm_accumulate_ring<WIDE, false, true>);
        else go(perm_accumulate_ring<WIDE, false>);
        return (int)hipGetLastError();
    });
}

static int perm(const gala_ctx *c, void *stream, const PermJob &job) {
    MaskJob mj{};
    mj.enabled = 0;
    return launch_perm(c, stream, job, mj);
}

static int perm_masked(const gala_ctx *c, void *stream, const PermJob &job, const FinalizeJob &fin) {
    MaskJob mj{};
    mj.enabled = 1;
    mj.first_chunk = !job.product_only && mask_in_first_chunk(job);
    const int used = job.nchunks + !mj.first_chunk;      // partial ciphertexts
    mj.nout = fin.nout;
    mj.r = fin.r;
    mj.r_stride = fin.r_stride;
    mj.mask_seed = fin.mask_seed;
    mj.layout = fin.mask;
    mj.pbits = c->pbits;
    mj.delta = as_words(c->delta_m);
    mj.Tp = make_tables(c->d_tw2p, c->ntt_p);
    mj.small = make_small(c);
    hipStream_t st = (hipStream_t)stream;
    const bool timed = c->prof_which == 0 && (size_t)(2 * c->prof_used + 1) < c->prof_events.size();
    if (timed) (void)hipEventRecord((hipEvent_t)c->prof_events[2 * c->prof_used], st);
    int rc;
    // One launch writes an item as soon as it is done, while other items are still read: only in place or with the inputs
    // and outputs apart, and not with the outputs over the shares r.  Otherwise the outputs are written by a second launch.
    const size_t span = (size_t)job.items * 2 * N;
    const bool apart = fin.ct_out == job.ct_in || fin.ct_out + span <= job.ct_in || job.ct_in + span <= fin.ct_out;
    const u64 *r_end = fin.r + (size_t)(job.items / fin.nout) * fin.r_stride;
    const bool r_apart = fin.ct_out + span <= fin.r || r_end <= fin.ct_out;
    const bool alone = job.product_only && apart && r_apart;
    if (alone) {
        rc = by_width(c, [&](auto width) {
            constexpr bool WIDE = decltype(width)::value;
            auto go = [&](auto kernel, int groups) {
                hipLaunchKernelGGL(kernel, dim3((unsigned)job.items), dim3(NT * groups), 0, st, job, make_tables(c->d_tw2, c->ntt_q),
                                   mj, fin.ct_out);
                return (int)hipGetLastError();
            };
#if GALA_LOGN <= 11
            if (few(2 * (size_t)job.items)) return go(scmult_masked_ring<WIDE, 2, true>, 2);
#endif
#if GALA_LOGN < 13       // a workgroup of n = 8192 leaves no registers idle
            if (few((size_t)job.items)) return go(scmult_masked_ring<WIDE, 1, true>, 1);
#endif
            return go(scmult_masked_ring<WIDE, 1, false>, 1);
        });
    } else {
        rc = launch_perm(c, stream, job, mj);
    }
    if (timed) (void)hipEventRecord((hipEvent_t)c->prof_events[2 * c->prof_used++ + 1], st);
    if (rc || alone) return rc;
    const size_t words = span;
    // many partials of few items: more wavefronts per word
    auto few_partials = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, job.partial, job.slots, used, fin.ct_out, words,
                           c->q);
    };
    if (used <= 2) few_partials(sum_few_partials_kernel<2>);
    else if (used <= 4) few_partials(sum_few_partials_kernel<4>);
    else if (used <= 8) few_partials(sum_few_partials_kernel<8>);
    else if (used > 64 && words / 64 < 2048)
        hipLaunchKernelGGL(sum_partials_kernel<16>, dim3((unsigned)(words / 64)), dim3(1024), 0, st, job.partial, job.slots,
                           used, fin.ct_out, words, c->q);
    else
        hipLaunchKernelGGL(sum_partials_kernel<4>, dim3((unsigned)(words / 64)), dim3(256), 0, st, job.partial, job.slots,
                           used, fin.ct_out, words, c->q);
    return (int)hipGetLastError();
}

template <bool WIDE>
static int decperm(const gala_ctx *c, hipStream_t st, const u64 *ct_in, size_t count, const RingTables &T, u64 *digits) {
    const size_t workgroups = count * (c->ndigits - 1);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)workgroups), dim3(NT), 0, st, ct_in, digits, T, c->gadget_bits, c->ndigits - 1);
    };
    // at n = 8192 all constants at the start spill 68 registers: eight rotations of eight inputs 47.3 us, 33.5 without
    if constexpr (LOGN < 13) {
        if (few(workgroups)) {
            go(decperm_ring<WIDE, true>);
            return (int)hipGetLastError();
        }
    }
    go(decperm_ring<WIDE, false>);
    return (int)hipGetLastError();
}
static int hoist_taps(const gala_ctx *c, void *stream, const u64 *ct_in, int batch, const TermList &terms,
                           bool any_rotation, const u64 *keys2, u64 *digits, u64 *xrot) {
    if (batch <= 0 || terms.nterm <= 0) return 0;
    const size_t count = (size_t)batch * terms.nin;
    const RingTables T = make_tables(c->d_tw2, c->ntt_q);
    hipStream_t st = (hipStream_t)stream;
    const dim3 per_term((unsigned)((size_t)batch * terms.nterm));
    return by_width(c, [&](auto width) {
        constexpr bool WIDE = decltype(width)::value;
#if GALA_LOGN < 13
        if (c->special) {     // digits[ct][j][modulus][N]: twice the digit storage of the one-prime form
            const SpecialJob S = make_special(c);
            if (any_rotation) {
                hipLaunchKernelGGL(decperm_special_ring<WIDE>, dim3((unsigned)(count * (2 * c->ndigits - 1))), dim3(NT), 0, st, ct_in,
                                   digits, T, S.TP, c->gadget_bits, c->ndigits);
                const int rc = (int)hipGetLastError();
                if (rc) return rc;
            }
            hipLaunchKernelGGL(hstperm_special_ring<WIDE>, dim3(per_term.x, 2), dim3(NT), 0, st, ct_in, digits, terms, keys2, xrot, T, S,
                               c->ndigits);
            return (int)hipGetLastError();
        }
#endif
        if (any_rotation && c->ndigits > 1) {
            const int rc = decperm<WIDE>(c, st, ct_in, count, T, digits);
            if (rc) return rc;
        }
        hipLaunchKernelGGL(hstperm_taps_ring<WIDE>, per_term, dim3(NT), 0, st, ct_in, digits, terms, keys2, xrot, T, c->ndigits);
        return (int)hipGetLastError();
    });
}

// DecPerm (when any term rotates) followed by the HstPerm of every term, written as the column image
static int hstperm_pack(const gala_ctx *c, void *stream, const u64 *ct_in, u64 *digits, int batch,
                             const TermList &terms, bool any_rotation, const u64 *keys2, u64 *xl) {
    if (batch <= 0 || terms.nterm <= 0) return 0;
    const RingTables T = make_tables(c->d_tw2, c->ntt_q);
    hipStream_t st = (hipStream_t)stream;
    const int eblocks = (terms.nterm + 15) / 16, kblocks = (terms.nterm + 63) / 64;
    const dim3 grid(N / 64, (unsigned)eblocks, (unsigned)((batch + 3) / 4));
    v4i_t *out = reinterpret_cast<v4i_t *>(xl);
    if (any_rotation && !keys2) return (int)hipErrorInvalidValue;
    return by_width(c, [&](auto width) {
        constexpr bool WIDE = decltype(width)::value;
        if (any_rotation && c->ndigits > 1) {
            const int rc = decperm<WIDE>(c, st, ct_in, (size_t)batch * terms.nin, T, digits);
            if (rc) return rc;
        }
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(PACK_THREADS), 0, st, ct_in, digits, terms, kblocks, keys2, out, T, c->ndigits, batch);
        };
        if (!any_rotation) go(hstperm_pack_ring<WIDE, 0, false>);
        else if (c->ndigits == 3) go(hstperm_pack_ring<WIDE, 3, true>);
        else go(hstperm_pack_ring<WIDE, 0, true>);
        return (int)hipGetLastError();
    });
}

static int ntt(const gala_ctx *c, void *stream, const u64 *src, u64 *dst, size_t count, int inverse, bool special) {
    if (!count) return 0;
    const RingTables T = special ? make_tables(c->d_tw2P, c->ntt_P) : make_tables(c->d_tw2, c->ntt_q);
    return by_width(c, [&](auto width) {
        constexpr bool WIDE = decltype(width)::value;
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)count), dim3(NT), 0, (hipStream_t)stream, src, dst, T);
        };
        if (inverse) go(ntt_ring<WIDE, true>);
        else go(ntt_ring<WIDE, false>);
        return (int)hipGetLastError();
    });
}

static int encrypt(const gala_ctx *c, void *stream, const MontPair *s_hat, const u64 *slots, const u64 *seeds, int count,
                        u64 *ct_out) {
    if (!count) return 0;
    return by_width(c, [&](auto width) {
        hipLaunchKernelGGL(encrypt_ring<decltype(width)::value>, dim3((unsigned)count), dim3(NT), 0, (hipStream_t)stream, slots, seeds,
                           reinterpret_cast<const ulonglong2 *>(s_hat), ct_out, make_tables(c->d_tw2, c->ntt_q),
                           make_tables(c->d_tw2p, c->ntt_p), make_small(c), c->d_slot_to_idx, gauss_buckets(), c->qbits,
                           as_words(c->delta_m));
        return (int)hipGetLastError();
    });
}
static int decrypt(const gala_ctx *c, void *stream, const MontPair *s_hat, const u64 *ct_in, int count, u64 *slots) {
    if (!count) return 0;
    return by_width(c, [&](auto width) {
        hipLaunchKernelGGL(decrypt_ring<decltype(width)::value>, dim3((unsigned)count), dim3(NT), 0, (hipStream_t)stream, ct_in,
                           reinterpret_cast<const ulonglong2 *>(s_hat), slots, make_tables(c->d_tw2, c->ntt_q),
                           make_tables(c->d_tw2p, c->ntt_p), make_small(c), c->d_slot_to_idx, (u64)(((u128)c->p << 64) / c->q));
        return (int)hipGetLastError();
    });
}

#define GALA_RING_OPS_(logn) ring_ops_##logn
#define GALA_RING_OPS(logn) GALA_RING_OPS_(logn)
const RingOps *GALA_RING_OPS(GALA_LOGN)() {
    static const RingOps ops = {ntt, perm, perm_masked, hoist_taps, hstperm_pack, encrypt, decrypt};
    return &ops;
}

}  // namespace gala
