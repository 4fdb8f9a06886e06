// Internal data structures of the library (host side) and the launch interface
// of the HIP kernels.  Nothing here is visible through the C ABI.
#pragma once
#include <cstddef>
#include <map>
#include <vector>

#include "../../include/gala.h"
#include "modarith.h"

namespace gala {

constexpr int kMaxDigits = 32;
constexpr int kMaxN = 8192;   // rings outside 1024 .. 8192 and moduli from 2^60 on run on the any-n kernels
constexpr int kGaussBound = 19;

// Cumulative table of the discrete Gaussian (passed to kernels by value) and the draw from it: one 64-bit word
// of the counter-based generator compared with the 38 thresholds.
struct GaussCdf {
    u64 t[2 * kGaussBound];   // floor(2^64 * P[X <= -bound + i])
};
// The same by the draw's top byte, for kernels that make many draws: how many thresholds the byte's whole range has passed, and
// kSeveral where more than one lies inside of it (the tails; elsewhere thresholds are further apart than a range is wide).
struct GaussBuckets {
    static constexpr unsigned char kSeveral = 64;
    u64 t[2 * kGaussBound];
    unsigned char passed[256];
};
GALA_HD int draw_gauss_cdf(const GaussCdf &cdf, u64 seed, u64 stream, u64 idx) {
    const u64 u = rand64(seed, stream, idx, 0);
    int x = -kGaussBound;
    for (int i = 0; i < 2 * kGaussBound; ++i) x += u >= cdf.t[i] ? 1 : 0;
    return x;
}

// Entries g0 .. g1-1 of a rotate-and-accumulate sum that chunk `chunk` of `nchunks` takes.  The first entry is the
// rotation by zero in he_fc and he_conv (a ScMult and no key switch): it rides with chunk 0, and the G-1 entries
// after it are spread evenly, so that no workgroup is launched for the cheap entry alone.
GALA_HD void chunk_range(int chunk, int nchunks, int G, int &g0, int &g1) {
    // 32 bits hold the products: chunk < G <= kMaxN; a workgroup starts with these divisions
    g0 = chunk ? 1 + (int)((u32)chunk * (u32)(G - 1) / (u32)nchunks) : 0;
    g1 = 1 + (int)((u32)(chunk + 1) * (u32)(G - 1) / (u32)nchunks);
}

// ---------------------------------------------------------------------------
// Negacyclic number-theoretic transform tables for one modulus.
// Forward: natural-order coefficients -> values a(psi^(2*brev(i)+1)) at index i.
// tw[m+i] = psi^brev(m+i) for the stage with m blocks; itw holds the inverses.
// The inverse folds n^-1 into its last stage (ninv, itw1n = itw[1]*ninv).
// ---------------------------------------------------------------------------
struct NttHost {
    int n = 0, logn = 0;
    Modulus mod{};
    u64 psi = 0;
    std::vector<u64> tw, tws, itw, itws;
    u64 ninv = 0, ninvs = 0, itw1n = 0, itw1ns = 0;
    u64 w8[3] = {0, 0, 0};                       // powers 1, 2, 3 of psi^(-2n/8)
    MontPair w8m[3] = {}, one_m{};               // ... and the constant 1 for the ring kernels
    bool digit_sums = false;                     // the context's gadget digits fit the ring kernels' sums of products (digit_pass_constants)

    void init(int n, u64 q, u64 psi);
    void forward(u64 *a) const;   // in place, canonical in -> canonical out
    void inverse(u64 *a) const;
};

// Device view of the same tables (pointers into one device allocation).
struct NttDev {
    const u64 *tw, *tws, *itw, *itws;
    u64 ninv, ninvs, itw1n, itw1ns;
    Modulus mod;
};

constexpr int kDigitPassWords = 22;
bool digit_pass_constants(const NttHost &h, int gadget_bits, u64 *words);

u64 pow_mod(u64 b, u64 e, u64 m);
u64 inv_mod(u64 a, u64 m);
u64 shoup_companion(u64 w, u64 q);
Reciprocal make_reciprocal(u64 q);
MontMaker make_mont(u64 m);
Modulus make_modulus(u64 q);
bool is_prime_u64(u64 v);
int bit_length(u64 v);
inline int brev(int v, int bits) {
    int r = 0;
    for (int b = 0; b < bits; ++b) r |= ((v >> b) & 1) << (bits - 1 - b);
    return r;
}

}  // namespace gala

// ---------------------------------------------------------------------------
// Handles
// ---------------------------------------------------------------------------
struct gala_ctx {
    int n = 0, logn = 0, gadget_bits = 0, ndigits = 0, pbits = 0, qbits = 0;
    gala::u64 q = 0, p = 0, delta = 0, delta_s = 0, zeta = 0;
    gala::NttHost ntt_q, ntt_p;
    // special prime of key switching (0: keys modulo q only)
    gala::u64 special = 0, Pq = 0, Pinv = 0;   // P mod q and P^-1 mod q
    gala::NttHost ntt_P;
    gala::MontPair delta_m{}, Pq_m{}, minus_Pinv_m{};   // delta, P and -P^-1 mod q for the ring kernels
    std::vector<int> slot_to_idx;      // slot s -> index of its value in the mod-p transform
    int device = 0;
    bool has_device = false;           // tables uploaded; false on a host without a HIP device
    gala::u64 *d_tables = nullptr;     // 8*n words: tw,tws,itw,itws for q then for p
    int *d_slot_to_idx = nullptr;
    gala::MontPair *d_tw2 = nullptr;        // ring kernels only: twiddles (MontPair) in the order of the radix-8 passes, forward then inverse
    gala::MontPair *d_tw2p = nullptr;       // the same for the plaintext modulus, or null when p < 2^26
    gala::u32 *d_tw32p = nullptr;      // ... with 32-bit words and companions floor(w 2^32 / p), when p < 2^26; else null
    gala::u64 *d_tablesP = nullptr;    // 4*n words: tw,tws,itw,itws for the special prime
    gala::MontPair *d_tw2P = nullptr;       // the same for the special prime
    gala::NttDev dev_q{}, dev_p{}, dev_P{};
    int key_polys() const { return special ? 4 : 2; }
    // measurement aid: event pairs recorded around rotate-and-accumulate launches
    mutable std::vector<void *> prof_events;   // 2*capacity hipEvent_t
    mutable int prof_used = 0;
    mutable int prof_which = 0;                // 0: rotate-and-accumulate launches, 1: convolution multiply-accumulate
};

struct gala_sk {
    std::vector<gala::u64> s;          // coefficients mod q (0, 1, q-1)
    std::vector<gala::u64> s_hat;      // forward transform of s
    gala::u64 *d_s_hat = nullptr;      // device copy of s_hat (null on a host without a device)
    gala::MontPair *d_s_pairs = nullptr;   // the same as MontPairs, for the ring kernels
};

struct gala_gk {
    const gala_ctx *ctx = nullptr;     // the context the keys were generated for (plans of another context refuse them)
    int n = 0, ndigits = 0, polys = 2; // polynomials per digit: (b, a) mod q, then (b, a) mod P with a special prime
    std::map<int, int> index_of;       // Galois element -> key index
    std::vector<int> elements;
    gala::u64 *d_keys = nullptr;       // nkeys x ndigits x polys x n, evaluation domain (b then a)
    gala::u64 *d_keys2 = nullptr;      // the folded keys as MontPairs for the ring kernels, or null
    int *d_elements = nullptr;         // nkeys Galois elements, device
    int *d_iota = nullptr;             // 0,1,2,... (key index of element k is k), device
    int *d_one = nullptr;              // the single value 1 (Galois element of the identity), device
    int *d_zeros = nullptr;            // nkeys zeros (every hoisted rotation reads input ciphertext 0 of its item), device
    size_t key_words() const { return (size_t)ndigits * polys * n; }
};

// A slot in one word: its position in the mod-p transform's input, its row, whether it is in a row at all and whether it
// is the row's first.
struct MaskSlot {
    static constexpr int kBits = 13, kFirst = 1 << 26, kInRow = 1 << 27;      // positions and rows are below n <= 8192
};

// Device description of how the server's mask is laid out in one output
// ciphertext: which slots are drawn from the generator and which absorb r.
struct MaskLayoutHost {
    int nout = 0;                      // output ciphertexts
    std::vector<int> row_ptr;          // nout x (n+1): CSR over the "rows" (outputs) of each ciphertext
    std::vector<int> row_slots;        // nout x n: slots of each row, first slot first
    std::vector<int> row_rindex;       // nout x n: index into r of each row
    std::vector<int> nrows;            // nout
    std::vector<unsigned char> is_first;  // nout x n: slot is the first of a real row (not drawn)
};
struct MaskLayoutDev {
    int *row_ptr = nullptr, *row_slots = nullptr, *row_rindex = nullptr, *nrows = nullptr;
    unsigned char *is_first = nullptr;
    int *slot_rowid = nullptr;         // nout x n: the row a slot belongs to, -1 for slots outside every row
    // nout x n pairs, by slot: what the ring kernels' masks need to know of it (MaskSlot), and the index into r of the row
    // whose first slot it is
    int *slot_mask = nullptr;
    int *row_first = nullptr;          // nout x n pairs, by row: the position of its first slot (-1: a row without slots) and its index into r
    bool sums = false;                 // some row has more than one slot
    bool strided = false;              // most slots of rows are n / 8 slots, a mask's threads, away from the next of their row
};

struct gala_fc_plan {
    gala_ctx *ctx = nullptr;
    int n_o = 0, n_i = 0, nop = 0, nip = 0, G = 0;
    bool big = false;
    std::vector<int> slot_row;         // padded row of each slot, -1 if it carries no weight
    std::vector<int> gal;              // Galois element of rotation g (gal[0] = 1)
    gala::u64 *d_w = nullptr;          // G x n encoded weights, evaluation domain
    gala::u64 *d_w2 = nullptr;         // the same as MontPairs for the ring kernels, or null: G polynomials in
                                       // natural order, then the same G in the threads' ownership order
    int *d_gal = nullptr;              // G Galois elements
    int *d_key_idx = nullptr;          // G key indices (valid once bound)
    const gala_gk *bound = nullptr;
    MaskLayoutHost mask_h;
    MaskLayoutDev mask_d;
};

// The hybrid matrix-vector product of Sec. III-A(2) (comparison schedule): G diagonal vectors that multiply the
// input rotated by 0..G-1, then rotate-and-sum steps on the running ciphertext.
struct gala_fc_hybrid_plan {
    gala_ctx *ctx = nullptr;
    int n_o = 0, n_i = 0, nop = 0, nip = 0, G = 0, R = 0;
    bool big = false;
    std::vector<int> in_gal;           // Galois elements of the input rotations g = 0..G-1 (in_gal[0] = 1)
    std::vector<int> ras_gal;          // Galois elements of the rotate-and-sum steps, in order
    std::vector<int> result_slot;      // slot that holds output t after the last step
    gala::u64 *d_w = nullptr;          // G x n diagonal vectors, evaluation domain
    int *d_in_ct = nullptr, *d_in_gal = nullptr, *d_in_key = nullptr;   // G each: the term list of the input rotations
    int *d_ras_gal = nullptr, *d_ras_key = nullptr;   // per step the pair (1, gal) / (-1, key index): 2 ints each
    const gala_gk *bound = nullptr;
    MaskLayoutHost mask_h;
    MaskLayoutDev mask_d;
};

struct gala_conv_plan {
    gala_ctx *ctx = nullptr;
    int c_o = 0, c_i = 0, k_h = 0, k_w = 0, u_h = 0, u_w = 0;
    int T = 0, cn = 0, hpos = 0, nin = 0, nout = 0, ntap = 0, centre = 0;
    std::vector<int> tap_gal, grp_gal; // Galois elements of taps (ntap) and kernel orders (cn)
    // Terms of the multiply-accumulate: the (input ciphertext, tap) pairs whose encoded kernels are not all zero,
    // in (tap, input) order: consecutive terms share their tap, i.e. their rotation and key, which the kernel that
    // rotates the inputs sixteen terms at a time loads once.  A dense kernel has nin*ntap of them.
    int nterm = 0, nrot_terms = 0, nrot_cts = 0;   // terms; those that rotate; input ciphertexts with a rotating term
    std::vector<int> term_ct, term_tap;
    int *d_term_ct = nullptr, *d_term_gal = nullptr, *d_term_key = nullptr;   // nterm each (key valid once bound)
    gala::u64 *d_w = nullptr;          // nout x cn x nterm x n encoded kernels, evaluation domain
    gala::u64 *d_wl = nullptr;         // the same as balanced base-256 digit planes for the matrix-core path, or null
    int *d_grp_gal = nullptr, *d_grp_key = nullptr;   // cn
    // output-rotation schedule (Sec. III-B(2)): entry gam * nin + I of an output ciphertext's sum is the block of input
    // ciphertext I in kernel order gam; seg_ptr[I] .. seg_ptr[I+1]-1 are the terms of input ciphertext I
    int *d_or_gal = nullptr, *d_or_key = nullptr;     // cn * nin
    int *d_seg_ptr = nullptr, *d_seg_terms = nullptr;  // nin + 1 offsets into the nterm term numbers grouped by input ciphertext
    const gala_gk *bound = nullptr;
    MaskLayoutHost mask_h;
    MaskLayoutDev mask_d;
};

// ---------------------------------------------------------------------------
// Kernel launchers (defined in gala_kernels.hip).  All return a hipError_t cast to int.
// ---------------------------------------------------------------------------
namespace gala {

// resolves, once per device, the device address of the fixed scratch array behind gala_he_fc_static (gala_api.cpp)
int static_scratch_init();

// batched transform of `count` polynomials of n words: inverse=0 forward.
int launch_ntt(const gala_ctx *ctx, void *stream, const u64 *src, u64 *dst, size_t count, int inverse);
// the same with the tables of another modulus of the context (dev_q, dev_p or dev_P)
int launch_ntt_mod(const gala_ctx *ctx, void *stream, const u64 *src, u64 *dst, size_t count, int inverse, const NttDev &T);
// Batched client steps on internal-form ciphertexts (one workgroup per ciphertext).
int launch_encrypt(const gala_ctx *ctx, void *stream, const gala_sk *sk, const u64 *slots, const u64 *seeds, int count,
                   u64 *ct_out);
int launch_decrypt(const gala_ctx *ctx, void *stream, const gala_sk *sk, const u64 *ct_in, int count, u64 *slots);
const u64 *gauss_cdf_table();
const GaussBuckets &gauss_buckets();
// Stand-alone Add / ScMult / plaintext operations on internal-form buffers (op: 0 add ct, 1 scmult, 2 sub plain, 3 add plain).
int launch_encode_plain(const gala_ctx *ctx, void *stream, const u64 *slots, int count, int mode, u64 *plain);
int launch_ct_op(const gala_ctx *ctx, void *stream, int op, const u64 *a, const u64 *b, size_t b_stride, int count, u64 *out);
// "encode" of a convolution plan on the device (Sec. III-B(3), kernel grouping): slot vectors of the encoded kernels
// `first` .. `first + count - 1` in (O, gamma, term) order, from the kernel tensor K (c_o x c_i x k_h x k_w, device)
struct ConvGeom {
    int c_o, c_i, k_h, k_w, u_h, u_w, T, cn, hpos, nterm, n;
    u64 p;
};
int launch_conv_weight_slots(const gala_ctx *ctx, void *stream, const u64 *K, const ConvGeom &g, const int *term_ct,
                             const int *term_tap, size_t first, size_t count, u64 *slots);
// "encode" of an FC plan on the device: slot vectors of the encoded weights g = 0..count-1 from W (n_o x n_i, device)
// and the plan's slot -> padded row table (n ints, device; -1: the slot carries no weight).  rotate_output: GALA's
// row-wise encoding (the product is rotated by g afterwards); otherwise the hybrid method's diagonals (the input is
// rotated by g before the product).
struct FcGeom {
    int n, n_o, n_i, nip, big, rotate_output;
    u64 p;
};
int launch_fc_weight_slots(const gala_ctx *ctx, void *stream, const u64 *W, const FcGeom &g, const int *slot_row, int count,
                           u64 *slots);
// out[b][rindex of row t] = sum of the row's slots mod p, for `count` items of nout slot vectors each
int launch_unpack_share(const gala_ctx *ctx, void *stream, const u64 *slots, int count, int nout, const MaskLayoutDev &layout,
                        size_t out_stride, u64 *out);

// key generation helper on `npairs` consecutive (t_hat, a_hat) pairs of n-word evaluation-domain
// polynomials: t_hat <- t_hat - a_hat * s_hat in place (s_hat shared by all pairs).
int launch_key_finish(const gala_ctx *ctx, void *stream, u64 *pairs, const u64 *s_hat, size_t npairs, const Modulus &mod);
// dst[i] = the MontPair of src[i] mod q for i < count: the constants that the ring kernels multiply by.
int launch_pair_pack(const gala_ctx *ctx, void *stream, const u64 *src, u64 *dst, size_t count);
// the same for nkeys whole key-switching keys, with the last digit's key folded into the others (key_pack_kernel)
int launch_key_pack(const gala_ctx *ctx, void *stream, const u64 *src, u64 *dst, size_t nkeys);
// dst[poly][512*(t/64) + 64*k + t%64] = src[poly][8*t + k] on 16-byte pairs of polynomials: the order in which
// the threads of the Perm kernel read the 8 consecutive coefficients they own - one coalesced load per k, the eight of
// a wavefront within 8 KiB
int launch_owner_order(void *stream, const u64 *src_pairs, u64 *dst_pairs, size_t npolys, int n);
// whether the context has kernels of its ring's own (ring_ops)
bool uses_fast_perm(const gala_ctx *ctx);

// One job of the rotate-and-accumulate kernel.  For item in [0,items), chunk in [0,nchunks):
//   partial[item][chunk] = sum over g in the chunk of Perm_{gal[g]}( in[item][g] (.) w[g] )
// where in[item][g] = ct_in + item*in_item_stride + g*in_g_stride (2n words each) and w[g] = w + g*n
// (w == nullptr: no ScMult).  gal[g] == 1 means no rotation.  key_idx[g] selects the key.
struct PermJob {
    const u64 *ct_in;
    size_t in_item_stride, in_g_stride;
    const u64 *w;
    const int *gal, *key_idx;
    const u64 *keys;
    const u64 *w2, *keys2;   // MontPair images of w and keys (ring kernels only)
    const int *in_g_index;   // optional: rotation g reads input number in_g_index[g] instead of g
    // ring kernels only, in8_S != 0: the inputs are the matrix-core product's sums in blocks of eight coefficients,
    // word (i/8)*in8_S + i%8 of a polynomial, c1 eight words after c0; item = b*in8_nout + O starts at
    // ct_in + O*in8_o_stride + 16*b and rotation g in_g_stride words further.
    size_t in8_S, in8_o_stride;
    int in8_nout;
    int G, items, nchunks;
    int slots;               // partial ciphertexts reserved per item (>= nchunks)
    u64 *partial;            // items x slots x 2n
    bool product_only;       // G = 1, gal[0] = 1 and weights: no rotation at all
};
int launch_perm_accumulate(const gala_ctx *ctx, void *stream, const PermJob &job);

// out[item] = sum_chunk partial[item][chunk] - mask(item) ; mask built from r and the generator.
struct FinalizeJob {
    const u64 *partial;
    int items, nchunks;
    int slots;               // partial ciphertexts reserved per item (>= nchunks)
    int nout;                // output ciphertexts per batch element (item = b*nout + O)
    const u64 *r;            // batch x r_stride values mod p (nullptr: no mask)
    size_t r_stride;
    u64 mask_seed;
    MaskLayoutDev mask;
    u64 *ct_out;             // items x 2n
};
int launch_finalize(const gala_ctx *ctx, void *stream, const FinalizeJob &job);
// Rotate-and-accumulate followed by share generation.  With the ring kernels the mask of every
// item is built by extra workgroups of the same launch (as one more partial ciphertext, slot
// `nchunks`, so job.slots must be >= nchunks + 1) and a light kernel adds the partials up;
// otherwise this is launch_perm_accumulate + launch_finalize.
int launch_perm_finalize(const gala_ctx *ctx, void *stream, const PermJob &job, const FinalizeJob &fin);

// DecPerm of `count` ciphertexts: digits[c][j] = forward(digit_j(inverse(c1))), j < ndigits.
int launch_decperm(const gala_ctx *ctx, void *stream, const u64 *ct_in, size_t count, u64 *digits);
#if defined(__HIPCC__)
// The digit planes of four balanced-digit words: out[u] = byte u of words a, b, c, d, in eight byte permutations.
__device__ __forceinline__ void transpose_bytes4(u32 a, u32 b, u32 c, u32 d, u32 (&out)[4]) {
    const u32 ab01 = __builtin_amdgcn_perm(b, a, 0x05010400), ab23 = __builtin_amdgcn_perm(b, a, 0x07030602);
    const u32 cd01 = __builtin_amdgcn_perm(d, c, 0x05010400), cd23 = __builtin_amdgcn_perm(d, c, 0x07030602);
    out[0] = __builtin_amdgcn_perm(cd01, ab01, 0x05040100);
    out[1] = __builtin_amdgcn_perm(cd01, ab01, 0x07060302);
    out[2] = __builtin_amdgcn_perm(cd23, ab23, 0x05040100);
    out[3] = __builtin_amdgcn_perm(cd23, ab23, 0x07060302);
}
// 16 balanced-digit words -> their eight digit chunks: chunk u holds byte u of every word
typedef int digit_chunk_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void digit_chunks(const u64 (&d)[16], digit_chunk_t (&c)[8]) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const u64 *t = d + 4 * w;
        u32 lo[4], hi[4];
        transpose_bytes4((u32)t[0], (u32)t[1], (u32)t[2], (u32)t[3], lo);
        transpose_bytes4((u32)(t[0] >> 32), (u32)(t[1] >> 32), (u32)(t[2] >> 32), (u32)(t[3] >> 32), hi);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            c[u][w] = (int)lo[u];
            c[4 + u][w] = (int)hi[u];
        }
    }
}
#endif

// The convolution's rotated inputs, one per (batch element, term): the description of the terms of a plan.
struct TermList {
    int nin, nterm;               // input ciphertexts per batch element, terms
    const int *ct, *gal, *key;    // per term: input ciphertext, Galois element of its tap, key index (device)
};
// HstPerm for the convolution's input rotations:
//   xrot[b][e] = HstPerm_{gal[e]}(ct_in[b*nin + ct[e]], its digits) ; a term with Galois element 1 is a copy.
int launch_hstperm_taps(const gala_ctx *ctx, void *stream, const u64 *ct_in, const u64 *digits, int batch,
                        const TermList &terms, const u64 *keys, u64 *xrot);
// acc[b][O][gam] = sum_{I,tap} w[O][gam][I][tap] (.) xrot[b][I][tap]   (both polynomials)
// seg_ptr (device, nseg + 1 ints) and seg_terms (device, term numbers) give nseg groups of terms sums of their own:
//   acc[b][O][gam][s] = sum over the terms seg_terms[seg_ptr[s] .. seg_ptr[s+1]-1]; nullptr: one sum over all terms
int launch_conv_mac(const gala_ctx *ctx, void *stream, const u64 *w, const u64 *xrot, int batch, int nout, int cn,
                    int nterm, u64 *acc, const int *seg_ptr = nullptr, const int *seg_terms = nullptr, int nseg = 1);

// Whether operands of this size, read once a launch, are worth keeping out of the caches: past the 256 MB of the
// last-level cache nothing of them is left for the next launch.  Below it they may be (13x11x24 to 40 channels at batch
// 5, 24 MB of kernels' digit planes: 81.2 us kept, 83.0 us not).
inline bool streams_past_cache(size_t bytes) { return bytes > ((size_t)256 << 20); }

// Matrix-core path of the convolution's multiply-accumulate (gala_conv_mfma.hip): digit-plane images of the
// encoded kernels (built once per plan) and of the rotated inputs (built per call), then one MFMA kernel.
void conv_mfma_geometry(int groups, int cols, int nterm, int *mtiles, int *ntiles, int *kblocks);
size_t conv_mfma_image_bytes(int n, int tiles, int kblocks);
int launch_limb_pack(const gala_ctx *ctx, void *stream, const u64 *src, int mode, int rows, int nterm, u64 *dst);
bool uses_fast_hoist(const gala_ctx *ctx);
size_t conv_mfma_tmp_bytes(int n, int mtiles, int ntiles);
// blocks_of_eight: tmp[(i/8)][row][column][i%8] instead of tmp[i][row][column] (what PermJob::in8_S describes)
int launch_conv_mfma(const gala_ctx *ctx, void *stream, const u64 *wl, const u64 *xl, int batch, int groups,
                     int nterm, u64 *tmp, bool blocks_of_eight = false);
int launch_conv_untranspose(const gala_ctx *ctx, void *stream, const u64 *tmp, int batch, int groups, u64 *acc);

// The launchers of one ring's own kernels (gala_ring_impl.h): rings of 1024 to 8192 slots, q < 2^60.
struct RingOps {
    // transform modulo q or modulo the special prime
    int (*ntt)(const gala_ctx *, void *stream, const u64 *src, u64 *dst, size_t count, int inverse, bool special);
    int (*perm)(const gala_ctx *, void *stream, const PermJob &);
    int (*perm_masked)(const gala_ctx *, void *stream, const PermJob &, const FinalizeJob &);
    // DecPerm (when any term rotates) and HstPerm of every term: as ciphertexts, or as the product's column image
    int (*hoist_taps)(const gala_ctx *, void *stream, const u64 *ct_in, int batch, const TermList &, bool any_rotation,
                      const u64 *keys2, u64 *digits, u64 *xrot);
    int (*hstperm_pack)(const gala_ctx *, void *stream, const u64 *ct_in, u64 *digits, int batch, const TermList &,
                        bool any_rotation, const u64 *keys2, u64 *xl);
    int (*encrypt)(const gala_ctx *, void *stream, const MontPair *s_hat, const u64 *slots, const u64 *seeds, int count, u64 *ct_out);
    int (*decrypt)(const gala_ctx *, void *stream, const MontPair *s_hat, const u64 *ct_in, int count, u64 *slots);
};
// the context's, or nullptr: its ring size or moduli have none and the any-n kernels serve it
const RingOps *ring_ops(const gala_ctx *ctx);

}  // namespace gala
