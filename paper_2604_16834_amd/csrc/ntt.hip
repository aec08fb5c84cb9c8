// Negacyclic NTT / inverse NTT over Z_q[X]/(X^N+1) for gfx950 (Background, "RNS Decomposition and
// NTT Optimization": the transform that makes ring multiplication quasi-linear).
//
// Forward: natural-order coefficients in, out[k] = a(psi^(2*bitrev(k)+1)).  The log2(N) radix-2
// stages are split into two passes; in each pass one 256-thread workgroup transforms a 2^11-point
// tile, every thread holding 8 points in registers:
//   hi pass : the first log_hi = log2(N) - 11 stages pair points 2^11 or more apart.  A tile is all
//             2^log_hi rows (rows are 2^11 elements apart) of a run of adjacent columns, so every
//             row segment is a contiguous, coalesced run.  Radix-8 in registers, one exchange through
//             LDS, then the remaining log_hi - 3 stages in registers.
//   lo pass : the last 11 stages act inside contiguous blocks of 2^11 points: radix 8, 8, 8, 4 in
//             registers with three exchanges through (padded, double-buffered) LDS.
// The bit-reversed output order falls out of this split with no transpose.  The inverse runs the
// mirrored lo pass first, then the mirrored hi pass, and folds the 1/N into its last store.
// Twiddles psi^bitrev(i) sit in one table per modulus, 16 bytes per entry; the index of the twiddle of
// a butterfly group obeys T(next stage) = 2*T + bit, so a thread needs only the index of its group at
// the first stage of a round.
//
// Two butterfly arithmetics, chosen per context (both give the same canonical residues):
//   ArithU64  any modulus below 2^58: 64-bit Shoup multiplication (twiddle + precomputed quotient), lazy
//             values (forward: below 60q < 2^64; inverse: kept in [0, 4q)).
//   ArithF64  every modulus below 2^50: residues are integers held in doubles and the twiddle product is
//             reduced with fused multiply-adds: for |y| < 2^51, h = y*w rounded, l = fma(y, w, -h) its
//             exact error, c = the integer nearest to y*(w/q) (one fma against 1.5*2^52), and
//             fma(-c, q, h) + l = y*w - c*q exactly: six double-precision
//             operations where the integer path spends more than twenty 32-bit ones, which moves the
//             lo pass from instruction issue to the HBM roof.  Twiddles are centred, |w| < q/2, so a multiplicand
//             may reach 4q and its product stays below q: values are brought back to |v| <= q/2 + 1 (three
//             operations) only where the bounds in f64mod.h ask for it, four of eight per forward round
//             and six of eight per inverse round; every sum stays below 2^53: all arithmetic is
//             exact.  Between the two passes the data sit in HBM as doubles below 4q.  (With every output of a
//             forward round and every sum of an inverse butterfly re-centred, 1920 limb-polys at N = 2^16: inverse lo
//             pass 486 us, now 444, forward 459 and 453; converting hi pass, 8 x 8 -> 19 limbs, 45.2 and 41.0.)
// Rings below 2^11 use a plain one-tile integer kernel.
#include <type_traits>

#include "ctx.h"
#include "convrule.h"
#include "f64mod.h"
#include "galois.h"
#include "shoup.h"

#define NTT_THREADS 256
#define NTT_TILE 2048
// Where point p of a tile sits in LDS.  A wavefront's 8-byte accesses are served sixteen lanes at a time, one per pair of
// 4-byte banks, so an access is conflict-free when the low four bits of the sixteen word indices are distinct.  The lo
// pass' four patterns spread the sixteen lanes over index bits {0,1,2,3} (thread-contiguous), {0,1,5,6} (round C),
// and {3,4,5,6} (eight consecutive points per thread); folding bits 4, 5, 6 into bits 1, 2, 3 and bit 6 also into
// bit 0 makes the low four bits a bijection of the lanes in all of them (measured: 6.2 cycles per wave-level 8-byte
// write in every pattern, against 8.1 with one padding word per eight in the two thread-contiguous ones).
#define LDS_PAD(p) ((p) ^ ((((p) >> 4) & 7u) << 1) ^ (((p) >> 6) & 1u))
#define LDS_PADDED_WORDS NTT_TILE

// ---- 64-bit integer arithmetic --------------------------------------------------------------------------
// Forward butterfly without a correction: the lazy Shoup product t (shoup.h) is in [0, 4q) for ANY 64-bit y, so
// both outputs stay non-negative and grow by at most 4q per stage: below 49q over the twelve stages of a whole ring in one
// kernel, below 25q over the up to six of a first pass, whose results are brought below 16q before the eleven that follow: 60q < 2^64 for
// every supported modulus (q < 2^58).  One word reduction at the very end.  The inverse keeps values in [0, 4q).
struct ArithU64 {
    typedef u64 E;
    typedef TwPair TW;
    typedef ModConst MC;
    static __device__ __forceinline__ E load_first(u64 raw, const MC&, bool /*inverse*/) { return raw; }
    static __device__ __forceinline__ E load_mid(u64 raw) { return raw; }
    static __device__ __forceinline__ u64 store_mid(E v) { return v; }
    static __device__ __forceinline__ u64 store_fwd_final(E v, const MC& m) { return reduce_word(v, m); }
    static __device__ __forceinline__ u64 store_inv_final(E v, const MC& m) { return mul_shoup(v, m.n_inv, m.n_inv_sh, m.q); }
    static __device__ __forceinline__ void fwd_bf(E& x, E& y, const TW w, const MC& m) {
        const u64 t = mul_shoup_lazy4(y, w.w, w.s, 0 - m.q);
        y = x + 4 * m.q - t;
        x = x + t;
    }
    static __device__ __forceinline__ void inv_bf(E& x, E& y, const TW w, const MC& m) {
        const u64 four_q = 4 * m.q;
        u64 s = x + y;
        if (s >= four_q) s -= four_q;
        const u64 d = x + four_q - y;
        x = s;
        y = mul_shoup_lazy4(d, w.w, w.s, 0 - m.q);
    }
    // between the passes of a forward transform: below 25q after up to six stages, 16q here, 60q after eleven more
    static __device__ __forceinline__ E load_second(u64 raw, const MC& m) { return raw >= 16 * m.q ? raw - 16 * m.q : raw; }
    static __device__ __forceinline__ void fwd_begin(E*, const MC&) {}
    static __device__ __forceinline__ void fwd_end(E*, const MC&) {}
    template <int KC>
    static __device__ __forceinline__ void inv_mid(E*, const MC&) {}
    static __device__ __forceinline__ void inv_end(E*, const MC&) {}
    static __device__ __forceinline__ void inv_end2(E*, const MC&) {}
};

// ---- double-precision arithmetic for moduli below 2^50 (the routines themselves: f64mod.h) -----------------------
struct ArithF64 {
    typedef double E;
    typedef TwF TW;
    typedef ModConstF MC;
    static __device__ __forceinline__ double round_mul(double v, double c) { return f64m_round_mul(v, c); }
    // v - q * round(v / q): |result| <= q/2 + 1 for integer |v| < 2^53
    static __device__ __forceinline__ double reduce(double v, const MC& m) { return f64m_reduce(v, m.q, m.qinv); }
    // y * w - q * c, c an integer within 3/4 of y * w / q: exact, magnitude below 0.75 q; needs |y| < 2^51, 0 <= w < q, wq = w / q rounded
    static __device__ __forceinline__ double mulmod(double y, double w, double wq, double q) { return f64m_mulmod(y, w, wq, q); }
    // the same for a multiplier without a precomputed w / q (a key word, a ciphertext residue): |y| < q, 0 <= w < q;
    // exact, magnitude below 0.75 q (0.63 q for |y| <= q/2 + 1)
    static __device__ __forceinline__ double mulmod_any(double y, double w, double q, double qinv) { return f64m_mulmod_any(y, w, q, qinv); }
    static __device__ __forceinline__ double from_u64(u64 raw) { return f64m_from_u64(raw); }
    static __device__ __forceinline__ u64 to_u64(double v) { return f64m_to_u64(v); }
    static __device__ __forceinline__ u64 canonical(double v, const MC& m) { return f64m_canonical(v, m.q); }  // |v| <= q/2 + 1 -> [0, q)
    static __device__ __forceinline__ E load_first(u64 raw, const MC&, bool) { return from_u64(raw); }  // canonical: in [0, q)
    static __device__ __forceinline__ E load_mid(u64 raw) { return __longlong_as_double((long long)raw); }
    static __device__ __forceinline__ E load_second(u64 raw, const MC&) { return load_mid(raw); }
    static __device__ __forceinline__ u64 store_mid(E v) { return (u64)__double_as_longlong(v); }
    static __device__ __forceinline__ u64 store_fwd_final(E v, const MC& m) { return canonical(v, m); }  // after fwd_end
    static __device__ __forceinline__ u64 store_inv_final(E v, const MC& m) { return canonical(mulmod(v, m.ninv, m.ninv_q, m.q), m); }
    static __device__ __forceinline__ void fwd_bf(E& x, E& y, const TW w, const MC& m) {
        const double t = mulmod(y, w.w, w.wq, m.q);
        y = x - t;
        x = x + t;
    }
    static __device__ __forceinline__ void inv_bf(E& x, E& y, const TW w, const MC& m) {
        const double s = x + y, d = x - y;
        x = s;
        y = mulmod(d, w.w, w.wq, m.q);
    }
    // the reductions (bounds: f64mod.h): before a forward round, after a transform's last one; after the first stage of an
    // inverse round, after its third, after the two-stage round that starts the inverse transform
    static __device__ __forceinline__ void fwd_begin(E* v, const MC& m) { f64m_fwd_begin(v, m.q, m.qinv); }
    static __device__ __forceinline__ void fwd_end(E* v, const MC& m) {
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = reduce(v[j], m);
    }
    template <int KC>
    static __device__ __forceinline__ void inv_mid(E* v, const MC& m) { f64m_inv_mid<KC>(v, m.q, m.qinv); }
    static __device__ __forceinline__ void inv_end(E* v, const MC& m) { f64m_inv_end(v, m.q, m.qinv); }
    static __device__ __forceinline__ void inv_end2(E* v, const MC& m) {
        v[0] = reduce(v[0], m);
        v[4] = reduce(v[4], m);
    }
};

// S radix-2 stages on 2^S "rows" of KC independent columns held in registers, v[row*KC + col];
// row bit S-1 is the largest distance.  T = twiddle index of this group at the first stage.
template <class A, int S, int KC>
__device__ __forceinline__ void fwd_rows(typename A::E* v, const typename A::TW* __restrict__ tw, u32 T, const typename A::MC& m) {
#pragma unroll
    for (int a = 0; a < S; a++) {
        const int half = (1 << S) >> (a + 1);
#pragma unroll
        for (int rr = 0; rr < (1 << S); rr++) {
            if (rr & half) continue;
            const typename A::TW w = tw[(T << a) + (rr >> (S - a))];
#pragma unroll
            for (int kc = 0; kc < KC; kc++) A::fwd_bf(v[rr * KC + kc], v[(rr + half) * KC + kc], w, m);
        }
    }
}

template <class A, int S, int KC>
__device__ __forceinline__ void inv_rows(typename A::E* v, const typename A::TW* __restrict__ tw, u32 T, const typename A::MC& m) {
#pragma unroll
    for (int a = S - 1; a >= 0; a--) {
        const int half = (1 << S) >> (a + 1);
#pragma unroll
        for (int rr = 0; rr < (1 << S); rr++) {
            if (rr & half) continue;
            const typename A::TW w = tw[(T << a) + (rr >> (S - a))];
#pragma unroll
            for (int kc = 0; kc < KC; kc++) A::inv_bf(v[rr * KC + kc], v[(rr + half) * KC + kc], w, m);
        }
        if (a == S - 1) A::template inv_mid<KC>(v, m);
    }
}

// Butterflies whose twiddle is the value alone (no twiddle / q): the quotient comes from the rounded product.  Half the
// registers and half the bytes per twiddle; the bounds in f64mod.h are for these.
struct ArithF64W : ArithF64 {
    typedef double TW;
    static __device__ __forceinline__ void fwd_bf(E& x, E& y, const double w, const MC& m) {
        const double t = mulmod_any(y, w, m.q, m.qinv);
        y = x - t;
        x = x + t;
    }
    static __device__ __forceinline__ void inv_bf(E& x, E& y, const double w, const MC& m) {
        const double s = x + y, d = x - y;
        x = s;
        y = mulmod_any(d, w, m.q, m.qinv);
    }
};
template <int S>
__device__ __forceinline__ void load_tw_w(const double* __restrict__ tw, u32 T, double* tv) {
#pragma unroll
    for (int a = 0; a < S; a++)
#pragma unroll
        for (int j = 0; j < (1 << a); j++) tv[(1 << a) - 1 + j] = tw[(T << a) + j];
}

// what the lo passes hold of a twiddle and how they multiply by it: the value alone in double precision
template <class A>
struct LoTw {
    typedef A AR;
    typedef typename A::TW TW;
};
template <>
struct LoTw<ArithF64> {
    typedef ArithF64W AR;
    typedef double TW;
};

// The same with the round's 2^S - 1 twiddles already in registers (tv[(1 << a) - 1 + j] = tw[(T << a) + j]):
// the lo pass requests the twiddles of the next round before it starts the current one, so their
// latency (they come from L2) hides behind a round of butterflies and an LDS exchange.
template <class A, int S>
__device__ __forceinline__ void load_tw(const typename A::TW* __restrict__ tw, u32 T, typename A::TW* tv) {
#pragma unroll
    for (int a = 0; a < S; a++)
#pragma unroll
        for (int j = 0; j < (1 << a); j++) tv[(1 << a) - 1 + j] = tw[(T << a) + j];
}

template <class A, int S>
__device__ __forceinline__ void fwd_rows_pre(typename A::E* v, const typename A::TW* tv, const typename A::MC& m) {
#pragma unroll
    for (int a = 0; a < S; a++) {
        const int half = (1 << S) >> (a + 1);
#pragma unroll
        for (int rr = 0; rr < (1 << S); rr++) {
            if (rr & half) continue;
            A::fwd_bf(v[rr], v[rr + half], tv[(1 << a) - 1 + (rr >> (S - a))], m);
        }
    }
}

template <class A, int S>
__device__ __forceinline__ void inv_rows_pre(typename A::E* v, const typename A::TW* tv, const typename A::MC& m) {
#pragma unroll
    for (int a = S - 1; a >= 0; a--) {
        const int half = (1 << S) >> (a + 1);
#pragma unroll
        for (int rr = 0; rr < (1 << S); rr++) {
            if (rr & half) continue;
            A::inv_bf(v[rr], v[rr + half], tv[(1 << a) - 1 + (rr >> (S - a))], m);
        }
        if (S == 3 && a == S - 1) A::template inv_mid<1>(v, m);
    }
}

struct NttArgs {
    const u64* src;
    u64* dst;
    size_t src_bstride;  // in limb-polys
    size_t dst_bstride;
    const void* mc;      // [M] ModConst or ModConstF
    const void* tw;      // [M][N] TwPair or TwF
    const double* tw_val;  // [M][N] the twiddles' values alone (lo passes in double precision), or null
    u32 log_n, log_lo, log_hi;
    u32 first;           // this pass reads the caller's canonical residues (else the other pass's intermediate form)
    u32 last;            // this pass writes the final result (canonical; inverse: times 1/N)
    u32 batch;           // batch items (each pl.n limb-polys)
    u32 lo_group;        // slices per group of the lo-pass numbering (0: plain)
    u32 use_src_list;    // batch item b reads src_list.p[b] instead of src + b*src_bstride*N
    PtrList8 src_list;
    PtrList8 mul_list;     // inverse, first pass, product variant: batch item b is src_list.p[b] (.) mul_list.p[b]
    u64 lin_ka, lin_kb;    // use_lin: ... is lin_ka * src_list.p[b] + lin_kb * mul_list.p[b] instead (one limb per item)
    u32 use_lin, pad2;
    // loop variant of the forward lo pass, ModUp: the items are (polynomial, digit) pairs, digits fastest, `beta` of them per
    // polynomial; limb e <= level is transformed for every digit but the one it belongs to, e / alpha (0: plain items)
    u32 beta, alpha, level, pad3;
    u32 gal[KS_MAX_BATCH];  // inverse, first pass, automorphism variant: batch item b is sigma_gal[b] of src_list.p[b]
    const TwF* inv_scale;  // inverse, last pass (double-precision arithmetic): the limb of modulus m is scaled by inv_scale[m]
                           // instead of 1/N and stored as the centred residue in a double (the form ModUp's conversion reads)
};

// Lo-pass workgroups are numbered in groups of `grp` consecutive (limb, block) slices, batch item by
// batch item: the `batch` tiles that use the same twiddle slice get ids that are a multiple of 8
// apart (same XCD) and close in time, so the slice comes from HBM once and from that XCD's L2 for the
// rest of the batch, while each batch item's `grp` tiles are one contiguous run of memory.
struct LoTile {
    u32 b, a, blk;
};
// grid = (grp, batch, slices / grp): linear id = x + grp * (y + batch * z), slice t = z * grp + x, item b = y
// (plain numbering when grp == 0: grid = (batch, slices), b = x, t = y)
__device__ __forceinline__ LoTile lo_tile(u32 log_hi, u32 grp) {
    const u32 t = grp ? blockIdx.z * grp + blockIdx.x : blockIdx.y;
    LoTile r;
    r.b = grp ? blockIdx.y : blockIdx.x;
    r.a = t >> log_hi;
    r.blk = t & ((1u << log_hi) - 1);
    return r;
}

// Entry i of one of a PolyList's byte arrays.  The list is a kernel argument and i is the same for the whole workgroup: read
// as the 32-bit word that holds it, this is a scalar load; a byte load is a vector load whose round trip to memory every
// address of the kernel then waits for.
__device__ __forceinline__ u32 pl_at(const unsigned char* arr, u32 i) {
    const u32 w = reinterpret_cast<const u32*>(arr)[i >> 2];
    return (w >> (8 * (i & 3))) & 0xffu;
}

// ModUp, all digits in one launch (launch_ntt_digits): whether entry a of row (polynomial, digit) is one of the digit's own limbs, which
// are not transformed
__device__ __forceinline__ bool own_limb(const NttArgs& args, u32 row, u32 a) {
    return args.beta && a <= args.level && a / args.alpha == row % args.beta;
}

template <class A>
struct PolyRef {
    const u64* src;
    u64* dst;
    const typename A::TW* tw;
    const double* tw_val;  // this modulus' row of NttArgs::tw_val
    typename A::MC mc;
};

// BYTES: read the list's entries with byte loads all the same (the converting hi pass: with scalar positions its tables of
// constants become scalar loads too, four limbs' worth of them more than the scalar registers hold: measured slower)
template <class A, bool BYTES = false>
__device__ __forceinline__ PolyRef<A> poly_ref(const NttArgs& args, const PolyList& pl, u32 b, u32 a) {
    const u32 m_idx = BYTES ? pl.mod[a] : pl_at(pl.mod, a);
    PolyRef<A> r;
    const u32 sp = BYTES ? pl.spos[a] : pl_at(pl.spos, a), dp = BYTES ? pl.dpos[a] : pl_at(pl.dpos, a);
    r.src = (args.use_src_list ? args.src_list.p[b] : args.src + (((size_t)b * args.src_bstride) << args.log_n)) + ((size_t)sp << args.log_n);
    r.dst = args.dst + (((size_t)b * args.dst_bstride + dp) << args.log_n);
    r.tw = (const typename A::TW*)args.tw + ((size_t)m_idx << args.log_n);
    r.tw_val = args.tw_val ? args.tw_val + ((size_t)m_idx << args.log_n) : nullptr;
    r.mc = ((const typename A::MC*)args.mc)[m_idx];
    return r;
}

template <class A, int S>
__device__ __forceinline__ void load_lo_tw(const PolyRef<A>& P, u32 T, typename LoTw<A>::TW* tv) {
    if constexpr (std::is_same<A, ArithF64>::value) load_tw_w<S>(P.tw_val, T, tv);
    else load_tw<A, S>(P.tw, T, tv);
}

// ================================ lo pass (contiguous 2^11 blocks) ================================
// positions inside the block: pos = d3*256 + d2*32 + d1*4 + d0 (d3,d2,d1 < 8, d0 < 4)
//   round A: thread = pos % 256,           points over d3          (distances 1024, 512, 256)
//   round B: thread = (d3, pos % 32),      points over d2          (distances 128, 64, 32)
//   round C: thread = (d3, d2, d0),        points over d1          (distances 16, 8, 4)
//   round D: thread = pos / 8,             8 consecutive points    (distances 2, 1)
// A workgroup transforms the same (limb, block) slice of IT consecutive batch items one after the other: the
// slice's twiddles (half as many bytes as the tile itself as values alone, as many with their quotients) are fetched once for
// all of them, and the next item's
// points are requested before the current item's butterflies start, so their latency hides behind a whole
// tile of work.  A buffer is rewritten only after a barrier that every reader of its old contents has passed: the
// forward pass has four exchanges per item (the last one turns each thread's 8 consecutive results into stores of
// 512 contiguous bytes per wave) and uses the two buffers in turn; the inverse pass has three, so its buffers swap
// roles from one item to the next.
template <class A>
__device__ __forceinline__ const u64* item_src(const NttArgs& args, const PolyList& pl, u32 b, u32 a) {
    return (args.use_src_list ? args.src_list.p[b] : args.src + (((size_t)b * args.src_bstride) << args.log_n)) + ((size_t)pl_at(pl.spos, a) << args.log_n);
}
__device__ __forceinline__ u64* item_dst(const NttArgs& args, const PolyList& pl, u32 b, u32 a) {
    return args.dst + (((size_t)b * args.dst_bstride + pl_at(pl.dpos, a)) << args.log_n);
}

// The last step of a division by dropped moduli on a slice of 2^11 results w that sit in LDS (buf, point p at LDS_PAD(p)) and
// are not stored: out = ((v - w) * cinv + addend) * mask + acc.  div_request asks for its operands, a round of butterflies
// ahead of div_store.
// EM: which of the optional operands the launch has: 0 = look at each item's pointers,
// 1 = every item has its addend (of component 0 at least) and nothing else, 2 = none has any, 3 = every item has the ciphertext
// `acc` and nothing else, 4 = every item has its mask and nothing else.  In all but case 0 the operand is requested with v, a
// round ahead of its use; behind a condition the compiler keeps each request next to its use, one round trip to memory per
// point (eight rotations of two limbs each at N = 2^16, sums added: 17.7 us in case 0, 14.2 us in case 3 with the rotated addend
// inside the inner product).
// i: limb (the list's dpos entry), bb: batch item (2 ciphertext + component), off: the slice's first point, t = 0..255
// EM_SUM*: one result for several items (launch_ntt_moddown_sum): v is the sum of ep.n_part partial sums, and one ciphertext is added, masked
// (EM_SUM_MASK), as it is (EM_SUM_ADD), or none.
#define EM_SUM 5
#define EM_SUM_ADD 6
#define EM_SUM_MASK 7
struct DivOperands {
    u64 v[8], v2[8], op[8];
    double vs[8];
};
template <class A, int EM>
__device__ __forceinline__ void div_request(const NttArgs& args, const FwdEpilogue& ep, u32 i, u32 bb, size_t off, u32 t, DivOperands& O) {
    const FinalItem& fi = ep.B.it[bb >> 1];
    if (EM == 1) {  // the addend, gathered through the item's automorphism; component 1 may have none
        const u64* add = (bb & 1) ? fi.add1 : fi.add0;
        if (add) {
            add += (size_t)i << args.log_n;
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const u32 x = (u32)off + t + 256 * j;
                O.op[j] = add[fi.g == 1 ? x : galois_gather_index(x, fi.g, args.log_n)];
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++) O.op[j] = 0;
        }
    } else if (EM == 3 || EM == 4 || EM == EM_SUM_ADD || EM == EM_SUM_MASK) {
        if (EM == EM_SUM_MASK) {
            const u64* mask = fi.mask + ((size_t)i << args.log_n) + off;
#pragma unroll
            for (int j = 0; j < 8; j++) O.v2[j] = mask[t + 256 * j];
        }
        const u64* op = (EM != 4 ? fi.acc + ((size_t)((bb & 1) * ep.n_out + i) << args.log_n) : fi.mask + ((size_t)i << args.log_n)) + off;
#pragma unroll
        for (int j = 0; j < 8; j++) O.op[j] = op[t + 256 * j];
    }
    if constexpr (EM >= EM_SUM) {  // residues below 2^50: four of them on a reduced sum stay below 2^53
        const u64* part = ep.v + (((size_t)bb * ep.E + i) << args.log_n) + off + t;
        const ModConstF mc = ((const ModConstF*)args.mc)[i];
#pragma unroll
        for (int j = 0; j < 8; j++) O.vs[j] = 0.0;
        auto add_parts = [&](auto many, u32 s) {  // so many parts' words requested together
            constexpr int M = decltype(many)::value;
            u64 w[M][8];
#pragma unroll
            for (int i = 0; i < M; i++)
#pragma unroll
                for (int j = 0; j < 8; j++) w[i][j] = (part + min(s + i, ep.n_part - 1) * ep.v_pstride)[256 * j];
#pragma unroll
            for (int j = 0; j < 8; j++) {
                double sum = O.vs[j];
#pragma unroll
                for (int i = 0; i < M; i++) sum += s + i < ep.n_part ? f64m_from_u64(w[i][j]) : 0.0;
                O.vs[j] = f64m_reduce(sum, mc.q, mc.qinv);
            }
        };
        if (ep.n_part <= 2) add_parts(std::integral_constant<int, 2>(), 0);
        else
            for (u32 s = 0; s < ep.n_part; s += 4) add_parts(std::integral_constant<int, 4>(), s);
        return;
    }
    const u64* vrow = (ep.use_vl ? ep.vl.p[bb >> 1] + (bb & 1) * ep.v_cstride + ((size_t)i << args.log_n)
                                 : ep.v + (((size_t)bb * ep.E + i) << args.log_n)) + off;
#pragma unroll
    for (int j = 0; j < 8; j++) O.v[j] = vrow[t + 256 * j];
    if constexpr (std::is_same<A, ArithF64>::value) {
        if (ep.use_vl == 2) {
            const u64* vrow2 = ep.vl2.p[bb >> 1] + (bb & 1) * ep.v2_cstride + ((size_t)i << args.log_n) + off;
#pragma unroll
            for (int j = 0; j < 8; j++) O.v2[j] = vrow2[t + 256 * j];
        }
    }
}
template <class A, int EM>
__device__ __forceinline__ void div_store(const NttArgs& args, const FwdEpilogue& ep, u32 i, u32 m_idx, u32 bb, size_t off, u32 t,
                                          const typename A::E* buf, const typename A::MC& mc, const DivOperands& O) {
    const u32 comp = bb & 1;
    const FinalItem fi = ep.B.it[bb >> 1];
    const u64 cv = ep.cinv[i];
    const u64* add = comp ? fi.add1 : fi.add0;
    u64* orow = fi.out + (((size_t)comp * ep.n_out + i) << args.log_n) + off;
    if constexpr (std::is_same<A, ArithF64>::value) {
        // in the transform's own arithmetic: v - w is an integer below 2q in magnitude, its product with the constant is
        // below 0.75 q, one more reduction after the addend; every value below is exact
        const double q = mc.q, cvd = A::from_u64(cv), cvq = cvd / q;
        double vd[8];
        if constexpr (EM >= EM_SUM) {
#pragma unroll
            for (int j = 0; j < 8; j++) vd[j] = O.vs[j];
        } else if (ep.use_vl == 2) {  // v = ka * x + kb * y
            const double ka = A::from_u64(ep.ka[i]), kb = A::from_u64(ep.kb[i]);
#pragma unroll
            for (int j = 0; j < 8; j++)
                vd[j] = A::reduce(A::mulmod_any(A::from_u64(O.v[j]), ka, q, mc.qinv) + A::mulmod_any(A::from_u64(O.v2[j]), kb, q, mc.qinv), mc);
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++) vd[j] = A::from_u64(O.v[j]);
        }
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const u32 p = t + 256 * j;
            double r = A::mulmod(vd[j] - buf[LDS_PAD(p)], cvd, cvq, q);
            if (EM == 1 || EM == 3 || EM == EM_SUM_ADD) {
                r = A::reduce(r + A::from_u64(O.op[j]), mc);
            } else if (EM == EM_SUM_MASK) {
                r = A::reduce(r + A::mulmod_any(A::from_u64(O.op[j]), A::from_u64(O.v2[j]), q, mc.qinv), mc);
            } else if (EM == 4) {
                r = A::mulmod_any(r, A::from_u64(O.op[j]), q, mc.qinv);
            } else if (EM == 0) {
                if (add) {
                    const u32 x = (u32)off + p;
                    const u32 xs = fi.g == 1 ? x : galois_gather_index(x, fi.g, args.log_n);
                    r = A::reduce(r + A::from_u64(add[((size_t)i << args.log_n) + xs]), mc);
                }
                if (fi.mask) r = A::mulmod_any(r, A::from_u64(fi.mask[((size_t)i << args.log_n) + off + p]), q, mc.qinv);
                if (fi.acc) r = A::reduce(r + A::from_u64(fi.acc[(((size_t)comp * ep.n_out + i) << args.log_n) + off + p]), mc);
            }
            orow[p] = A::canonical(r, mc);
        }
    } else {
        const ModConst mi = ep.mci[m_idx];
        const u64 cvs = ep.cinv[ep.num_q + i];
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const u32 p = t + 256 * j;
            const u64 w = A::store_fwd_final(buf[LDS_PAD(p)], mc);
            u64 r = mul_shoup(sub_mod(O.v[j], w, mi.q), cv, cvs, mi.q);
            if (EM == 1 || EM == 3) {
                r = add_mod(r, O.op[j], mi.q);
            } else if (EM == 4) {
                r = mulmod_barrett(r, O.op[j], mi);
            } else if (EM == 0) {
                if (add) {
                    const u32 x = (u32)off + p;
                    const u32 xs = fi.g == 1 ? x : galois_gather_index(x, fi.g, args.log_n);
                    r = add_mod(r, add[((size_t)i << args.log_n) + xs], mi.q);
                }
                if (fi.mask) r = mulmod_barrett(r, fi.mask[((size_t)i << args.log_n) + off + p], mi);
                if (fi.acc) r = add_mod(r, fi.acc[(((size_t)comp * ep.n_out + i) << args.log_n) + off + p], mi.q);
            }
            orow[p] = r;
        }
    }
}

// The plain forward lo pass with the workgroup's batch items in a loop: items tile.b, tile.b + (the grid's extent over
// items), ... of the same 2^11-point slice.  The slice's 27 twiddles per thread are 216 bytes (432 with their quotients) against the 128 bytes of
// an item's points and results, so a workgroup that fetches them for two items still moves more twiddles than data through
// the CU's cache; this one fetches them once for all its items and requests an item's points while the previous one is
// transformed.  Same rounds, same LDS exchanges as fwd_lo_body.
template <class A>
__global__ __launch_bounds__(NTT_THREADS) void ntt_fwd_lo_loop_kernel(NttArgs args, PolyList pl) {
    typedef typename A::E E;
    typedef typename LoTw<A>::TW TW;
    typedef typename LoTw<A>::AR AR;
    __shared__ E lds0[LDS_PADDED_WORDS];
    __shared__ E lds1[LDS_PADDED_WORDS];
    const u32 tid = threadIdx.x;
    const LoTile tile = lo_tile(args.log_hi, args.lo_group);
    const u32 b_step = args.lo_group ? gridDim.y : gridDim.x;
    const u32 blk = tile.blk;
    const bool digits = args.beta != 0;
    const u32 own = digits && tile.a <= args.level ? tile.a / args.alpha : 0xffffffffu;
    const u32 per = digits ? args.beta - (own < args.beta ? 1 : 0) : 1;  // items per polynomial of this limb
    const u32 n_items = digits ? args.batch / args.beta * per : args.batch;
    if (tile.b >= n_items) return;  // whole workgroup
    auto row_of = [&](u32 i) {  // batch row of this limb's item i
        if (!digits) return i;
        const u32 p = i / per, j = i - p * per;
        return p * args.beta + j + (j >= own ? 1 : 0);
    };
    const PolyRef<A> P = poly_ref<A>(args, pl, row_of(tile.b), tile.a);
    const size_t off = (size_t)blk << 11;
    const u32 TA = (1u << args.log_hi) + blk;
    const u32 d3 = tid >> 5, x5 = tid & 31, d2 = (tid >> 2) & 7, d0 = tid & 3;
    E v[8];
    u64 raw[8];
    TW wa[7], wb[7], wc[7], wd[6];
    load_lo_tw<A, 3>(P, TA, wa);
    {
        const u64* src = P.src + off;
#pragma unroll
        for (int j = 0; j < 8; j++) raw[j] = src[tid + 256 * j];
    }
    load_lo_tw<A, 3>(P, 8 * TA + d3, wb);
    load_lo_tw<A, 3>(P, 64 * TA + 8 * d3 + d2, wc);
    load_lo_tw<A, 2>(P, 512 * TA + 2 * tid, wd);
    load_lo_tw<A, 2>(P, 512 * TA + 2 * tid + 1, wd + 3);
    for (u32 b = tile.b; b < n_items; b += b_step) {
        if (args.first) {
#pragma unroll
            for (int j = 0; j < 8; j++) v[j] = A::load_first(raw[j], P.mc, false);
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++) v[j] = A::load_second(raw[j], P.mc);
        }
        if (b + b_step < n_items) {  // the next item's points, a tile ahead
            const u64* src = item_src<A>(args, pl, row_of(b + b_step), tile.a) + off;
#pragma unroll
            for (int j = 0; j < 8; j++) raw[j] = src[tid + 256 * j];
        }
        A::fwd_begin(v, P.mc);
        fwd_rows_pre<AR, 3>(v, wa, P.mc);
#pragma unroll
        for (int j = 0; j < 8; j++) lds0[LDS_PAD(tid + 256 * j)] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = lds0[LDS_PAD(d3 * 256 + 32 * j + x5)];
        A::fwd_begin(v, P.mc);
        fwd_rows_pre<AR, 3>(v, wb, P.mc);
#pragma unroll
        for (int j = 0; j < 8; j++) lds1[LDS_PAD(d3 * 256 + 32 * j + x5)] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = lds1[LDS_PAD(d3 * 256 + d2 * 32 + 4 * j + d0)];
        A::fwd_begin(v, P.mc);
        fwd_rows_pre<AR, 3>(v, wc, P.mc);
#pragma unroll
        for (int j = 0; j < 8; j++) lds0[LDS_PAD(d3 * 256 + d2 * 32 + 4 * j + d0)] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = lds0[LDS_PAD(8 * tid + j)];
        fwd_rows_pre<AR, 2>(v, wd, P.mc);
        fwd_rows_pre<AR, 2>(v + 4, wd + 3, P.mc);
        A::fwd_end(v, P.mc);
        // back through LDS so that a wave stores 512 contiguous bytes per instruction
#pragma unroll
        for (int j = 0; j < 8; j++) lds1[LDS_PAD(8 * tid + j)] = v[j];
        __syncthreads();
        u64* dst = item_dst(args, pl, row_of(b), tile.a) + off;
#pragma unroll
        for (int j = 0; j < 8; j++) dst[tid + 256 * j] = A::store_fwd_final(lds1[LDS_PAD(tid + 256 * j)], P.mc);
        // (no barrier between items: the next item's first exchange writes lds0, whose last read is behind the barrier above,
        // and its first barrier stands between these reads of lds1 and the next writes to it)
    }
}

// the lo pass as the last kernel of a division by dropped moduli: one batch item per workgroup
template <class A, int EM>
__global__ __launch_bounds__(NTT_THREADS) void ntt_fwd_lo_div_kernel(NttArgs args, PolyList pl, FwdEpilogue ep) {
    typedef typename A::E E;
    typedef typename LoTw<A>::TW TW;
    typedef typename LoTw<A>::AR AR;
    __shared__ E lds0[LDS_PADDED_WORDS];
    __shared__ E lds1[LDS_PADDED_WORDS];
    const u32 tid = threadIdx.x;
    const LoTile tile = lo_tile(args.log_hi, args.lo_group);
    const u32 blk = tile.blk, b = tile.b;
    const PolyRef<A> P = poly_ref<A>(args, pl, b, tile.a);
    const size_t off = (size_t)blk << 11;
    const u32 TA = (1u << args.log_hi) + blk;
    const u32 d3 = tid >> 5, x5 = tid & 31, d2 = (tid >> 2) & 7, d0 = tid & 3;
    E v[8];
    u64 raw[8];
    TW wa[7], wb[7], wc[7], wd[6];
    load_lo_tw<A, 3>(P, TA, wa);
    load_lo_tw<A, 3>(P, 8 * TA + d3, wb);
#pragma unroll
    for (int j = 0; j < 8; j++) raw[j] = P.src[off + tid + 256 * j];
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = A::load_second(raw[j], P.mc);
    A::fwd_begin(v, P.mc);
    fwd_rows_pre<AR, 3>(v, wa, P.mc);
    load_lo_tw<A, 3>(P, 64 * TA + 8 * d3 + d2, wc);
#pragma unroll
    for (int j = 0; j < 8; j++) lds0[LDS_PAD(tid + 256 * j)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = lds0[LDS_PAD(d3 * 256 + 32 * j + x5)];
    A::fwd_begin(v, P.mc);
    fwd_rows_pre<AR, 3>(v, wb, P.mc);
    load_lo_tw<A, 2>(P, 512 * TA + 2 * tid, wd);
    load_lo_tw<A, 2>(P, 512 * TA + 2 * tid + 1, wd + 3);
#pragma unroll
    for (int j = 0; j < 8; j++) lds1[LDS_PAD(d3 * 256 + 32 * j + x5)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = lds1[LDS_PAD(d3 * 256 + d2 * 32 + 4 * j + d0)];
    A::fwd_begin(v, P.mc);
    fwd_rows_pre<AR, 3>(v, wc, P.mc);
#pragma unroll
    for (int j = 0; j < 8; j++) lds0[LDS_PAD(d3 * 256 + d2 * 32 + 4 * j + d0)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = lds0[LDS_PAD(8 * tid + j)];
    DivOperands O;
    const u32 i = pl_at(pl.dpos, tile.a);
    div_request<A, EM>(args, ep, i, b, off, tid, O);
    fwd_rows_pre<AR, 2>(v, wd, P.mc);
    fwd_rows_pre<AR, 2>(v + 4, wd + 3, P.mc);
    A::fwd_end(v, P.mc);
    // back through LDS so that a wave stores 512 contiguous bytes per instruction
#pragma unroll
    for (int j = 0; j < 8; j++) lds1[LDS_PAD(8 * tid + j)] = v[j];
    __syncthreads();
    div_store<A, EM>(args, ep, i, pl_at(pl.mod, tile.a), b, off, tid, lds1, P.mc, O);
}

// The lo pass of ModUp's forward transforms with the inner product with the switching key in place of its stores.
// A workgroup owns one 2^11-point slice of one position e of the extended basis of one batch item: it transforms that
// slice of every digit whose limb e went through the converting hi pass (all live digits but the one e belongs to; the
// slice's twiddles are fetched once for all of them), multiplies each result by the two key words of (digit, e) as it
// comes out, adds the product of the digit that owns e (its limb is the decomposed polynomial's own, never transformed)
// and stores the two components of the inner product: the extended
// digits are never written in evaluation form nor read back.  All sums are exact integers in doubles for any number of digits:
// they are reduced at every eighth digit (f64m_sum_due).
struct MacEpilogue {
    DigitSrc D;           // D.digits: rows (j*E + e) hold the hi pass' output (doubles); D.own: the decomposed polynomials
    PtrList8 key;         // per batch item: [dnum][2][M][N] (the same pointer for a shared key)
    OutList8 out;         // per batch item: [2][E][N]
    const u64* negp;      // [num_q]: -P mod q_i
    u32 level, M, E, beta;
    // the positions from inv_from on are what a division that follows drops: their sums leave in the form between the two passes of an
    // inverse transform (E: none of them)
    const double* itw_val;  // [M][N], NttArgs::tw_val of inverse transforms
    // SUM (with ROT): the other positions' sums of all items of a workgroup are added up and stored once, as item tile.b's
    u32 inv_from, first;  // first: the position that the grid's first slices belong to
    // PROD: the decomposed polynomial is d2 = a1 (.) b1 of the ciphertext product (a0, a1) x (b0, b1), which exists
    // nowhere in evaluation form: the own-limb term is formed from a1, b1 ([level+1][N] each, per batch item), and the
    // addends are d0 = a0 (.) b0 and d1 = a0 (.) b1 + a1 (.) b0 (D.own is not read)
    PtrList8 a0, a1, b0, b1;
    // ROT: item b is a rotation by gal[b] of the ciphertext (a0, D.own): the digits are those of sigma(D.own), the own-limb term and the
    // addend P sigma(a0) are gathered as they are read
    u32 gal[KS_MAX_BATCH];
    // HOIST (with ROT): the digits are those of D.own.p[0] itself, one set for all items, finished (launch_ntt_modup without hi_only) and read through
    // the item's automorphism
    // LIN (with PROD): the addends are ka * x + kb * y of two more ciphertexts (component 1 at + x_cstride, y_cstride)
    PtrList8 lx, ly;
    size_t x_cstride, y_cstride;
    u64 ka[CKKS_MAX_MODULI], kb[CKKS_MAX_MODULI];
    // MASK (with SUM): the rotated ciphertext is the product of (a0, D.own) with mask [level+1][N]
    const u64* mask;
    // DIV: the division's last step instead of stores: w are the converted dropped parts behind the first pass of their forward transform
    // ([2 * item + component][n_out][N]), cinv the multipliers (FwdEpilogue), res the results, add what is added to them (entries may be null)
    const double* w;
    const u64* cinv;
    PtrList8 add;
    OutList8 res;
};

// poly[x] through a wave-uniform base and a 32-bit offset (a polynomial is at most 1 MiB): half the address registers
__device__ __forceinline__ u64 word_at(const u64* poly, u32 x) { return *reinterpret_cast<const u64*>(reinterpret_cast<const char*>(poly) + 8 * x); }

// The inverse lo pass of a slice whose points tid + 256 i the workgroup's threads hold, |v| <= q / 2 + 1 (ntt_inv_lo_kernel's rounds
// behind one more exchange), for both components of an inner product one after the other: the slice's inverse twiddles are fetched
// once for the two.  The sums of the limbs that a division drops are read by nothing but the inverse transform, whose first pass
// owns the same slices: kept here, they are neither written nor read in between, and a launch goes.  At N = 2^16, 13 + 8 limbs, a
// product with its rescale 122 -> 113 us (117 with these limbs' workgroups, the longer ones, last in the launch instead of first);
// three rotations of 19 + 8 limbs 363 -> 355, the activation of sixteen ciphertexts of 20 + 7 limbs 4646 -> 4585, six rotations of 7 + 3
// limbs at N = 2^13 52.9 -> 51.1.  (Both components side by side in two buffers spill: activation 4914.)
__device__ __forceinline__ void mac_inverse_lo(double (&r0)[8], double (&r1)[8], double* lds0, double* lds1, const double* __restrict__ itw, u32 TA, u32 tid,
                                               const ModConstF& mc, u64* __restrict__ o0, u64* __restrict__ o1) {
    typedef ArithF64 A;
    typedef ArithF64W AW;
    const u32 d3 = tid >> 5, x5 = tid & 31, d2 = (tid >> 2) & 7, d0 = tid & 3;
    double wa[7], wb[7], wc[7], wd[6];
    load_tw_w<2>(itw, 512 * TA + 2 * tid, wd);
    load_tw_w<2>(itw, 512 * TA + 2 * tid + 1, wd + 3);
    load_tw_w<3>(itw, 64 * TA + 8 * d3 + d2, wc);
    load_tw_w<3>(itw, 8 * TA + d3, wb);
    load_tw_w<3>(itw, TA, wa);
#pragma unroll
    for (int comp = 0; comp < 2; comp++) {
        double v[8];
        // (lds0: its last readers are behind a barrier, the last digit's or the other component's last one)
#pragma unroll
        for (int j = 0; j < 8; j++) lds0[LDS_PAD(tid + 256 * j)] = comp ? r1[j] : r0[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = lds0[LDS_PAD(8 * tid + j)];
        inv_rows_pre<AW, 2>(v, wd, mc);
        inv_rows_pre<AW, 2>(v + 4, wd + 3, mc);
        A::inv_end2(v, mc);
#pragma unroll
        for (int j = 0; j < 8; j++) lds1[LDS_PAD(8 * tid + j)] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = lds1[LDS_PAD(d3 * 256 + d2 * 32 + 4 * j + d0)];
        inv_rows_pre<AW, 3>(v, wc, mc);
        A::inv_end(v, mc);
#pragma unroll
        for (int j = 0; j < 8; j++) lds0[LDS_PAD(d3 * 256 + d2 * 32 + 4 * j + d0)] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = lds0[LDS_PAD(d3 * 256 + 32 * j + x5)];
        inv_rows_pre<AW, 3>(v, wb, mc);
        A::inv_end(v, mc);
#pragma unroll
        for (int j = 0; j < 8; j++) lds1[LDS_PAD(d3 * 256 + 32 * j + x5)] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = lds1[LDS_PAD(tid + 256 * j)];
        inv_rows_pre<AW, 3>(v, wa, mc);
        A::inv_end(v, mc);
        u64* o = comp ? o1 : o0;
#pragma unroll
        for (int j = 0; j < 8; j++) o[tid + 256 * j] = A::store_mid(v[j]);
    }
}

// The forward lo pass' four rounds on v; the results sit in lds1, point p at LDS_PAD(p), behind a barrier.
__device__ __forceinline__ void fwd_lo_rounds(double (&v)[8], double* lds0, double* lds1, u32 tid, const double (&wa)[7], const double (&wb)[7],
                                              const double (&wc)[7], const double (&wd)[6], const ModConstF& mc) {
    typedef ArithF64 A;
    typedef ArithF64W AW;
    const u32 d3 = tid >> 5, x5 = tid & 31, d2 = (tid >> 2) & 7, d0 = tid & 3;
    A::fwd_begin(v, mc);
    fwd_rows_pre<AW, 3>(v, wa, mc);
#pragma unroll
    for (int i = 0; i < 8; i++) lds0[LDS_PAD(tid + 256 * i)] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = lds0[LDS_PAD(d3 * 256 + 32 * i + x5)];
    A::fwd_begin(v, mc);
    fwd_rows_pre<AW, 3>(v, wb, mc);
#pragma unroll
    for (int i = 0; i < 8; i++) lds1[LDS_PAD(d3 * 256 + 32 * i + x5)] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = lds1[LDS_PAD(d3 * 256 + d2 * 32 + 4 * i + d0)];
    A::fwd_begin(v, mc);
    fwd_rows_pre<AW, 3>(v, wc, mc);
#pragma unroll
    for (int i = 0; i < 8; i++) lds0[LDS_PAD(d3 * 256 + d2 * 32 + 4 * i + d0)] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = lds0[LDS_PAD(8 * tid + i)];
    fwd_rows_pre<AW, 2>(v, wd, mc);
    fwd_rows_pre<AW, 2>(v + 4, wd + 3, mc);
    A::fwd_end(v, mc);
#pragma unroll
    for (int i = 0; i < 8; i++) lds1[LDS_PAD(8 * tid + i)] = v[i];
    __syncthreads();
}

// PROD, LIN, ROT, SUM, MASK, DIV, HOIST (see MacEpilogue) are template arguments so that what follows the digits is straight-line code: with the
// operands behind conditions, even ones that are the same for the whole launch, the compiler keeps each request next to its
// use, one round trip to memory per point.
template <bool PROD, bool LIN, bool ROT, bool SUM = false, bool MASK = false, bool DIV = false, bool HOIST = false>
__global__ __launch_bounds__(NTT_THREADS) void ntt_fwd_lo_mac_kernel(NttArgs args, PolyList pl, MacEpilogue ep) {
    typedef ArithF64 A;
    typedef double E;
    __shared__ E lds0[LDS_PADDED_WORDS];
    __shared__ E lds1[LDS_PADDED_WORDS];
    const u32 tid = threadIdx.x;
    const LoTile tile = lo_tile(args.log_hi, args.lo_group);
    static_assert((!DIV || !SUM) && (!HOIST || (ROT && !SUM)), "");
    const u32 e_at = tile.a + ep.first, e = e_at < ep.E ? e_at : e_at - ep.E;  // the dropped limbs, the longer work, first
    const u32 blk = tile.blk, m_idx = pl_at(pl.mod, e);
    // the batch items of this workgroup: tile.b, tile.b + (the grid's extent over items), ...: a workgroup that takes several
    // fetches the slice's twiddles (half as many bytes as an item's points) once for all of them and requests an item's first
    // points before it is done with the previous item
    const u32 b_step = args.lo_group ? gridDim.y : gridDim.x;
    const size_t N = (size_t)1 << args.log_n, off = (size_t)blk << 11;
    const double* tw = args.tw_val + ((size_t)m_idx << args.log_n);
    const ModConstF mc = ((const ModConstF*)args.mc)[m_idx];
    const u32 own = e <= ep.level ? e / ep.D.alpha : 0xffffffffu;  // the digit that limb e belongs to
    const u32 TA = (1u << args.log_hi) + blk;
    const u32 d3 = tid >> 5, x5 = tid & 31, d2 = (tid >> 2) & 7, d0 = tid & 3;
    const size_t kstride = (size_t)ep.M * N;  // between the b and the a part of a digit's key; two of them per digit
    const size_t dstride = (size_t)ep.E * N;
    typedef ArithF64W AW;
    double wa[7], wb[7], wc[7], wd[6];  // the slice's twiddles, fetched once for all digits of all items
    if (!HOIST || DIV) {
        load_tw_w<3>(tw, TA, wa);
        load_tw_w<3>(tw, 8 * TA + d3, wb);
        load_tw_w<3>(tw, 64 * TA + 8 * d3 + d2, wc);
        load_tw_w<2>(tw, 512 * TA + 2 * tid, wd);
        load_tw_w<2>(tw, 512 * TA + 2 * tid + 1, wd + 3);
    }
    const u32 j0 = HOIST ? ep.beta : (own == 0 ? 1 : 0);  // first digit to transform
    E v[8], raw[8];
    // DIV: the converted parts of item b
    auto request_w = [&](u32 b, u32 comp) {
        const double* w = ep.w + ((size_t)(2 * b + comp) * ep.inv_from + e) * N + off;
#pragma unroll
        for (int i = 0; i < 8; i++) raw[i] = w[tid + 256 * i];
    };
    auto request_first = [&](u32 b) {  // the first points of item b
        if (j0 < ep.beta) {
            const double* hi0 = (const double*)(ep.D.digits + b * ep.D.bstride) + (size_t)e * N + off;
#pragma unroll
            for (int i = 0; i < 8; i++) raw[i] = hi0[(size_t)j0 * dstride + tid + 256 * i];
        } else if (DIV && !LIN) {
            request_w(b, 0);
        }
    };
    request_first(tile.b);
    const double cvd = DIV ? A::from_u64(ep.cinv[e]) : 0.0, cvq = DIV ? cvd / mc.q : 0.0;
    const bool summed = SUM && e < ep.inv_from;
    E acc0[8], acc1[8];
    for (u32 b = tile.b; b < args.batch; b += b_step) {
    const u64* key = ep.key.p[b] + (size_t)m_idx * N + off;
    const double* hi = (const double*)(ep.D.digits + b * ep.D.bstride) + (size_t)e * N + off;
    if (!SUM || b == tile.b || !summed) {  // a sum over items starts from the last one's reduced sum (f64m_sum_due: so it may)
#pragma unroll
        for (int j = 0; j < 8; j++) acc0[j] = acc1[j] = 0.0;
    }
    u32 j = j0;
    while (j < ep.beta) {
        u32 jn = j + 1;
        if (jn == own) jn++;
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] = raw[i];
        if (jn < ep.beta) {  // the next digit's points, a tile ahead
#pragma unroll
            for (int i = 0; i < 8; i++) raw[i] = hi[(size_t)jn * dstride + tid + 256 * i];
        } else if (DIV && !LIN) {
            request_w(b, 0);
        }
        A::fwd_begin(v, mc);
        fwd_rows_pre<AW, 3>(v, wa, mc);
#pragma unroll
        for (int i = 0; i < 8; i++) lds0[LDS_PAD(tid + 256 * i)] = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] = lds0[LDS_PAD(d3 * 256 + 32 * i + x5)];
        A::fwd_begin(v, mc);
        fwd_rows_pre<AW, 3>(v, wb, mc);
#pragma unroll
        for (int i = 0; i < 8; i++) lds1[LDS_PAD(d3 * 256 + 32 * i + x5)] = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] = lds1[LDS_PAD(d3 * 256 + d2 * 32 + 4 * i + d0)];
        A::fwd_begin(v, mc);
        fwd_rows_pre<AW, 3>(v, wc, mc);
#pragma unroll
        for (int i = 0; i < 8; i++) lds0[LDS_PAD(d3 * 256 + d2 * 32 + 4 * i + d0)] = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] = lds0[LDS_PAD(8 * tid + i)];
        // the key words of this digit at the points this thread ends up with: requested now, needed after the last round
        u64 k0[8], k1[8];
        {
            const u64* kj = key + (size_t)j * 2 * kstride;
#pragma unroll
            for (int i = 0; i < 8; i++) {
                k0[i] = kj[tid + 256 * i];
                k1[i] = kj[kstride + tid + 256 * i];
            }
        }
        fwd_rows_pre<AW, 2>(v, wd, mc);
        fwd_rows_pre<AW, 2>(v + 4, wd + 3, mc);
        A::fwd_end(v, mc);
        // back through LDS: point tid + 256 i of the slice, where the key words were fetched
#pragma unroll
        for (int i = 0; i < 8; i++) lds1[LDS_PAD(8 * tid + i)] = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const double y = lds1[LDS_PAD(tid + 256 * i)];
            acc0[i] += A::mulmod_any(y, A::from_u64(k0[i]), mc.q, mc.qinv);
            acc1[i] += A::mulmod_any(y, A::from_u64(k1[i]), mc.q, mc.qinv);
        }
        if (f64m_sum_due(j, jn)) {  // uniform; never with seven digits or fewer
#pragma unroll
            for (int i = 0; i < 8; i++) acc0[i] = A::reduce(acc0[i], mc), acc1[i] = A::reduce(acc1[i], mc);
        }
        j = jn;
    }
    // the next item's first points: requested before the operands of what follows, or, where those leave no registers (the
    // linear combination's twelve operands per point), after them
    auto request_next = [&]() {
        if (b + b_step < args.batch) request_first(b + b_step);
    };
    if (!LIN && !DIV) request_next();
    if (PROD && e <= ep.level) {
        // the tensor product of this slice, formed here: d2 feeds the digit that owns the limb, P d0 and P d1 join the sums
        const u64* kj = key + (size_t)own * 2 * kstride;
        const size_t po = (size_t)e * N + off;
        const u64 *pa0 = ep.a0.p[b] + po, *pa1 = ep.a1.p[b] + po, *pb0 = ep.b0.p[b] + po, *pb1 = ep.b1.p[b] + po;
        const double pres = mc.q - A::from_u64(ep.negp[e]);  // P mod q_e
        const u64* lx = LIN ? ep.lx.p[b] + po : nullptr;
        const u64* ly = LIN ? ep.ly.p[b] + po : nullptr;
        const double ka = LIN ? A::from_u64(ep.ka[e]) : 0.0, kb = LIN ? A::from_u64(ep.kb[e]) : 0.0;
        // four points at a time (two with the linear combination: the twiddles stay in registers for the next item and leave
        // room for 24 operands): six to ten operands per point, requested before the first is used
        constexpr int HP = LIN ? 2 : 4;
#pragma unroll
        for (int h = 0; h < 8; h += HP) {
            u64 ra0[HP], ra1[HP], rb0[HP], rb1[HP], rk0[HP], rk1[HP], rx0[HP], rx1[HP], ry0[HP], ry1[HP];
#pragma unroll
            for (int i = 0; i < HP; i++) {
                const u32 x = tid + 256 * (h + i);
                ra0[i] = pa0[x], ra1[i] = pa1[x], rb0[i] = pb0[x], rb1[i] = pb1[x];
                rk0[i] = kj[x], rk1[i] = kj[kstride + x];
                if (LIN) rx0[i] = lx[x], rx1[i] = lx[ep.x_cstride + x], ry0[i] = ly[x], ry1[i] = ly[ep.y_cstride + x];
            }
#pragma unroll
            for (int i = 0; i < HP; i++) {
                const double A0 = A::from_u64(ra0[i]), A1 = A::from_u64(ra1[i]), B0 = A::from_u64(rb0[i]), B1 = A::from_u64(rb1[i]);
                const double dd2 = A::mulmod_any(A1, B1, mc.q, mc.qinv);
                double dd0 = A::mulmod_any(A0, B0, mc.q, mc.qinv);
                double dd1 = A::mulmod_any(A0, B1, mc.q, mc.qinv) + A::mulmod_any(A1, B0, mc.q, mc.qinv);
                if (LIN) {  // at most 0.75 q more per term: both sums stay below 2^53
                    dd0 += A::mulmod_any(A::from_u64(rx0[i]), ka, mc.q, mc.qinv) + A::mulmod_any(A::from_u64(ry0[i]), kb, mc.q, mc.qinv);
                    dd1 += A::mulmod_any(A::from_u64(rx1[i]), ka, mc.q, mc.qinv) + A::mulmod_any(A::from_u64(ry1[i]), kb, mc.q, mc.qinv);
                }
                dd0 = A::reduce(dd0, mc);  // back below q / 2 + 1 as multiplicands
                dd1 = A::reduce(dd1, mc);
                acc0[h + i] += A::mulmod_any(dd2, A::from_u64(rk0[i]), mc.q, mc.qinv) + A::mulmod_any(dd0, pres, mc.q, mc.qinv);
                acc1[h + i] += A::mulmod_any(dd2, A::from_u64(rk1[i]), mc.q, mc.qinv) + A::mulmod_any(dd1, pres, mc.q, mc.qinv);
            }
        }
    } else if constexpr (HOIST) {
        // every digit, whole, and c0 through the rotation: a slice's sources are one slice, a wavefront's 64 points an aligned run of them
        const u64* co = ep.a0.p[b] + (size_t)e * N;
        const bool live = e <= ep.level;  // uniform
        const double pres = live ? mc.q - A::from_u64(ep.negp[e]) : 0.0;
        u32 x0 = (u32)off + tid;
        asm volatile("" : "+v"(x0));  // (see below)
        u32 xs[8];
#pragma unroll
        for (int i = 0; i < 8; i++) xs[i] = galois_gather_index(x0 + 256 * i, ep.gal[b], args.log_n);
        if (live) {
            u64 rc[8];
#pragma unroll
            for (int i = 0; i < 8; i++) rc[i] = word_at(co, xs[i]);
#pragma unroll
            for (int i = 0; i < 8; i++) acc0[i] = A::mulmod_any(A::from_u64(rc[i]), pres, mc.q, mc.qinv);
        }
        for (u32 d = 0; d < ep.beta; d++) {
            const u64* row = d == own ? ep.D.own.p[0] + (size_t)e * N : ep.D.digits + ((size_t)d * ep.E + e) * N;
            const u64* kj = key + (size_t)d * 2 * kstride;
            u64 ry[8], rk0[8], rk1[8];
#pragma unroll
            for (int i = 0; i < 8; i++) ry[i] = word_at(row, xs[i]), rk0[i] = kj[tid + 256 * i], rk1[i] = kj[kstride + tid + 256 * i];
#pragma unroll
            for (int i = 0; i < 8; i++) {
                const double y = A::from_u64(ry[i]);
                acc0[i] += A::mulmod_any(y, A::from_u64(rk0[i]), mc.q, mc.qinv);
                acc1[i] += A::mulmod_any(y, A::from_u64(rk1[i]), mc.q, mc.qinv);
            }
            if ((d & 3) == 3) {  // products of residues that are not reduced: 0.75 q each
#pragma unroll
                for (int i = 0; i < 8; i++) acc0[i] = A::reduce(acc0[i], mc), acc1[i] = A::reduce(acc1[i], mc);
            }
        }
    } else if (!PROD && e <= ep.level) {
        // the digit that owns this limb
        const u64* kj = key + (size_t)own * 2 * kstride;
        const u64* yo = ep.D.own.p[b] + (size_t)e * N;
        const u64* co = ROT ? ep.a0.p[b] + (size_t)e * N : nullptr;
        const u64* mo = MASK ? ep.mask + (size_t)e * N : nullptr;
        const u32 g = ROT ? ep.gal[b] : 1;
        const double pres = ROT ? mc.q - A::from_u64(ep.negp[e]) : 0.0;  // P mod q_e
        u32 x0 = (u32)off + tid;
        if (ROT) asm volatile("" : "+v"(x0));  // not the same for every item as far as the compiler can tell: it would keep what the index is made of
        constexpr int HP = ROT ? 4 : 8;  // points requested before the first is used
#pragma unroll
        for (int h = 0; h < 8; h += HP) {
            u64 ry[HP], rc[HP], rm[HP], rk0[HP], rk1[HP];
#pragma unroll
            for (int i = 0; i < HP; i++) {
                const u32 x = tid + 256 * (h + i);
                if (ROT) {
                    const u32 xs = galois_gather_index(x0 + 256 * (h + i), g, args.log_n);
                    ry[i] = word_at(yo, xs), rc[i] = word_at(co, xs);
                    if (MASK) rm[i] = word_at(mo, xs);
                } else {
                    ry[i] = yo[off + x];
                }
                rk0[i] = kj[x], rk1[i] = kj[kstride + x];
            }
#pragma unroll
            for (int i = 0; i < HP; i++) {
                double y = A::from_u64(ry[i]), cc = ROT ? A::from_u64(rc[i]) : 0.0;
                if (MASK) {  // below 0.75 q
                    const double m = A::from_u64(rm[i]);
                    y = A::mulmod_any(y, m, mc.q, mc.qinv);
                    cc = A::mulmod_any(cc, m, mc.q, mc.qinv);
                }
                acc0[h + i] += A::mulmod_any(y, A::from_u64(rk0[i]), mc.q, mc.qinv);
                if (ROT) acc0[h + i] += A::mulmod_any(cc, pres, mc.q, mc.qinv);
                acc1[h + i] += A::mulmod_any(y, A::from_u64(rk1[i]), mc.q, mc.qinv);
            }
        }
    }
    if (LIN && DIV) request_w(b, 0);
    if (LIN && !DIV) request_next();
    u64* o0 = ep.out.p[summed ? tile.b : b] + (size_t)e * N + off;
    u64* o1 = o0 + (size_t)ep.E * N;
#pragma unroll
    for (int i = 0; i < 8; i++) acc0[i] = A::reduce(acc0[i], mc), acc1[i] = A::reduce(acc1[i], mc);
    if (SUM && summed && b + b_step < args.batch) continue;  // uniform over the workgroup
    if constexpr (DIV) {  // (v - w) cinv, and what is added
        const u64* add = ep.add.p[b];
        u64* res = ep.res.p[b] + (size_t)e * N + off;
#pragma unroll
        for (int comp = 0; comp < 2; comp++) {
#pragma unroll
            for (int i = 0; i < 8; i++) v[i] = raw[i];
            if (comp == 0) request_w(b, 1);
            else request_next();
            fwd_lo_rounds(v, lds0, lds1, tid, wa, wb, wc, wd, mc);
            const size_t at = (size_t)comp * ep.inv_from * N;
            double r[8];
#pragma unroll
            for (int i = 0; i < 8; i++) r[i] = A::mulmod((comp ? acc1[i] : acc0[i]) - lds1[LDS_PAD(tid + 256 * i)], cvd, cvq, mc.q);
            if (add) {  // uniform
                const u64* ad = add + at + (size_t)e * N + off;
                u64 ra[8];
#pragma unroll
                for (int i = 0; i < 8; i++) ra[i] = ad[tid + 256 * i];
#pragma unroll
                for (int i = 0; i < 8; i++) r[i] = A::reduce(r[i] + A::from_u64(ra[i]), mc);
            }
#pragma unroll
            for (int i = 0; i < 8; i++) res[at + tid + 256 * i] = A::canonical(r[i], mc);
        }
        continue;
    }
    if (e >= ep.inv_from) {
        mac_inverse_lo(acc0, acc1, lds0, lds1, ep.itw_val + ((size_t)m_idx << args.log_n), TA, tid, mc, o0, o1);
    } else {
#pragma unroll
        for (int i = 0; i < 8; i++) {
            o0[tid + 256 * i] = A::canonical(acc0[i], mc);
            o1[tid + 256 * i] = A::canonical(acc1[i], mc);
        }
    }
    // (no barrier between items: the next item's first exchange writes lds0, and its barrier stands between the last item's
    // reads of lds1 and the next writes to it)
    }
}

// the first points of an inverse transform: canonical residues, or (MUL) the product or linear combination of two operands
template <class A, bool MUL>
__device__ __forceinline__ void inv_first_points(const NttArgs& args, const typename A::MC& mc, const ulonglong2* raw, const ulonglong2* raw2, typename A::E* v) {
    if constexpr (MUL) {
        if (args.use_lin) {  // uniform
            const double ka = A::from_u64(args.lin_ka), kb = A::from_u64(args.lin_kb);
#pragma unroll
            for (int j = 0; j < 4; j++) {
                v[2 * j] = A::reduce(A::mulmod_any(A::from_u64(raw[j].x), ka, mc.q, mc.qinv) + A::mulmod_any(A::from_u64(raw2[j].x), kb, mc.q, mc.qinv), mc);
                v[2 * j + 1] = A::reduce(A::mulmod_any(A::from_u64(raw[j].y), ka, mc.q, mc.qinv) + A::mulmod_any(A::from_u64(raw2[j].y), kb, mc.q, mc.qinv), mc);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; j++) {
                v[2 * j] = A::mulmod_any(A::from_u64(raw[j].x), A::from_u64(raw2[j].x), mc.q, mc.qinv);
                v[2 * j + 1] = A::mulmod_any(A::from_u64(raw[j].y), A::from_u64(raw2[j].y), mc.q, mc.qinv);
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; j++) {
            v[2 * j] = A::load_first(raw[j].x, mc, true);
            v[2 * j + 1] = A::load_first(raw[j].y, mc, true);
        }
    }
}

// the eight points 8 t + j of a slice of sigma_g of a polynomial: the map takes them to an aligned run of eight
__device__ __forceinline__ void load_permuted(const u64* __restrict__ poly, u32 x0, u32 g, u32 log_n, ulonglong2* raw) {
#pragma unroll
    for (int j = 0; j < 4; j++) {
        raw[j].x = word_at(poly, galois_gather_index(x0 + 2 * j, g, log_n));
        raw[j].y = word_at(poly, galois_gather_index(x0 + 2 * j + 1, g, log_n));
    }
}

// MUL (double-precision arithmetic, first pass, source list): the transform's input is the pointwise product of two
// polynomials (the d2 = a1 (.) b1 of a ciphertext product), formed as the points are loaded: d2 itself is never stored.
// GAL (likewise): it is the polynomial under the item's automorphism, gathered as it is loaded (with MUL: the product under it).
template <class A, int IT, bool MUL = false, bool GAL = false>
__global__ __launch_bounds__(NTT_THREADS) __attribute__((amdgpu_waves_per_eu(3, 8))) void ntt_inv_lo_kernel(NttArgs args, PolyList pl) {
    static_assert(!MUL || IT == 1, "the variants with two operands take one item");
    typedef typename A::E E;
    __shared__ E lds0[LDS_PADDED_WORDS];
    __shared__ E lds1[LDS_PADDED_WORDS];
    const u32 tid = threadIdx.x;
    const LoTile tile = lo_tile(args.log_hi, args.lo_group);
    const u32 blk = tile.blk, b0 = tile.b * IT;
    const u32 cnt = args.batch - b0 < (u32)IT ? args.batch - b0 : (u32)IT;
    const PolyRef<A> P = poly_ref<A>(args, pl, b0, tile.a);
    const size_t off = (size_t)blk << 11;
    const u32 TA = (1u << args.log_hi) + blk;
    const u32 d3 = tid >> 5, x5 = tid & 31, d2 = (tid >> 2) & 7, d0 = tid & 3;
    typedef typename LoTw<A>::TW TW;
    typedef typename LoTw<A>::AR AR;
    E v[8];
    ulonglong2 raw[4], raw2[MUL ? 4 : 1];
    TW wa[7], wb[7], wc[7], wd[6];
    load_lo_tw<A, 2>(P, 512 * TA + 2 * tid, wd);
    load_lo_tw<A, 2>(P, 512 * TA + 2 * tid + 1, wd + 3);
    load_lo_tw<A, 3>(P, 64 * TA + 8 * d3 + d2, wc);
    const size_t moff = ((size_t)pl_at(pl.spos, tile.a) << args.log_n) + off + 8 * tid;  // MUL: the multiplier's point
    if constexpr (GAL) {
        load_permuted(P.src, (u32)off + 8 * tid, args.gal[b0], args.log_n, raw);
        if constexpr (MUL) load_permuted(args.mul_list.p[b0] + ((size_t)pl_at(pl.spos, tile.a) << args.log_n), (u32)off + 8 * tid, args.gal[b0], args.log_n, raw2);
    } else {
        const ulonglong2* in = reinterpret_cast<const ulonglong2*>(P.src + off + 8 * tid);
#pragma unroll
        for (int j = 0; j < 4; j++) raw[j] = in[j];
        if constexpr (MUL) {
            const ulonglong2* in2 = reinterpret_cast<const ulonglong2*>(args.mul_list.p[b0] + moff);
#pragma unroll
            for (int j = 0; j < 4; j++) raw2[j] = in2[j];
        }
    }
#pragma unroll
    for (int it = 0; it < IT; it++) {
        if ((u32)it >= cnt) break;
        E* buf0 = (it & 1) ? lds1 : lds0;  // three exchanges per item: the buffers swap roles from item to item
        E* buf1 = (it & 1) ? lds0 : lds1;
        inv_first_points<A, MUL>(args, P.mc, raw, raw2, v);
        if (it + 1 < IT && (u32)(it + 1) < cnt) {  // the next item's points, a tile ahead
            const u64* next = item_src<A>(args, pl, b0 + it + 1, tile.a);
            if constexpr (GAL) {
                load_permuted(next, (u32)off + 8 * tid, args.gal[b0 + it + 1], args.log_n, raw);
            } else {
                const ulonglong2* in = reinterpret_cast<const ulonglong2*>(next + off + 8 * tid);
#pragma unroll
                for (int j = 0; j < 4; j++) raw[j] = in[j];
            }
        }
        inv_rows_pre<AR, 2>(v, wd, P.mc);
        inv_rows_pre<AR, 2>(v + 4, wd + 3, P.mc);
        A::inv_end2(v, P.mc);
        if (it == 0) load_lo_tw<A, 3>(P, 8 * TA + d3, wb);
#pragma unroll
        for (int j = 0; j < 8; j++) buf0[LDS_PAD(8 * tid + j)] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = buf0[LDS_PAD(d3 * 256 + d2 * 32 + 4 * j + d0)];
        inv_rows_pre<AR, 3>(v, wc, P.mc);
        A::inv_end(v, P.mc);
        if (it == 0) load_lo_tw<A, 3>(P, TA, wa);
#pragma unroll
        for (int j = 0; j < 8; j++) buf1[LDS_PAD(d3 * 256 + d2 * 32 + 4 * j + d0)] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = buf1[LDS_PAD(d3 * 256 + 32 * j + x5)];
        inv_rows_pre<AR, 3>(v, wb, P.mc);
        A::inv_end(v, P.mc);
#pragma unroll
        for (int j = 0; j < 8; j++) buf0[LDS_PAD(d3 * 256 + 32 * j + x5)] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = buf0[LDS_PAD(tid + 256 * j)];
        inv_rows_pre<AR, 3>(v, wa, P.mc);
        A::inv_end(v, P.mc);
        u64* dst = item_dst(args, pl, b0 + it, tile.a) + off;
        if (args.last) {
#pragma unroll
            for (int j = 0; j < 8; j++) dst[tid + 256 * j] = A::store_inv_final(v[j], P.mc);
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++) dst[tid + 256 * j] = A::store_mid(v[j]);  // the hi pass follows
        }
    }
}

// ============================ hi pass (rows 2^11 apart, adjacent columns) ============================
// tile = R = 2^LOG_HI rows x CC = 2048/R columns; element (row, col) lives at (row << 11) + col0 + col.
// LOG_HI <= 3: a thread holds all R rows of 8/R columns (no exchange).
// LOG_HI >= 4: round 1 = radix 8 over rows r0 + (R/8)*j of one column; exchange through LDS;
//              round 2 = the remaining LOG_HI-3 stages over R/8 consecutive rows of 64/R adjacent columns.
// The forward hi pass is the first pass of a transform (reads canonical residues, writes the
// intermediate form); the inverse hi pass is the last one.
template <class A, int LOG_HI>
__global__ __launch_bounds__(NTT_THREADS) void ntt_fwd_hi_kernel(NttArgs args, PolyList pl) {
    typedef typename A::E E;
    constexpr int R = 1 << LOG_HI, CC = NTT_TILE / R;
    const u32 tid = threadIdx.x, row = blockIdx.y / pl.n, a = blockIdx.y % pl.n;
    if constexpr (!std::is_same<A, ArithF64>::value)
        if (own_limb(args, row, a)) return;  // whole workgroup
    const PolyRef<A> P = poly_ref<A>(args, pl, row, a);
    const u64* src = P.src + (size_t)blockIdx.x * CC;
    u64* dst = P.dst + (size_t)blockIdx.x * CC;
    E v[8];
    if constexpr (LOG_HI <= 3) {
        constexpr int KC = 8 / R;
#pragma unroll
        for (int rr = 0; rr < R; rr++)
#pragma unroll
            for (int kc = 0; kc < KC; kc++) v[rr * KC + kc] = A::load_first(src[((size_t)rr << 11) + kc * 256 + tid], P.mc, false);
        fwd_rows<A, LOG_HI, KC>(v, P.tw, 1, P.mc);
#pragma unroll
        for (int rr = 0; rr < R; rr++)
#pragma unroll
            for (int kc = 0; kc < KC; kc++) dst[((size_t)rr << 11) + kc * 256 + tid] = A::store_mid(v[rr * KC + kc]);
    } else {
        __shared__ __attribute__((aligned(16))) E lds[NTT_TILE];
        constexpr int R8 = R / 8, S2 = LOG_HI - 3, KC2 = 8 / R8;
        const u32 r0 = tid / CC, col = tid % CC;
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = A::load_first(src[((size_t)(r0 + R8 * j) << 11) + col], P.mc, false);
        fwd_rows<A, 3, 1>(v, P.tw, 1, P.mc);
#pragma unroll
        for (int j = 0; j < 8; j++) lds[(r0 + R8 * j) * CC + col] = v[j];
        __syncthreads();
        const u32 G = tid >> 5, cg = tid & 31;
#pragma unroll
        for (int rr = 0; rr < R8; rr++)
#pragma unroll
            for (int kc = 0; kc < KC2; kc++) v[rr * KC2 + kc] = lds[(G * R8 + rr) * CC + cg * KC2 + kc];
        A::fwd_begin(v, P.mc);
        fwd_rows<A, S2, KC2>(v, P.tw, 8 + G, P.mc);
#pragma unroll
        for (int rr = 0; rr < R8; rr++)
#pragma unroll
            for (int kc = 0; kc < KC2; kc++) dst[((size_t)(G * R8 + rr) << 11) + cg * KC2 + kc] = A::store_mid(v[rr * KC2 + kc]);
    }
}

// The forward hi pass with a basis conversion (ModUp's or ModDown's) in front of it: the points of the target limb at
// position e = pl.dpos[a] are
//   sum_i yhat_i * [B/b_i]_{q_e}  mod q_e
// evaluated from the source basis' centred residues yhat (doubles, nd limbs from position lo of each batch item of y)
// as the tile is loaded: the converted polynomial is never written in coefficient form.
// convf: [position][ap] (constant, constant / q_e), rows padded with zeros to ap = 4, 8, 12 or 16 entries.
// alpha != 0 (ModUp): the digits of a polynomial in one launch, blockIdx.z = digit j.  Digit j has the source limbs
// [j alpha, (j + 1) alpha) of the n_src there are, its table at convf + j * convf_dstride, its results at dst + j * dst_dstride,
// and every entry of the list but its own limbs as targets.
struct ConvPrologue {
    const double* y;
    size_t y_bstride;  // elements
    const TwF* convf;
    u32 lo, nd;
    u32 ap, groups;    // groups: workgroups per tile and polynomial (T targets each)
    u32 alpha, n_src, digit0, per;  // digit0: the launch's first digit; per: targets per workgroup (ntt_mid_conv_kernel)
    size_t convf_dstride, dst_dstride;
};

// the source residues of one point: no branch around the loads (entries beyond the nd source limbs re-read the last
// one against a zero constant)
// ND <= AP: the entries that are read and multiplied (a row of the constants has AP, the last AP - ND of them zero)
template <int AP, int ND>
__device__ __forceinline__ void conv_load(double (&yv)[AP], const double* __restrict__ yp, size_t N, u32 nd) {
#pragma unroll
    for (int a = 0; a < ND; a++) yv[a] = yp[(size_t)((u32)a < nd ? a : nd - 1) * N];
}
template <int AP, int ND>
__device__ __forceinline__ double conv_sum(const double (&yv)[AP], const double* cw, double q, double qinv) {
    static_assert(ND <= 8 || AP > 8, "rows of more than eight entries are padded to twelve or sixteen");
    return f64m_dot_w<ND>(yv, cw, q, qinv);
}

// The source limbs of a conversion that are still to go through the last pass of their inverse transform.
struct MidPrologue {
    const TwF* itw;     // [M][N] inverse twiddles, and their values alone
    const double* itw_val;
    const TwF* scale;   // by modulus: what the inverse transform's last step multiplies by
    u32 first, next;    // source limb k has the modulus k ? next + k - 1 : first (a digit's first limb is added to both)
};

// One workgroup converts and transforms the same tile of T target limbs: the source residues are fetched once for all T
// (the fetch, from L2 after the first, is what bounds a one-target-per-workgroup version).
// MID (one source limb, LOG_HI >= 4): the source is what the inverse transform's first pass left, and goes through its second here, on the
// same tile.
template <int LOG_HI, int AP, int T, int ND = AP, bool MID = false>
__global__ __launch_bounds__(NTT_THREADS) void ntt_fwd_hi_conv_kernel(NttArgs args, PolyList pl, ConvPrologue cp, MidPrologue mp) {
    static_assert(!MID || (ND == 1 && LOG_HI >= 4), "");
    typedef ArithF64 A;
    typedef double E;
    constexpr int R = 1 << LOG_HI, CC = NTT_TILE / R;
    const u32 tid = threadIdx.x, tile = blockIdx.x, b = blockIdx.y / cp.groups, a0 = (blockIdx.y % cp.groups) * T;
    const size_t N = (size_t)1 << args.log_n;
    const u32 dig = cp.digit0 + blockIdx.z, lo = cp.lo + dig * cp.alpha;
    const u32 nd = cp.alpha ? min(cp.alpha, cp.n_src - lo) : cp.nd;
    const u32 n_targets = cp.alpha ? pl.n - nd : pl.n;
    if (a0 >= n_targets) return;  // whole workgroup: a digit with more limbs has fewer targets
    const TwF* convf = cp.convf + dig * cp.convf_dstride;
    const double* y = cp.y + b * cp.y_bstride + (size_t)lo * N + (size_t)tile * CC;
    PolyRef<A> P[T];
    double cw[T][ND];  // the centred constants (the tables' quotients by the modulus are not read)
#pragma unroll
    for (int t = 0; t < T; t++) {
        u32 a_idx = a0 + t < n_targets ? a0 + t : n_targets - 1;  // a ragged last group repeats its last limb and skips the store
        if (cp.alpha && a_idx >= lo) a_idx += nd;
        P[t] = poly_ref<A, true>(args, pl, b, a_idx);
        P[t].dst += dig * cp.dst_dstride;
        const TwF* ce = convf + (size_t)pl.dpos[a_idx] * AP;
#pragma unroll
        for (int a = 0; a < ND; a++) cw[t][a] = ce[a].w;
    }
    E v[T][8];
    if constexpr (LOG_HI <= 3) {
        constexpr int KC = 8 / R;
#pragma unroll
        for (int rr = 0; rr < R; rr++)
#pragma unroll
            for (int kc = 0; kc < KC; kc++) {
                double yv[AP];
                conv_load<AP, ND>(yv, y + ((size_t)rr << 11) + kc * 256 + tid, N, nd);
#pragma unroll
                for (int t = 0; t < T; t++) v[t][rr * KC + kc] = conv_sum<AP, ND>(yv, cw[t], P[t].mc.q, P[t].mc.qinv);
            }
#pragma unroll
        for (int t = 0; t < T; t++) {
            if (a0 + t >= n_targets) break;
            u64* dst = P[t].dst + (size_t)tile * CC;
            fwd_rows<A, LOG_HI, KC>(v[t], P[t].tw, 1, P[t].mc);
#pragma unroll
            for (int rr = 0; rr < R; rr++)
#pragma unroll
                for (int kc = 0; kc < KC; kc++) dst[((size_t)rr << 11) + kc * 256 + tid] = A::store_mid(v[t][rr * KC + kc]);
        }
    } else {
        __shared__ __attribute__((aligned(16))) E lds[NTT_TILE];
        constexpr int R8 = R / 8, S2 = LOG_HI - 3, KC2 = 8 / R8;
        const u32 r0 = tid / CC, col = tid % CC, G = tid >> 5, cg = tid & 31;
        if constexpr (MID) {  // ntt_inv_hi_kernel's two rounds
            const u32 m_src = dig * cp.alpha + mp.first;
            const ModConstF mc = ((const ModConstF*)args.mc)[m_src];
            const TwF scale = mp.scale[m_src];
            const TwF* tw = mp.itw + ((size_t)m_src << args.log_n);
            E u[8];
#pragma unroll
            for (int rr = 0; rr < R8; rr++)
#pragma unroll
                for (int kc = 0; kc < KC2; kc++) u[rr * KC2 + kc] = y[((size_t)(G * R8 + rr) << 11) + cg * KC2 + kc];
            inv_rows<A, S2, KC2>(u, tw, 8 + G, mc);
            if (S2 == 3) A::inv_end(u, mc);
#pragma unroll
            for (int rr = 0; rr < R8; rr++)
#pragma unroll
                for (int kc = 0; kc < KC2; kc++) lds[(G * R8 + rr) * CC + cg * KC2 + kc] = u[rr * KC2 + kc];
            __syncthreads();
#pragma unroll
            for (int j = 0; j < 8; j++) u[j] = lds[(r0 + R8 * j) * CC + col];
            inv_rows<A, 3, 1>(u, tw, 1, mc);
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const double yv[1] = {f64m_centre(A::mulmod(u[j], scale.w, scale.wq, mc.q), mc.q)};
#pragma unroll
                for (int t = 0; t < T; t++) v[t][j] = f64m_dot_w<1>(yv, cw[t], P[t].mc.q, P[t].mc.qinv);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++) {
                double yv[AP];
                conv_load<AP, ND>(yv, y + ((size_t)(r0 + R8 * j) << 11) + col, N, nd);
#pragma unroll
                for (int t = 0; t < T; t++) v[t][j] = conv_sum<AP, ND>(yv, cw[t], P[t].mc.q, P[t].mc.qinv);
            }
        }
#pragma unroll
        for (int t = 0; t < T; t++) {
            if (a0 + t >= n_targets) break;  // uniform over the workgroup
            u64* dst = P[t].dst + (size_t)tile * CC;
            if (t || MID) __syncthreads();  // the previous exchange has been read
            fwd_rows<A, 3, 1>(v[t], P[t].tw, 1, P[t].mc);
#pragma unroll
            for (int j = 0; j < 8; j++) lds[(r0 + R8 * j) * CC + col] = v[t][j];
            __syncthreads();
#pragma unroll
            for (int rr = 0; rr < R8; rr++)
#pragma unroll
                for (int kc = 0; kc < KC2; kc++) v[t][rr * KC2 + kc] = lds[(G * R8 + rr) * CC + cg * KC2 + kc];
            A::fwd_begin(v[t], P[t].mc);
            fwd_rows<A, S2, KC2>(v[t], P[t].tw, 8 + G, P[t].mc);
#pragma unroll
            for (int rr = 0; rr < R8; rr++)
#pragma unroll
                for (int kc = 0; kc < KC2; kc++) dst[((size_t)(G * R8 + rr) << 11) + cg * KC2 + kc] = A::store_mid(v[t][rr * KC2 + kc]);
        }
    }
}

// The converting hi pass of the larger rings (LOG_HI >= 4) as two phases through LDS.  Its time is arithmetic, about 70
// double-precision operations per point and target: 40 for a sum of eight terms, the rest butterflies.  With a thread holding
// its eight points of several targets through both (the kernel above), most of 210 registers are points that wait and
// the targets' constants overflow the scalar registers (two waves per SIMD, 50 scalar spills).  Here a workgroup of
// 512 threads first converts its tile for four targets, one target at a time (a thread's points: tid + 512 i; the target's
// constants are wide scalar loads), into 64 KB of LDS, then each half of the workgroup transforms two of the targets in
// place.  Nothing but the source residues lives across targets: at most 128 registers, four waves per SIMD from two workgroups
// whose phases interleave, and a small launch's workgroup is done sooner.  8 -> 13 and 5 -> 16 limbs of one polynomial at
// N = 2^16 (a digit each): 17.5 us a launch and digit with the kernel above, 13 us for both; launches that fill the chip several
// times gain little (8 polynomials, 8 -> 19 limbs: 47.8 and 45.2 us; vector units 68 % busy while a CU has work, which it
// has 72 % of the time).  A workgroup that goes on with more sets of its tile is slower (52 us).
// The tables are read through the constant address space: behind the stores to LDS the compiler would otherwise fetch
// wave-uniform constants with vector loads.
#define HC_THREADS 512
#define HC_T 4
template <class V>
using ConstPtr = const __attribute__((address_space(4))) V*;
template <class V>
__device__ __forceinline__ ConstPtr<V> const_ptr(const V* p) { return (ConstPtr<V>)p; }
// MID: the source limbs are what the inverse transform's first pass left and go through its second here first, four at a time: each half of
// the workgroup takes two through the two rounds of ntt_inv_hi_kernel in the buffers that the targets use afterwards.
template <int LOG_HI, int AP, int ND, bool MID>
__global__ __launch_bounds__(HC_THREADS) __attribute__((amdgpu_waves_per_eu(4, 4))) void ntt_fwd_hi_conv_lds_kernel(NttArgs args, PolyList pl, ConvPrologue cp,
                                                                                                                   MidPrologue mp) {
    static_assert(!MID || ND <= CONV_MID_TERMS, "");
    typedef ArithF64 A;
    constexpr int R = 1 << LOG_HI, CC = NTT_TILE / R, PTS = NTT_TILE / HC_THREADS, PP = ND <= 9 ? PTS : 2;
    constexpr int R8 = R / 8, S2 = LOG_HI - 3, KC2 = 8 / R8;
    __shared__ __attribute__((aligned(16))) double lds[HC_T][NTT_TILE];
    const u32 tid = threadIdx.x, tile = blockIdx.x, b = blockIdx.y / cp.groups, a0 = (blockIdx.y % cp.groups) * HC_T;
    const size_t N = (size_t)1 << args.log_n;
    const u32 dig = cp.digit0 + blockIdx.z, lo = cp.lo + dig * cp.alpha;
    const u32 nd = cp.alpha ? min(cp.alpha, cp.n_src - lo) : cp.nd;
    const u32 n_targets = cp.alpha ? pl.n - nd : pl.n;
    if (a0 >= n_targets) return;  // whole workgroup: a digit with more limbs has fewer targets
    const u32 cnt = min((u32)HC_T, n_targets - a0);
    const TwF* convf = cp.convf + dig * cp.convf_dstride;
    const double* y = cp.y + b * cp.y_bstride + (size_t)lo * N + (size_t)tile * CC;
    u64* dst0 = args.dst + (((size_t)b * args.dst_bstride) << args.log_n) + dig * cp.dst_dstride + (size_t)tile * CC;
    auto entry = [&](u32 a) { return cp.alpha && a >= lo ? a + nd : a; };  // list entry of target a: past the digit's own limbs
    const u32 half = __builtin_amdgcn_readfirstlane(tid >> 8), lt = tid & 255;
    const u32 r0 = lt / CC, col = lt % CC, G = lt >> 5, cg = lt & 31;
#pragma unroll
    for (int h = 0; h < PTS; h += PP) {
        double yv[PP][AP];
#pragma unroll
        for (int i = 0; i < PP; i++) {
            const u32 p = tid + HC_THREADS * (h + i), off = ((p / CC) << 11) + p % CC;
            if constexpr (!MID)
#pragma unroll
                for (int k = 0; k < ND; k++) yv[i][k] = (y + (size_t)((u32)k < nd ? k : nd - 1) * N)[off];  // see conv_load
        }
        if constexpr (MID) {
#pragma unroll
            for (int k0 = 0; k0 < ND; k0 += HC_T) {
                double u[2][8];
                auto source = [&](int s) { return min((u32)k0 + half + 2 * s, nd - 1); };  // see conv_load
                auto modulus = [&](u32 k) { return dig * cp.alpha + (k ? mp.next + k - 1 : mp.first); };
                if (k0) __syncthreads();  // the last four have been read
#pragma unroll
                for (int s = 0; s < 2; s++)
                    if (k0 + 2 * s < ND) {
                        const double* ys = y + (size_t)source(s) * N;
#pragma unroll
                        for (int rr = 0; rr < R8; rr++)
#pragma unroll
                            for (int kc = 0; kc < KC2; kc++) u[s][rr * KC2 + kc] = ys[((G * R8 + rr) << 11) + cg * KC2 + kc];
                    }
#pragma unroll
                for (int s = 0; s < 2; s++)
                    if (k0 + 2 * s < ND) {
                        const u32 m_idx = modulus(source(s));
                        ConstPtr<ModConstF> pm = const_ptr((const ModConstF*)args.mc + m_idx);
                        const ModConstF mc = {pm->q, pm->qinv, 0.0, 0.0};
                        inv_rows<A, S2, KC2>(u[s], mp.itw + ((size_t)m_idx << args.log_n), 8 + G, mc);
                        if (S2 == 3) A::inv_end(u[s], mc);
#pragma unroll
                        for (int rr = 0; rr < R8; rr++)
#pragma unroll
                            for (int kc = 0; kc < KC2; kc++) lds[half + 2 * s][(G * R8 + rr) * CC + cg * KC2 + kc] = u[s][rr * KC2 + kc];
                    }
                __syncthreads();
#pragma unroll
                for (int s = 0; s < 2; s++)
                    if (k0 + 2 * s < ND) {
                        const u32 m_idx = modulus(source(s));
                        ConstPtr<ModConstF> pm = const_ptr((const ModConstF*)args.mc + m_idx);
                        ConstPtr<TwF> ps = const_ptr(mp.scale + m_idx), tw = const_ptr(mp.itw + ((size_t)m_idx << args.log_n));
                        const ModConstF mc = {pm->q, pm->qinv, 0.0, 0.0};
                        const TwF scale = {ps->w, ps->wq};
                        TwF w1[7];
#pragma unroll
                        for (int i = 0; i < 7; i++) w1[i] = TwF{tw[1 + i].w, tw[1 + i].wq};
                        double* buf = lds[half + 2 * s];  // a thread writes back what it has read
#pragma unroll
                        for (int j = 0; j < 8; j++) u[s][j] = buf[(r0 + R8 * j) * CC + col];
                        inv_rows_pre<A, 3>(u[s], w1, mc);
#pragma unroll
                        for (int j = 0; j < 8; j++) buf[(r0 + R8 * j) * CC + col] = f64m_centre(A::mulmod(u[s][j], scale.w, scale.wq, mc.q), mc.q);
                    }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < PP; i++)
#pragma unroll
                    for (int k = k0; k < k0 + HC_T && k < ND; k++) yv[i][k] = lds[k - k0][tid + HC_THREADS * i];
            }
        }
#pragma unroll 1
        for (u32 t = 0; t < cnt; t++) {
            const u32 a = entry(a0 + t), m_idx = pl_at(pl.mod, a);
            ConstPtr<TwF> ce = const_ptr(convf + (size_t)pl_at(pl.dpos, a) * AP);
            ConstPtr<ModConstF> mc = const_ptr((const ModConstF*)args.mc + m_idx);
            const double q = mc->q, qinv = mc->qinv;
            double cw[ND];
#pragma unroll
            for (int k = 0; k < ND; k++) cw[k] = ce[k].w;
#pragma unroll
            for (int i = 0; i < PP; i++) lds[t][tid + HC_THREADS * (h + i)] = conv_sum<AP, ND>(yv[i], cw, q, qinv);
        }
    }
    __syncthreads();
#pragma unroll 1
    for (u32 t = half; t < cnt; t += 2) {
        const u32 m_idx = pl_at(pl.mod, entry(a0 + t));
        const TwF* tw = (const TwF*)args.tw + ((size_t)m_idx << args.log_n);
        ConstPtr<ModConstF> pm = const_ptr((const ModConstF*)args.mc + m_idx);
        const ModConstF mc = {pm->q, pm->qinv, 0.0, 0.0};
        double v[8];
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = lds[t][(r0 + R8 * j) * CC + col];
        TwF w1[7];
#pragma unroll
        for (int i = 0; i < 7; i++) w1[i] = TwF{const_ptr(tw + 1 + i)->w, const_ptr(tw + 1 + i)->wq};
        fwd_rows_pre<A, 3>(v, w1, mc);
#pragma unroll
        for (int j = 0; j < 8; j++) lds[t][(r0 + R8 * j) * CC + col] = v[j];
    }
    __syncthreads();
#pragma unroll 1
    for (u32 t = half; t < cnt; t += 2) {
        const u32 a = entry(a0 + t), m_idx = pl_at(pl.mod, a);
        const TwF* tw = (const TwF*)args.tw + ((size_t)m_idx << args.log_n);
        ConstPtr<ModConstF> pm = const_ptr((const ModConstF*)args.mc + m_idx);
        const ModConstF mc = {pm->q, pm->qinv, 0.0, 0.0};
        u64* dst = dst0 + ((size_t)pl_at(pl.dpos, a) << args.log_n);
        double v[8];
#pragma unroll
        for (int rr = 0; rr < R8; rr++)
#pragma unroll
            for (int kc = 0; kc < KC2; kc++) v[rr * KC2 + kc] = lds[t][(G * R8 + rr) * CC + cg * KC2 + kc];
        A::fwd_begin(v, mc);
        fwd_rows<A, S2, KC2>(v, tw, 8 + G, mc);
#pragma unroll
        for (int rr = 0; rr < R8; rr++)
#pragma unroll
            for (int kc = 0; kc < KC2; kc++) dst[((size_t)(G * R8 + rr) << 11) + cg * KC2 + kc] = A::store_mid(v[rr * KC2 + kc]);
    }
}

// The inverse transform's last store: times 1/N, canonical; or (double-precision arithmetic only) times *scale and centred,
// as a double: |t| < 0.75 q after the exact product, so the centred representative is t, t - q or t + q.
template <class A>
__device__ __forceinline__ u64 inv_last_store(typename A::E v, const typename A::MC& m, const TwF* scale) {
    if constexpr (std::is_same<A, ArithF64>::value) {
        if (scale) {
            const TwF k = *scale;
            const double t = f64m_centre(ArithF64::mulmod(v, k.w, k.wq, m.q), m.q);
            return (u64)__double_as_longlong(t);
        }
    }
    return A::store_inv_final(v, m);
}

template <class A, int LOG_HI>
__global__ __launch_bounds__(NTT_THREADS) void ntt_inv_hi_kernel(NttArgs args, PolyList pl) {
    typedef typename A::E E;
    constexpr int R = 1 << LOG_HI, CC = NTT_TILE / R;
    const u32 tid = threadIdx.x;
    const PolyRef<A> P = poly_ref<A>(args, pl, blockIdx.y / pl.n, blockIdx.y % pl.n);
    u64* dst = P.dst + (size_t)blockIdx.x * CC;  // the lo pass has already moved the data to dst
    const TwF* scale = args.inv_scale ? args.inv_scale + pl_at(pl.mod, blockIdx.y % pl.n) : nullptr;
    E v[8];
    if constexpr (LOG_HI <= 3) {
        constexpr int KC = 8 / R;
#pragma unroll
        for (int rr = 0; rr < R; rr++)
#pragma unroll
            for (int kc = 0; kc < KC; kc++) v[rr * KC + kc] = A::load_mid(dst[((size_t)rr << 11) + kc * 256 + tid]);
        inv_rows<A, LOG_HI, KC>(v, P.tw, 1, P.mc);
#pragma unroll
        for (int rr = 0; rr < R; rr++)
#pragma unroll
            for (int kc = 0; kc < KC; kc++) dst[((size_t)rr << 11) + kc * 256 + tid] = inv_last_store<A>(v[rr * KC + kc], P.mc, scale);
    } else {
        __shared__ __attribute__((aligned(16))) E lds[NTT_TILE];
        constexpr int R8 = R / 8, S2 = LOG_HI - 3, KC2 = 8 / R8;
        const u32 G = tid >> 5, cg = tid & 31;
#pragma unroll
        for (int rr = 0; rr < R8; rr++)
#pragma unroll
            for (int kc = 0; kc < KC2; kc++) v[rr * KC2 + kc] = A::load_mid(dst[((size_t)(G * R8 + rr) << 11) + cg * KC2 + kc]);
        inv_rows<A, S2, KC2>(v, P.tw, 8 + G, P.mc);
        if (S2 == 3) A::inv_end(v, P.mc);
#pragma unroll
        for (int rr = 0; rr < R8; rr++)
#pragma unroll
            for (int kc = 0; kc < KC2; kc++) lds[(G * R8 + rr) * CC + cg * KC2 + kc] = v[rr * KC2 + kc];
        __syncthreads();
        const u32 r0 = tid / CC, col = tid % CC;
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = lds[(r0 + R8 * j) * CC + col];
        inv_rows<A, 3, 1>(v, P.tw, 1, P.mc);
#pragma unroll
        for (int j = 0; j < 8; j++) dst[((size_t)(r0 + R8 * j) << 11) + col] = inv_last_store<A>(v[j], P.mc, scale);
    }
}

// Division of a SUM of items by dropped moduli (launch_ntt_moddown_sum).  Each item rounds by itself, so each one's dropped limbs go through
// their inverse transform and are centred; from there on the division is linear: sum_r (v_r - NTT(conv(y_r))) / P = (sum_r v_r - NTT(conv(sum_r y_r))) / P,
// limb by limb modulo q_i.  So the centred residues are added up as integers (at most 16 of them, below 2^53) and there is one conversion and one
// forward transform for all items, where each had its own.  Four blocks of 19 + 8 limbs merged at N = 2^16: 352 -> 283 us (a rotation's product with
// its mask is formed as it is read, too).
// The inverse transform's last pass of the items 2 r + comp, r < n_items, added up into item comp.  grid = (tiles, components x list)
template <int LOG_HI>
__global__ __launch_bounds__(NTT_THREADS) void ntt_inv_hi_sum_kernel(NttArgs args, PolyList pl, u32 n_items) {
    typedef ArithF64 A;
    constexpr int R = 1 << LOG_HI, CC = NTT_TILE / R;
    const u32 tid = threadIdx.x, comp = blockIdx.y / pl.n, a = blockIdx.y % pl.n;
    const PolyRef<A> P = poly_ref<A>(args, pl, comp, a);
    u64* dst = P.dst + (size_t)blockIdx.x * CC;
    const size_t item = (2 * args.dst_bstride) << args.log_n;
    const TwF scale = args.inv_scale[pl_at(pl.mod, a)];
    double raw[8], sum[8];
    if constexpr (LOG_HI <= 3) {
        constexpr int KC = 8 / R;
        auto load = [&](u32 r) {
#pragma unroll
            for (int i = 0; i < 8; i++) raw[i] = A::load_mid((dst + r * item)[((size_t)(i / KC) << 11) + (i % KC) * 256 + tid]);
        };
        load(0);
        for (u32 r = 0; r < n_items; r++) {
            double v[8];
#pragma unroll
            for (int i = 0; i < 8; i++) v[i] = raw[i];
            if (r + 1 < n_items) load(r + 1);
            inv_rows<A, LOG_HI, KC>(v, P.tw, 1, P.mc);
#pragma unroll
            for (int i = 0; i < 8; i++) {
                const double t = f64m_centre(A::mulmod(v[i], scale.w, scale.wq, P.mc.q), P.mc.q);
                sum[i] = r ? sum[i] + t : t;
            }
        }
#pragma unroll
        for (int i = 0; i < 8; i++) dst[((size_t)(i / KC) << 11) + (i % KC) * 256 + tid] = A::store_mid(sum[i]);
    } else {
        __shared__ __attribute__((aligned(16))) double lds[2][NTT_TILE];  // in turn: an item's reads and the next one's writes do not meet
        constexpr int R8 = R / 8, S2 = LOG_HI - 3, KC2 = 8 / R8;
        const u32 G = tid >> 5, cg = tid & 31, r0 = tid / CC, col = tid % CC;
        auto load = [&](u32 r) {
#pragma unroll
            for (int i = 0; i < 8; i++) raw[i] = A::load_mid((dst + r * item)[((size_t)(G * R8 + i / KC2) << 11) + cg * KC2 + i % KC2]);
        };
        load(0);
        for (u32 r = 0; r < n_items; r++) {
            double v[8];
            double* buf = lds[r & 1];
#pragma unroll
            for (int i = 0; i < 8; i++) v[i] = raw[i];
            if (r + 1 < n_items) load(r + 1);
            inv_rows<A, S2, KC2>(v, P.tw, 8 + G, P.mc);
            if (S2 == 3) A::inv_end(v, P.mc);
#pragma unroll
            for (int i = 0; i < 8; i++) buf[(G * R8 + i / KC2) * CC + cg * KC2 + i % KC2] = v[i];
            __syncthreads();
#pragma unroll
            for (int j = 0; j < 8; j++) v[j] = buf[(r0 + R8 * j) * CC + col];
            inv_rows<A, 3, 1>(v, P.tw, 1, P.mc);
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const double t = f64m_centre(A::mulmod(v[j], scale.w, scale.wq, P.mc.q), P.mc.q);
                sum[j] = r ? sum[j] + t : t;
            }
        }
        // (item 0's points of this tile were all read before the first barrier)
#pragma unroll
        for (int j = 0; j < 8; j++) dst[((size_t)(r0 + R8 * j) << 11) + col] = A::store_mid(sum[j]);
    }
}

// The conversion of such a sum with the first pass of its forward transform, a target limb per workgroup.  The sums, up to 2^53, are reduced modulo the
// target first; the constants' rows are taken four at a time (padded with zeros).  One launch of a kind per sum: neither source limbs that
// several targets share (two: 21.8 us for 2 x 8 -> 19 limbs at N = 2^16, one: 20.9, twice the waves) nor numbers of terms known to the
// compiler, as the kernel for every item has them, are worth their instantiations here.
// grid = (tiles, targets x components)
template <int LOG_HI>
__global__ __launch_bounds__(NTT_THREADS) void ntt_fwd_hi_conv_sum_kernel(NttArgs args, PolyList pl, ConvPrologue cp) {
    typedef ArithF64 A;
    constexpr int R = 1 << LOG_HI, CC = NTT_TILE / R, KC = LOG_HI <= 3 ? 8 / R : 1, R8 = LOG_HI <= 3 ? 1 : R / 8, S2 = LOG_HI <= 3 ? 1 : LOG_HI - 3, KC2 = 8 / R8;
    const u32 tid = threadIdx.x, b = blockIdx.y / pl.n, a = blockIdx.y % pl.n, m_idx = pl_at(pl.mod, a), pos = pl_at(pl.dpos, a);
    const size_t N = (size_t)1 << args.log_n;
    const u32 r0 = tid / CC, col = tid % CC;
    auto at = [&](int j) { return LOG_HI <= 3 ? ((u32)(j / KC) << 11) + (j % KC) * 256 + tid : ((r0 + R8 * j) << 11) + col; };
    const double* y = cp.y + b * cp.y_bstride + (size_t)cp.lo * N + (size_t)blockIdx.x * CC;
    ConstPtr<ModConstF> pm = const_ptr((const ModConstF*)args.mc + m_idx);
    const ModConstF mc = {pm->q, pm->qinv, 0.0, 0.0};
    ConstPtr<TwF> ce = const_ptr(cp.convf + (size_t)pos * cp.ap);
    double v[8];
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = 0.0;
    for (u32 k8 = 0; k8 < cp.nd; k8 += 8) {  // a chain takes eight terms
        double s[8], lo[8];
#pragma unroll
        for (int j = 0; j < 8; j++) s[j] = F64M_DOT_BASE, lo[j] = 0.0;
        for (u32 k0 = k8; k0 < k8 + 8 && k0 < cp.nd; k0 += 4) {
            double yv[4][8];
#pragma unroll
            for (int k = 0; k < 4; k++)
#pragma unroll
                for (int j = 0; j < 8; j++) yv[k][j] = y[(size_t)min(k0 + k, cp.nd - 1) * N + at(j)];
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const double w = ce[k0 + k].w;
#pragma unroll
                for (int j = 0; j < 8; j++) f64m_chain_add(s[j], lo[j], f64m_reduce(yv[k][j], mc.q, mc.qinv), w);
            }
        }
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = f64m_reduce(v[j] + f64m_chain_join(s[j], lo[j], mc.q, mc.qinv), mc.q, mc.qinv);
    }
    const TwF* tw = (const TwF*)args.tw + ((size_t)m_idx << args.log_n);
    u64* dst = args.dst + (((size_t)b * args.dst_bstride + pos) << args.log_n) + (size_t)blockIdx.x * CC;
    if constexpr (LOG_HI <= 3) {
        fwd_rows<A, LOG_HI, KC>(v, tw, 1, mc);
#pragma unroll
        for (int j = 0; j < 8; j++) dst[at(j)] = A::store_mid(v[j]);
    } else {
        __shared__ __attribute__((aligned(16))) double lds[NTT_TILE];
        const u32 G = tid >> 5, cg = tid & 31;
        fwd_rows<A, 3, 1>(v, tw, 1, mc);
#pragma unroll
        for (int j = 0; j < 8; j++) lds[(r0 + R8 * j) * CC + col] = v[j];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] = lds[(G * R8 + i / KC2) * CC + cg * KC2 + i % KC2];
        A::fwd_begin(v, mc);
        fwd_rows<A, S2, KC2>(v, tw, 8 + G, mc);
#pragma unroll
        for (int i = 0; i < 8; i++) dst[((size_t)(G * R8 + i / KC2) << 11) + cg * KC2 + i % KC2] = A::store_mid(v[i]);
    }
}

// The last pass of an inverse transform, a basis conversion and the first pass of the forward transforms of its targets in one
// kernel, for the rings of 2^13 and 2^14 points: a thread owns the R = 2^LOG_HI points of one column, which is all that the three act
// on, so nothing goes through LDS.  It takes the column of every source limb through the inverse pass' LOG_HI stages (scaled and
// centred as inv_last_store does), and per target the conversion sum and the forward pass' stages.  The inverse stages are repeated by
// every group of cp.per targets (mid_conv_per: when, and figures).
// grid = (2^11 columns / NTT_THREADS, groups x polynomials, digits)
// A column's stages, twiddles tw[1..2^S - 1] through the scalar path; the inverse reduces the sums of its first stage (bounds: f64mod.h)
template <int S>
__device__ __forceinline__ void load_column_tw(ConstPtr<TwF> tw, TwF* w) {
#pragma unroll
    for (int i = 0; i < (1 << S) - 1; i++) w[i] = TwF{tw[1 + i].w, tw[1 + i].wq};
}
template <int S>
__device__ __forceinline__ void inv_column(double* v, ConstPtr<TwF> tw, const ModConstF& m) {
    typedef ArithF64 A;
    TwF w[(1 << S) - 1];
    load_column_tw<S>(tw, w);
#pragma unroll
    for (int a = S - 1; a >= 0; a--) {
        const int half = (1 << S) >> (a + 1);
#pragma unroll
        for (int rr = 0; rr < (1 << S); rr++) {
            if (rr & half) continue;
            A::inv_bf(v[rr], v[rr + half], w[(1 << a) - 1 + (rr >> (S - a))], m);
            if (a == S - 1) v[rr] = A::reduce(v[rr], m);
        }
    }
}
template <int S>
__device__ __forceinline__ void fwd_column(double* v, ConstPtr<TwF> tw, const ModConstF& m) {
    TwF w[(1 << S) - 1];
    load_column_tw<S>(tw, w);
    fwd_rows_pre<ArithF64, S>(v, w, m);
}
template <int LOG_HI, int ND>
__global__ __launch_bounds__(NTT_THREADS) void ntt_mid_conv_kernel(NttArgs args, PolyList pl, ConvPrologue cp, MidPrologue mp) {
    typedef ArithF64 A;
    constexpr int R = 1 << LOG_HI;
    const u32 col = blockIdx.x * NTT_THREADS + threadIdx.x, b = blockIdx.y / cp.groups, a0 = (blockIdx.y % cp.groups) * cp.per;
    const size_t N = (size_t)1 << args.log_n;
    const u32 dig = cp.digit0 + blockIdx.z, lo = dig * cp.alpha;
    const u32 nd = cp.alpha ? min(cp.alpha, cp.n_src - lo) : cp.nd;
    const u32 n_targets = cp.alpha ? pl.n - nd : pl.n;
    if (a0 >= n_targets) return;  // whole workgroup: a digit with more limbs has fewer targets
    const u32 a1 = min(a0 + cp.per, n_targets);
    const double* y = cp.y + b * cp.y_bstride + (size_t)(cp.lo + lo) * N + col;
    u64* dst0 = args.dst + (((size_t)b * args.dst_bstride) << args.log_n) + dig * cp.dst_dstride + col;
    const TwF* convf = cp.convf + dig * cp.convf_dstride;
    double yv[R][ND];
#pragma unroll
    for (int k = 0; k < ND; k++) {
        const size_t row = (size_t)((u32)k < nd ? k : nd - 1) * N;  // see conv_load
#pragma unroll
        for (int r = 0; r < R; r++) yv[r][k] = y[row + ((size_t)r << 11)];
    }
#pragma unroll
    for (int k = 0; k < ND; k++) {
        const u32 kk = (u32)k < nd ? k : nd - 1, m_idx = lo + (kk ? mp.next + kk - 1 : mp.first);
        ConstPtr<ModConstF> pm = const_ptr((const ModConstF*)args.mc + m_idx);
        ConstPtr<TwF> ps = const_ptr(mp.scale + m_idx), tw = const_ptr(mp.itw + ((size_t)m_idx << args.log_n));
        const ModConstF mc = {pm->q, pm->qinv, 0.0, 0.0};
        const TwF scale = {ps->w, ps->wq};
        double v[R];
#pragma unroll
        for (int r = 0; r < R; r++) v[r] = yv[r][k];
        inv_column<LOG_HI>(v, tw, mc);
#pragma unroll
        for (int r = 0; r < R; r++) yv[r][k] = f64m_centre(A::mulmod(v[r], scale.w, scale.wq, mc.q), mc.q);
    }
#pragma unroll 1
    for (u32 t = a0; t < a1; t++) {
        const u32 a = cp.alpha && t >= lo ? t + nd : t, m_idx = pl_at(pl.mod, a), pos = pl_at(pl.dpos, a);  // past the digit's own limbs
        ConstPtr<ModConstF> pm = const_ptr((const ModConstF*)args.mc + m_idx);
        ConstPtr<TwF> ce = const_ptr(convf + (size_t)pos * cp.ap), tw = const_ptr((const TwF*)args.tw + ((size_t)m_idx << args.log_n));
        const ModConstF mc = {pm->q, pm->qinv, 0.0, 0.0};
        double cw[ND], v[R];
#pragma unroll
        for (int k = 0; k < ND; k++) cw[k] = ce[k].w;
#pragma unroll
        for (int r = 0; r < R; r++) v[r] = f64m_dot_w<ND>(yv[r], cw, mc.q, mc.qinv);
        fwd_column<LOG_HI>(v, tw, mc);
        u64* dst = dst0 + ((size_t)pos << args.log_n);
#pragma unroll
        for (int r = 0; r < R; r++) dst[(size_t)r << 11] = A::store_mid(v[r]);
    }
}

// ============================ rings of 2^12 points: the whole transform in one workgroup ============================
// 256 R threads (R = 2 blocks of 2^11 points, eight points per thread) hold a whole limb-poly: the hi pass' stage acts
// on the R points of a thread's columns, one more exchange through LDS takes the place of the trip through memory, and the lo
// pass' rounds follow, 256 threads per block.  On this ring a call is a chain of launches that leave most of the chip idle;
// each is worth a launch (about 2 us) and a chain of dependent loads (1 to 2 us) whatever it computes: a rescale in two
// kernels instead of four takes 14.2 us instead of 20.7, five limbs forward and back 17.4 instead of 23.5, and a filled chip gains
// the memory traffic (1536 limb-polys 58 us instead of 88).  With four blocks (2^13 points) the
// compute units next door, which the two passes use, are missed more than the launches: key switches 58 -> 64 us.  What a round waits
// for through the scalar path (the outer stage's twiddle, the scale) is asked for before the first round: requested at its use each was a round
// trip of 0.6 to 1 us (direct convolution of five channels, 14 + 4 limbs, 306 -> 294 us).
// AP: 0 = the source is a polynomial, else rows of conversion constants as in ntt_fwd_hi_conv_kernel, ND of them real.  DIV: the
// results go through a division's last step (em as in div_request) instead of being stored.
// grid = (entries of the list, batch)
#define RING_LOG_HI 1
#define RING_THREADS (NTT_THREADS << RING_LOG_HI)
// the inverse transform likewise: the lo pass' rounds mirrored, an exchange, the hi pass' stages; v[j] ends as the ring's point
// ((j / KC) << 11) + (j % KC) * THREADS + tid, to be scaled.  src: the limb-poly; tw, tw_val: its modulus' inverse twiddles.  The last
// reads of LDS are of lds1.
#define RING_R (1 << RING_LOG_HI)
template <class A>
__device__ __forceinline__ void inv_ring_rounds(const u64* src, const PolyRef<A>& P, typename A::E* lds0, typename A::E* lds1, u32 tid, typename A::E* v) {
    typedef typename LoTw<A>::TW TW;
    typedef typename LoTw<A>::AR AR;
    constexpr int R = RING_R, KC = 8 / R, THREADS = RING_THREADS;
    const u32 blk = __builtin_amdgcn_readfirstlane(tid >> 8), t = tid & 255;
    const size_t off = (size_t)blk << 11;
    const u32 TA = R + blk;
    const u32 d3 = t >> 5, x5 = t & 31, d2 = (t >> 2) & 7, d0 = t & 3;
    typename A::E* buf0 = lds0 + blk * LDS_PADDED_WORDS;
    typename A::E* buf1 = lds1 + blk * LDS_PADDED_WORDS;
    TW wa[7], wb[7], wc[7], wd[6];
    load_lo_tw<A, 2>(P, 512 * TA + 2 * t, wd);
    load_lo_tw<A, 2>(P, 512 * TA + 2 * t + 1, wd + 3);
    load_lo_tw<A, 3>(P, 64 * TA + 8 * d3 + d2, wc);
    ulonglong2 raw[4];
    const ulonglong2* in = reinterpret_cast<const ulonglong2*>(src + off + 8 * t);
#pragma unroll
    for (int j = 0; j < 4; j++) raw[j] = in[j];
    typename A::TW wl[R - 1];  // the last stage's: asked for now, a scalar load at its use is a round trip to memory
#pragma unroll
    for (int i = 0; i < R - 1; i++) wl[i] = P.tw[1 + i];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        v[2 * j] = A::load_first(raw[j].x, P.mc, true);
        v[2 * j + 1] = A::load_first(raw[j].y, P.mc, true);
    }
    inv_rows_pre<AR, 2>(v, wd, P.mc);
    inv_rows_pre<AR, 2>(v + 4, wd + 3, P.mc);
    A::inv_end2(v, P.mc);
    load_lo_tw<A, 3>(P, 8 * TA + d3, wb);
#pragma unroll
    for (int j = 0; j < 8; j++) buf0[LDS_PAD(8 * t + j)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = buf0[LDS_PAD(d3 * 256 + d2 * 32 + 4 * j + d0)];
    inv_rows_pre<AR, 3>(v, wc, P.mc);
    A::inv_end(v, P.mc);
    load_lo_tw<A, 3>(P, TA, wa);
#pragma unroll
    for (int j = 0; j < 8; j++) buf1[LDS_PAD(d3 * 256 + d2 * 32 + 4 * j + d0)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = buf1[LDS_PAD(d3 * 256 + 32 * j + x5)];
    inv_rows_pre<AR, 3>(v, wb, P.mc);
    A::inv_end(v, P.mc);
#pragma unroll
    for (int j = 0; j < 8; j++) buf0[LDS_PAD(d3 * 256 + 32 * j + x5)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = buf0[LDS_PAD(t + 256 * j)];
    inv_rows_pre<AR, 3>(v, wa, P.mc);
    A::inv_end(v, P.mc);
#pragma unroll
    for (int j = 0; j < 8; j++) buf1[LDS_PAD(t + 256 * j)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = lds1[(j / KC) * LDS_PADDED_WORDS + LDS_PAD((j % KC) * THREADS + tid)];
    static_assert(R == 2, "one stage");
#pragma unroll
    for (int kc = 0; kc < KC; kc++) A::inv_bf(v[kc], v[KC + kc], wl[0], P.mc);
    A::template inv_mid<KC>(v, P.mc);
}
// grid = (entries of the list, batch)
template <class A>
__global__ __launch_bounds__(RING_THREADS) void ntt_inv_ring_kernel(NttArgs args, PolyList pl) {
    typedef typename A::E E;
    constexpr int R = RING_R, KC = 8 / R, THREADS = RING_THREADS;
    __shared__ E lds0[R * LDS_PADDED_WORDS];
    __shared__ E lds1[R * LDS_PADDED_WORDS];
    const u32 tid = threadIdx.x, a = blockIdx.x;
    const PolyRef<A> P = poly_ref<A>(args, pl, blockIdx.y, a);
    const bool scaled = std::is_same<A, ArithF64>::value && args.inv_scale;
    const TwF scale = scaled ? args.inv_scale[pl_at(pl.mod, a)] : TwF{0.0, 0.0};
    E v[8];
    inv_ring_rounds<A>(P.src, P, lds0, lds1, tid, v);
#pragma unroll
    for (int j = 0; j < 8; j++) P.dst[((size_t)(j / KC) << 11) + (j % KC) * THREADS + tid] = inv_last_store<A>(v[j], P.mc, scaled ? &scale : nullptr);
}

// MID: the source is one limb in evaluation form that goes through its whole inverse transform here first (a rescale in one launch).
template <class A, int AP, int ND, bool DIV, bool MID>
__device__ __forceinline__ void fwd_ring_body(const NttArgs& args, const PolyList& pl, const ConvPrologue& cp, const FwdEpilogue* ep, int em, const MidPrologue& mp) {
    typedef typename A::E E;
    typedef typename LoTw<A>::TW TW;
    typedef typename LoTw<A>::AR AR;
    constexpr int R = RING_R, KC = 8 / R, THREADS = RING_THREADS;
    __shared__ E lds_a[R * LDS_PADDED_WORDS];
    __shared__ E lds_b[R * LDS_PADDED_WORDS];
    E* lds0 = MID ? lds_b : lds_a;  // (the inverse rounds read lds_b last: the first write here goes to the other one)
    E* lds1 = MID ? lds_a : lds_b;
    const u32 tid = threadIdx.x, b = blockIdx.y, a = blockIdx.x;
    if constexpr (AP == 0 && !std::is_same<A, ArithF64>::value) {
        if (own_limb(args, b, a)) return;  // whole workgroup
    }
    const PolyRef<A> P = poly_ref<A>(args, pl, b, a);
    const u32 blk = __builtin_amdgcn_readfirstlane(tid >> 8), t = tid & 255;
    const size_t N = (size_t)1 << args.log_n, off = (size_t)blk << 11;
    const u32 TA = R + blk;
    const u32 d3 = t >> 5, x5 = t & 31, d2 = (t >> 2) & 7, d0 = t & 3;
    TW wa[7], wb[7], wc[7], wd[6];
    load_lo_tw<A, 3>(P, TA, wa);
    load_lo_tw<A, 3>(P, 8 * TA + d3, wb);
    E v[8];
    typename A::TW wl[R - 1];  // the first stage's (see inv_ring_rounds)
#pragma unroll
    for (int i = 0; i < R - 1; i++) wl[i] = P.tw[1 + i];
    if constexpr (MID) {
        PolyRef<A> S;
        S.tw = mp.itw + ((size_t)mp.first << args.log_n);
        S.tw_val = mp.itw_val + ((size_t)mp.first << args.log_n);
        S.mc = ((const ModConstF*)args.mc)[mp.first];
        const TwF scale = mp.scale[mp.first];
        const double cw[1] = {(cp.convf + (size_t)pl_at(pl.dpos, a) * AP)->w};
        inv_ring_rounds<A>(args.src_list.p[b], S, lds_a, lds_b, tid, v);
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const double yv[1] = {f64m_centre(A::mulmod(v[j], scale.w, scale.wq, S.mc.q), S.mc.q)};
            v[j] = f64m_dot_w<1>(yv, cw, P.mc.q, P.mc.qinv);
        }
    } else if constexpr (AP > 0) {
        const double* y = cp.y + b * cp.y_bstride + (size_t)cp.lo * N;
        const TwF* ce = cp.convf + (size_t)pl_at(pl.dpos, a) * AP;
        const u32 nd = cp.nd;
        double cw[ND];
#pragma unroll
        for (int k = 0; k < ND; k++) cw[k] = ce[k].w;
#pragma unroll
        for (int j = 0; j < 8; j++) {
            double yv[AP];
            conv_load<AP, ND>(yv, y + ((size_t)(j / KC) << 11) + (j % KC) * THREADS + tid, N, nd);
            v[j] = conv_sum<AP, ND>(yv, cw, P.mc.q, P.mc.qinv);
        }
    } else {
        u64 raw[8];
#pragma unroll
        for (int j = 0; j < 8; j++) raw[j] = P.src[((size_t)(j / KC) << 11) + (j % KC) * THREADS + tid];
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = A::load_first(raw[j], P.mc, false);
    }
    static_assert(R == 2, "one stage");
#pragma unroll
    for (int kc = 0; kc < KC; kc++) A::fwd_bf(v[kc], v[KC + kc], wl[0], P.mc);
    E* buf0 = lds0 + blk * LDS_PADDED_WORDS;
    E* buf1 = lds1 + blk * LDS_PADDED_WORDS;
#pragma unroll
    for (int j = 0; j < 8; j++) lds1[(j / KC) * LDS_PADDED_WORDS + LDS_PAD((j % KC) * THREADS + tid)] = v[j];
    load_lo_tw<A, 3>(P, 64 * TA + 8 * d3 + d2, wc);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = buf1[LDS_PAD(t + 256 * j)];
    A::fwd_begin(v, P.mc);
    fwd_rows_pre<AR, 3>(v, wa, P.mc);
#pragma unroll
    for (int j = 0; j < 8; j++) buf0[LDS_PAD(t + 256 * j)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = buf0[LDS_PAD(d3 * 256 + 32 * j + x5)];
    A::fwd_begin(v, P.mc);
    fwd_rows_pre<AR, 3>(v, wb, P.mc);
    load_lo_tw<A, 2>(P, 512 * TA + 2 * t, wd);
    load_lo_tw<A, 2>(P, 512 * TA + 2 * t + 1, wd + 3);
#pragma unroll
    for (int j = 0; j < 8; j++) buf1[LDS_PAD(d3 * 256 + 32 * j + x5)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = buf1[LDS_PAD(d3 * 256 + d2 * 32 + 4 * j + d0)];
    A::fwd_begin(v, P.mc);
    fwd_rows_pre<AR, 3>(v, wc, P.mc);
    DivOperands O;
    const u32 i = pl_at(pl.dpos, a);
    if constexpr (DIV) {
        if (em == 1) div_request<A, 1>(args, *ep, i, b, off, t, O);
        else if (em == 3) div_request<A, 3>(args, *ep, i, b, off, t, O);
        else if (em == 4) div_request<A, 4>(args, *ep, i, b, off, t, O);
        else div_request<A, 2>(args, *ep, i, b, off, t, O);
    }
#pragma unroll
    for (int j = 0; j < 8; j++) buf0[LDS_PAD(d3 * 256 + d2 * 32 + 4 * j + d0)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = buf0[LDS_PAD(8 * t + j)];
    fwd_rows_pre<AR, 2>(v, wd, P.mc);
    fwd_rows_pre<AR, 2>(v + 4, wd + 3, P.mc);
    A::fwd_end(v, P.mc);
#pragma unroll
    for (int j = 0; j < 8; j++) buf1[LDS_PAD(8 * t + j)] = v[j];
    __syncthreads();
    if constexpr (DIV) {
        const u32 m_idx = pl_at(pl.mod, a);
        if (em == 1 || em == 3) div_store<A, 1>(args, *ep, i, m_idx, b, off, t, buf1, P.mc, O);
        else if (em == 4) div_store<A, 4>(args, *ep, i, m_idx, b, off, t, buf1, P.mc, O);
        else if (em == 2) div_store<A, 2>(args, *ep, i, m_idx, b, off, t, buf1, P.mc, O);
        else div_store<A, 0>(args, *ep, i, m_idx, b, off, t, buf1, P.mc, O);
    } else {
        u64* dst = P.dst + off;
#pragma unroll
        for (int j = 0; j < 8; j++) dst[t + 256 * j] = A::store_fwd_final(buf1[LDS_PAD(t + 256 * j)], P.mc);
    }
}
template <class A>
__global__ __launch_bounds__(RING_THREADS) void ntt_fwd_ring_kernel(NttArgs args, PolyList pl) {
    fwd_ring_body<A, 0, 1, false, false>(args, pl, ConvPrologue{}, nullptr, 0, MidPrologue{});
}
template <class A, int AP, int ND, bool MID>
__global__ __launch_bounds__(RING_THREADS) void ntt_fwd_ring_div_kernel(NttArgs args, PolyList pl, ConvPrologue cp, FwdEpilogue ep, int em, MidPrologue mp) {
    fwd_ring_body<A, AP, ND, true, MID>(args, pl, cp, &ep, em, mp);
}

// ================================= rings below 2^11: one tile per poly (integer arithmetic) ==============
template <bool INVERSE>
__global__ __launch_bounds__(NTT_THREADS) void ntt_small_kernel(NttArgs args, PolyList pl) {
    typedef ArithU64 A;
    __shared__ u64 lds[NTT_TILE];
    const u32 tid = threadIdx.x;
    const PolyRef<A> P = poly_ref<A>(args, pl, blockIdx.y / pl.n, blockIdx.y % pl.n);
    const u32 n = 1u << args.log_n;
    for (u32 e = tid; e < n; e += NTT_THREADS) lds[e] = P.src[e];
    __syncthreads();
    for (u32 st = 0; st < args.log_n; st++) {
        const u32 r = INVERSE ? args.log_n - 1 - st : st;  // stage with 2^r groups
        const u32 lt = args.log_n - 1 - r;                 // log2 of the pair distance
        for (u32 bf = tid; bf < n / 2; bf += NTT_THREADS) {
            const u32 i = bf >> lt;
            const u32 i0 = (i << (lt + 1)) + (bf & ((1u << lt) - 1)), i1 = i0 + (1u << lt);
            u64 x = lds[i0], y = lds[i1];
            if (INVERSE) A::inv_bf(x, y, P.tw[(1u << r) + i], P.mc); else A::fwd_bf(x, y, P.tw[(1u << r) + i], P.mc);
            lds[i0] = x;
            lds[i1] = y;
        }
        __syncthreads();
    }
    for (u32 e = tid; e < n; e += NTT_THREADS) P.dst[e] = INVERSE ? A::store_inv_final(lds[e], P.mc) : A::store_fwd_final(lds[e], P.mc);
}

template <class A, int LOG_HI>
static void launch_hi(bool inverse, dim3 grid, hipStream_t st, const NttArgs& args, const PolyList& pl) {
    if (inverse) hipLaunchKernelGGL((ntt_inv_hi_kernel<A, LOG_HI>), grid, dim3(NTT_THREADS), 0, st, args, pl);
    else hipLaunchKernelGGL((ntt_fwd_hi_kernel<A, LOG_HI>), grid, dim3(NTT_THREADS), 0, st, args, pl);
}

template <class A>
static void launch_hi_any(u32 log_hi, bool inverse, dim3 grid, hipStream_t st, const NttArgs& args, const PolyList& pl) {
    switch (log_hi) {
        case 2: launch_hi<A, 2>(inverse, grid, st, args, pl); break;
        case 3: launch_hi<A, 3>(inverse, grid, st, args, pl); break;
        case 4: launch_hi<A, 4>(inverse, grid, st, args, pl); break;
        case 5: launch_hi<A, 5>(inverse, grid, st, args, pl); break;
        default: launch_hi<A, 6>(inverse, grid, st, args, pl); break;
    }
}

// Batch items a lo-pass workgroup takes one after the other: as many as leave LO_FILL workgroups, at most `most`.  Sharing a
// slice's twiddles saves cache traffic only once the chip is full; below that the items of a workgroup are a serial chain of
// tiles next to idle CUs.  The line is the number of workgroups the chip holds at once (three waves per SIMD, 256 CUs); 512,
// 1024 and 2048 measure the same.  A small launch's time is its longest workgroup: five polynomials of 13 limbs at N = 2^14
// (520 slices of work), forward and inverse, 52 -> 41 us; six key switches of 10 limbs at N = 2^13, 101 -> 83 us; launches of
// 768 slices and more are unchanged.
#define LO_FILL 768
static u32 lo_items(u32 slices, u32 batch, u32 most) {
    const u32 n = (u32)((u64)slices * batch / LO_FILL);
    return n < 1 ? 1 : (n < most ? n : most);
}

template <class A, int IT>
static void launch_inv_lo_it(dim3 grid, hipStream_t st, const NttArgs& args, const PolyList& pl, bool mul, bool gal) {
    if constexpr (std::is_same<A, ArithF64>::value) {
        if constexpr (IT == 1) {
            if (gal && mul) {
                hipLaunchKernelGGL((ntt_inv_lo_kernel<A, IT, true, true>), grid, dim3(NTT_THREADS), 0, st, args, pl);
                return;
            }
        }
        if (gal) {
            hipLaunchKernelGGL((ntt_inv_lo_kernel<A, IT, false, true>), grid, dim3(NTT_THREADS), 0, st, args, pl);
            return;
        }
    }
    if constexpr (std::is_same<A, ArithF64>::value && IT == 1) {  // the product-forming variant takes one item
        if (mul) {
            hipLaunchKernelGGL((ntt_inv_lo_kernel<A, IT, true>), grid, dim3(NTT_THREADS), 0, st, args, pl);
            return;
        }
    }
    hipLaunchKernelGGL((ntt_inv_lo_kernel<A, IT>), grid, dim3(NTT_THREADS), 0, st, args, pl);
}
// The plain forward lo pass: workgroups that loop over their items, up to eight each where the launch is large (measured at N = 2^16: 2, 4, 8 and 16
// items give 2.04, 2.06, 2.08 and 2.10e6 limb transforms per second against 1.97e6 with one fetch of the twiddles per two
// items; eight still leaves the layer's batches of eight a grid of one workgroup per slice).  `grid` is a lo pass' grid,
// whose extent over items is set here.
template <class A>
static void launch_fwd_lo_loop(u32 batch, dim3 grid, hipStream_t st, const NttArgs& args, const PolyList& pl) {
    const u32 per_wg = lo_items(pl.n << args.log_hi, batch, 8);
    const u32 ext = (batch + per_wg - 1) / per_wg;
    if (args.lo_group) grid.y = ext;
    else grid.x = ext;
    hipLaunchKernelGGL((ntt_fwd_lo_loop_kernel<A>), grid, dim3(NTT_THREADS), 0, st, args, pl);
}
// which optional operands the division's last step has: the same for the whole launch (see div_request)
static int div_operands(const NttArgs& args, const FwdEpilogue& ep) {
    u32 n_add0 = 0, n_add1 = 0, n_mask = 0, n_acc = 0;
    const u32 n_ct = (args.batch + 1) / 2;
    for (u32 r = 0; r < n_ct; r++) {
        const FinalItem& fi = ep.B.it[r];
        n_add0 += fi.add0 ? 1 : 0;
        n_add1 += fi.add1 ? 1 : 0;
        n_mask += fi.mask ? 1 : 0;
        n_acc += fi.acc ? 1 : 0;
    }
    if (n_mask + n_acc == 0) return n_add0 == n_ct ? 1 : (n_add0 + n_add1 == 0 ? 2 : 0);
    if (n_add0 + n_add1 == 0) return n_acc == n_ct && !n_mask ? 3 : (n_mask == n_ct && !n_acc ? 4 : 0);
    return 0;
}
template <class A>
static void launch_lo_div(dim3 grid, hipStream_t st, const NttArgs& args, const PolyList& pl, const FwdEpilogue& ep) {
    const int em = div_operands(args, ep);
    // one instantiation per case; one batch item per workgroup (see per_wg in launch_ntt_any)
#define LO_DIV_LAUNCH(EM) hipLaunchKernelGGL((ntt_fwd_lo_div_kernel<A, EM>), grid, dim3(NTT_THREADS), 0, st, args, pl, ep)
    if (em == 1) LO_DIV_LAUNCH(1);
    else if (em == 2) LO_DIV_LAUNCH(2);
    else if (em == 3) LO_DIV_LAUNCH(3);
    else if (em == 4) LO_DIV_LAUNCH(4);
    else LO_DIV_LAUNCH(0);
#undef LO_DIV_LAUNCH
}
template <class A>
static void launch_inv_lo(u32 items, dim3 grid, hipStream_t st, const NttArgs& args, const PolyList& pl, bool mul, bool gal) {
    if (items == 2 && !mul) launch_inv_lo_it<A, 2>(grid, st, args, pl, false, gal);
    else launch_inv_lo_it<A, 1>(grid, st, args, pl, mul, gal);
}

// Target limbs per workgroup: four share one fetch of the source residues; in a launch that would not give every CU two
// workgroups, two or one, each done sooner (one polynomial pair's rescale at N = 2^16, 12 limbs: 13.1 us with four, 8.9 with one; six
// decompositions of digits of three limbs at N = 2^13: 9.3 and 6.6).
template <int LOG_HI, int AP, int ND, bool MID>
static void launch_hi_conv_regs_as(u32 n_targets, u32 digits, u32 batch, hipStream_t st, const NttArgs& args, const PolyList& pl, ConvPrologue cp, const MidPrologue& mp) {
    u32 t = 4;
    while (t > 1 && ((n_targets + t - 1) / t * batch * digits << LOG_HI) < 512) t >>= 1;
    cp.groups = (n_targets + t - 1) / t;
    const dim3 grid(1u << LOG_HI, cp.groups * batch, digits), block(NTT_THREADS);
    if (t == 4) hipLaunchKernelGGL((ntt_fwd_hi_conv_kernel<LOG_HI, AP, 4, ND, MID>), grid, block, 0, st, args, pl, cp, mp);
    else if (t == 2) hipLaunchKernelGGL((ntt_fwd_hi_conv_kernel<LOG_HI, AP, 2, ND, MID>), grid, block, 0, st, args, pl, cp, mp);
    else hipLaunchKernelGGL((ntt_fwd_hi_conv_kernel<LOG_HI, AP, 1, ND, MID>), grid, block, 0, st, args, pl, cp, mp);
}
template <int LOG_HI, int AP, int ND>
static void launch_hi_conv_regs(u32 n_targets, u32 digits, u32 batch, hipStream_t st, const NttArgs& args, const PolyList& pl, const ConvPrologue& cp, const MidPrologue* mp) {
    if constexpr (LOG_HI >= 4 && ND == 1) {
        if (mp) {
            launch_hi_conv_regs_as<LOG_HI, AP, ND, true>(n_targets, digits, batch, st, args, pl, cp, *mp);
            return;
        }
    }
    launch_hi_conv_regs_as<LOG_HI, AP, ND, false>(n_targets, digits, batch, st, args, pl, cp, MidPrologue{});
}
template <int LOG_HI, int AP, int ND>
static void launch_hi_conv_lds(u32 n_targets, u32 digits, u32 batch, hipStream_t st, const NttArgs& args, const PolyList& pl, ConvPrologue cp, const MidPrologue* mp) {
    cp.groups = (n_targets + HC_T - 1) / HC_T;
    const dim3 grid(1u << LOG_HI, cp.groups * batch, digits), block(HC_THREADS);
    if constexpr (ND <= CONV_MID_TERMS) {
        if (mp) {
            hipLaunchKernelGGL((ntt_fwd_hi_conv_lds_kernel<LOG_HI, AP, ND, true>), grid, block, 0, st, args, pl, cp, *mp);
            return;
        }
    }
    hipLaunchKernelGGL((ntt_fwd_hi_conv_lds_kernel<LOG_HI, AP, ND, false>), grid, block, 0, st, args, pl, cp, MidPrologue{});
}
// n_targets: the most targets a digit of the launch has
template <int LOG_HI>
static hipError_t launch_hi_conv_ap(u32 n_targets, u32 digits, u32 batch, hipStream_t st, const NttArgs& args, const PolyList& pl, const ConvPrologue& cp, const MidPrologue* mp) {
    if (mp && !conv_has_mid(LOG_HI, cp.ap, cp.nd)) return hipErrorInvalidValue;
    const u32 terms = hi_conv_terms(LOG_HI, cp.ap, cp.nd);
#define HI_CONV(AP, ND)                                                                                                              \
    if constexpr (hi_conv_terms(LOG_HI, AP, ND) == ND) {                                                                             \
        if (cp.ap == AP && terms == ND) {                                                                                            \
            if constexpr (LOG_HI < 4 || (AP == 4 && ND == 1)) launch_hi_conv_regs<LOG_HI, AP, ND>(n_targets, digits, batch, st, args, pl, cp, mp); \
            else launch_hi_conv_lds<LOG_HI, AP, ND>(n_targets, digits, batch, st, args, pl, cp, mp);                                 \
            return hipSuccess;                                                                                                       \
        }                                                                                                                            \
    }
    HI_CONV(4, 1) HI_CONV(4, 2) HI_CONV(4, 3) HI_CONV(4, 4)
    HI_CONV(8, 4) HI_CONV(8, 5) HI_CONV(8, 6) HI_CONV(8, 7) HI_CONV(8, 8)
    HI_CONV(12, 9) HI_CONV(12, 10) HI_CONV(12, 12)
    HI_CONV(16, 8) HI_CONV(16, 10) HI_CONV(16, 12) HI_CONV(16, 16)
#undef HI_CONV
    return hipErrorInvalidValue;
}
static u32 mid_conv_per_of(const ckks_ctx* c, u32 nd, u32 ap, u32 n_targets, u32 rows) {
    return ntt_has_modup(c) ? mid_conv_per(c->log_hi, nd, ap, n_targets, rows) : 0;
}
u32 ntt_mid_modup(const ckks_ctx* c, u32 level, u32 n) {
    const u32 nd = c->alpha < level + 1 ? c->alpha : level + 1;
    return mid_conv_per_of(c, nd, c->alpha_pad, c->ext_limbs(level) - nd, n * c->live_digits(level));
}
// Rings of 2^12 points: a division that starts from whole sums (lo_done: they have been through the inverse transform's first pass) takes
// the whole-ring kernels where they give between half of the CUs and every CU a limb-poly of the result.  Pass by pass / whole ring in us, limb-polys of the largest
// batch in brackets: direct convolutions of one channel of 16 + 6 limbs (256) 67.7 / 66.0, two of 7 + 4 (224) 63.7 / 62.3, five of 8 + 4 (240) 134 / 128, five of 7 + 4 (210)
// 129 / 126; with four keys, one of 21 + 8 limbs 121 / 116, of 24 + 8 122 / 118; eight hoisted rotations of 14 + 2 limbs in seven digits (224) 91.7 / 90.9.  (Hoisted rotations
// of up to four digits come with lo_done.)  At the window's ends, measured on hoisted rotations that came this way then: 84 36.0 / 37.6, 112 38.5 / 39.0, 336 53.9 / 58.2
u32 ntt_mid_moddown(const ckks_ctx* c, u32 level, bool merged, u32 polys, bool lo_done) {
    const u32 n_out = merged ? level : level + 1;
    if (ntt_one_pass(c) && !lo_done && n_out * polys > 112 && n_out * polys <= 256) return 0;
    return mid_conv_per_of(c, c->num_p + (merged ? 1 : 0), merged ? c->k2_pad : c->k_pad, n_out, polys);
}
u32 ntt_mid_rescale(const ckks_ctx* c, u32 level, u32 polys) { return mid_conv_per_of(c, 1, 4, level, polys); }
// The rescale of a ring of 2^12 points in one launch, the dropped limb's inverse transform repeated by every target's workgroup, while every
// limb-poly of the result has a CU of its own: one ciphertext of 4 limbs 14.2 us in two launches (or three: pass by pass), 10.5 in one
bool ntt_rescale_one_launch(const ckks_ctx* c, u32 level, u32 polys) { return ntt_has_modup(c) && ntt_one_pass(c) && level * polys <= 256; }

template <int LOG_HI>
static hipError_t launch_mid_conv_hi(dim3 grid, hipStream_t st, const NttArgs& args, const PolyList& pl, const ConvPrologue& cp, const MidPrologue& mp) {
    const u32 terms = mid_conv_terms(LOG_HI, cp.nd);
#define MID_CONV(ND)                                                                                                                 \
    if constexpr (mid_conv_terms(LOG_HI, ND) == ND) {                                                                                \
        if (terms == ND) {                                                                                                           \
            hipLaunchKernelGGL((ntt_mid_conv_kernel<LOG_HI, ND>), grid, dim3(NTT_THREADS), 0, st, args, pl, cp, mp);                 \
            return hipSuccess;                                                                                                       \
        }                                                                                                                            \
    }
    MID_CONV(1) MID_CONV(2) MID_CONV(3) MID_CONV(4) MID_CONV(5) MID_CONV(6) MID_CONV(7) MID_CONV(8) MID_CONV(9) MID_CONV(10) MID_CONV(12) MID_CONV(16)
#undef MID_CONV
    return hipErrorInvalidValue;
}
static hipError_t launch_mid_conv(u32 log_hi, u32 n_targets, u32 digits, u32 batch, hipStream_t st, const NttArgs& args, const PolyList& pl, ConvPrologue cp, const MidPrologue& mp) {
    cp.groups = (n_targets + cp.per - 1) / cp.per;
    const dim3 grid((1u << CKKS_TILE_LOG) / NTT_THREADS, cp.groups * batch, digits);
    switch (log_hi) {
        case 1: return launch_mid_conv_hi<1>(grid, st, args, pl, cp, mp);
        case 2: return launch_mid_conv_hi<2>(grid, st, args, pl, cp, mp);
        case 3: return launch_mid_conv_hi<3>(grid, st, args, pl, cp, mp);
        default: return hipErrorInvalidValue;
    }
}

static hipError_t launch_hi_conv(u32 log_hi, u32 n_targets, u32 digits, u32 batch, hipStream_t st, const NttArgs& args, const PolyList& pl, const ConvPrologue& cp,
                                 const MidPrologue* mp) {
    if (mp && !cp.per) return hipErrorInvalidValue;
    if (mp && log_hi <= 3) return launch_mid_conv(log_hi, n_targets, digits, batch, st, args, pl, cp, *mp);
    switch (log_hi) {
        case 2: return launch_hi_conv_ap<2>(n_targets, digits, batch, st, args, pl, cp, mp);
        case 3: return launch_hi_conv_ap<3>(n_targets, digits, batch, st, args, pl, cp, mp);
        case 4: return launch_hi_conv_ap<4>(n_targets, digits, batch, st, args, pl, cp, mp);
        case 5: return launch_hi_conv_ap<5>(n_targets, digits, batch, st, args, pl, cp, mp);
        case 6: return launch_hi_conv_ap<6>(n_targets, digits, batch, st, args, pl, cp, mp);
        default: return hipErrorInvalidValue;  // a ring of 2^12 points has no converting pass of its own
    }
}

// The whole-ring kernels: a workgroup per entry of the list and batch item.
template <class A>
static void launch_ring_as(bool inverse, u32 entries, hipStream_t st, const NttArgs& args, const PolyList& pl, const ConvPrologue* conv, const FwdEpilogue* ep,
                           const MidPrologue* mid) {
    const dim3 grid(entries, args.batch), block(RING_THREADS);
    if (inverse) {
        hipLaunchKernelGGL((ntt_inv_ring_kernel<A>), grid, block, 0, st, args, pl);
        return;
    }
    if (!ep) {
        hipLaunchKernelGGL((ntt_fwd_ring_kernel<A>), grid, block, 0, st, args, pl);
        return;
    }
    const ConvPrologue cp = conv ? *conv : ConvPrologue{};
    const MidPrologue mp = mid ? *mid : MidPrologue{};
    const int em = div_operands(args, *ep);
#define RING_LAUNCH(AP, ND, MID) hipLaunchKernelGGL((ntt_fwd_ring_div_kernel<A, AP, ND, MID>), grid, block, 0, st, args, pl, cp, *ep, em, mp)
    if constexpr (std::is_same<A, ArithF64>::value) {
        if (conv) {
            if (mid) RING_LAUNCH(4, 1, true);
            else if (cp.ap == 4) RING_LAUNCH(4, 4, false);
            else if (cp.ap == 8) RING_LAUNCH(8, 8, false);
            else if (cp.ap == 12 && cp.nd == 9) RING_LAUNCH(12, 9, false);
            else if (cp.ap == 12) RING_LAUNCH(12, 12, false);
            else RING_LAUNCH(16, 16, false);
            return;
        }
    }
    RING_LAUNCH(0, 1, false);
#undef RING_LAUNCH
}
static void launch_ring(const ckks_ctx* c, bool inverse, u32 entries, hipStream_t st, const NttArgs& args, const PolyList& pl, const ConvPrologue* conv,
                        const FwdEpilogue* ep, const MidPrologue* mid = nullptr) {
    if (c->ntt_f64) launch_ring_as<ArithF64>(inverse, entries, st, args, pl, conv, ep, mid);
    else launch_ring_as<ArithU64>(inverse, entries, st, args, pl, conv, ep, mid);
}

static hipError_t launch_ntt_any(const ckks_ctx* c, bool inverse, const u64* src, size_t src_bstride, u64* dst,
                                 size_t dst_bstride, const PolyList& pl, u32 batch, hipStream_t st, const u64* const* src_ptrs,
                                 const FwdEpilogue* epilogue, const TwF* inv_scale, const ConvPrologue* conv,
                                 const u64* const* mul_ptrs = nullptr, const u64* lin_k = nullptr, NttPasses passes = NTT_BOTH,
                                 const MidPrologue* mid = nullptr, const u32* gals = nullptr) {
    if (pl.n == 0 || batch == 0) return hipSuccess;
    if (passes != NTT_BOTH && ((!inverse && (!conv || epilogue || passes != NTT_HI)) || c->log_hi < 1)) return hipErrorInvalidValue;
    if (passes == NTT_HI && (src != dst || src_ptrs || (ntt_one_pass(c) && !mid))) return hipErrorInvalidValue;
    if ((mul_ptrs || gals) && ntt_one_pass(c) && passes != NTT_LO) return hipErrorInvalidValue;
    if (mid && (!conv || !conv->per || c->log_hi < 1)) return hipErrorInvalidValue;
    if (mul_ptrs && (!inverse || !src_ptrs || !ntt_has_modup(c))) return hipErrorInvalidValue;
    if (lin_k && (!mul_ptrs || pl.n != 1)) return hipErrorInvalidValue;
    if (gals && (!inverse || !src_ptrs || lin_k || !ntt_has_modup(c))) return hipErrorInvalidValue;
    if (epilogue && epilogue->use_vl == 2 && !c->ntt_f64) return hipErrorInvalidValue;
    if (src_ptrs && batch > KS_MAX_BATCH) return hipErrorInvalidValue;
    if (epilogue && (inverse || !ntt_has_epilogue(c) || batch > 2 * KS_MAX_BATCH)) return hipErrorInvalidValue;
    if ((inv_scale && !inverse) || (conv && inverse) || ((inv_scale || conv) && !ntt_has_modup(c))) return hipErrorInvalidValue;
    if (conv && (conv->nd == 0 || conv->nd > conv->ap || (conv->ap != 4 && conv->ap != 8 && conv->ap != 12 && conv->ap != 16)))
        return hipErrorInvalidValue;
    const bool f64 = c->ntt_f64;
    NttArgs args;
    args.src = src;
    args.dst = dst;
    args.src_bstride = src_bstride;
    args.dst_bstride = dst_bstride;
    args.mc = f64 ? (const void*)c->d_mcf : (const void*)c->d_mc;
    args.tw = f64 ? (const void*)(inverse ? c->d_itwf : c->d_twf) : (const void*)(inverse ? c->d_itw : c->d_tw);
    args.tw_val = f64 ? (inverse ? c->d_itwf_val : c->d_twf_val) : nullptr;
    args.log_n = c->log_n;
    args.log_lo = c->log_lo;
    args.log_hi = c->log_hi;
    args.first = 1;
    args.last = 1;
    args.batch = batch;
    {
        const u32 slices = pl.n << c->log_hi;
        args.lo_group = 0;
        for (u32 g = 64; g >= 8; g >>= 1)
            if (slices % g == 0) { args.lo_group = g; break; }
    }
    args.use_src_list = src_ptrs ? 1 : 0;
    for (u32 b = 0; b < KS_MAX_BATCH; b++) {
        args.src_list.p[b] = (src_ptrs && b < batch) ? src_ptrs[b] : nullptr;
        args.mul_list.p[b] = (mul_ptrs && b < batch) ? mul_ptrs[b] : nullptr;
        args.gal[b] = (gals && b < batch) ? gals[b] : 1;
    }
    args.inv_scale = inv_scale;
    args.use_lin = lin_k ? 1 : 0;
    args.lin_ka = lin_k ? lin_k[0] : 0;
    args.lin_kb = lin_k ? lin_k[1] : 0;
    args.pad2 = 0;
    args.beta = args.alpha = args.level = args.pad3 = 0;
    const u32 polys = pl.n * batch;
    const dim3 block(NTT_THREADS);
    const double pass_bytes = 16.0 * polys * c->N;
    if (c->log_n < CKKS_TILE_LOG) {
        ProfScope ps__(c, inverse ? K_NTT_INV_LO : K_NTT_FWD_LO, st, pass_bytes, 0.5 * polys * c->N * c->log_n);
        if (inverse) hipLaunchKernelGGL(ntt_small_kernel<true>, dim3(1, polys), block, 0, st, args, pl);
        else hipLaunchKernelGGL(ntt_small_kernel<false>, dim3(1, polys), block, 0, st, args, pl);
        return hipGetLastError();
    }
    if (ntt_one_pass(c) && passes == NTT_BOTH && !mid) {
        const double ring_bytes = conv ? 8.0 * c->N * batch * ((double)conv->nd + (epilogue ? 2.0 : 1.0) * pl.n) : (epilogue ? 1.5 : 1.0) * pass_bytes;
        ProfScope ps__(c, inverse ? K_NTT_INV_LO : K_NTT_FWD_LO, st, ring_bytes, 0.5 * polys * c->N * c->log_n);
        launch_ring(c, inverse, pl.n, st, args, pl, conv, epilogue);
        return hipGetLastError();
    }
    const dim3 grid(c->N >> CKKS_TILE_LOG, polys);  // hi pass: one workgroup per 2^11 points
    const u32 slices = pl.n << c->log_hi;
    // batch items per lo-pass workgroup: in the inverse pass of a large launch two share one fetch of the twiddles (an unrolled four cost too many
    // registers, and a loop over the items as in the plain forward pass spills in the variant that forms a product as it
    // loads, 4.7 -> 6.3 ms per step of the block slice; that variant takes one item: with two it holds two operands' points a
    // tile ahead and spills at three waves per SIMD, 4.7 against 4.2 ms per step for the class); the pass that ends a division takes one (with its epilogue's operands
    // two items leave only two waves per SIMD, which costs more than the second fetch of the twiddles); the plain forward
    // pass sets its own extent (launch_fwd_lo_loop)
    const u32 per_wg = epilogue ? 1 : lo_items(slices, batch, 2);
    const u32 lo_wgs = (batch + per_wg - 1) / per_wg;
    const dim3 grid_lo = args.lo_group ? dim3(args.lo_group, lo_wgs, slices / args.lo_group) : dim3(lo_wgs, slices);  // see lo_tile()
    const double lo_ops = 0.5 * polys * c->N * c->log_lo, hi_ops = 0.5 * polys * c->N * c->log_hi;
    // the second pass of either direction continues in place on dst
    NttArgs second = args;
    second.src = dst;
    second.src_bstride = dst_bstride;
    second.use_src_list = 0;
    second.first = 0;
    PolyList pd = pl;
    for (u32 i = 0; i < pl.n; i++) pd.spos[i] = pl.dpos[i];
    auto hi = [&](const NttArgs& a, const PolyList& l) { if (f64) launch_hi_any<ArithF64>(c->log_hi, inverse, grid, st, a, l); else launch_hi_any<ArithU64>(c->log_hi, inverse, grid, st, a, l); };
    auto lo = [&](const NttArgs& a, const PolyList& l) {
        if (!inverse) {
            if (f64) launch_fwd_lo_loop<ArithF64>(batch, grid_lo, st, a, l);
            else launch_fwd_lo_loop<ArithU64>(batch, grid_lo, st, a, l);
        } else {
            if (f64) launch_inv_lo<ArithF64>(per_wg, grid_lo, st, a, l, false, gals != nullptr);
            else launch_inv_lo<ArithU64>(per_wg, grid_lo, st, a, l, false, false);
        }
    };
    if (!inverse) {
        if (c->log_hi > 0) {
            args.last = 0;
            if (conv) {  // reads the digit's nd limbs for every target limb (from cache after the first), writes the target limbs
                ProfScope ps__(c, K_NTT_FWD_HI, st, 8.0 * c->N * batch * ((double)conv->nd + pl.n), hi_ops);
                if (hipError_t e = launch_hi_conv(c->log_hi, pl.n, 1, batch, st, args, pl, *conv, mid); e != hipSuccess) return e;
                if (passes == NTT_HI) return hipGetLastError();
            } else {
                ProfScope ps__(c, K_NTT_FWD_HI, st, pass_bytes, hi_ops);
                hi(args, pl);
            }
            if (epilogue) {  // reads w and v, writes the quotients (plus the addends it reads)
                ProfScope ps__(c, K_NTT_FWD_LO, st, (epilogue->use_vl == 2 ? 2.0 : 1.5) * pass_bytes, lo_ops);
                if (f64) launch_lo_div<ArithF64>(grid_lo, st, second, pd, *epilogue);
                else launch_lo_div<ArithU64>(grid_lo, st, second, pd, *epilogue);
            } else {
                ProfScope ps__(c, K_NTT_FWD_LO, st, pass_bytes, lo_ops);
                lo(second, pd);
            }
        } else {
            ProfScope ps__(c, K_NTT_FWD_LO, st, pass_bytes, lo_ops);
            lo(args, pl);
        }
    } else {
        args.last = c->log_hi == 0;
        if (passes != NTT_HI) {
            ProfScope ps__(c, K_NTT_INV_LO, st, mul_ptrs ? 1.5 * pass_bytes : pass_bytes, lo_ops);
            if (mul_ptrs) {  // one item per workgroup (see lo_items)
                dim3 g1 = grid_lo;
                if (args.lo_group) g1.y = batch;
                else g1.x = batch;
                launch_inv_lo<ArithF64>(1, g1, st, args, pl, true, gals != nullptr);
            }
            else lo(args, pl);
        }
        if (c->log_hi > 0 && passes != NTT_LO) { ProfScope ps__(c, K_NTT_INV_HI, st, pass_bytes, hi_ops); hi(second, pd); }
    }
    return hipGetLastError();
}

hipError_t launch_ntt(const ckks_ctx* c, bool inverse, const u64* src, size_t src_bstride, u64* dst, size_t dst_bstride,
                      const PolyList& pl, u32 batch, hipStream_t st, const u64* const* src_ptrs, const FwdEpilogue* epilogue,
                      const TwF* inv_scale, const u64* const* mul_ptrs, const u64* lin_k, NttPasses passes, const u32* gals) {
    return launch_ntt_any(c, inverse, src, src_bstride, dst, dst_bstride, pl, batch, st, src_ptrs, epilogue, inv_scale, nullptr, mul_ptrs, lin_k, passes, nullptr, gals);
}

// Small launches take all digits at once: one converting hi pass and (unless the inner product takes it from there) one lo pass,
// instead of a launch per digit that leaves most of the chip idle (one polynomial of 13 limbs in digits of 8 and 5 at N = 2^16:
// 17.5 us per digit; a product with its rescale 167 -> 153 us, six unhoisted rotations at N = 2^13 83 -> 70 us).  From 768
// workgroups per digit on, a digit fills the chip by itself and goes through its two passes alone: what the second reads is
// then still in the last-level cache, and the other stream's kernels get their turn between the launches (all digits at once:
// 1 % slower for 64 channels, 2 % for the sixteen-channel activation).
hipError_t launch_ntt_modup(const ckks_ctx* c, u32 level, const double* y, size_t y_bstride, u64* digits, u32 n, hipStream_t st, bool hi_only, u32 mid_per) {
    if (!ntt_has_modup(c) || n == 0) return hipErrorInvalidValue;
    const u32 E = c->ext_limbs(level), beta = c->live_digits(level), L1 = level + 1;
    ConvPrologue cp;
    cp.y = y;
    cp.y_bstride = y_bstride;
    cp.convf = c->modup_table_f(level, 0);
    cp.lo = 0;
    cp.nd = c->alpha < L1 ? c->alpha : L1;
    cp.ap = c->alpha_pad;
    cp.groups = 0;
    cp.alpha = c->alpha;
    cp.n_src = L1;
    cp.digit0 = cp.per = 0;
    cp.convf_dstride = (size_t)c->M * c->alpha_pad;
    cp.dst_dstride = (size_t)E * c->N;
    PolyList all;
    all.n = E;
    for (u32 e = 0; e < CKKS_MAX_MODULI; e++) {
        all.spos[e] = all.dpos[e] = (unsigned char)(e < E ? e : 0);
        all.mod[e] = (unsigned char)(e < E ? c->ext_modulus(level, e) : 0);
    }
    NttArgs args = {};
    args.mc = c->d_mcf;
    args.tw = c->d_twf;
    args.tw_val = c->d_twf_val;
    args.log_n = c->log_n;
    args.log_lo = c->log_lo;
    args.log_hi = c->log_hi;
    const MidPrologue mp = {c->d_itwf, c->d_itwf_val, c->d_modup_prep_f + (size_t)level * c->num_q, 0, 1};
    cp.per = mid_per;
    const bool together = (mid_per && c->log_hi <= 3) || ((E - cp.nd + 3) / 4 * n << c->log_hi) < 768;
    for (u32 j0 = 0; j0 < beta; j0 += together ? beta : 1) {
        const u32 nj = together ? beta : 1;
        double rows = 0.0;  // transformed limb-polys
        u32 most = 0;       // targets of one digit
        cp.nd = c->digit_hi(j0, level) - c->digit_lo(j0);  // most source limbs of a digit (the last one may have fewer)
        for (u32 j = j0; j < j0 + nj; j++) {
            const u32 t = E - (c->digit_hi(j, level) - c->digit_lo(j));
            rows += (double)n * t;
            most = t > most ? t : most;
        }
        cp.digit0 = j0;
        args.src = nullptr;
        args.dst = digits;
        args.src_bstride = args.dst_bstride = (size_t)beta * E;
        args.first = 1;
        args.last = 0;
        args.batch = n;
        args.beta = 0;
        {
            ProfScope ps__(c, K_NTT_FWD_HI, st, 8.0 * c->N * (n * (together ? (double)L1 : (double)(E - most)) + rows), 0.5 * rows * c->N * c->log_hi);
            if (hipError_t e = launch_hi_conv(c->log_hi, most, nj, n, st, args, all, cp, mid_per ? &mp : nullptr); e != hipSuccess) return e;
        }
        if (hi_only) continue;  // the caller's own lo pass follows (launch_ntt_lo_mac)
        PolyList pl = all;
        args.dst = digits + (size_t)j0 * E * c->N;
        if (together) {  // rows (polynomial, digit) at a stride of E limb-polys
            args.dst_bstride = E;
            args.batch = n * beta;
            args.beta = beta;
            args.alpha = c->alpha;
            args.level = level;
        } else {  // the digit's own limbs are not in the list
            const u32 lo = c->digit_lo(j0), nd = E - most;
            for (u32 a = lo; a + nd < E; a++) {
                pl.spos[a] = pl.dpos[a] = all.dpos[a + nd];
                pl.mod[a] = all.mod[a + nd];
            }
            pl.n = most;
        }
        args.src = args.dst;
        args.src_bstride = args.dst_bstride;
        args.first = 0;
        args.last = 1;
        const u32 slices = pl.n << c->log_hi;
        args.lo_group = 0;
        for (u32 g = 64; g >= 8; g >>= 1)
            if (slices % g == 0) { args.lo_group = g; break; }
        const dim3 grid = args.lo_group ? dim3(args.lo_group, 1, slices / args.lo_group) : dim3(1, slices);
        ProfScope ps__(c, K_NTT_FWD_LO, st, 16.0 * rows * c->N, 0.5 * rows * c->N * c->log_lo);
        launch_fwd_lo_loop<ArithF64>(args.batch, grid, st, args, pl);
    }
    return hipGetLastError();
}

// The forward transforms of all digits of a ModUp with 64-bit integer butterflies (the conversions have written their target
// limbs in coefficient form): rows (polynomial, digit), a digit's own limbs skipped.  One launch per pass for all digits at every size: the
// passes are bound by instruction issue, so nothing is lost by a first pass that ends before the second starts, and a digit
// alone ends with a part of the chip idle.  56-bit moduli, a launch per digit and pass (conversion included) and now, in us: one
// unhoisted rotation of 7 limbs at N = 2^12 89.5 and 65.6, at 2^13 107.8 and 75.8, of 24 limbs at 2^16 293 and 257, four of those
// 784 and 724; a product of 24 limbs 365 and 329.
hipError_t launch_ntt_digits(const ckks_ctx* c, u32 level, u64* digits, u32 n, hipStream_t st) {
    if (c->ntt_f64 || c->log_hi == 0 || n == 0) return hipErrorInvalidValue;
    const u32 E = c->ext_limbs(level), beta = c->live_digits(level);
    PolyList all;
    all.n = E;
    for (u32 e = 0; e < CKKS_MAX_MODULI; e++) {
        all.spos[e] = all.dpos[e] = (unsigned char)(e < E ? e : 0);
        all.mod[e] = (unsigned char)(e < E ? c->ext_modulus(level, e) : 0);
    }
    NttArgs args = {};
    args.mc = c->d_mc;
    args.tw = c->d_tw;
    args.log_n = c->log_n;
    args.log_lo = c->log_lo;
    args.log_hi = c->log_hi;
    args.src = args.dst = digits;  // rows (polynomial, digit) at a stride of E limb-polys
    args.src_bstride = args.dst_bstride = E;
    args.batch = n * beta;
    args.beta = beta;
    args.alpha = c->alpha;
    args.level = level;
    args.first = 1;
    const double rows = n * ((double)beta * E - (level + 1.0));
    if (ntt_one_pass(c)) {
        args.last = 1;
        ProfScope ps__(c, K_NTT_FWD_LO, st, 16.0 * rows * c->N, 0.5 * rows * c->N * c->log_n);
        launch_ring(c, false, E, st, args, all, nullptr, nullptr);
        return hipGetLastError();
    }
    {
        ProfScope ps__(c, K_NTT_FWD_HI, st, 16.0 * rows * c->N, 0.5 * rows * c->N * c->log_hi);
        launch_hi_any<ArithU64>(c->log_hi, false, dim3(c->N >> CKKS_TILE_LOG, E * args.batch), st, args, all);
    }
    args.first = 0;
    args.last = 1;
    const u32 slices = E << c->log_hi;
    for (u32 g = 64; g >= 8; g >>= 1)
        if (slices % g == 0) { args.lo_group = g; break; }
    const dim3 grid = args.lo_group ? dim3(args.lo_group, 1, slices / args.lo_group) : dim3(1, slices);
    ProfScope ps__(c, K_NTT_FWD_LO, st, 16.0 * rows * c->N, 0.5 * rows * c->N * c->log_lo);
    launch_fwd_lo_loop<ArithU64>(args.batch, grid, st, args, all);
    return hipGetLastError();
}

hipError_t launch_ntt_rescale(const ckks_ctx* c, u32 level, const double* y, u64* dst, u32 batch, hipStream_t st,
                              const FwdEpilogue* epilogue, u32 mid_per, const u64* const* dropped) {
    if (level == 0 || !c->d_rescale_conv_f) return hipErrorInvalidValue;
    if (dropped && (!ntt_rescale_one_launch(c, level, batch) || batch > KS_MAX_BATCH || epilogue->use_vl == 2)) return hipErrorInvalidValue;
    ConvPrologue cp;
    cp.y = y;
    cp.y_bstride = c->N;  // one limb per batch item
    cp.convf = c->d_rescale_conv_f;
    cp.lo = 0;
    cp.nd = 1;
    cp.ap = 4;
    cp.alpha = cp.n_src = cp.digit0 = cp.per = 0;
    cp.convf_dstride = cp.dst_dstride = 0;
    PolyList pl;
    for (u32 a = 0; a < CKKS_MAX_MODULI; a++) pl.spos[a] = pl.dpos[a] = pl.mod[a] = (unsigned char)(a < level ? a : 0);
    pl.n = level;
    const MidPrologue mp = {c->d_itwf, c->d_itwf_val, c->d_rescale_prep_f, level, level};
    if (dropped) {
        NttArgs args = {};
        args.mc = c->d_mcf;
        args.tw = c->d_twf;
        args.tw_val = c->d_twf_val;
        args.log_n = c->log_n;
        args.log_lo = c->log_lo;
        args.log_hi = c->log_hi;
        args.batch = batch;
        for (u32 b = 0; b < batch; b++) args.src_list.p[b] = dropped[b];
        // in: the dropped limbs and the others, out: the quotients
        ProfScope ps__(c, K_NTT_FWD_LO, st, 8.0 * c->N * batch * (1.0 + 2.0 * level), 0.5 * batch * (1.0 + level) * c->N * c->log_n);
        launch_ring(c, false, level, st, args, pl, &cp, epilogue, &mp);
        return hipGetLastError();
    }
    cp.per = mid_per;
    return launch_ntt_any(c, false, dst, level, dst, level, pl, batch, st, nullptr, epilogue, nullptr, &cp, nullptr, nullptr, NTT_BOTH, mid_per ? &mp : nullptr);
}

hipError_t launch_ntt_lo_mac(const ckks_ctx* c, u32 level, const DigitSrc& digits, const u64* const* keys, u64* const* outs, u32 n,
                             hipStream_t st, u32 inv_from, const MacProduct* prod, const MacRotate* rot, u32* n_part, const MacDivide* div, bool dropped_only) {
    if ((div || dropped_only) && (n_part || inv_from == 0 || inv_from >= c->ext_limbs(level) || (!prod && !rot))) return hipErrorInvalidValue;
    if (!ntt_has_modup(c) || (n_part && !rot) || (rot && rot->mask && !n_part) || (rot && rot->hoisted && n_part) || c->log_hi == 0 || n == 0 || n > KS_MAX_BATCH || (prod && rot)) return hipErrorInvalidValue;
    const u32 E = c->ext_limbs(level), beta = c->live_digits(level);
    NttArgs args = {};
    args.mc = c->d_mcf;
    args.tw = c->d_twf;
    args.tw_val = c->d_twf_val;
    args.log_n = c->log_n;
    args.log_lo = c->log_lo;
    args.log_hi = c->log_hi;
    args.batch = n;
    const u32 slices = (div ? inv_from : (dropped_only ? E - inv_from : E)) << c->log_hi;
    args.lo_group = 0;
    for (u32 g = 64; g >= 8; g >>= 1)
        if (slices % g == 0) { args.lo_group = g; break; }
    PolyList pl;
    pl.n = E;
    for (u32 e = 0; e < CKKS_MAX_MODULI; e++) pl.spos[e] = pl.dpos[e] = pl.mod[e] = (unsigned char)(e < E ? c->ext_modulus(level, e) : 0);
    MacEpilogue ep;
    ep.D = digits;
    double n_add = 0.0, n_keys = 0.0, n_src = 0.0;
    for (u32 b = 0; b < KS_MAX_BATCH; b++) {
        ep.key.p[b] = b < n ? keys[b] : nullptr;
        ep.out.p[b] = b < n ? outs[b] : nullptr;
        if (b < n && !ep.key.p[b]) return hipErrorInvalidValue;
        ep.a0.p[b] = b < n ? (prod ? prod->a0[b] : (rot ? rot->c0[b] : nullptr)) : nullptr;
        ep.gal[b] = (rot && b < n) ? rot->gs[b] : 1;
        if (rot && b < n && !ep.a0.p[b]) return hipErrorInvalidValue;
        ep.a1.p[b] = (prod && b < n) ? prod->a1[b] : nullptr;
        ep.b0.p[b] = (prod && b < n) ? prod->b0[b] : nullptr;
        ep.b1.p[b] = (prod && b < n) ? prod->b1[b] : nullptr;
        if (prod && b < n && (!ep.a0.p[b] || !ep.a1.p[b] || !ep.b0.p[b] || !ep.b1.p[b])) return hipErrorInvalidValue;
        if (b < n && (b == 0 || keys[b] != keys[b - 1])) n_keys += 1.0;
        if (rot && b < n && (b == 0 || rot->c0[b] != rot->c0[b - 1])) n_src += 1.0;
    }
    ep.negp = c->d_moddown + 2 * c->k_pad + (size_t)c->k_pad * c->num_q + 2 * c->num_q;
    ep.level = level;
    ep.M = c->M;
    ep.E = E;
    ep.beta = beta;
    ep.itw_val = c->d_itwf_val;
    ep.inv_from = inv_from;
    ep.first = div ? 0 : (inv_from < E ? inv_from : 0);
    ep.w = div ? div->w : nullptr;
    ep.cinv = div ? div->cinv : nullptr;
    for (u32 b = 0; b < KS_MAX_BATCH; b++) {
        ep.add.p[b] = div && div->adds && b < n ? div->adds[b] : nullptr;
        ep.res.p[b] = div && b < n ? div->outs[b] : nullptr;
        if (ep.add.p[b]) n_add += 1.0;
    }
    ep.mask = rot ? rot->mask : nullptr;
    const bool lin = prod && prod->lin_x;
    if (lin && (!prod->lin_y || !prod->ka || !prod->kb)) return hipErrorInvalidValue;
    ep.x_cstride = lin ? prod->x_cstride : 0;
    ep.y_cstride = lin ? prod->y_cstride : 0;
    for (u32 b = 0; b < KS_MAX_BATCH; b++) {
        ep.lx.p[b] = (lin && b < n) ? prod->lin_x[b] : nullptr;
        ep.ly.p[b] = (lin && b < n) ? prod->lin_y[b] : nullptr;
        if (lin && b < n && (!ep.lx.p[b] || !ep.ly.p[b])) return hipErrorInvalidValue;
    }
    for (u32 i = 0; i < CKKS_MAX_MODULI; i++) {
        ep.ka[i] = (lin && i <= level) ? prod->ka[i] : 0;
        ep.kb[i] = (lin && i <= level) ? prod->kb[i] : 0;
    }
    // the grid's extent over the batch: two, i.e. four items per workgroup in a batch of eight (measured: 16.5 ms per step for
    // the lo-pass class with one item per workgroup, 16.35 with all eight, 16.15 with four, which still leave the chip's 256
    // CUs, two workgroups each, four rounds of workgroups); more of them where the launch is small (see lo_items)
    const u32 items = lo_items(slices, n, 4), b_least = n < 2 ? n : 2;
    const u32 b_ext = (n + items - 1) / items < b_least ? b_least : (n + items - 1) / items;
    const dim3 grid = args.lo_group ? dim3(args.lo_group, b_ext, slices / args.lo_group) : dim3(b_ext, slices);
    if (n_part) *n_part = b_ext;
    // What this launch covers: np positions, `live` of them ciphertext limbs, `inverse` of them dropped limbs that go on into their inverse
    // transform.  In: per item every (digit, position) row but the digits' own limbs, which come from the decomposed polynomial (finished digits once for all
    // items), the operands at the live limbs (once per distinct ciphertext of a rotation), the keys (once per distinct key), the mask; for a division the converted
    // parts and what is added.  Out: two components per item, of a sum the partial sums.
    const bool hoisted = rot && rot->hoisted;
    const double np = div ? inv_from : (dropped_only ? E - inv_from : E), kept = dropped_only ? 0.0 : (inv_from < E ? inv_from : E), inverse = div ? 0.0 : np - kept;
    const double live = div ? inv_from : (dropped_only ? level + 1.0 - inv_from : level + 1.0);
    const double rows = beta * np - live, n_tr = hoisted ? 0.0 : n * rows;  // n_tr: transformed
    double words = (hoisted ? 1.0 : (double)n) * rows + n_keys * 2.0 * beta * np + (rot && rot->mask ? live : 0.0);
    words += live * (prod ? (lin ? 8.0 : 4.0) * n : (rot ? 2.0 * n_src : 1.0 * n));  // (lin: two components of two ciphertexts)
    words += 2.0 * (n * inverse + (n_part ? b_ext : n) * kept);
    if (div) words += 2.0 * kept * (n + n_add);
    ProfScope ps__(c, K_NTT_FWD_LO, st, 8.0 * c->N * words, 0.5 * c->N * c->log_lo * (n_tr + 2.0 * n * (inverse + (div ? kept : 0.0))));
    // which operands join after the digits is the same for the whole launch: one instantiation per case
#define LO_MAC_LAUNCH(...) hipLaunchKernelGGL((ntt_fwd_lo_mac_kernel<__VA_ARGS__>), grid, dim3(NTT_THREADS), 0, st, args, pl, ep)
    if (rot && rot->hoisted) {
        if (div) LO_MAC_LAUNCH(false, false, true, false, false, true, true);
        else LO_MAC_LAUNCH(false, false, true, false, false, false, true);
        return hipGetLastError();
    }
    if (div) {
        if (lin) LO_MAC_LAUNCH(true, true, false, false, false, true);
        else if (prod) LO_MAC_LAUNCH(true, false, false, false, false, true);
        else LO_MAC_LAUNCH(false, false, true, false, false, true);
        return hipGetLastError();
    }
    if (lin) LO_MAC_LAUNCH(true, true, false);
    else if (prod) LO_MAC_LAUNCH(true, false, false);
    else if (rot && rot->mask) LO_MAC_LAUNCH(false, false, true, true, true);
    else if (n_part) LO_MAC_LAUNCH(false, false, true, true);
    else if (rot) LO_MAC_LAUNCH(false, false, true);
    else LO_MAC_LAUNCH(false, false, false);
#undef LO_MAC_LAUNCH
    return hipGetLastError();
}

hipError_t launch_ntt_moddown(const ckks_ctx* c, u32 level, bool merged, const double* y, u64* dst, u32 batch, hipStream_t st,
                              const FwdEpilogue* epilogue, u32 mid_per) {
    if (merged && level == 0) return hipErrorInvalidValue;
    const u32 n_out = merged ? level : level + 1;
    ConvPrologue cp;
    cp.y = y;
    cp.y_bstride = (size_t)c->ext_limbs(level) * c->N;
    cp.convf = merged ? c->moddown_rs_table_f(level) : c->d_moddown_f;
    cp.lo = merged ? level : level + 1;  // the dropped limbs sit at consecutive positions of the extended polynomial
    cp.nd = merged ? c->num_p + 1 : c->num_p;
    cp.ap = merged ? c->k2_pad : c->k_pad;
    cp.alpha = cp.n_src = cp.digit0 = cp.per = 0;
    cp.convf_dstride = cp.dst_dstride = 0;
    PolyList pl;
    for (u32 a = 0; a < CKKS_MAX_MODULI; a++) pl.spos[a] = pl.dpos[a] = pl.mod[a] = (unsigned char)(a < n_out ? a : 0);
    pl.n = n_out;
    const MidPrologue mp = {c->d_itwf, c->d_itwf_val, merged ? c->d_moddown_rs_prep_f + (size_t)level * c->M : c->d_moddown_prep_f, merged ? level : c->num_q,
                            merged ? c->num_q : c->num_q + 1};
    cp.per = mid_per;
    return launch_ntt_any(c, false, dst, n_out, dst, n_out, pl, batch, st, nullptr, epilogue, nullptr, &cp, nullptr, nullptr, epilogue ? NTT_BOTH : NTT_HI, mid_per ? &mp : nullptr);
}

// v: [2][E][N] per item, v_bstride apart: the items' dropped limbs have been through the first pass of their inverse transform, their other limbs are
// n_part partial sums in the places of the first n_part items (launch_ntt_lo_mac with n_part).  w: [2][level+1][N] scratch.
hipError_t launch_ntt_moddown_sum(const ckks_ctx* c, u32 level, u64* v, size_t v_bstride, u32 n, u32 n_part, u64* w, const FinalItem& item, hipStream_t st) {
    const u32 E = c->ext_limbs(level), n_out = level + 1, k = c->num_p;
    if (!ntt_has_modup(c) || n == 0 || n > KS_MAX_BATCH || n_part == 0 || n_part > n || (item.mask && !item.acc) || item.add0 || item.add1 || v_bstride != 2 * (size_t)E * c->N)
        return hipErrorInvalidValue;
    NttArgs args = {};
    args.mc = c->d_mcf;
    args.log_n = c->log_n;
    args.log_lo = c->log_lo;
    args.log_hi = c->log_hi;
    PolyList dropped, pl;
    for (u32 a = 0; a < CKKS_MAX_MODULI; a++) {
        dropped.spos[a] = dropped.dpos[a] = (unsigned char)(a < k ? n_out + a : 0);
        dropped.mod[a] = (unsigned char)(a < k ? c->num_q + a : 0);
        pl.spos[a] = pl.dpos[a] = pl.mod[a] = (unsigned char)(a < n_out ? a : 0);
    }
    dropped.n = k;
    pl.n = n_out;
    ConvPrologue cp = {};
    cp.y = (const double*)v;
    cp.y_bstride = (size_t)E * c->N;
    cp.convf = c->d_moddown_f;
    cp.lo = n_out;
    cp.nd = k;
    cp.ap = c->k_pad;
    const u32 tiles = c->N >> CKKS_TILE_LOG;
    const dim3 block(NTT_THREADS);
#define BY_LOG_HI(LAUNCH)                     \
    switch (c->log_hi) {                      \
        case 1: LAUNCH(1); break;             \
        case 2: LAUNCH(2); break;             \
        case 3: LAUNCH(3); break;             \
        case 4: LAUNCH(4); break;             \
        case 5: LAUNCH(5); break;             \
        case 6: LAUNCH(6); break;             \
        default: return hipErrorInvalidValue; \
    }
    {
        args.tw = c->d_itwf;
        args.src = args.dst = v;
        args.src_bstride = args.dst_bstride = E;
        args.inv_scale = c->d_moddown_prep_f;
        ProfScope ps__(c, K_NTT_INV_HI, st, 16.0 * c->N * k * (n + 1.0), (double)n * c->N * k * c->log_hi);
#define INV_HI_SUM(H) hipLaunchKernelGGL((ntt_inv_hi_sum_kernel<H>), dim3(tiles, 2 * k), block, 0, st, args, dropped, n)
        BY_LOG_HI(INV_HI_SUM)
#undef INV_HI_SUM
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    args.tw = c->d_twf;
    args.tw_val = c->d_twf_val;
    args.src = args.dst = w;
    args.src_bstride = args.dst_bstride = n_out;
    args.inv_scale = nullptr;
    args.batch = 2;
    {
        ProfScope ps__(c, K_NTT_FWD_HI, st, 16.0 * c->N * ((double)k + n_out), (double)c->N * n_out * c->log_hi);
#define CONV_SUM(H) hipLaunchKernelGGL((ntt_fwd_hi_conv_sum_kernel<H>), dim3(tiles, 2 * n_out), block, 0, st, args, pl, cp)
        BY_LOG_HI(CONV_SUM)
#undef CONV_SUM
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
#undef BY_LOG_HI
    FwdEpilogue ep = {};
    ep.v = v;
    ep.cinv = c->d_moddown + 2 * c->k_pad + (size_t)c->k_pad * c->num_q;
    ep.mci = c->d_mc;
    ep.E = E;
    ep.n_out = n_out;
    ep.num_q = c->num_q;
    ep.n_part = n_part;
    ep.v_pstride = v_bstride;
    ep.B.it[0] = item;
    const u32 slices = n_out << c->log_hi;
    for (u32 g = 64; g >= 8; g >>= 1)
        if (slices % g == 0) { args.lo_group = g; break; }
    const dim3 grid = args.lo_group ? dim3(args.lo_group, 2, slices / args.lo_group) : dim3(2, slices);
    ProfScope ps__(c, K_NTT_FWD_LO, st, 8.0 * c->N * n_out * (4.0 + 2.0 * n_part + (item.acc ? 2.0 : 0.0) + (item.mask ? 1.0 : 0.0)), (double)c->N * n_out * c->log_lo);
    if (item.mask) hipLaunchKernelGGL((ntt_fwd_lo_div_kernel<ArithF64, EM_SUM_MASK>), grid, block, 0, st, args, pl, ep);
    else if (item.acc) hipLaunchKernelGGL((ntt_fwd_lo_div_kernel<ArithF64, EM_SUM_ADD>), grid, block, 0, st, args, pl, ep);
    else hipLaunchKernelGGL((ntt_fwd_lo_div_kernel<ArithF64, EM_SUM>), grid, block, 0, st, args, pl, ep);
    return hipGetLastError();
}
