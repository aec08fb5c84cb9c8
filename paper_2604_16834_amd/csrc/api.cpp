// The C boundary: argument checks, workspace carving and the order of kernel launches of every
// exported operation.  No arithmetic happens on the host; no call here allocates or synchronises.
//
// Work is batched wherever operands are independent: the channel ciphertexts of a layer share their
// rotation and relinearisation keys, so eight or sixteen of them (see ks_batch) go through every kernel of a
// key switch together (the key streams from HBM once per batch, NTT launches are large enough to fill
// the chip); the rotations of one ciphertext share its extended digits (hoisting).
#include <cstdio>
#include <new>
#include <vector>

#include "ctx.h"

namespace {

int set_err(const ckks_ctx* c, int code, const char* msg) {
    if (c) c->err = msg;
    return code;
}

#define HIP_TRY(expr)                                                              \
    do {                                                                           \
        hipError_t e__ = (expr);                                                   \
        if (e__ != hipSuccess) {                                                   \
            c->err = std::string(#expr ": ") + hipGetErrorString(e__);             \
            return CKKS_ERR_HIP;                                                   \
        }                                                                          \
    } while (0)

// bump allocator over the caller's workspace (256-byte aligned blocks of u64)
int set_hip_err(const ckks_ctx* c, hipError_t e) {
    c->err = std::string("HIP: ") + hipGetErrorString(e);
    return CKKS_ERR_HIP;
}

struct Arena {
    char* base;
    size_t cap, used;
    Arena(void* p, size_t n) : base((char*)p), cap(n), used(0) {}
    u64* take(size_t elems) {
        size_t bytes = (elems * sizeof(u64) + 255) & ~(size_t)255;
        if (!base || used + bytes > cap) { used = cap + 1; return nullptr; }
        u64* r = (u64*)(base + used);
        used += bytes;
        return r;
    }
    bool ok() const { return used <= cap; }
    Arena rest() const { return ok() ? Arena(base + used, cap - used) : Arena(nullptr, 0); }
};
size_t blk(size_t elems) { return (elems * sizeof(u64) + 255) & ~(size_t)255; }

PolyList range_list(u32 first_pos, u32 count, u32 first_mod) {
    PolyList pl;
    pl.n = count;
    for (u32 a = 0; a < CKKS_MAX_MODULI; a++) {
        pl.spos[a] = pl.dpos[a] = (unsigned char)(a < count ? first_pos + a : 0);
        pl.mod[a] = (unsigned char)(a < count ? first_mod + a : 0);
    }
    return pl;
}

PtrList8 ptr_list(const u64* const* p, u32 n) {
    PtrList8 l;
    for (u32 b = 0; b < KS_MAX_BATCH; b++) l.p[b] = b < n ? p[b] : nullptr;
    return l;
}
OutList8 out_list(u64* const* p, u32 n) {
    OutList8 l;
    for (u32 b = 0; b < KS_MAX_BATCH; b++) l.p[b] = b < n ? p[b] : nullptr;
    return l;
}

bool level_ok(const ckks_ctx* c, u32 level) { return level < c->num_q; }

// ---- key-switch workspace: n_dig polynomials being decomposed, n_v key switches in flight ----------
struct KsWs {
    u64 *y, *digits, *v, *w;
    size_t y_b, dig_b, v_b, w_b;  // per-item strides in elements
    mutable const u64* own[KS_MAX_BATCH] = {};  // the polynomials run_modup decomposed last (the digits' own limbs stay there)
};
// the digits of items b0, b0 + 1, ... of the batch in ws, as the inner-product kernels take them
DigitSrc dsrc(const ckks_ctx* c, const KsWs& ws, u32 b0) {
    DigitSrc d;
    d.digits = ws.digits + b0 * ws.dig_b;
    d.bstride = ws.dig_b;
    for (u32 b = 0; b < KS_MAX_BATCH; b++) d.own.p[b] = b0 + b < KS_MAX_BATCH ? ws.own[b0 + b] : nullptr;
    d.alpha = c->alpha;
    d.pad = 0;
    return d;
}
size_t ws_ks(const ckks_ctx* c, u32 level, u32 n_dig, u32 n_v) {
    const size_t N = c->N, L1 = level + 1, E = c->ext_limbs(level), beta = c->live_digits(level);
    return blk(n_dig * L1 * N) + blk(n_dig * beta * E * N) + blk(n_v * 2 * E * N) + blk(n_v * 2 * L1 * N);
}
bool carve_ks(const ckks_ctx* c, u32 level, u32 n_dig, u32 n_v, Arena& ar, KsWs& b) {
    const size_t N = c->N, L1 = level + 1, E = c->ext_limbs(level), beta = c->live_digits(level);
    b.y_b = L1 * N;
    b.dig_b = beta * E * N;
    b.v_b = 2 * E * N;
    b.w_b = 2 * L1 * N;
    b.y = ar.take(n_dig * b.y_b);
    b.digits = ar.take(n_dig * b.dig_b);
    b.v = ar.take(n_v * b.v_b);
    b.w = ar.take(n_v * b.w_b);
    return ar.ok();
}
// Most key switches that go through the kernels together: as many as the pointer lists hold.  A small launch takes as long as its longest
// workgroup, so a second batch costs nearly what the first does, and large ones share the keys and the twiddles of twice as many.
// Sixteen unhoisted rotations in batches of eight / together in us: N = 2^12, 7 + 3 limbs 82 / 46, 2^14 140 / 112, 2^16 477 / 443,
// 21 + 8 limbs 1353 / 1310; activation of eight, x^3 and x^4 in one batch: 2^12, 7 + 3 limbs 169 / 134, 2^16, 21 + 8 2681 / 2619.
// (Eight with integer arithmetic, whose inner-product launch takes no more.)
u32 ks_batch(const ckks_ctx* c) { return ntt_has_modup(c) ? KS_MAX_BATCH : CT_BATCH; }
// Calls with more than eight independent items: together on the caller's stream while a polynomial of the extended basis has no more
// coefficients than `limit`, in batches of eight that alternate between two streams above.  A fork and a join are worth 45 us; from some size on
// the kernels of one batch beside another's are worth more, and the sooner where sixteen are not all of them: several batches on one
// stream come one after the other.
bool together(const ckks_ctx* c, u32 level, size_t limit) { return ntt_has_modup(c) && (size_t)c->ext_limbs(level) * c->N <= limit; }
// Hoisted rotations, two streams / together in us, 12 / 16: N = 2^12, 7 + 3 limbs 101 / 46, 105 / 47, 24 + 8 (0.13 M coefficients) 99 / 79, 106 / 90,
// 2^14, 14 + 6 (0.33 M) 158 / 157, 189 / 190, 2^15, 7 + 3 (0.33 M) 156 / 152, 191 / 185, 2^14, 24 + 8 (0.52 M) 221 / 227, 275 / 277;
// 17 / 24 / 64: 2^12, 7 + 3 (0.04 M) 115 / 66, 124 / 74, 238 / 157, 24 + 8 (0.13 M) 122 / 113, 135 / 132, 276 / 303, 2^13, 14 + 6 (0.16 M) 133 / 128, 147 / 151,
// 321 / 348, 2^14, 14 + 6 211 / 220, 275 / 283, 631 / 678
bool rotations_together(const ckks_ctx* c, u32 level, u32 n) { return together(c, level, n <= KS_MAX_BATCH ? (size_t)3 << 17 : (size_t)1 << 17); }
size_t ws_rescale(const ckks_ctx* c, u32 level, u32 n) { return blk(2 * (size_t)n * c->N) + blk(2 * (size_t)n * level * c->N); }
// n unhoisted rotations: their key switches, and a permuted copy of each polynomial where no transform gathers it (run_rotate_batch)
size_t ws_permuted(const ckks_ctx* c, u32 level, u32 n) { return ntt_has_modup(c) ? 0 : blk((size_t)n * (level + 1) * c->N); }
size_t ws_rotate_unhoisted(const ckks_ctx* c, u32 level, u32 n) { return ws_ks(c, level, n, n) + ws_permuted(c, level, n); }
// a product's scratch: the key switch's, and the three polynomials of the tensor product where a kernel forms them (elsewhere they
// are not stored: run_product)
size_t ws_ctct(const ckks_ctx* c, u32 level, u32 n) {
    return (ntt_has_modup(c) ? 0 : 3 * blk((size_t)n * (level + 1) * c->N)) + ws_ks(c, level, n, n);
}

// Decompose + ModUp of n <= ks_batch polynomials srcs[b] ([level+1][N], NTT form) into
// ws.digits + b*ws.dig_b ([beta][E][N], NTT form).
// hi_only (double-precision transforms only): the forward transforms stop after their first pass; the caller finishes them
// inside the inner product (launch_ntt_lo_mac).
// muls (with hi_only): the polynomial to decompose is srcs[b] (.) muls[b], formed as the inverse transform loads it.
// gals (with hi_only, ntt_has_modup): it is sigma_gals[b](srcs[b]); the own limbs stay where they are, not permuted.
int run_modup(const ckks_ctx* c, u32 level, const u64* const* srcs, u32 n, const KsWs& ws, hipStream_t st, bool hi_only = false,
              const u64* const* muls = nullptr, const u32* gals = nullptr) {
    const u32 N = c->N, L1 = level + 1, E = c->ext_limbs(level), beta = c->live_digits(level);
    for (u32 b = 0; b < KS_MAX_BATCH; b++) ws.own[b] = (b < n && !muls) ? srcs[b] : nullptr;  // a product has no stored own limbs
    if (muls && !hi_only) return set_err(c, CKKS_ERR_INVALID_ARG, "internal: product source without the fused inner product");
    // all live limbs of every polynomial to coefficient form at once.  With double-precision transforms the inverse scales
    // limb i by N^-1 (Q_j/q_i)^-1 and leaves the centred residue as a double, and each digit's basis conversion happens
    // inside the first pass of the forward transforms of its target limbs (no conversion kernel, no coefficient-form copy
    // of the extended digit).
    const bool fused = ntt_has_modup(c);
    if (hi_only && !fused) return set_err(c, CKKS_ERR_INVALID_ARG, "internal: fused inner product without fused ModUp");
    const u32 mid = ntt_mid_modup(c, level, n);  // the inverse's second pass inside the converting one
    HIP_TRY(launch_ntt(c, true, nullptr, 0, ws.y, L1, range_list(0, L1, 0), n, st, srcs, nullptr,
                       fused ? c->d_modup_prep_f + (size_t)level * c->num_q : nullptr, muls, nullptr, mid ? NTT_LO : NTT_BOTH, gals));  // (positions 0..level are moduli 0..level)
    if (fused) {
        HIP_TRY(launch_ntt_modup(c, level, (const double*)ws.y, ws.y_b, ws.digits, n, st, hi_only, mid));
        return CKKS_OK;
    }
    if (!c->small_q && c->log_hi > 0) {  // all digits together (see launch_ntt_digits)
        HIP_TRY(launch_modup_conv(c, level, 0, beta, ws.y, ws.y_b, ws.digits, ws.dig_b, n, st));
        HIP_TRY(launch_ntt_digits(c, level, ws.digits, n, st));
        return CKKS_OK;
    }
    for (u32 j = 0; j < beta; j++) {
        const u32 lo = c->digit_lo(j), hi = c->digit_hi(j, level);
        u64* digit = ws.digits + (size_t)j * E * N;
        HIP_TRY(launch_modup_conv(c, level, j, 1, ws.y, ws.y_b, ws.digits, ws.dig_b, n, st));
        PolyList pl;
        pl.n = 0;
        for (u32 e = 0; e < E; e++) {
            const u32 t = c->ext_modulus(level, e);
            if (t >= lo && t < hi) continue;
            pl.spos[pl.n] = pl.dpos[pl.n] = (unsigned char)e;
            pl.mod[pl.n] = (unsigned char)t;
            pl.n++;
        }
        for (u32 a = pl.n; a < CKKS_MAX_MODULI; a++) pl.spos[a] = pl.dpos[a] = pl.mod[a] = 0;
        HIP_TRY(launch_ntt(c, false, digit, (size_t)beta * E, digit, (size_t)beta * E, pl, n, st));
    }
    return CKKS_OK;
}

// What the forward transform of the converted dropped part does to its results instead of storing them (see FwdEpilogue).
FwdEpilogue moddown_epilogue(const ckks_ctx* c, u32 level, bool merged, const u64* v, const FinalItem* items, u32 n) {
    FwdEpilogue ep;
    const u32 kp = merged ? c->k2_pad : c->k_pad;
    const u64* tab = merged ? c->moddown_rs_table(level) : c->d_moddown;
    ep.v = v;
    ep.cinv = tab + 2 * kp + (size_t)kp * c->num_q;
    ep.mci = c->d_mc;
    ep.E = c->ext_limbs(level);
    ep.n_out = merged ? level : level + 1;
    ep.num_q = c->num_q;
    ep.use_vl = 0;
    ep.v_cstride = ep.v2_cstride = 0;
    for (u32 r = 0; r < KS_MAX_BATCH; r++) ep.vl.p[r] = ep.vl2.p[r] = nullptr;
    for (u32 r = 0; r < KS_MAX_BATCH; r++) ep.B.it[r] = r < n ? items[r] : FinalItem{nullptr, nullptr, nullptr, nullptr, 1, 0};
    return ep;
}

// The first of the extended basis' positions that a division drops: the special primes', or (merged) limb `level` in front of them.
u32 dropped_from(u32 level, bool merged) { return merged ? level : level + 1; }

// ModDown of the n inner products sitting in ws.v: one pass of each kernel over the whole batch.
// items[r] says what is added to / multiplied into the r-th result and where it goes ([2][level+1][N]).
// merged: the division is by P*q_level (ModDown and rescale in one): the dropped limbs are position
// level and the special primes, the results are [2][level][N].
// items null (with lo_done): all but the second pass of the converted parts' forward transforms and the last step (run_inner_divide).
// lo_done: the dropped limbs have been through the first pass of their inverse transform (launch_ntt_lo_mac with inv_from).
int run_moddown(const ckks_ctx* c, u32 level, const KsWs& ws, u32 n, const FinalItem* items, hipStream_t st, bool merged = false,
                bool lo_done = false) {
    const u32 L1 = level + 1, E = c->ext_limbs(level), k = c->num_p;
    const u32 mid = ntt_mid_moddown(c, level, merged, 2 * n, lo_done);
    if (merged) {
        PolyList dl = range_list(level, k + 1, c->num_q - 1);  // positions level.. ; moduli fixed up below
        dl.mod[0] = (unsigned char)level;
        for (u32 a = 1; a <= k; a++) dl.mod[a] = (unsigned char)(c->num_q + a - 1);
        if (ntt_has_modup(c)) {  // conversion inside the forward transform's first pass, last step inside its second
            if (!lo_done || !mid)
                HIP_TRY(launch_ntt(c, true, ws.v, E, ws.v, E, dl, 2 * n, st, nullptr, nullptr, c->d_moddown_rs_prep_f + (size_t)level * c->M,
                                   nullptr, nullptr, lo_done ? NTT_HI : (mid ? NTT_LO : NTT_BOTH)));
            if (!items) {
                HIP_TRY(launch_ntt_moddown(c, level, true, (const double*)ws.v, ws.w, 2 * n, st, nullptr, mid));
                return CKKS_OK;
            }
            const FwdEpilogue ep = moddown_epilogue(c, level, true, ws.v, items, n);
            HIP_TRY(launch_ntt_moddown(c, level, true, (const double*)ws.v, ws.w, 2 * n, st, &ep, mid));
            return CKKS_OK;
        }
        HIP_TRY(launch_ntt(c, true, ws.v, E, ws.v, E, dl, 2 * n, st));
        HIP_TRY(launch_moddown_conv(c, level, true, ws.v, ws.w, 2 * n, st));
        if (ntt_has_epilogue(c)) {  // the last step rides on the transform's stores
            const FwdEpilogue ep = moddown_epilogue(c, level, true, ws.v, items, n);
            HIP_TRY(launch_ntt(c, false, ws.w, level, ws.w, level, range_list(0, level, 0), 2 * n, st, nullptr, &ep));
            return CKKS_OK;
        }
        HIP_TRY(launch_ntt(c, false, ws.w, level, ws.w, level, range_list(0, level, 0), 2 * n, st));
        HIP_TRY(launch_moddown_final(c, level, true, ws.v, ws.w, items, n, st));
        return CKKS_OK;
    }
    if (ntt_has_modup(c)) {
        if (!lo_done || !mid)
            HIP_TRY(launch_ntt(c, true, ws.v, E, ws.v, E, range_list(L1, k, c->num_q), 2 * n, st, nullptr, nullptr, c->d_moddown_prep_f, nullptr, nullptr,
                               lo_done ? NTT_HI : (mid ? NTT_LO : NTT_BOTH)));
        if (!items) {
            HIP_TRY(launch_ntt_moddown(c, level, false, (const double*)ws.v, ws.w, 2 * n, st, nullptr, mid));
            return CKKS_OK;
        }
        const FwdEpilogue ep = moddown_epilogue(c, level, false, ws.v, items, n);
        HIP_TRY(launch_ntt_moddown(c, level, false, (const double*)ws.v, ws.w, 2 * n, st, &ep, mid));
        return CKKS_OK;
    }
    HIP_TRY(launch_ntt(c, true, ws.v, E, ws.v, E, range_list(L1, k, c->num_q), 2 * n, st));  // P-part -> coefficients
    HIP_TRY(launch_moddown_conv(c, level, false, ws.v, ws.w, 2 * n, st));
    if (ntt_has_epilogue(c)) {
        const FwdEpilogue ep = moddown_epilogue(c, level, false, ws.v, items, n);
        HIP_TRY(launch_ntt(c, false, ws.w, L1, ws.w, L1, range_list(0, L1, 0), 2 * n, st, nullptr, &ep));
        return CKKS_OK;
    }
    HIP_TRY(launch_ntt(c, false, ws.w, L1, ws.w, L1, range_list(0, L1, 0), 2 * n, st));
    HIP_TRY(launch_moddown_final(c, level, false, ws.v, ws.w, items, n, st));
    return CKKS_OK;
}

// Inner products (launch_ntt_lo_mac: prod or rot) and their division, outs[b] = (..) / P + accs[b] (merged: / (P q_level)).  Large launches take the inner
// products of the limbs that stay inside the division's last pass, when the converted dropped limbs are there: the sums are neither written
// nor read back, and one fetch of a slice's twiddles serves the digits and both components of the converted part.  Small ones take
// all positions at once, as the dropped limbs' launch alone leaves CUs idle and the other limbs' digits wait behind it.  All at once / inside the division in us,
// by slices (limbs that stay x items x blocks of 2^11): six rotations at N = 2^13, 7 + 3 limbs (168) 42 / 52, one at 2^15, 14 + 5 (208) 60 / 68, a product at
// 2^16, 13 + 8 (416) 101 / 103, twelve rotations at 2^13, 14 + 7 (624) 83 / 86; a product at 2^16, 24 + 8 (768) 163 / 159, six rotations, 6 + 3 (960) 130 / 125,
// twelve at 2^14, 14 + 5 (1248) 166 / 158, at 2^16, 21 + 8 (8064) 981 / 935, activations of sixteen, 20 + 7, 2^14 (1152) 1151 / 1061, 2^16 (4608) 4443 / 4107
#define DIVIDE_INSIDE_SLICES 768
// Hoisted rotations likewise, whose finished digits are read through the rotation: a kernel of its own that scattered every position's sums, four launches behind the
// digits / all at once, three launches / inside the division, in us: one at N = 2^12, 5 + 3 limbs (10) 33.9 / 32.1 / 36, three at 2^15, 7 + 3 (336)
// 63.7 / 60.5 / 66.8, sixteen at 2^13, 14 + 7 (832) 88.3 / 82.2 / 85; six at 2^16, 6 + 2 (960) 104 / 107 / 102.5, two of 24 + 8 (1536) 204 / 194 / 181,
// sixteen (6144 a batch) 993 / 981 / 840
#define DIVIDE_INSIDE_HOISTED 900
int run_inner_divide(const ckks_ctx* c, u32 level, const KsWs& ws, const u64* const* keys, u32 n, u64* const* outs, const u64* const* accs, hipStream_t st,
                     bool merged, const MacProduct* prod, const MacRotate* rot) {
    u64* vs[KS_MAX_BATCH];
    for (u32 b = 0; b < n; b++) vs[b] = ws.v + b * ws.v_b;
    const u32 from = dropped_from(level, merged);
    const u32 slices = from * n << c->log_hi;
    if (rot && rot->hoisted ? slices < DIVIDE_INSIDE_HOISTED : c->log_hi < 2 || slices < DIVIDE_INSIDE_SLICES) {
        HIP_TRY(launch_ntt_lo_mac(c, level, dsrc(c, ws, 0), keys, vs, n, st, from, prod, rot));
        FinalItem items[KS_MAX_BATCH];
        for (u32 b = 0; b < n; b++) items[b] = FinalItem{nullptr, nullptr, nullptr, outs[b], 1, 0, accs ? accs[b] : nullptr};
        return run_moddown(c, level, ws, n, items, st, merged, true);
    }
    HIP_TRY(launch_ntt_lo_mac(c, level, dsrc(c, ws, 0), keys, vs, n, st, from, prod, rot, nullptr, nullptr, true));
    if (int rc = run_moddown(c, level, ws, n, nullptr, st, merged, true)) return rc;
    const u64* tab = merged ? c->moddown_rs_table(level) : c->d_moddown;
    const u32 kp = merged ? c->k2_pad : c->k_pad;
    const MacDivide div = {(const double*)ws.w, tab + 2 * kp + (size_t)kp * c->num_q, outs, accs};
    HIP_TRY(launch_ntt_lo_mac(c, level, dsrc(c, ws, 0), keys, vs, n, st, from, prod, rot, nullptr, &div));
    return CKKS_OK;
}

// Whether n rotations of one ciphertext's finished digits in a layout take that kernel.  More than four digits, a launch of key_inner_items_kernel per rotation / this,
// in us: sixteen at N = 2^12, 10 + 2 limbs in five digits 133 / 50, 24 + 1 in 24 391 / 215, 2^14, 24 + 3 in eight 356 / 334, 2^16, 24 + 3 in eight 1448 / 1230; four
// 54 / 38, 106 / 77, 144 / 128, 491 / 418; but one, whose workgroups take the digits in turn, 34.4 / 35.3, 57.1 / 61.4, 73.2 / 71.1, 205 / 202.  Up to four digits: see
// DIVIDE_INSIDE_HOISTED.  (ckks_rotate_hoisted keeps a launch per rotation with more than four digits.)
bool hoisted_inside(const ckks_ctx* c, u32 level, u32 n) { return ntt_has_modup(c) && (n > 1 || c->live_digits(level) <= 4); }

// n <= CT_BATCH ciphertexts cts[b] (component stride ct_cstride) rescaled from `level` into outs[b]
int run_rescale(const ckks_ctx* c, u32 level, const u64* const* cts, size_t ct_cstride, u64* const* outs, u32 n, Arena ar,
                hipStream_t st) {
    const size_t N = c->N;
    u64* r = ar.take(2 * (size_t)n * N);
    u64* w = ar.take(2 * (size_t)n * level * N);
    if (!ar.ok()) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for rescale");
    const u32 mid = ntt_mid_rescale(c, level, 2 * n);  // the inverse's second pass inside the converting one
    const u64* last[KS_MAX_BATCH];  // the dropped limb of every component
    for (u32 b = 0; b < n; b++) {
        last[2 * b] = cts[b] + (size_t)level * N;
        last[2 * b + 1] = cts[b] + ct_cstride + (size_t)level * N;
    }
    if (ntt_has_modup(c)) {
        // the rescale as a division by one dropped limb through the fused passes: the inverse transform leaves centred doubles,
        // the forward transform reduces them modulo each remaining limb as it loads and applies (c_i - w_i) q_level^-1 as it stores
        const bool one = ntt_rescale_one_launch(c, level, 2 * n);
        if (!one) HIP_TRY(launch_ntt(c, true, nullptr, 0, r, 1, range_list(0, 1, level), 2 * n, st, last, nullptr, c->d_rescale_prep_f, nullptr, nullptr, mid ? NTT_LO : NTT_BOTH));
        FwdEpilogue ep;
        ep.v = nullptr;
        ep.cinv = c->d_rescale_ep + (size_t)level * 2 * c->num_q;
        ep.mci = c->d_mc;
        ep.E = 0;
        ep.n_out = level;
        ep.num_q = c->num_q;
        ep.use_vl = 1;
        ep.v_cstride = ct_cstride;
        ep.v2_cstride = 0;
        for (u32 b = 0; b < KS_MAX_BATCH; b++) {
            ep.vl2.p[b] = nullptr;
            ep.vl.p[b] = b < n ? cts[b] : nullptr;
            ep.B.it[b] = b < n ? FinalItem{nullptr, nullptr, nullptr, outs[b], 1, 0} : FinalItem{nullptr, nullptr, nullptr, nullptr, 1, 0};
        }
        HIP_TRY(launch_ntt_rescale(c, level, (const double*)r, w, 2 * n, st, &ep, mid, one ? last : nullptr));
        return CKKS_OK;
    }
    HIP_TRY(launch_ntt(c, true, nullptr, 0, r, 1, range_list(0, 1, level), 2 * n, st, last));
    HIP_TRY(launch_rescale_conv(c, level, r, w, 2 * n, st));
    HIP_TRY(launch_ntt(c, false, w, level, w, level, range_list(0, level, 0), 2 * n, st));
    HIP_TRY(launch_rescale_final(c, level, ptr_list(cts, n), ct_cstride, w, out_list(outs, n), n, st));
    return CKKS_OK;
}

// The same for Rescale(ka * x[b] + kb * y[b]) (double-precision contexts with the fused passes): the linear combination is
// formed where it is read, in the inverse transform of the dropped limb and in the division's last step.
int run_rescale_lin(const ckks_ctx* c, u32 level, const u64* const* xs, size_t x_cstride, const u64* ka, const u64* const* ys,
                    size_t y_cstride, const u64* kb, u64* const* outs, u32 n, Arena ar, hipStream_t st) {
    if (!ntt_has_modup(c)) return set_err(c, CKKS_ERR_INVALID_ARG, "internal: fused rescale of a linear combination");
    const size_t N = c->N;
    u64* r = ar.take(2 * (size_t)n * N);
    u64* w = ar.take(2 * (size_t)n * level * N);
    if (!ar.ok()) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for rescale");
    const u32 mid = ntt_mid_rescale(c, level, 2 * n);
    const u64 *last[KS_MAX_BATCH], *last2[KS_MAX_BATCH];
    for (u32 b = 0; b < n; b++) {
        last[2 * b] = xs[b] + (size_t)level * N;
        last[2 * b + 1] = xs[b] + x_cstride + (size_t)level * N;
        last2[2 * b] = ys[b] + (size_t)level * N;
        last2[2 * b + 1] = ys[b] + y_cstride + (size_t)level * N;
    }
    const u64 lin_k[2] = {ka[level], kb[level]};
    HIP_TRY(launch_ntt(c, true, nullptr, 0, r, 1, range_list(0, 1, level), 2 * n, st, last, nullptr, c->d_rescale_prep_f, last2, lin_k, mid ? NTT_LO : NTT_BOTH));
    FwdEpilogue ep;
    ep.v = nullptr;
    ep.cinv = c->d_rescale_ep + (size_t)level * 2 * c->num_q;
    ep.mci = c->d_mc;
    ep.E = 0;
    ep.n_out = level;
    ep.num_q = c->num_q;
    ep.use_vl = 2;
    ep.v_cstride = x_cstride;
    ep.v2_cstride = y_cstride;
    for (u32 b = 0; b < KS_MAX_BATCH; b++) {
        ep.vl.p[b] = b < n ? xs[b] : nullptr;
        ep.vl2.p[b] = b < n ? ys[b] : nullptr;
        ep.B.it[b] = b < n ? FinalItem{nullptr, nullptr, nullptr, outs[b], 1, 0} : FinalItem{nullptr, nullptr, nullptr, nullptr, 1, 0};
    }
    for (u32 i = 0; i < CKKS_MAX_MODULI; i++) {
        ep.ka[i] = i < level ? ka[i] : 0;
        ep.kb[i] = i < level ? kb[i] : 0;
    }
    HIP_TRY(launch_ntt_rescale(c, level, (const double*)r, w, 2 * n, st, &ep, mid));
    return CKKS_OK;
}

// lin (optional): an addend ka * x + kb * y of a ciphertext product, formed on the fly.
struct LinAddend {
    const u64* const* x;
    size_t x_cstride;
    const u64* ka;
    const u64* const* y;
    size_t y_cstride;
    const u64* kb;
};

// n <= ks_batch ciphertext products with relinearisation in contexts with the fused inner product: no tensor-product kernel, d2 =
// a1 (.) b1 is formed as the inverse transform loads it, P d0, P d1 and the own-limb term as the inner product's last terms, all
// from the operands themselves (b, b1: the two components of the second one); dividing the sums by P (merged: by P*q_level) is then the whole product.
int run_product(const ckks_ctx* c, u32 level, const u64* const* a, size_t a_cstride, const u64* const* b, const u64* const* b1, const u64* d_rlk,
                u64* const* outs, u32 n, const KsWs& ws, hipStream_t st, bool merged, const LinAddend* lin = nullptr) {
    const u64 *a1[KS_MAX_BATCH], *keys[KS_MAX_BATCH];
    for (u32 i = 0; i < n; i++) {
        a1[i] = a[i] + a_cstride;
        keys[i] = d_rlk;
    }
    int rc = run_modup(c, level, a1, n, ws, st, true, b1);
    if (rc) return rc;
    MacProduct prod = {a, a1, b, b1};
    if (lin) {
        prod.lin_x = lin->x;
        prod.x_cstride = lin->x_cstride;
        prod.ka = lin->ka;
        prod.lin_y = lin->y;
        prod.y_cstride = lin->y_cstride;
        prod.kb = lin->kb;
    }
    return run_inner_divide(c, level, ws, keys, n, outs, nullptr, st, merged, &prod, nullptr);
}

// n products a[b]*b[b] (as many as ks_batch, CT_BATCH without the fused inner product) with relinearisation (operands possibly at a higher level:
// component strides given); outs[b] = [2][level+1][N]
int run_ctct(const ckks_ctx* c, u32 level, const u64* const* a, size_t a_cstride, const u64* const* b, size_t b_cstride,
             const u64* d_rlk, u64* const* outs, u32 n, Arena ar, hipStream_t st) {
    const size_t N = c->N, L1 = level + 1;
    KsWs ws;
    if (!carve_ks(c, level, n, n, ar, ws)) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for ct-ct multiply");
    const u64* b1[KS_MAX_BATCH];
    for (u32 i = 0; i < n; i++) b1[i] = b[i] + b_cstride;
    if (ntt_has_modup(c)) return run_product(c, level, a, a_cstride, b, b1, d_rlk, outs, n, ws, st, false);
    u64* d0 = ar.take(n * L1 * N);
    u64* d1 = ar.take(n * L1 * N);
    u64* d2 = ar.take(n * L1 * N);
    if (!ar.ok()) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for ct-ct multiply");
    HIP_TRY(launch_tensor(c, level, ptr_list(a, n), a_cstride, ptr_list(b, n), b_cstride, d0, d1, d2, n, nullptr, 0, st));
    const u64 *d2s[CT_BATCH], *keys[CT_BATCH];
    u32 gs[CT_BATCH];
    FinalItem items[CT_BATCH];
    for (u32 i = 0; i < n; i++) {
        d2s[i] = d2 + i * L1 * N;
        keys[i] = d_rlk;
        gs[i] = 1;
        items[i] = FinalItem{d0 + i * L1 * N, d1 + i * L1 * N, nullptr, outs[i], 1, 0};
    }
    int rc = run_modup(c, level, d2s, n, ws, st);
    if (rc) return rc;
    HIP_TRY(launch_key_inner_items(c, level, dsrc(c, ws, 0), keys, gs, nullptr, ws.v, ws.v_b, n, st));
    return run_moddown(c, level, ws, n, items, st);
}

// n <= CT_BATCH products Rescale(a[b]*b[b] + addend[b]) with the relinearisation's ModDown and the rescale merged into
// one division by P*q_level: the tensor product's d0, d1 (plus the addend) enter the extended basis as P times
// themselves inside the inner-product kernel.  addend (optional): n ciphertexts [2][level+1][N], item stride
// add_bstride; in contexts with the fused inner product it is given as lin instead.  outs[b] = [2][level][N].
int run_ctct_merged(const ckks_ctx* c, u32 level, const u64* const* a, size_t a_cstride, const u64* const* b, size_t b_cstride,
                    const u64* addend, size_t add_bstride, const u64* d_rlk, u64* const* outs, u32 n, Arena ar, hipStream_t st,
                    const LinAddend* lin = nullptr) {
    const size_t N = c->N, L1 = level + 1;
    KsWs ws;
    if (!carve_ks(c, level, n, n, ar, ws)) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for ct-ct multiply");
    const bool mac = ntt_has_modup(c);  // the inner product inside the forward transforms' second pass
    if (lin && (!mac || addend)) return set_err(c, CKKS_ERR_INVALID_ARG, "internal: linear addend without the fused inner product");
    if (mac && addend) return set_err(c, CKKS_ERR_INVALID_ARG, "internal: with the fused inner product the addend is given as a linear combination");
    const u64* b1[KS_MAX_BATCH];
    for (u32 i = 0; i < n; i++) b1[i] = b[i] + b_cstride;
    if (mac) return run_product(c, level, a, a_cstride, b, b1, d_rlk, outs, n, ws, st, true, lin);
    u64* d0 = ar.take(n * L1 * N);
    u64* d1 = ar.take(n * L1 * N);
    u64* d2 = ar.take(n * L1 * N);
    if (!ar.ok()) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for ct-ct multiply");
    const u64 *d2s[CT_BATCH], *add0[CT_BATCH], *add1[CT_BATCH];
    u64* vs[CT_BATCH];
    FinalItem items[CT_BATCH];
    HIP_TRY(launch_tensor(c, level, ptr_list(a, n), a_cstride, ptr_list(b, n), b_cstride, d0, d1, d2, n, addend, add_bstride, st));
    for (u32 i = 0; i < n; i++) {
        d2s[i] = d2 + i * L1 * N;
        add0[i] = d0 + i * L1 * N;
        add1[i] = d1 + i * L1 * N;
        vs[i] = ws.v + i * ws.v_b;
        items[i] = FinalItem{nullptr, nullptr, nullptr, outs[i], 1, 0};
    }
    int rc = run_modup(c, level, d2s, n, ws, st);
    if (rc) return rc;
    HIP_TRY(launch_key_inner_ext(c, level, dsrc(c, ws, 0), d_rlk, 1, add0, add1, nullptr, vs, n, st));
    return run_moddown(c, level, ws, n, items, st, true);
}

// whether x^3 = x^2 x and x^4 = x^2 x^2 of n ciphertexts go through the kernels as one batch of products (merged divisions)
bool act_pairs(const ckks_ctx* c, u32 n) { return ntt_has_modup(c) && 2 * n <= ks_batch(c); }
size_t ws_poly_act_in(const ckks_ctx* c, u32 level, u32 n, bool pairs) {
    const size_t N = c->N, one = ws_ctct(c, level, n) + ws_rescale(c, level, n), two = pairs ? ws_ctct(c, level - 1, 2 * n) : 0;
    return blk(2 * (size_t)n * level * N) + 2 * blk(2 * (size_t)n * (level - 1) * N) + blk(2 * (size_t)n * (level - 2) * N) +
           blk(2 * (size_t)n * (level + 1) * N) + (one > two ? one : two);
}
size_t ws_poly_act(const ckks_ctx* c, u32 level, u32 n) { return ws_poly_act_in(c, level, n, act_pairs(c, n)); }
// ciphertexts of a batch of the activation with merged divisions, of n_ct in all: sixteen together leave no room for the pairs of products.  Two
// streams with pairs / together in us, 9 / 12 / 16: N = 2^12, 5 + 2 limbs (0.03 M coefficients) 211 / 161, 216 / 165, 226 / 174, 7 + 3 204 / 181, 211 / 187,
// 219 / 197, 10 + 4 (0.06 M) 206 / 205, 219 / 225, 226 / 243, 2^13, 5 + 2 (0.06 M) 209 / 181, 216 / 187, 220 / 212, 2^12, 14 + 6 (0.08 M) 206 / 242, 225 / 265, 268 / 327,
// 2^14, 7 + 3 (0.16 M) 264 / 312, 290 / 353, 348 / 415; in two batches, 24: 2^12, 5 + 2 269 / 321, 7 + 3 307 / 362, 2^14, 7 + 3 587 / 694
u32 act_batch(const ckks_ctx* c, u32 level, u32 n_ct) {
    return n_ct > CT_BATCH && n_ct <= KS_MAX_BATCH && together(c, level, (size_t)1 << 16) ? KS_MAX_BATCH : CT_BATCH;
}

// The convolution with one division by P per output channel: every aligned copy stays on the extended
// basis Q_level P (inner product + P * sigma_g(c0), times the tap's mask), the sum over (input channel,
// tap) is taken there, and only the C_out sums go through ModDown and the rescale.  gs: Galois
// elements of the nine taps (1 = no rotation); masks [9][E][N], w_res [C_out][C_in][9][E].
// per-lane scratch of the deferred convolution: the key-switch buffers, a batch of un-rescaled outputs, the rescale's scratch
size_t ws_conv_lane(const ckks_ctx* c, u32 level, u32 kb) {
    return ws_ks(c, level, kb, kb) + blk((size_t)kb * 2 * (level + 1) * c->N) + ws_rescale(c, level, CT_BATCH);
}
// Two streams / together in us, merged: 9 -> 4 channels at N = 2^12, 4 + 2 limbs (0.02 M coefficients) 94 / 63, 24 + 8 (0.13 M) 183 / 169, 16 -> 16 162 / 108,
// 372 / 359, 16 -> 32 with 7 + 3 limbs 232 / 210, 24 + 8 461 / 455; more than sixteen inputs: 4 + 2 limbs 17 -> 4 116 / 107, 24 -> 8 137 / 144, 64 -> 64 411 / 399,
// 7 + 3 (0.04 M) 162 / 171, 217 / 227, 565 / 586, 24 + 8 296 / 314, 429 / 443, 1182 / 1239; only the divisions in two batches, 3 -> 12: 7 + 3 97 / 55, 2^14, 14 + 6
// (0.33 M) 259 / 248, 24 + 8 (0.52 M) 388 / 382, but with a rescale of its own 2^12, 24 + 8 158 / 158, 2^13, 14 + 6 (0.16 M) 177 / 185, 24 + 8 255 / 261
bool conv_together(const ckks_ctx* c, const he_conv_desc* d) {
    const bool one_division = d->c_in <= CT_BATCH && d->c_out <= KS_MAX_BATCH && d->alignment == HE_CONV_DEFERRED_MERGED;
    return together(c, d->level, d->c_in > KS_MAX_BATCH ? (size_t)1 << 15 : (one_division ? (size_t)1 << 19 : (size_t)1 << 17));
}
// channels of a batch, and whether two batches are in flight when there is more than one
u32 conv_batch(const ckks_ctx* c, const he_conv_desc* d) { return conv_together(c, d) && (d->c_in > CT_BATCH || d->c_out > CT_BATCH) ? KS_MAX_BATCH : CT_BATCH; }

// Whether the inner products and the weighted sum of a deferred convolution are one kernel that stores no aligned copies (launch_key_inner_sum):
// with up to four outputs, whose sums a thread holds; on small rings with up to eight, in two groups that form the inner products twice.  Merged
// convolutions, copies and sum / one kernel in us: N = 2^12, 5 + 2 limbs, 1 -> 1 37.9 / 33.5, 4 -> 4 51.6 / 44.4, 16 -> 4 101.8 / 74.0, 64 -> 1 352 / 224, 8 -> 8 69.4 / 62.0,
// 2^13, 5 + 2, 3 -> 2 56.9 / 44.8, 2^14, 12 + 4, 4 -> 4 158 / 133, 2^15, 9 + 3, 16 -> 4 675 / 510, 2^16, 24 + 8, 1 -> 1 453 / 351, 5 -> 3 1196 / 934, 16 -> 1 3069 / 2017,
// 64 -> 1 11770 / 7420; eight outputs above 2^15 coefficients 2^12, 10 + 5, 1 -> 8 50.7 / 54.2, 2^16, 24 + 8, 8 -> 8 2027 / 2303
bool conv_summed(const ckks_ctx* c, const he_conv_desc* d) {
    if (!c->small_q || c->live_digits(d->level) > 4 || c->N % 64) return false;
    return d->c_out <= 4 || (d->c_out <= 8 && (size_t)c->ext_limbs(d->level) * c->N <= (size_t)1 << 15);
}

// sets of scratch that a deferred convolution can use: two where batches run side by side (one kernel's sums over the channels go into the same place)
u32 conv_lanes(const ckks_ctx* c, const he_conv_desc* d) {
    return (!conv_summed(c, d) && !conv_together(c, d) && c->side && (d->c_in > CT_BATCH || d->c_out > CT_BATCH)) ? 2 : 1;
}
// words of its aligned copies on the extended basis, and of the scratch of the kernel that sums them: none where they are not stored
size_t conv_copies(const ckks_ctx* c, const he_conv_desc* d) {
    return conv_summed(c, d) ? 0 : (size_t)d->c_in * 9 * 2 * c->ext_limbs(d->level) * c->N;
}
size_t conv_sum_scratch(const ckks_ctx* c, const he_conv_desc* d) {
    return conv_summed(c, d) ? 0 : weighted_sum_scratch_elems(c, c->ext_limbs(d->level), d->c_in * 9, d->c_out);
}

// the schedules that divide every rotation by P, kb of them at a time
size_t ws_conv_rotated(const ckks_ctx* c, const he_conv_desc* d, u32 kb) {
    const size_t N = c->N, L1 = d->level + 1;
    return ws_ks(c, d->level, CT_BATCH, kb) + blk((size_t)d->c_in * 9 * 2 * L1 * N) + blk((size_t)d->c_out * 2 * L1 * N) +
           blk(weighted_sum_scratch_elems(c, (u32)L1, d->c_in * 9, d->c_out)) + ws_rescale(c, d->level, CT_BATCH) +
           (d->alignment == HE_CONV_ALIGN_FOUR_KEYS ? 2 * blk((size_t)CT_BATCH * 2 * L1 * N) : 0);
}

int conv_deferred(const ckks_ctx* c, const he_conv_desc* d, const u32* gs, const uint64_t* const* h_d_in,
                  const ckks_key* const* rot_keys, const u64* masks, const u64* w_res, uint64_t* const* h_d_out, void* d_ws,
                  size_t ws_bytes, hipStream_t st0) {
    const u32 level = d->level, E = c->ext_limbs(level);
    const bool merged = d->alignment == HE_CONV_DEFERRED_MERGED;  // ModDown and rescale of the sums as one division
    const size_t N = c->N, L1 = level + 1, ct_elems = 2 * L1 * N, x_elems = 2 * (size_t)E * N;
    Arena ar(d_ws, ws_bytes);
    u64* xs = ar.take(conv_copies(c, d));
    u64* acc = ar.take((size_t)d->c_out * x_elems);
    u64* wscratch = ar.take(conv_sum_scratch(c, d));
    // Batches of input channels (alignment) and of output channels (division) are independent: with room for two sets of
    // scratch every other batch runs on the library's side stream, between a fork and a join on the caller's stream.
    u32 kb = conv_batch(c, d);
    if (ar.ok() && ar.used + ws_conv_lane(c, level, kb) > ar.cap) kb = CT_BATCH;  // in a smaller workspace
    const size_t lane_bytes = ws_conv_lane(c, level, kb);
    const u32 n_lanes = (conv_lanes(c, d) == 2 && c->side_stream() && ar.ok() && ar.used + 2 * lane_bytes <= ar.cap) ? 2 : 1;
    struct Lane {
        KsWs ws;
        u64* tmp;
        Arena rest;
        hipStream_t st;
    };
    Lane lanes[2] = {{KsWs{}, nullptr, Arena(nullptr, 0), st0}, {KsWs{}, nullptr, Arena(nullptr, 0), c->side}};
    bool ok = ar.ok();
    for (u32 l = 0; l < n_lanes && ok; l++) {
        ok = carve_ks(c, level, kb, kb, ar, lanes[l].ws);
        lanes[l].tmp = ar.take((size_t)kb * ct_elems);
        u64* r = ar.take(ws_rescale(c, level, CT_BATCH) / sizeof(u64));
        lanes[l].rest = Arena(r, ws_rescale(c, level, CT_BATCH));
        ok = ok && ar.ok();
    }
    if (!ok) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for the convolution");
    // the aligned copies are stored term-innermost when the fused inner product can write them that way
    const bool fused_taps = c->live_digits(level) <= 4;
    const XLayout xl = (fused_taps && N % 64 == 0) ? XLayout::tiled((size_t)d->c_in * 9, N) : XLayout::classic(E, N);
    const bool summed = conv_summed(c, d);
    bool forked = false;
    auto fork = [&]() -> int {
        if (n_lanes < 2 || forked) return CKKS_OK;
        HIP_TRY(hipEventRecord(c->ev_fork, st0));
        HIP_TRY(hipStreamWaitEvent(c->side, c->ev_fork, 0));
        forked = true;
        return CKKS_OK;
    };
    auto join = [&](int rc) -> int {  // also on the error paths: the caller's stream never runs ahead of the side stream
        if (!forked) return rc;
        forked = false;
        hipError_t e = hipEventRecord(c->ev_join, c->side);
        if (e == hipSuccess) e = hipStreamWaitEvent(st0, c->ev_join, 0);
        return (e != hipSuccess && rc == CKKS_OK) ? set_hip_err(c, e) : rc;
    };
    auto align_batch = [&](u32 c0, const Lane& L) -> int {
        const KsWs& ws = L.ws;
        hipStream_t st = L.st;
        const u32 n = d->c_in - c0 < kb ? d->c_in - c0 : kb;
        const u64 *in[KS_MAX_BATCH], *c1s[KS_MAX_BATCH];
        for (u32 b = 0; b < n; b++) {
            in[b] = (const u64*)h_d_in[c0 + b];
            c1s[b] = in[b] + L1 * N;
        }
        int rc = run_modup(c, level, c1s, n, ws, st);
        if (rc) return rc;
        if (summed) {
            const u64* skeys[9];
            for (u32 t = 0; t < 9; t++) skeys[t] = gs[t] == 1 ? nullptr : rot_keys[t]->d_key;
            HIP_TRY(launch_key_inner_sum(c, level, dsrc(c, ws, 0), skeys, gs, masks, in, n, w_res, c0, d->c_in, d->c_out, acc, st));
            return CKKS_OK;
        }
        // taps without a rotation (the centre) are a product with the mask; all the others go through one launch
        const u64 *tkeys[8], *tmasks[8], *centre_mask = nullptr;
        u32 tg[8], ttap[8], n_taps = 0, centre_tap = 0, n_centre = 0;
        for (u32 t = 0; t < 9; t++) n_centre += gs[t] == 1 ? 1 : 0;
        for (u32 t = 0; t < 9; t++) {
            const u64* mask = masks + (size_t)t * E * N;
            if (gs[t] == 1) {
                if (fused_taps && n_centre == 1) {  // the tap without a rotation rides on the fused launch
                    centre_mask = mask;
                    centre_tap = t;
                } else {
                    for (u32 b = 0; b < n; b++) HIP_TRY(launch_centre_ext(c, level, mask, in[b], xs, xl, (c0 + b) * 9 + t, st));
                }
                continue;
            }
            tkeys[n_taps] = rot_keys[t]->d_key;
            tmasks[n_taps] = mask;
            tg[n_taps] = gs[t];
            ttap[n_taps++] = t;
        }
        if (fused_taps) {
            for (u32 b0 = 0; b0 < n; b0 += CT_BATCH)
                HIP_TRY(launch_key_inner_taps(c, level, dsrc(c, ws, b0), tkeys, tg, tmasks, ttap, n_taps, in + b0, xs, xl, (c0 + b0) * 9, 9,
                                              n - b0 < CT_BATCH ? n - b0 : CT_BATCH, st, centre_mask, centre_tap));
        } else {  // many digits: one launch per tap (classic layout: every term is a [2][E][N] array)
            for (u32 i = 0; i < n_taps; i++)
                for (u32 b0 = 0; b0 < n; b0 += CT_BATCH) {
                    const u32 m = n - b0 < CT_BATCH ? n - b0 : CT_BATCH;
                    u64* outs[CT_BATCH];
                    for (u32 b = 0; b < m; b++) outs[b] = xs + ((size_t)(c0 + b0 + b) * 9 + ttap[i]) * x_elems;
                    HIP_TRY(launch_key_inner_ext(c, level, dsrc(c, ws, b0), tkeys[i], tg[i], in + b0, nullptr, tmasks[i], outs, m, st));
                }
        }
        return CKKS_OK;
    };
    int rc;
    if (d->c_in > kb && (rc = fork())) return rc;
    for (u32 c0 = 0, k = 0; c0 < d->c_in; c0 += kb, k++)
        if ((rc = align_batch(c0, lanes[forked ? k & 1 : 0]))) return join(rc);
    if ((rc = join(CKKS_OK))) return rc;
    if (!summed) HIP_TRY(launch_weighted_sum(c, level, true, xs, xl, d->c_in * 9, w_res, d->c_out, acc, wscratch, d->weight_bits, st0));
    if (d->c_out > kb && (rc = fork())) return rc;
    for (u32 o0 = 0, k = 0; o0 < d->c_out; o0 += kb, k++) {
        const Lane& L = lanes[forked ? k & 1 : 0];
        const u32 n = d->c_out - o0 < kb ? d->c_out - o0 : kb;
        KsWs wd = L.ws;
        wd.v = acc + (size_t)o0 * x_elems;  // the sums take the place of a batch of inner products
        wd.v_b = x_elems;
        FinalItem items[KS_MAX_BATCH];
        const u64* ins[KS_MAX_BATCH];
        u64* outs[KS_MAX_BATCH];
        for (u32 b = 0; b < n; b++) {
            ins[b] = L.tmp + (size_t)b * ct_elems;
            outs[b] = (u64*)h_d_out[o0 + b];
            items[b] = FinalItem{nullptr, nullptr, nullptr, merged ? outs[b] : L.tmp + (size_t)b * ct_elems, 1, 0};
        }
        if ((rc = run_moddown(c, level, wd, n, items, L.st, merged))) return join(rc);
        for (u32 b0 = 0; b0 < n && !merged; b0 += CT_BATCH)
            if ((rc = run_rescale(c, level, ins + b0, L1 * N, outs + b0, n - b0 < CT_BATCH ? n - b0 : CT_BATCH, L.rest, L.st))) return join(rc);
    }
    return join(CKKS_OK);
}

// Inner products of n_taps rotations of the same n ciphertexts, whose digits are in ws: P sigma_g(c0) + <sigma_g(digits), key> of
// tap i and ciphertext b at ws.v + (pos[i] + b) * ws.v_b.  One launch that reads the digits once for its taps where their count
// allows it, else one per tap.
hipError_t rotated_inner(const ckks_ctx* c, u32 level, const KsWs& ws, const u64* const* cts, u32 n, const u64* const* keys, const u32* gs,
                         const u32* pos, u32 n_taps, hipStream_t st) {
    if (c->live_digits(level) <= 4) {
        for (u32 i0 = 0; i0 < n_taps; i0 += 8) {
            const u32 m = n_taps - i0 < 8 ? n_taps - i0 : 8;
            if (hipError_t e = launch_key_inner_taps(c, level, dsrc(c, ws, 0), keys + i0, gs + i0, nullptr, pos + i0, m, cts, ws.v,
                                                     XLayout::classic(c->ext_limbs(level), c->N), 0, 1, n, st); e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    for (u32 i = 0; i < n_taps; i++) {
        const u64* k[CT_BATCH];
        u32 g[CT_BATCH];
        for (u32 b = 0; b < n; b++) k[b] = keys[i], g[b] = gs[i];
        if (hipError_t e = launch_key_inner_items(c, level, dsrc(c, ws, 0), k, g, cts, ws.v + (size_t)pos[i] * ws.v_b, ws.v_b, n, st); e != hipSuccess) return e;
    }
    return hipSuccess;
}

// n <= ks_batch ciphertexts srcs[b] ([2][level+1][N]) rotated, outs[b] = Rot(srcs[b]) with keys[b] / gal[b] ([2][level+1][N], no
// overlap).  Where a key switch takes its inner product inside the forward transforms' second pass, the permuted polynomial is
// decomposed (the digits of a permuted polynomial are the permuted digits), gathered as the inverse transform loads it: no
// kernel for the automorphism, the extended digits are never written in evaluation form.  Elsewhere one inner-product launch for all of them reads
// the digits through sigma (a key streams once for neighbouring items that share it).  Either adds P sigma(c0), so that the
// division by P is the rotation.  At N = 2^16, two to four limbs, eight rotations in us, digits read through sigma / permuted: 143 / 118.
// accs (optional): outs[b] = Rot(srcs[b]) + accs[b], the sum formed by the division's last step.
int run_rotate_batch(const ckks_ctx* c, u32 level, u32 n, const u64* const* srcs, const ckks_key* const* keys, const u32* gal,
                     u64* const* outs, const KsWs& ws, hipStream_t st, const u64* const* accs = nullptr) {
    const size_t L1 = level + 1;
    const bool mac = ntt_has_modup(c);
    const u64 *c1s[KS_MAX_BATCH], *kd[KS_MAX_BATCH];
    FinalItem items[KS_MAX_BATCH];
    for (u32 b = 0; b < n; b++) {
        c1s[b] = srcs[b] + L1 * c->N;
        kd[b] = keys[b]->d_key;
        items[b] = FinalItem{nullptr, nullptr, nullptr, outs[b], 1, 0, accs ? accs[b] : nullptr};
    }
    int rc = run_modup(c, level, c1s, n, ws, st, mac, nullptr, mac ? gal : nullptr);
    if (rc) return rc;
    if (mac) {
        const MacRotate rot = {srcs, gal};
        return run_inner_divide(c, level, ws, kd, n, outs, accs, st, false, nullptr, &rot);
    }
    HIP_TRY(launch_key_inner_items(c, level, dsrc(c, ws, 0), kd, gal, srcs, ws.v, ws.v_b, n, st));
    return run_moddown(c, level, ws, n, items, st);
}

// out = sum_b Rot(srcs[b] (.) mask) + add (.) add_mask for n <= ks_batch ciphertexts (mask, add, add_mask optional), where a key switch takes its
// inner product inside the forward transforms' second pass: the products with the mask are formed as they are read, the inner products and, past
// each item's rounding, the divisions by P are added up (launch_ntt_moddown_sum).  out may be add.
int run_rotate_sum(const ckks_ctx* c, u32 level, u32 n, const u64* const* srcs, const ckks_key* const* keys, const u32* gal, const u64* mask, const u64* add,
                   const u64* add_mask, u64* out, const KsWs& ws, hipStream_t st) {
    const u64 *c1s[KS_MAX_BATCH], *kd[KS_MAX_BATCH], *masks[KS_MAX_BATCH];
    u64* vs[KS_MAX_BATCH];
    for (u32 b = 0; b < n; b++) {
        c1s[b] = srcs[b] + (size_t)(level + 1) * c->N;
        kd[b] = keys[b]->d_key;
        masks[b] = mask;
        vs[b] = ws.v + b * ws.v_b;
    }
    if (int rc = run_modup(c, level, c1s, n, ws, st, true, mask ? masks : nullptr, gal)) return rc;
    for (u32 b = 0; b < n; b++) ws.own[b] = c1s[b];  // (their products with the mask are formed where they are read)
    const MacRotate rot = {srcs, gal, mask};
    u32 n_part = 0;
    HIP_TRY(launch_ntt_lo_mac(c, level, dsrc(c, ws, 0), kd, vs, n, st, dropped_from(level, false), nullptr, &rot, &n_part));
    HIP_TRY(launch_ntt_moddown_sum(c, level, ws.v, ws.v_b, n, n_part, ws.w, FinalItem{nullptr, nullptr, add_mask, out, 1, 0, add}, st));
    return CKKS_OK;
}

// Whether sums of rotations share a division: with less to do, the items that one workgroup takes in turn are a longer chain than the launches that
// go.  By coefficients of the extended basis, one by one / together in us: merges at N = 2^12, 7 + 4 limbs, eight (0.04 M) 53.6 / 54.6, 2^13, 7 + 3, five
// (0.08 M) 60.5 / 62.7, 2^14, 6 + 3, eight (0.15 M) 79 / 73, 2^13, 14 + 7, eight (0.15 M) 82.5 / 76, 2^12, 24 + 8, eight (0.12 M) 78.7 / 73, 2^16, 19 + 8, four (1.8 M) 352 / 283;
// fully connected layers 2^12, 7 + 3 291 / 300, 2^13, 8 + 3 402 / 415, 2^14, 6 + 3 (0.10 M) 426 / 423, 16 + 8 (0.18 M) 765 / 749, 2^16, 24 + 8 2131 / 2080
bool sums_together(const ckks_ctx* c, u32 level) { return ntt_has_modup(c) && (size_t)c->ext_limbs(level) * c->N >= (size_t)3 << 15; }

// rotations of a merge of g blocks that share their launches, at most `most`
u32 merge_batch(u32 g, u32 most) { return g - 1 < most ? (g > 1 ? g - 1 : 1) : most; }
size_t ws_merge_in(const ckks_ctx* c, u32 level, u32 g, u32 nb) {
    const size_t N = c->N, L1 = level + 1;
    return ws_ks(c, level, nb, nb) + (sums_together(c, level) ? 0 : 2 * blk((size_t)g * 2 * L1 * N)) + blk(2 * L1 * N) + ws_rescale(c, level, 1);
}
size_t ws_merge(const ckks_ctx* c, u32 level, u32 g) { return ws_merge_in(c, level, g, merge_batch(g, ks_batch(c))); }

// out = Rescale( sum_{i<g} Rot(cts[i] (.) mask, -i*sts) ), g <= KS_MAX_BATCH; keys[i] / gal[i] for i >= 1 (validated by the caller)
int run_merge(const ckks_ctx* c, const u64* const* cts, u32 g, u32 level, const u64* mask, const ckks_key* const* keys, const u32* gal,
              u64* out, Arena ar, hipStream_t st) {
    const size_t N = c->N, L1 = level + 1, ct_elems = 2 * L1 * N;
    u32 nb = merge_batch(g, ks_batch(c));
    if (ar.used + ws_merge_in(c, level, g, nb) > ar.cap) nb = merge_batch(g, CT_BATCH);  // in a smaller workspace
    KsWs ws;
    bool ok = carve_ks(c, level, nb, nb, ar, ws);
    const bool sums = sums_together(c, level);                      // run_rotate_sum
    u64* masked = sums ? nullptr : ar.take((size_t)g * ct_elems);   // C_i (.) M
    u64* rotated = sums ? nullptr : ar.take((size_t)g * ct_elems);  // Rot(C_i (.) M, -i*sts), i >= 1
    u64* total = ar.take(ct_elems);
    if (!ok || !ar.ok() || ar.used + ws_rescale(c, level, 1) > ar.cap)
        return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for the merge");
    const u64* in = total;
    if (sums) {
        for (u32 i0 = 1; i0 < g; i0 += nb) {
            const u32 n = g - i0 < nb ? g - i0 : nb;
            if (int rc = run_rotate_sum(c, level, n, cts + i0, keys + i0, gal + i0, mask, i0 == 1 ? cts[0] : total, i0 == 1 ? mask : nullptr, total, ws, st))
                return rc;
        }
        if (g == 1) HIP_TRY(launch_mask_mul(c, level, &mask, cts, &total, 1, st));
        return run_rescale(c, level, &in, L1 * N, &out, 1, ar.rest(), st);
    }
    const u64* masks[KS_MAX_BATCH];
    u64* mouts[KS_MAX_BATCH];
    for (u32 i = 0; i < g; i++) masks[i] = mask, mouts[i] = masked + i * ct_elems;
    HIP_TRY(launch_mask_mul(c, level, masks, cts, mouts, g, st));
    // blocks 1..g-1: every block has its own key; a batch shares the decomposition and ModDown launches
    for (u32 i0 = 1; i0 < g; i0 += nb) {
        const u32 n = g - i0 < nb ? g - i0 : nb;
        const u64* srcs[KS_MAX_BATCH];
        u64* outs[KS_MAX_BATCH];
        for (u32 b = 0; b < n; b++) {
            srcs[b] = masked + (i0 + b) * ct_elems;
            outs[b] = rotated + (i0 + b) * ct_elems;
        }
        if (int rc = run_rotate_batch(c, level, n, srcs, keys + i0, gal + i0, outs, ws, st)) return rc;
    }
    const u64* terms[KS_MAX_BATCH];
    terms[0] = masked;
    for (u32 i = 1; i < g; i++) terms[i] = rotated + i * ct_elems;
    HIP_TRY(launch_ct_sum(c, level, ptr_list(terms, g), g, total, st));
    return run_rescale(c, level, &in, L1 * N, &out, 1, ar.rest(), st);
}

// Slot re-layout with two rotations per element, for the n_ct ciphertexts of a channel vector (level `level`):
//   outs[b] = sum_h Rot( Rescale( sum_l masks[h*n_lo+l] (.) Rot(cts[b], lo_l) ), hi_h )        ([2][level][N])
// g_lo / g_hi: Galois elements (1 = no rotation, key ignored); masks: device pointers [level+1][N] or null; every h has
// at least one mask (validated by the caller).  First rotations: one decomposition per ciphertext, every key read once per
// batch of up to CT_BATCH (ciphertext, offset) pairs; second rotations batched the same way over (h, ciphertext).
// the key-switch buffers of both levels, `most` (ciphertext, offset) pairs at a time
size_t ws_relayout_ks(const ckks_ctx* c, u32 level, u32 most) {
    const size_t lo = ws_ks(c, level, CT_BATCH, most), hi = ws_ks(c, level - 1, most, most);
    return lo > hi ? lo : hi;
}
// words of the second rotations' results: one ciphertext's that share a division are not stored
size_t relayout_rotated(const ckks_ctx* c, u32 level, u32 n_ct, u32 n_hi) {
    const size_t nb = n_ct < CT_BATCH ? n_ct : CT_BATCH;
    return n_ct == 1 && sums_together(c, level - 1) ? 0 : nb * n_hi * 2 * (size_t)level * c->N;
}
size_t ws_relayout_in(const ckks_ctx* c, u32 level, u32 n_ct, u32 n_lo, u32 n_hi, u32 most) {
    const size_t N = c->N, ctl = 2 * (size_t)(level + 1) * N, ctl1 = 2 * (size_t)level * N;
    const size_t nb = n_ct < CT_BATCH ? n_ct : CT_BATCH;
    return blk(nb * n_lo * ctl) + blk(nb * n_hi * ctl) + blk(nb * n_hi * ctl1) + blk(relayout_rotated(c, level, n_ct, n_hi)) + ws_relayout_ks(c, level, most) + ws_rescale(c, level, CT_BATCH);
}
size_t ws_relayout(const ckks_ctx* c, u32 level, u32 n_ct, u32 n_lo, u32 n_hi) {
    return ws_relayout_in(c, level, n_ct, n_lo, n_hi, ks_batch(c));
}

int run_relayout(const ckks_ctx* c, u32 level, u32 n_ct, const u64* const* cts, u32 n_lo, const ckks_key* const* lo_keys, const u32* g_lo,
                 u32 n_hi, const ckks_key* const* hi_keys, const u32* g_hi, const u64* const* masks, u64* const* outs, Arena ar,
                 hipStream_t st) {
    const size_t N = c->N, ctl = 2 * (size_t)(level + 1) * N, ctl1 = 2 * (size_t)level * N;
    const u32 nb_max = n_ct < CT_BATCH ? n_ct : CT_BATCH, l1 = level - 1;
    u64* R = ar.take((size_t)nb_max * n_lo * ctl);      // Rot(ct_b, lo_l)
    u64* Vacc = ar.take((size_t)nb_max * n_hi * ctl);   // masked sums before their rescale
    u64* V = ar.take((size_t)nb_max * n_hi * ctl1);     // level-1
    u64* Vrot = ar.take(relayout_rotated(c, level, n_ct, n_hi));
    u32 kb = ks_batch(c);  // rotations at a time
    if (ar.ok() && ar.used + ws_relayout_ks(c, level, kb) + ws_rescale(c, level, CT_BATCH) > ar.cap) kb = CT_BATCH;  // in a smaller workspace
    const size_t ks_bytes = ws_relayout_ks(c, level, kb);
    u64* ks_region = ar.take(ks_bytes / sizeof(u64));
    if (!ar.ok() || ar.used + ws_rescale(c, level, CT_BATCH) > ar.cap)
        return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for the re-layout");
    KsWs ws;
    auto ks_at = [&](u32 lv, u32 n_dig) {  // the key-switch buffers are carved again for the lower level
        Arena sub(ks_region, ks_bytes);
        return carve_ks(c, lv, n_dig, kb, sub, ws);
    };
    int rc;
    for (u32 c0 = 0; c0 < n_ct; c0 += CT_BATCH) {
        const u32 n = n_ct - c0 < CT_BATCH ? n_ct - c0 : CT_BATCH;
        auto r_at = [&](u32 b, u32 l) { return R + ((size_t)b * n_lo + l) * ctl; };
        // first rotations
        ks_at(level, CT_BATCH);
        const u64* c1s[CT_BATCH];
        for (u32 b = 0; b < n; b++) c1s[b] = cts[c0 + b] + (size_t)(level + 1) * N;
        if ((rc = run_modup(c, level, c1s, n, ws, st))) return rc;
        const u32 per = kb / n;  // offsets per ModDown batch
        for (u32 la = 0; la < n_lo; la += per) {
            FinalItem items[KS_MAX_BATCH];
            const u64* tkeys[KS_MAX_BATCH];
            u32 tg[KS_MAX_BATCH], pos[KS_MAX_BATCH], nt = 0, nk = 0;
            for (u32 l = la; l < n_lo && l < la + per; l++) {
                if (g_lo[l] == 1) {
                    for (u32 b = 0; b < n; b++) HIP_TRY(launch_copy(cts[c0 + b], r_at(b, l), ctl, st));
                    continue;
                }
                tkeys[nt] = lo_keys[l]->d_key;
                tg[nt] = g_lo[l];
                pos[nt++] = nk;
                for (u32 b = 0; b < n; b++) items[nk++] = FinalItem{nullptr, nullptr, nullptr, r_at(b, l), 1, 0};
            }
            if (n == 1 && nt && hoisted_inside(c, level, nt)) {
                const u64* same[KS_MAX_BATCH];
                u64* to[KS_MAX_BATCH];
                for (u32 i = 0; i < nt; i++) same[i] = cts[c0], to[i] = items[i].out;
                const MacRotate rot = {same, tg, nullptr, true};
                if ((rc = run_inner_divide(c, level, ws, tkeys, nt, to, nullptr, st, false, nullptr, &rot))) return rc;
                continue;
            }
            HIP_TRY(rotated_inner(c, level, ws, cts + c0, n, tkeys, tg, pos, nt, st));
            if (nk && (rc = run_moddown(c, level, ws, nk, items, st))) return rc;
        }
        // masked sums, one per (ciphertext, h), and their rescale
        HIP_TRY(launch_relayout_mac(c, level, false, R, masks, Vacc, n, n_lo, n_hi, st));
        const u32 n_v = n * n_hi;
        for (u32 i0 = 0; i0 < n_v; i0 += CT_BATCH) {
            const u32 m = n_v - i0 < CT_BATCH ? n_v - i0 : CT_BATCH;
            const u64* pv[CT_BATCH];
            u64* ov[CT_BATCH];
            for (u32 i = 0; i < m; i++) {
                pv[i] = Vacc + (size_t)(i0 + i) * ctl;
                ov[i] = V + (size_t)(i0 + i) * ctl1;
            }
            if ((rc = run_rescale(c, level, pv, (size_t)(level + 1) * N, ov, m, ar.rest(), st))) return rc;
        }
        // second rotations, ordered by h so that the ciphertexts of a batch share each key
        ks_at(l1, kb);
        const u64* srcs[KS_MAX_BATCH];
        const ckks_key* ks[KS_MAX_BATCH];
        u32 gs[KS_MAX_BATCH], nk = 0;
        u64* dsts[KS_MAX_BATCH];
        if (n == 1 && sums_together(c, l1)) {  // (several ciphertexts share each key instead)
            const u64* terms[KS_MAX_BATCH];
            u64* out = outs[c0];
            const u64* add = nullptr;  // the blocks that stay where they are
            u32 nt = 0;
            for (u32 h = 0; h <= n_hi; h++) {
                if (h < n_hi && g_hi[h] == 1) terms[nt++] = V + (size_t)h * ctl1;
                if (nt == KS_MAX_BATCH || (h == n_hi && nt > 1) || (h == n_hi && nt == 1 && n_hi == 1)) {
                    HIP_TRY(launch_ct_sum(c, l1, ptr_list(terms, nt), nt, out, st));
                    add = terms[0] = out;
                    nt = 1;
                } else if (h == n_hi && nt == 1) {
                    add = terms[0];
                }
            }
            for (u32 h = 0; h <= n_hi; h++) {
                if (h < n_hi && g_hi[h] != 1) {
                    srcs[nk] = V + (size_t)h * ctl1;
                    ks[nk] = hi_keys[h];
                    gs[nk++] = g_hi[h];
                }
                if (nk == kb || (h == n_hi && nk)) {
                    if ((rc = run_rotate_sum(c, l1, nk, srcs, ks, gs, nullptr, add, nullptr, out, ws, st))) return rc;
                    add = out;
                    nk = 0;
                }
            }
            continue;
        }
        for (u32 h = 0; h < n_hi; h++) {
            if (g_hi[h] == 1) continue;
            for (u32 b = 0; b < n; b++) {
                srcs[nk] = V + ((size_t)b * n_hi + h) * ctl1;
                dsts[nk] = Vrot + ((size_t)b * n_hi + h) * ctl1;
                ks[nk] = hi_keys[h];
                gs[nk++] = g_hi[h];
                if (nk == kb) {
                    if ((rc = run_rotate_batch(c, l1, nk, srcs, ks, gs, dsts, ws, st))) return rc;
                    nk = 0;
                }
            }
        }
        if (nk && (rc = run_rotate_batch(c, l1, nk, srcs, ks, gs, dsts, ws, st))) return rc;
        // the sums; the running sum is one of the terms of every launch after the first
        for (u32 b = 0; b < n; b++) {
            u64* out = outs[c0 + b];
            for (u32 h = 0; h < n_hi;) {
                const u64* terms[KS_MAX_BATCH];
                u32 nt = 0;
                if (h) terms[nt++] = out;
                for (; h < n_hi && nt < KS_MAX_BATCH; h++) terms[nt++] = (g_hi[h] == 1 ? V : Vrot) + ((size_t)b * n_hi + h) * ctl1;
                HIP_TRY(launch_ct_sum(c, l1, ptr_list(terms, nt), nt, out, st));
            }
        }
    }
    return CKKS_OK;
}

// The same re-layout with the divisions by P deferred past the sums (masks on the extended basis, [level+1+k][N]):
//   X_l = (P sigma(c0) + v0, v1) for the first rotations (inner products only), V_h = (sum_l M[h][l] (.) X_l) / (P q_level),
//   out = ModDown( sum_h X'_h ) with X'_h the pre-division copy of Rot(V_h, hi_h).
size_t ws_relayout_deferred(const ckks_ctx* c, u32 level, u32 n_ct, u32 n_lo, u32 n_hi) {
    const size_t N = c->N, xel = 2 * (size_t)c->ext_limbs(level) * N, xel1 = 2 * (size_t)c->ext_limbs(level - 1) * N, ctl1 = 2 * (size_t)level * N;
    const size_t nb = n_ct < CT_BATCH ? n_ct : CT_BATCH;
    return blk(nb * n_lo * xel) + blk(nb * n_hi * xel) + blk(nb * n_hi * ctl1) + blk(nb * n_hi * xel1) + blk(nb * xel1) +
           ws_ks(c, level, CT_BATCH, CT_BATCH);
}

int run_relayout_deferred(const ckks_ctx* c, u32 level, u32 n_ct, const u64* const* cts, u32 n_lo, const ckks_key* const* lo_keys,
                          const u32* g_lo, u32 n_hi, const ckks_key* const* hi_keys, const u32* g_hi, const u64* const* masks,
                          u64* const* outs, Arena ar, hipStream_t st) {
    const u32 l1 = level - 1, nb_max = n_ct < CT_BATCH ? n_ct : CT_BATCH;
    const size_t N = c->N, xel = 2 * (size_t)c->ext_limbs(level) * N, xel1 = 2 * (size_t)c->ext_limbs(l1) * N, ctl1 = 2 * (size_t)level * N;
    u64* X = ar.take((size_t)nb_max * n_lo * xel);     // first rotations before their division
    u64* Vacc = ar.take((size_t)nb_max * n_hi * xel);  // masked sums on the extended basis
    u64* V = ar.take((size_t)nb_max * n_hi * ctl1);    // divided by P q_level: level-1
    u64* Xh = ar.take((size_t)nb_max * n_hi * xel1);   // second rotations before their division
    u64* W = ar.take((size_t)nb_max * xel1);           // their sums
    KsWs ws;
    const size_t ks_bytes = ws_ks(c, level, CT_BATCH, CT_BATCH);
    u64* ks_region = ar.take(ks_bytes / sizeof(u64));
    // Up to eight first rotations of a batch of ciphertexts in one launch (the digits are read once for the eight, not once
    // per rotation): the keyed offsets in groups of eight.
    const bool fused_lo = c->live_digits(level) <= 4;
    std::vector<u32> keyed;
    for (u32 l = 0; l < n_lo; l++)
        if (g_lo[l] != 1) keyed.push_back(l);
    const u32 n_groups = fused_lo ? (u32)((keyed.size() + 7) / 8) : 0;
    if (!ar.ok()) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for the re-layout");
    auto ks_at = [&](u32 lv) {
        Arena sub(ks_region, ks_bytes);
        return carve_ks(c, lv, CT_BATCH, CT_BATCH, sub, ws);
    };
    int rc;
    for (u32 c0 = 0; c0 < n_ct; c0 += CT_BATCH) {
        const u32 n = n_ct - c0 < CT_BATCH ? n_ct - c0 : CT_BATCH;
        ks_at(level);
        const u64 *in[CT_BATCH], *c1s[CT_BATCH];
        for (u32 b = 0; b < n; b++) {
            in[b] = cts[c0 + b];
            c1s[b] = in[b] + (size_t)(level + 1) * N;
        }
        if ((rc = run_modup(c, level, c1s, n, ws, st))) return rc;
        for (u32 l = 0; l < n_lo; l++) {
            u64* xo[CT_BATCH];
            for (u32 b = 0; b < n; b++) xo[b] = X + ((size_t)b * n_lo + l) * xel;
            if (g_lo[l] == 1) {
                for (u32 b = 0; b < n; b++) HIP_TRY(launch_scale_p_ext(c, level, in[b], xo[b], st));
            } else if (!fused_lo) {
                HIP_TRY(launch_key_inner_ext(c, level, dsrc(c, ws, 0), lo_keys[l]->d_key, g_lo[l], in, nullptr, nullptr, xo, n, st));
            }
        }
        for (u32 g = 0; g < n_groups; g++) {  // X[b][l] = term b * n_lo + l of a [2][E][N] array per term
            const u64* tkeys[8];
            u32 tg[8], ttap[8], nt = 0;
            for (size_t i = (size_t)g * 8; i < keyed.size() && nt < 8; i++) {
                const u32 l = keyed[i];
                tkeys[nt] = lo_keys[l]->d_key;
                tg[nt] = g_lo[l];
                ttap[nt++] = l;
            }
            HIP_TRY(launch_key_inner_taps(c, level, dsrc(c, ws, 0), tkeys, tg, nullptr, ttap, nt, in, X, XLayout::classic(c->ext_limbs(level), N), 0,
                                          n_lo, n, st));
        }
        HIP_TRY(launch_relayout_mac(c, level, true, X, masks, Vacc, n, n_lo, n_hi, st));
        const u32 n_v = n * n_hi;
        for (u32 i0 = 0; i0 < n_v; i0 += CT_BATCH) {  // one division by P q_level per sum
            const u32 m = n_v - i0 < CT_BATCH ? n_v - i0 : CT_BATCH;
            KsWs wd = ws;
            wd.v = Vacc + (size_t)i0 * xel;
            wd.v_b = xel;
            FinalItem items[CT_BATCH];
            for (u32 i = 0; i < m; i++) items[i] = FinalItem{nullptr, nullptr, nullptr, V + (size_t)(i0 + i) * ctl1, 1, 0};
            if ((rc = run_moddown(c, level, wd, m, items, st, true))) return rc;
        }
        // second rotations on the extended basis of level-1, ordered by h so that the ciphertexts of a batch share each key
        ks_at(l1);
        const u64 *src[CT_BATCH], *sc1[CT_BATCH];
        const ckks_key* ks[CT_BATCH];
        u32 gs[CT_BATCH], nk = 0;
        u64* dst[CT_BATCH];
        auto flush = [&]() -> int {
            int r = run_modup(c, l1, sc1, nk, ws, st);
            if (r) return r;
            for (u32 b0 = 0; b0 < nk;) {
                u32 b1 = b0 + 1;
                while (b1 < nk && ks[b1] == ks[b0]) b1++;
                HIP_TRY(launch_key_inner_ext(c, l1, dsrc(c, ws, b0), ks[b0]->d_key, gs[b0], src + b0, nullptr, nullptr,
                                             dst + b0, b1 - b0, st));
                b0 = b1;
            }
            nk = 0;
            return CKKS_OK;
        };
        for (u32 h = 0; h < n_hi; h++)
            for (u32 b = 0; b < n; b++) {
                const u64* v = V + ((size_t)b * n_hi + h) * ctl1;
                u64* xh = Xh + ((size_t)b * n_hi + h) * xel1;
                if (g_hi[h] == 1) {
                    HIP_TRY(launch_scale_p_ext(c, l1, v, xh, st));
                    continue;
                }
                src[nk] = v;
                sc1[nk] = v + (size_t)level * N;
                dst[nk] = xh;
                ks[nk] = hi_keys[h];
                gs[nk++] = g_hi[h];
                if (nk == CT_BATCH && (rc = flush())) return rc;
            }
        if (nk && (rc = flush())) return rc;
        // sums on the extended basis, then one ModDown per ciphertext
        for (u32 b = 0; b < n; b++) {
            u64* w = W + (size_t)b * xel1;
            for (u32 h = 0; h < n_hi;) {
                const u64* terms[KS_MAX_BATCH];
                u32 nt = 0;
                if (h) terms[nt++] = w;
                for (; h < n_hi && nt < KS_MAX_BATCH; h++) terms[nt++] = Xh + ((size_t)b * n_hi + h) * xel1;
                HIP_TRY(launch_ct_sum(c, l1, ptr_list(terms, nt), nt, w, st, true));
            }
        }
        KsWs wd = ws;
        wd.v = W;
        wd.v_b = xel1;
        FinalItem items[CT_BATCH];
        for (u32 b = 0; b < n; b++) items[b] = FinalItem{nullptr, nullptr, nullptr, outs[c0 + b], 1, 0};
        if ((rc = run_moddown(c, l1, wd, n, items, st))) return rc;
    }
    return CKKS_OK;
}

u32 ilog2(u32 v) { u32 r = 0; while ((1u << (r + 1)) <= v) r++; return r; }

}  // namespace

extern "C" {

size_t ckks_workspace_bytes(const ckks_ctx* c, int op, uint32_t level, uint32_t count) {
    if (!c || !level_ok(c, level)) return 0;
    const size_t N = c->N, L1 = level + 1;
    const u32 nb = count < 1 ? 1 : (count > CT_BATCH ? CT_BATCH : count);
    switch (op) {
        case CKKS_OP_KEYSWITCH: return c->dnum ? ws_ks(c, level, 1, 1) : 0;
        case CKKS_OP_ROTATE: {
            if (!c->dnum) return 0;
            // hoisted, more than one batch: a second set of inner-product and conversion buffers (two batches in flight);
            // unhoisted: every rotation of a batch has its own digits
            const size_t hoisted = ws_ks(c, level, 1, nb) +
                                   (count > CT_BATCH && c->side ? blk((size_t)nb * 2 * c->ext_limbs(level) * N) + blk((size_t)nb * 2 * L1 * N) : 0);
            const u32 most = ks_batch(c), ub = count < most ? (count ? count : 1) : most;
            const size_t unhoisted = ws_rotate_unhoisted(c, level, ub);
            return hoisted > unhoisted ? hoisted : unhoisted;
        }
        case CKKS_OP_RESCALE: return level >= 1 ? ws_rescale(c, level, 1) : 0;
        case CKKS_OP_CTCT_MUL_RELIN: return c->dnum ? ws_ctct(c, level, 1) : 0;
        // more than one batch of channels: two batches in flight (one on the library's side stream), each with its own scratch
        case CKKS_OP_POLY_ACT: {
            if (!c->dnum || level < 4) return 0;
            const size_t lanes = ws_poly_act(c, level, nb) * (count > CT_BATCH && c->side ? 2 : 1);  // sized for overlap on
            const u32 most = act_batch(c, level, count);
            const size_t one = ws_poly_act(c, level, count < most ? (count ? count : 1) : most);
            return one > lanes ? one : lanes;
        }
        default: return 0;
    }
}

size_t he_conv_workspace_bytes(const ckks_ctx* c, const he_conv_desc* d) {
    if (!c || !d || !c->dnum || !level_ok(c, d->level) || d->level < 1) return 0;
    const size_t N = c->N;
    if (d->alignment == HE_CONV_DEFERRED_MODDOWN || d->alignment == HE_CONV_DEFERRED_MERGED) {
        const size_t E = c->ext_limbs(d->level);
        return conv_lanes(c, d) * ws_conv_lane(c, d->level, conv_batch(c, d)) + blk(conv_copies(c, d)) + blk((size_t)d->c_out * 2 * E * N) + blk(conv_sum_scratch(c, d));
    }
    return ws_conv_rotated(c, d, ks_batch(c));
}

int ckks_ctx_set_overlap(ckks_ctx* c, int on) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    c->overlap = on != 0;
    return CKKS_OK;
}

uint32_t ckks_galois_element(const ckks_ctx* c, int32_t offset) {
    if (!c) return 0;
    const long n = (long)(c->N / 2);
    long r = offset % n;
    if (r < 0) r += n;
    const u64 two_n = 2ull * c->N;
    u64 g = 1, base = 5;
    for (; r; r >>= 1) {
        if (r & 1) g = g * base % two_n;
        base = base * base % two_n;
    }
    return (uint32_t)g;
}

// Polynomials of a large batch that go through both passes before the next ones do.  The first pass writes what the second reads: 240 MB of
// it stay in the 256 MB last-level cache in between, at the price of a drain and a fill of the chip per launch (about 8 us).  Forward and inverse
// together in us, all at once / in parts of about 240 MB: N = 2^16, 30 limbs, 472 MB 666 / 655, 692 MB 1016 / 959, 991 MB 1468 / 1381; 2^15, 24 limbs,
// 478 MB 664 / 657, 994 MB 1423 / 1365; 2^13 480 MB 668 / 632, 999 MB 1451 / 1317; the same calls over eight buffers in turn, which are not in any cache before: 2^16
// 535 MB 784 / 744, 692 MB 1017 / 962, 1007 MB 1491 / 1369, 2^15 1007 MB 1442 / 1355, 2^13 944 MB 1386 / 1238; parts of 170 MB of 346 MB 467 / 497, of 126 MB of 991 MB 1493, so a
// batch is cut from 444 MB on.  With 64-bit integer butterflies, which are bound by instruction issue: 994 MB 1868 / 1891, not cut.
static u32 ntt_cached_batch(const ckks_ctx* c, u32 n_limbs, u32 batch) {
    if (!c->ntt_f64 || c->log_hi == 0 || ntt_one_pass(c)) return batch;
    const u64 part = 240000000, total = (u64)batch * n_limbs * c->N * sizeof(u64), parts = (total + part * 15 / 100) / part;
    return parts > 1 ? (u32)((batch + parts - 1) / parts) : batch;
}

static int ntt_entry(const ckks_ctx* c, bool inverse, uint64_t* d_polys, const uint32_t* h_idx, uint32_t n_limbs, uint32_t batch,
                     void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!d_polys || !h_idx || n_limbs == 0 || batch == 0) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer or empty batch");
    if (n_limbs > CKKS_MAX_MODULI) return set_err(c, CKKS_ERR_INVALID_ARG, "at most 64 limbs per polynomial");
    PolyList pl;
    pl.n = n_limbs;
    for (u32 a = 0; a < CKKS_MAX_MODULI; a++) {
        if (a < n_limbs && h_idx[a] >= c->M) return set_err(c, CKKS_ERR_INVALID_ARG, "modulus index out of range");
        pl.spos[a] = pl.dpos[a] = (unsigned char)(a < n_limbs ? a : 0);
        pl.mod[a] = (unsigned char)(a < n_limbs ? h_idx[a] : 0);
    }
    u32 max_batch = 65535 / n_limbs;  // grid.y limit
    if (const u32 part = ntt_cached_batch(c, n_limbs, batch); part < max_batch) max_batch = part;
    u64* p = (u64*)d_polys;
    for (u32 b0 = 0; b0 < batch; b0 += max_batch) {
        const u32 nb = batch - b0 < max_batch ? batch - b0 : max_batch;
        u64* base = p + (size_t)b0 * n_limbs * c->N;
        HIP_TRY(launch_ntt(c, inverse, base, n_limbs, base, n_limbs, pl, nb, (hipStream_t)stream));
    }
    return CKKS_OK;
}

int ckks_ntt_fwd(const ckks_ctx* c, uint64_t* d_polys, const uint32_t* h_idx, uint32_t n_limbs, uint32_t batch, void* stream) {
    return ntt_entry(c, false, d_polys, h_idx, n_limbs, batch, stream);
}
int ckks_ntt_inv(const ckks_ctx* c, uint64_t* d_polys, const uint32_t* h_idx, uint32_t n_limbs, uint32_t batch, void* stream) {
    return ntt_entry(c, true, d_polys, h_idx, n_limbs, batch, stream);
}

int ckks_key_load(const ckks_ctx* c, const uint64_t* d_key, uint32_t galois_elt, ckks_key** out) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!d_key || !out) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer");
    if (!c->dnum) return set_err(c, CKKS_ERR_UNSUPPORTED_PARAMS, "context has no key-switching digits");
    if (galois_elt != 0 && ((galois_elt & 1) == 0 || galois_elt >= 2 * c->N)) return set_err(c, CKKS_ERR_INVALID_ARG, "Galois element must be odd and below 2N");
    ckks_key* k = new (std::nothrow) ckks_key;
    if (!k) return set_err(c, CKKS_ERR_INVALID_ARG, "out of host memory");
    k->d_key = (const u64*)d_key;
    k->galois_elt = galois_elt;
    *out = k;
    return CKKS_OK;
}
void ckks_key_free(ckks_key* k) { delete k; }

int ckks_key_expand_a(const ckks_ctx* c, uint64_t a_seed, uint64_t* d_key, void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!d_key) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer");
    if (!c->dnum) return set_err(c, CKKS_ERR_UNSUPPORTED_PARAMS, "context has no key-switching digits");
    HIP_TRY(launch_key_expand_a(c, a_seed, (u64*)d_key, (hipStream_t)stream));
    return CKKS_OK;
}

int ckks_keyset_stage(const ckks_ctx* c, const uint64_t* const* h_b, const uint64_t* h_a_seeds, uint64_t* const* h_d_keys,
                      uint32_t n_keys, void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!h_b || !h_a_seeds || !h_d_keys) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer");
    if (!c->dnum) return set_err(c, CKKS_ERR_UNSUPPORTED_PARAMS, "context has no key-switching digits");
    for (u32 i = 0; i < n_keys; i++)
        if (!h_b[i] || !h_d_keys[i]) return set_err(c, CKKS_ERR_INVALID_ARG, "null key pointer");
    const size_t half = (size_t)c->M * c->N * sizeof(u64);  // one digit's b (or a) part
    hipStream_t st = (hipStream_t)stream;
    for (u32 i = 0; i < n_keys; i++) {
        // the b halves: dnum rows of `half` bytes, densely packed on the host, every other row of the device key
        HIP_TRY(hipMemcpy2DAsync(h_d_keys[i], 2 * half, h_b[i], half, half, c->dnum, hipMemcpyHostToDevice, st));
        HIP_TRY(launch_key_expand_a(c, h_a_seeds[i], (u64*)h_d_keys[i], st));
    }
    return CKKS_OK;
}

int ckks_keyswitch(const ckks_ctx* c, const uint64_t* d_c, uint32_t level, const ckks_key* key, uint64_t* d_out, void* d_ws,
                   size_t ws_bytes, void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!d_c || !d_out) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer");
    if (!key) return set_err(c, CKKS_ERR_NO_KEY, "no key");
    if (!c->dnum) return set_err(c, CKKS_ERR_UNSUPPORTED_PARAMS, "context has no key-switching digits");
    if (!level_ok(c, level)) return set_err(c, CKKS_ERR_LEVEL_MISMATCH, "level out of range");
    Arena ar(d_ws, ws_bytes);
    KsWs ws;
    if (!carve_ks(c, level, 1, 1, ar, ws)) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for key switch");
    hipStream_t st = (hipStream_t)stream;
    const u64* src = (const u64*)d_c;
    const bool mac = ntt_has_modup(c);
    int rc = run_modup(c, level, &src, 1, ws, st, mac);
    if (rc) return rc;
    if (mac) {
        const u64* k = key->d_key;
        HIP_TRY(launch_ntt_lo_mac(c, level, dsrc(c, ws, 0), &k, &ws.v, 1, st, dropped_from(level, false)));
    } else {
        const u64* k = key->d_key;
        const u32 g = 1;
        HIP_TRY(launch_key_inner_items(c, level, dsrc(c, ws, 0), &k, &g, nullptr, ws.v, ws.v_b, 1, st));
    }
    const FinalItem item = {nullptr, nullptr, nullptr, (u64*)d_out, 1, 0};
    return run_moddown(c, level, ws, 1, &item, st, false, mac);
}

int ckks_rotate_hoisted(const ckks_ctx* c, const uint64_t* d_ct, uint32_t level, const int32_t* h_offsets, uint32_t n_rot,
                        const ckks_key* const* keys, uint64_t* const* h_d_outs, int hoisted, void* d_ws, size_t ws_bytes,
                        void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!d_ct || !h_offsets || !h_d_outs || n_rot == 0) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer or no rotations");
    if (!c->dnum) return set_err(c, CKKS_ERR_UNSUPPORTED_PARAMS, "context has no key-switching digits");
    if (!level_ok(c, level)) return set_err(c, CKKS_ERR_LEVEL_MISMATCH, "level out of range");
    const size_t N = c->N, L1 = level + 1;
    // validate everything before the first launch
    u32 n_keyed = 0;
    for (u32 t = 0; t < n_rot; t++) {
        if (!h_d_outs[t]) return set_err(c, CKKS_ERR_INVALID_ARG, "null output pointer");
        const u32 g = ckks_galois_element(c, h_offsets[t]);
        if (g == 1) continue;
        n_keyed++;
        if (!keys || !keys[t]) return set_err(c, CKKS_ERR_NO_KEY, "rotation key missing");
        if (keys[t]->galois_elt != g) return set_err(c, CKKS_ERR_NO_KEY, "rotation key was made for another offset");
    }
    // rotations go through the kernels in batches of up to ks_batch (hoisted: see rotations_together): hoisted ones share the digits and batch their
    // ModDown; unhoisted ones each have their own digits, of the permuted polynomial, and share every launch, in batches as large as the
    // workspace holds (one at a time in the smallest workspace that is accepted)
    const bool one_stream = rotations_together(c, level, n_keyed);
    const u32 most = hoisted && !one_stream ? CT_BATCH : ks_batch(c);
    u32 rb = n_keyed < most ? (n_keyed ? n_keyed : 1) : most;
    Arena ar(d_ws, ws_bytes);
    KsWs ws = {};
    u64* pc1 = nullptr;
    if (n_keyed) {
        if (hoisted) {
            if (rb > CT_BATCH && ws_bytes < ws_ks(c, level, 1, rb)) rb = CT_BATCH;  // in a smaller workspace
            if (!carve_ks(c, level, 1, rb, ar, ws)) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for rotation");
        } else {
            while (rb > 1 && ws_bytes < ws_rotate_unhoisted(c, level, rb)) rb--;
            if (!carve_ks(c, level, rb, rb, ar, ws)) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for rotation");
            if (!ntt_has_modup(c)) pc1 = ar.take((size_t)rb * L1 * N);
            if (!ar.ok()) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for rotation");
        }
    }
    hipStream_t st = (hipStream_t)stream;
    // More than one batch of hoisted rotations: with room for a second set of inner-product and conversion buffers, every
    // other batch runs on the context's second stream (its traffic-bound inner products next to the other batch's ModDown).
    KsWs lane_ws[2] = {ws, ws};
    bool two_lanes = false;
    if (hoisted && n_keyed > rb && c->side_stream() && !one_stream) {
        Arena extra = ar;
        lane_ws[1].v = extra.take(rb * ws.v_b);
        lane_ws[1].w = extra.take(rb * ws.w_b);
        two_lanes = extra.ok();
    }
    const u64* ct = (const u64*)d_ct;
    const u64* c0 = ct;
    const u64* c1 = ct + L1 * N;
    if (n_keyed && hoisted) {
        int rc = run_modup(c, level, &c1, 1, ws, st);
        if (rc) return rc;
        for (u32 l = 0; l < 2; l++) lane_ws[l].own[0] = ws.own[0];  // both lanes read the same digits
    }
    if (two_lanes) {
        HIP_TRY(hipEventRecord(c->ev_fork, st));
        HIP_TRY(hipStreamWaitEvent(c->side, c->ev_fork, 0));
    }
    auto join = [&](int rc) -> int {  // also on the error paths
        if (!two_lanes) return rc;
        hipError_t e = hipEventRecord(c->ev_join, c->side);
        if (e == hipSuccess) e = hipStreamWaitEvent(st, c->ev_join, 0);
        return (e != hipSuccess && rc == CKKS_OK) ? set_hip_err(c, e) : rc;
    };
    FinalItem items[KS_MAX_BATCH];
    const ckks_key* pend_key[KS_MAX_BATCH];
    u32 nb = 0, lane = 0;
    // the pending unhoisted rotations: one decomposition of sigma_g(c1) per rotation and one ModDown for the batch
    auto flush_unhoisted = [&]() -> int {
        const u64 *srcs[KS_MAX_BATCH], *ks[KS_MAX_BATCH];
        u64* outs[KS_MAX_BATCH];
        u32 gs[KS_MAX_BATCH];
        const u32 n = nb;
        nb = 0;
        for (u32 b = 0; b < n; b++) {
            gs[b] = items[b].g;
            ks[b] = pend_key[b]->d_key;
            outs[b] = items[b].out;
            srcs[b] = ntt_has_modup(c) ? ct : pc1 + (size_t)b * L1 * N;
        }
        if (ntt_has_modup(c)) return run_rotate_batch(c, level, n, srcs, pend_key, gs, outs, ws, st);
        HIP_TRY(launch_automorph(c, (u32)L1, c1, gs, n, pc1, st));
        if (int rc = run_modup(c, level, srcs, n, ws, st)) return rc;
        for (u32 b = 0; b < n; b++) gs[b] = 1;  // the digits already belong to sigma_g(c1): no gather in the inner product, only on c0
        HIP_TRY(launch_key_inner_items(c, level, dsrc(c, ws, 0), ks, gs, nullptr, ws.v, ws.v_b, n, st));
        return run_moddown(c, level, ws, n, items, st);
    };
    const bool fused_hoist = hoisted && c->live_digits(level) <= 4;
    auto flush_hoisted = [&]() -> int {
        const KsWs& lw = lane_ws[lane];
        hipStream_t ls = lane ? c->side : st;
        const u64 *tkeys[KS_MAX_BATCH], *cts[KS_MAX_BATCH];
        u64* outs[KS_MAX_BATCH];
        u32 tg[KS_MAX_BATCH], ttap[KS_MAX_BATCH];
        for (u32 b = 0; b < nb; b++) {
            tkeys[b] = pend_key[b]->d_key;
            tg[b] = items[b].g;
            ttap[b] = b;
            cts[b] = ct;
            outs[b] = items[b].out;
            items[b].g = 1;  // the division's last step adds nothing: c0 is inside the sum already
        }
        if (ntt_has_modup(c)) {
            const MacRotate rot = {cts, tg, nullptr, true};
            int rc = run_inner_divide(c, level, lw, tkeys, nb, outs, nullptr, ls, false, nullptr, &rot);
            nb = 0;
            if (two_lanes) lane ^= 1;
            return rc;
        }
        if (hipError_t e = rotated_inner(c, level, lw, &ct, 1, tkeys, tg, ttap, nb, ls); e != hipSuccess) return set_hip_err(c, e);
        int rc = run_moddown(c, level, lw, nb, items, ls);
        nb = 0;
        if (two_lanes) lane ^= 1;
        return rc;
    };
    for (u32 t = 0; t < n_rot; t++) {
        const u32 g = ckks_galois_element(c, h_offsets[t]);
        u64* out = (u64*)h_d_outs[t];
        if (g == 1) {
            if (hipError_t e = launch_copy(ct, out, 2 * L1 * N, st); e != hipSuccess) return join(set_hip_err(c, e));
            continue;
        }
        if (hoisted && fused_hoist) {
            // same digits, one key per rotation: the rotations of a batch share their launches, each reads the digits through its automorphism, and the
            // sums P sigma_g(c0) + inner product make the division by P the rotation, c0 included (run_inner_divide; moduli above 2^50 and rings up to
            // 2^11: rotated_inner, which reads the digits once for all)
            pend_key[nb] = keys[t];
            items[nb] = FinalItem{nullptr, nullptr, nullptr, out, g, 0};
            if (++nb == rb) {
                if (int rc = flush_hoisted()) return join(rc);
            }
        } else if (hoisted) {
            // many digits: one launch per rotation; the digits are read through sigma_g
            const KsWs& lw = lane_ws[lane];
            hipStream_t ls = lane ? c->side : st;
            const u64* k = keys[t]->d_key;
            if (hipError_t e = launch_key_inner_items(c, level, dsrc(c, lw, 0), &k, &g, &c0, lw.v + nb * lw.v_b, lw.v_b, 1, ls); e != hipSuccess)
                return join(set_hip_err(c, e));
            items[nb] = FinalItem{nullptr, nullptr, nullptr, out, 1, 0};
            if (++nb == rb) {
                int rc = run_moddown(c, level, lw, nb, items, ls);
                if (rc) return join(rc);
                nb = 0;
                if (two_lanes) lane ^= 1;
            }
        } else {
            items[nb] = FinalItem{c0, nullptr, nullptr, out, g, 0};
            pend_key[nb] = keys[t];
            if (++nb == rb)
                if (int rc = flush_unhoisted()) return rc;
        }
    }
    if (nb && !hoisted) {
        if (int rc = flush_unhoisted()) return rc;
    } else if (nb && fused_hoist) {
        if (int rc = flush_hoisted()) return join(rc);
    } else if (nb) {
        int rc = run_moddown(c, level, lane_ws[lane], nb, items, lane ? c->side : st);
        if (rc) return join(rc);
    }
    return join(CKKS_OK);
}

int ckks_ptct_mac(const ckks_ctx* c, const uint64_t* const* h_d_pts, const uint64_t* const* h_d_cts, uint32_t n_terms,
                  uint32_t level, uint64_t* d_acc, int accumulate, void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!h_d_pts || !h_d_cts || !d_acc || n_terms == 0) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer or no terms");
    if (!level_ok(c, level)) return set_err(c, CKKS_ERR_LEVEL_MISMATCH, "level out of range");
    for (u32 k = 0; k < n_terms; k++)
        if (!h_d_pts[k] || !h_d_cts[k]) return set_err(c, CKKS_ERR_INVALID_ARG, "null operand pointer");
    HIP_TRY(launch_ptct_mac(c, level, (const u64* const*)h_d_pts, (const u64* const*)h_d_cts, n_terms, (u64*)d_acc, accumulate,
                            (hipStream_t)stream));
    return CKKS_OK;
}

int ckks_rescale(const ckks_ctx* c, const uint64_t* d_ct, uint32_t level, uint64_t* d_out, void* d_ws, size_t ws_bytes, void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!d_ct || !d_out) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer");
    if (!level_ok(c, level) || level < 1) return set_err(c, CKKS_ERR_LEVEL_MISMATCH, "rescale needs 1 <= level < num_q");
    const u64* ct = (const u64*)d_ct;
    u64* out = (u64*)d_out;
    return run_rescale(c, level, &ct, (size_t)(level + 1) * c->N, &out, 1, Arena(d_ws, ws_bytes), (hipStream_t)stream);
}

int ckks_ctct_mul_relin(const ckks_ctx* c, const uint64_t* d_a, const uint64_t* d_b, uint32_t level, const ckks_key* rlk,
                        uint64_t* d_out, void* d_ws, size_t ws_bytes, void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!d_a || !d_b || !d_out) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer");
    if (!c->dnum) return set_err(c, CKKS_ERR_UNSUPPORTED_PARAMS, "context has no key-switching digits");
    if (!rlk) return set_err(c, CKKS_ERR_NO_KEY, "no relinearisation key");
    if (rlk->galois_elt != 0) return set_err(c, CKKS_ERR_NO_KEY, "key is a rotation key, not the relinearisation key");
    if (!level_ok(c, level)) return set_err(c, CKKS_ERR_LEVEL_MISMATCH, "level out of range");
    const size_t cs = (size_t)(level + 1) * c->N;
    const u64* a = (const u64*)d_a;
    const u64* b = (const u64*)d_b;
    u64* out = (u64*)d_out;
    return run_ctct(c, level, &a, cs, &b, cs, rlk->d_key, &out, 1, Arena(d_ws, ws_bytes), (hipStream_t)stream);
}

int he_conv_check_weights(const ckks_ctx* c, const he_conv_desc* d, const uint64_t* d_w_res, void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!d || !d_w_res) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer");
    if (d->c_in == 0 || d->c_out == 0) return set_err(c, CKKS_ERR_INVALID_ARG, "empty convolution shape");
    if (!level_ok(c, d->level)) return set_err(c, CKKS_ERR_LEVEL_MISMATCH, "level out of range");
    if (d->alignment > HE_CONV_DEFERRED_MERGED) return set_err(c, CKKS_ERR_INVALID_ARG, "unknown alignment");
    if (d->weight_bits == 0) return CKKS_OK;  // nothing promised
    const bool ext = d->alignment == HE_CONV_DEFERRED_MODDOWN || d->alignment == HE_CONV_DEFERRED_MERGED;
    hipStream_t st = (hipStream_t)stream;
    HIP_TRY(launch_weight_check(c, d->level, ext, (const u64*)d_w_res, (size_t)d->c_out * d->c_in * 9, d->weight_bits, c->d_check, st));
    u32 bad = 0;
    HIP_TRY(hipMemcpyAsync(&bad, c->d_check, sizeof(bad), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    if (bad) {
        c->err = std::to_string(bad) + " weight residues are not integers below 2^(weight_bits-1) = 2^" + std::to_string(d->weight_bits - 1) +
                 " in magnitude: he_conv_batched would return wrong residues with this weight_bits";
        return CKKS_ERR_INVALID_ARG;
    }
    return CKKS_OK;
}

int he_conv_batched(const ckks_ctx* c, const he_conv_desc* d, const uint64_t* const* h_d_in, const ckks_key* const* rot_keys,
                    const uint64_t* d_tap_masks, const uint64_t* d_w_res, uint64_t* const* h_d_out, void* d_ws, size_t ws_bytes,
                    void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!d || !h_d_in || !rot_keys || !d_tap_masks || !d_w_res || !h_d_out) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer");
    if (!c->dnum) return set_err(c, CKKS_ERR_UNSUPPORTED_PARAMS, "context has no key-switching digits");
    if (d->c_in == 0 || d->c_out == 0 || d->height == 0 || d->width == 0 || d->batch == 0)
        return set_err(c, CKKS_ERR_INVALID_ARG, "empty convolution shape");
    if (!level_ok(c, d->level) || d->level < 1) return set_err(c, CKKS_ERR_LEVEL_MISMATCH, "convolution needs 1 <= level < num_q");
    if ((u64)d->height * d->width * d->batch > c->N / 2) return set_err(c, CKKS_ERR_INVALID_ARG, "H*W*batch exceeds the N/2 slots");
    if (d->alignment > HE_CONV_DEFERRED_MERGED) return set_err(c, CKKS_ERR_INVALID_ARG, "unknown alignment");
    const bool four = d->alignment == HE_CONV_ALIGN_FOUR_KEYS;
    const u32 level = d->level;
    const size_t N = c->N, L1 = level + 1, ct_elems = 2 * L1 * N;
    u32 gs[9];
    {
        u32 t = 0;
        for (int dy = -1; dy <= 1; dy++)
            for (int dx = -1; dx <= 1; dx++, t++) {
                gs[t] = ckks_galois_element(c, dy * (int32_t)d->width + dx);
                if (gs[t] == 1) continue;
                if (four && (t & 1) == 0) continue;  // the corner taps are reached in two steps: no key of their own
                if (!rot_keys[t]) return set_err(c, CKKS_ERR_NO_KEY, "rotation key missing for a tap");
                if (rot_keys[t]->galois_elt != gs[t]) return set_err(c, CKKS_ERR_NO_KEY, "rotation key does not match its tap offset");
            }
    }
    for (u32 i = 0; i < d->c_in; i++) if (!h_d_in[i]) return set_err(c, CKKS_ERR_INVALID_ARG, "null input ciphertext");
    for (u32 o = 0; o < d->c_out; o++) if (!h_d_out[o]) return set_err(c, CKKS_ERR_INVALID_ARG, "null output ciphertext");

    if (d->alignment == HE_CONV_DEFERRED_MODDOWN || d->alignment == HE_CONV_DEFERRED_MERGED)
        return conv_deferred(c, d, gs, h_d_in, rot_keys, (const u64*)d_tap_masks, (const u64*)d_w_res, h_d_out, d_ws, ws_bytes,
                             (hipStream_t)stream);
    Arena ar(d_ws, ws_bytes);
    KsWs ws;
    u32 kb = ks_batch(c);  // rotations divided at a time
    if (ws_bytes < ws_conv_rotated(c, d, kb)) kb = CT_BATCH;  // in a smaller workspace
    bool ok = carve_ks(c, level, CT_BATCH, kb, ar, ws);
    u64* xs = ar.take((size_t)d->c_in * 9 * ct_elems);
    u64* acc = ar.take((size_t)d->c_out * ct_elems);
    u64* wscratch = ar.take(weighted_sum_scratch_elems(c, (u32)L1, d->c_in * 9, d->c_out));
    u64* side[2] = {nullptr, nullptr};  // C^-1 and C^+1 of the current batch (four-key alignment)
    if (four) {
        side[0] = ar.take((size_t)CT_BATCH * ct_elems);
        side[1] = ar.take((size_t)CT_BATCH * ct_elems);
    }
    if (!ok || !ar.ok() || ar.used + ws_rescale(c, level, CT_BATCH) > ar.cap)
        return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for the convolution");
    hipStream_t st = (hipStream_t)stream;

    // input alignment: nine aligned copies of every input channel, each times its tap mask.  Channels
    // go in batches: one shared pass of the decomposition kernels, then inner products that stream each
    // tap's key once for the whole batch and batched ModDowns (a single channel: one of each for its eight taps).
    auto mask_of = [&](u32 t) { return (const u64*)d_tap_masks + (size_t)t * L1 * N; };
    auto slot = [&](u32 ch, u32 t) { return xs + ((size_t)ch * 9 + t) * ct_elems; };
    // One rotation of every ciphertext of a batch: by the offset of tap kt, times masks[b] (or unmasked), to outs[b].
    struct TapJob {
        u32 kt;
        u64* outs[CT_BATCH];
        const u64* masks[CT_BATCH];
    };
    // The rotations `jobs` of the n ciphertexts `base`, whose digits are in ws: as many taps at a time as fill a batch of
    // kb key switches (all eight for one or two channels, two for eight).
    auto rotate_jobs = [&](const u64* const* base, u32 n, const TapJob* jobs, u32 n_jobs) -> int {
        const u32 per = kb / n;
        for (u32 j0 = 0; j0 < n_jobs; j0 += per) {
            const u32 m = n_jobs - j0 < per ? n_jobs - j0 : per;
            FinalItem items[KS_MAX_BATCH];
            const u64* keys[KS_MAX_BATCH];
            u32 g[KS_MAX_BATCH], pos[KS_MAX_BATCH];
            for (u32 j = 0; j < m; j++) {
                const TapJob& job = jobs[j0 + j];
                keys[j] = rot_keys[job.kt]->d_key;
                g[j] = gs[job.kt];
                pos[j] = j * n;
                for (u32 b = 0; b < n; b++) items[pos[j] + b] = FinalItem{nullptr, nullptr, job.masks[b], job.outs[b], 1, 0};
            }
            HIP_TRY(rotated_inner(c, level, ws, base, n, keys, g, pos, m, st));  // P sigma_g(c0) included: dividing it by P is the rotation
            if (int rc = run_moddown(c, level, ws, m * n, items, st)) return rc;
        }
        return CKKS_OK;
    };
    // copies that only take their tap's mask: noted, then multiplied in as few launches as their number allows
    const u64 *mm_masks[9 * CT_BATCH], *mm_cts[9 * CT_BATCH];
    u64* mm_outs[9 * CT_BATCH];
    u32 n_mm = 0;
    auto masked = [&](const u64* m, const u64* ct, u64* out) { mm_masks[n_mm] = m, mm_cts[n_mm] = ct, mm_outs[n_mm++] = out; };
    auto flush_masked = [&]() -> int {
        HIP_TRY(launch_mask_mul(c, level, mm_masks, mm_cts, mm_outs, n_mm, st));
        n_mm = 0;
        return CKKS_OK;
    };
    for (u32 c0 = 0; c0 < d->c_in; c0 += CT_BATCH) {
        const u32 n = d->c_in - c0 < CT_BATCH ? d->c_in - c0 : CT_BATCH;
        const u64 *in[CT_BATCH], *c1s[CT_BATCH];
        TapJob jobs[8];
        u32 nj = 0;
        for (u32 b = 0; b < n; b++) {
            in[b] = (const u64*)h_d_in[c0 + b];
            c1s[b] = in[b] + L1 * N;
        }
        int rc = run_modup(c, level, c1s, n, ws, st);
        if (rc) return rc;
        if (!four) {
            for (u32 t = 0; t < 9; t++) {
                if (gs[t] == 1) {
                    for (u32 b = 0; b < n; b++) masked(mask_of(t), in[b], slot(c0 + b, t));
                    continue;
                }
                TapJob& job = jobs[nj++];
                job.kt = t;
                for (u32 b = 0; b < n; b++) job.outs[b] = slot(c0 + b, t), job.masks[b] = mask_of(t);
            }
            if ((rc = flush_masked())) return rc;
            if ((rc = rotate_jobs(in, n, jobs, nj))) return rc;
            continue;
        }
        // four-key alignment, first stage: the input rotated by -1, +1 (kept unmasked for the second
        // stage) and by -W, +W (final), all from the one decomposition of the input
        const u64* base[2 * CT_BATCH];  // C^-1 of the batch, then C^+1
        for (u32 sd = 0; sd < 2; sd++) {
            const u32 kt = sd == 0 ? 3 : 5;
            u64* outs[CT_BATCH];
            for (u32 b = 0; b < n; b++) base[sd * n + b] = outs[b] = side[sd] + (size_t)b * ct_elems;
            if (gs[kt] == 1) {
                for (u32 b = 0; b < n; b++) HIP_TRY(launch_copy(in[b], outs[b], ct_elems, st));
                continue;
            }
            TapJob& job = jobs[nj++];
            job.kt = kt;
            for (u32 b = 0; b < n; b++) job.outs[b] = outs[b], job.masks[b] = nullptr;
        }
        for (u32 kt = 1; kt <= 7; kt += 6) {
            if (gs[kt] == 1) {
                for (u32 b = 0; b < n; b++) masked(mask_of(kt), in[b], slot(c0 + b, kt));
                continue;
            }
            TapJob& job = jobs[nj++];
            job.kt = kt;
            for (u32 b = 0; b < n; b++) job.outs[b] = slot(c0 + b, kt), job.masks[b] = mask_of(kt);
        }
        if ((rc = rotate_jobs(in, n, jobs, nj))) return rc;
        for (u32 b = 0; b < n; b++) {
            masked(mask_of(4), in[b], slot(c0 + b, 4));
            masked(mask_of(3), side[0] + (size_t)b * ct_elems, slot(c0 + b, 3));
            masked(mask_of(5), side[1] + (size_t)b * ct_elems, slot(c0 + b, 5));
        }
        // second stage: C^-1 and C^+1 rotated by -W and +W (their own decompositions; both in one batch where they fit)
        const u32 n2 = 2 * n <= CT_BATCH ? 2 * n : n;
        for (u32 b0 = 0; b0 < 2 * n; b0 += n2) {
            for (u32 b = 0; b < n2; b++) c1s[b] = base[b0 + b] + L1 * N;
            if ((rc = run_modup(c, level, c1s, n2, ws, st))) return rc;
            nj = 0;
            for (u32 kt = 1; kt <= 7; kt += 6) {
                TapJob job;
                job.kt = kt;
                for (u32 b = 0; b < n2; b++) {
                    const u32 sd = (b0 + b) / n, t = (kt == 1 ? 0 : 6) + 2 * sd;  // corner taps 0, 2 (row -1) and 6, 8 (row +1)
                    job.outs[b] = slot(c0 + (b0 + b) % n, t);
                    job.masks[b] = mask_of(t);
                    if (gs[kt] == 1) masked(job.masks[b], base[b0 + b], job.outs[b]);
                }
                if (gs[kt] != 1) jobs[nj++] = job;
            }
            if ((rc = rotate_jobs(base + b0, n2, jobs, nj))) return rc;
        }
        if ((rc = flush_masked())) return rc;
    }
    // convolution evaluation: integer-weighted sum over (input channel, tap) for every output channel
    HIP_TRY(launch_weighted_sum(c, level, false, xs, XLayout::classic(L1, N), d->c_in * 9, (const u64*)d_w_res, d->c_out, acc, wscratch, d->weight_bits, st));
    for (u32 o0 = 0; o0 < d->c_out; o0 += CT_BATCH) {
        const u32 n = d->c_out - o0 < CT_BATCH ? d->c_out - o0 : CT_BATCH;
        const u64* ins[CT_BATCH];
        u64* outs[CT_BATCH];
        for (u32 b = 0; b < n; b++) {
            ins[b] = acc + (size_t)(o0 + b) * ct_elems;
            outs[b] = (u64*)h_d_out[o0 + b];
        }
        int rc = run_rescale(c, level, ins, L1 * N, outs, n, ar.rest(), st);
        if (rc) return rc;
    }
    return CKKS_OK;
}

size_t he_accumulator_workspace_bytes(const ckks_ctx* c, uint32_t level, uint32_t g) {
    if (!c || !c->dnum || !level_ok(c, level) || level < 1 || g == 0 || g > KS_MAX_BATCH) return 0;
    return ws_merge(c, level, g);
}

int he_accumulator_merge(const ckks_ctx* c, const uint64_t* const* h_d_cts, uint32_t g, uint32_t level, uint32_t sts,
                         const uint64_t* d_mask, const ckks_key* const* keys, uint64_t* d_out, void* d_ws, size_t ws_bytes,
                         void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!h_d_cts || !d_mask || !d_out || g == 0) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer or no ciphertexts");
    if (g > KS_MAX_BATCH) return set_err(c, CKKS_ERR_INVALID_ARG, "at most 16 ciphertexts per merge");
    if (!c->dnum) return set_err(c, CKKS_ERR_UNSUPPORTED_PARAMS, "context has no key-switching digits");
    if (!level_ok(c, level) || level < 1) return set_err(c, CKKS_ERR_LEVEL_MISMATCH, "merge needs 1 <= level < num_q");
    if (sts == 0 || (u64)g * sts > c->N / 2) return set_err(c, CKKS_ERR_INVALID_ARG, "g * sts exceeds the N/2 slots");
    u32 gal[KS_MAX_BATCH];
    for (u32 i = 0; i < g; i++) {
        if (!h_d_cts[i]) return set_err(c, CKKS_ERR_INVALID_ARG, "null ciphertext pointer");
        gal[i] = ckks_galois_element(c, -(int32_t)(i * sts));
        if (i == 0) continue;
        if (!keys || !keys[i]) return set_err(c, CKKS_ERR_NO_KEY, "rotation key missing for a block");
        if (keys[i]->galois_elt != gal[i]) return set_err(c, CKKS_ERR_NO_KEY, "rotation key does not match the block's offset");
    }
    return run_merge(c, (const u64* const*)h_d_cts, g, level, (const u64*)d_mask, keys, gal, (u64*)d_out, Arena(d_ws, ws_bytes),
                     (hipStream_t)stream);
}

// ---- slot re-layout with two rotations per element (down-sampling compaction, FC output reconstruction) ----
size_t he_relayout_workspace_bytes(const ckks_ctx* c, uint32_t level, uint32_t n_ct, uint32_t n_lo, uint32_t n_hi, uint32_t schedule) {
    if (!c || !c->dnum || !level_ok(c, level) || level < 1 || n_ct == 0 || n_lo == 0 || n_hi == 0 || schedule > HE_RELAYOUT_DEFERRED) return 0;
    return schedule == HE_RELAYOUT_DEFERRED ? ws_relayout_deferred(c, level, n_ct, n_lo, n_hi) : ws_relayout(c, level, n_ct, n_lo, n_hi);
}

int he_relayout_two_rotations(const ckks_ctx* c, const uint64_t* const* h_d_cts, uint32_t n_ct, uint32_t level, const int32_t* h_lo,
                              uint32_t n_lo, const ckks_key* const* lo_keys, const int32_t* h_hi, uint32_t n_hi,
                              const ckks_key* const* hi_keys, const uint64_t* const* h_d_masks, uint32_t schedule,
                              uint64_t* const* h_d_outs, void* d_ws, size_t ws_bytes, void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!h_d_cts || !h_lo || !h_hi || !h_d_masks || !h_d_outs || n_ct == 0 || n_lo == 0 || n_hi == 0)
        return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer or an empty list");
    if (schedule > HE_RELAYOUT_DEFERRED) return set_err(c, CKKS_ERR_INVALID_ARG, "unknown schedule");
    if (!c->dnum) return set_err(c, CKKS_ERR_UNSUPPORTED_PARAMS, "context has no key-switching digits");
    if (!level_ok(c, level) || level < 1) return set_err(c, CKKS_ERR_LEVEL_MISMATCH, "the re-layout needs 1 <= level < num_q");
    if ((u64)n_lo * n_hi > (u64)c->N) return set_err(c, CKKS_ERR_INVALID_ARG, "more (lo, hi) pairs than coefficients");
    for (u32 b = 0; b < n_ct; b++)
        if (!h_d_cts[b] || !h_d_outs[b]) return set_err(c, CKKS_ERR_INVALID_ARG, "null ciphertext pointer");
    std::vector<u32> g_lo(n_lo), g_hi(n_hi);
    for (u32 l = 0; l < n_lo; l++) {
        g_lo[l] = ckks_galois_element(c, h_lo[l]);
        if (g_lo[l] != 1 && (!lo_keys || !lo_keys[l] || lo_keys[l]->galois_elt != g_lo[l]))
            return set_err(c, CKKS_ERR_NO_KEY, "key of a first rotation missing or made for another offset");
    }
    for (u32 h = 0; h < n_hi; h++) {
        g_hi[h] = ckks_galois_element(c, h_hi[h]);
        if (g_hi[h] != 1 && (!hi_keys || !hi_keys[h] || hi_keys[h]->galois_elt != g_hi[h]))
            return set_err(c, CKKS_ERR_NO_KEY, "key of a second rotation missing or made for another offset");
        bool any = false;
        for (u32 l = 0; l < n_lo; l++) any = any || h_d_masks[(size_t)h * n_lo + l];
        if (!any) return set_err(c, CKKS_ERR_INVALID_ARG, "a second rotation has no mask at all");
    }
    return (schedule == HE_RELAYOUT_DEFERRED ? run_relayout_deferred : run_relayout)(
        c, level, n_ct, (const u64* const*)h_d_cts, n_lo, lo_keys, g_lo.data(), n_hi, hi_keys, g_hi.data(), (const u64* const*)h_d_masks,
        (u64* const*)h_d_outs, Arena(d_ws, ws_bytes), (hipStream_t)stream);
}

// ---- batched fully connected layer ------------------------------------------------------------------
static u32 fc_base(const he_fc_desc* d) {
    if (d->base) return d->base;
    u32 b = 1;
    while (b * b < d->batch) b++;
    return b;
}

static size_t max3(size_t a, size_t b, size_t c3) { return a > b ? (a > c3 ? a : c3) : (b > c3 ? b : c3); }

// inner sums that share their launches
static u32 fc_batch(const ckks_ctx* c, const he_fc_desc* d) {
    const u32 most = ks_batch(c);
    return d->d_out > CT_BATCH ? (d->d_out < most ? d->d_out : most) : CT_BATCH;
}
// nb inner sums, mb rotations of the merge and rb of the layout at a time
static size_t fc_workspace_in(const ckks_ctx* c, const he_fc_desc* d, u32 nb, u32 mb, u32 rb) {
    const size_t N = c->N;
    const u32 level = d->level, base = fc_base(d), n_lo = base < d->batch ? base : d->batch, n_hi = (d->batch + base - 1) / base;
    const size_t ct0 = 2 * (size_t)(level + 1) * N, ct1 = 2 * (size_t)level * N, ct2 = 2 * (size_t)(level - 1) * N;
    return blk(CT_BATCH * ct0) + blk(d->d_out * ct1) + blk(nb * ct1) + blk(ct2) + ws_ks(c, level - 1, nb, nb) +
           max3(ws_merge_in(c, level - 1, d->d_out, merge_batch(d->d_out, mb)), ws_rescale(c, level, CT_BATCH), ws_relayout_in(c, level - 2, 1, n_lo, n_hi, rb));
}
size_t he_fc_workspace_bytes(const ckks_ctx* c, const he_fc_desc* d) {
    if (!c || !d || !c->dnum || !level_ok(c, d->level) || d->level < 3 || d->d_out == 0 || d->d_out > KS_MAX_BATCH || d->batch == 0) return 0;
    return fc_workspace_in(c, d, fc_batch(c, d), ks_batch(c), ks_batch(c));
}

int he_fc_batched(const ckks_ctx* c, const he_fc_desc* d, const uint64_t* d_in, const uint64_t* d_w_enc, const ckks_key* const* sum_keys,
                  const ckks_key* const* merge_keys, const uint64_t* d_merge_mask, const uint64_t* d_place_masks,
                  const ckks_key* const* lo_keys, const ckks_key* const* hi_keys, const uint64_t* d_bias, uint64_t* d_out, void* d_ws,
                  size_t ws_bytes, void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!d || !d_in || !d_w_enc || !d_merge_mask || !d_place_masks || !d_bias || !d_out) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer");
    if (!c->dnum) return set_err(c, CKKS_ERR_UNSUPPORTED_PARAMS, "context has no key-switching digits");
    if (!level_ok(c, d->level) || d->level < 3) return set_err(c, CKKS_ERR_LEVEL_MISMATCH, "the layer needs 3 <= level < num_q");
    if (d->d_in == 0 || (d->d_in & (d->d_in - 1)) || d->d_out == 0 || d->d_out > d->d_in || d->batch == 0)
        return set_err(c, CKKS_ERR_INVALID_ARG, "d_in must be a power of two and 1 <= d_out <= d_in");
    if (d->d_out > KS_MAX_BATCH) return set_err(c, CKKS_ERR_UNSUPPORTED_PARAMS, "at most 16 outputs per call");
    if ((u64)d->batch * d->d_in > c->N / 2) return set_err(c, CKKS_ERR_INVALID_ARG, "batch * d_in exceeds the N/2 slots");
    const u32 level = d->level, l1 = level - 1, l2 = level - 2, l3 = level - 3;
    const u32 base = fc_base(d), n_lo = base < d->batch ? base : d->batch, n_hi = (d->batch + base - 1) / base;
    const u32 delta = d->d_in - d->d_out, n_sum = ilog2(d->d_in);
    // Galois elements and keys of every rotation, checked before the first launch
    u32 g_sum[32], g_merge[KS_MAX_BATCH];
    for (u32 s = 0; s < n_sum; s++) {
        g_sum[s] = ckks_galois_element(c, (int32_t)(1u << s));
        if (!sum_keys || !sum_keys[s] || sum_keys[s]->galois_elt != g_sum[s]) return set_err(c, CKKS_ERR_NO_KEY, "key of an inner-sum rotation missing or wrong");
    }
    for (u32 i = 0; i < d->d_out; i++) {
        g_merge[i] = ckks_galois_element(c, -(int32_t)i);
        if (i && (!merge_keys || !merge_keys[i] || merge_keys[i]->galois_elt != g_merge[i]))
            return set_err(c, CKKS_ERR_NO_KEY, "key of a merge rotation missing or wrong");
    }
    std::vector<u32> g_lo(n_lo), g_hi(n_hi);
    for (u32 l = 0; l < n_lo; l++) {
        g_lo[l] = ckks_galois_element(c, (int32_t)(l * delta));
        if (g_lo[l] != 1 && (!lo_keys || !lo_keys[l] || lo_keys[l]->galois_elt != g_lo[l]))
            return set_err(c, CKKS_ERR_NO_KEY, "key of a layout rotation (mod_idx) missing or wrong");
    }
    for (u32 h = 0; h < n_hi; h++) {
        g_hi[h] = ckks_galois_element(c, (int32_t)(h * base * delta));
        if (g_hi[h] != 1 && (!hi_keys || !hi_keys[h] || hi_keys[h]->galois_elt != g_hi[h]))
            return set_err(c, CKKS_ERR_NO_KEY, "key of a layout rotation (base_idx) missing or wrong");
    }
    const size_t N = c->N;
    const size_t ct0 = 2 * (size_t)(level + 1) * N, ct1 = 2 * (size_t)(l1 + 1) * N, ct2 = 2 * (size_t)(l2 + 1) * N, ct3 = 2 * (size_t)(l3 + 1) * N;
    if (!d_ws || ws_bytes < fc_workspace_in(c, d, CT_BATCH, CT_BATCH, CT_BATCH))  // what every batch of eight needs
        return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for the layer");
    // all inner sums together where the workspace is as large as asked for (the merge and the layout look at what is left themselves)
    const u32 nb = ws_bytes >= fc_workspace_in(c, d, fc_batch(c, d), CT_BATCH, CT_BATCH) ? fc_batch(c, d) : CT_BATCH;
    Arena ar(d_ws, ws_bytes);
    u64* prod = ar.take(CT_BATCH * ct0);        // C_in (.) w_i before its rescale
    u64* S = ar.take(d->d_out * ct1);           // running inner sums, level-1
    u64* Srot = ar.take(nb * ct1);              // their rotations
    u64* U = ar.take(ct2);                      // merged, level-2
    KsWs ws;
    if (!carve_ks(c, l1, nb, nb, ar, ws))
        return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for the layer");
    hipStream_t st = (hipStream_t)stream;
    const u64* in = (const u64*)d_in;
    int rc;
    // 1. per-output products and their rescale
    for (u32 i0 = 0; i0 < d->d_out; i0 += CT_BATCH) {
        const u32 n = d->d_out - i0 < CT_BATCH ? d->d_out - i0 : CT_BATCH;
        const u64 *pp[CT_BATCH], *mm[CT_BATCH], *mi[CT_BATCH];
        u64 *os[CT_BATCH], *mo[CT_BATCH];
        for (u32 b = 0; b < n; b++) {
            mm[b] = (const u64*)d_w_enc + (size_t)(i0 + b) * (level + 1) * N;
            mi[b] = in;
            pp[b] = mo[b] = prod + b * ct0;
            os[b] = S + (i0 + b) * ct1;
        }
        HIP_TRY(launch_mask_mul(c, level, mm, mi, mo, n, st));
        if ((rc = run_rescale(c, level, pp, (size_t)(level + 1) * N, os, n, ar.rest(), st))) return rc;
    }
    // inner sums over d_in slots (all outputs of a batch share each rotation key): T <- T + Rot(T, 2^s), the sum rides on the
    // rotation's last kernel, the running sums alternate between two buffers
    for (u32 i0 = 0; i0 < d->d_out; i0 += nb) {
        const u32 n = d->d_out - i0 < nb ? d->d_out - i0 : nb;
        const u64* cur[KS_MAX_BATCH];
        u64 *nxt[KS_MAX_BATCH], *os[KS_MAX_BATCH], *orot[KS_MAX_BATCH];
        for (u32 b = 0; b < n; b++) {
            cur[b] = os[b] = S + (i0 + b) * ct1;
            orot[b] = Srot + b * ct1;
        }
        for (u32 s = 0; s < n_sum; s++) {
            const ckks_key* ks[KS_MAX_BATCH];
            u32 gs[KS_MAX_BATCH];
            for (u32 b = 0; b < n; b++) {
                ks[b] = sum_keys[s];
                gs[b] = g_sum[s];
                nxt[b] = (s & 1) ? os[b] : orot[b];
            }
            if ((rc = run_rotate_batch(c, l1, n, cur, ks, gs, nxt, ws, st, cur))) return rc;
            for (u32 b = 0; b < n; b++) cur[b] = nxt[b];
        }
        if (n_sum & 1)  // an odd number of steps ends in the second buffer
            HIP_TRY(launch_copy(Srot, os[0], n * ct1, st));
    }
    // 2. merge over the outputs: element (j, i) to slot j*d_in + i
    {
        const u64* cts[KS_MAX_BATCH];
        for (u32 i = 0; i < d->d_out; i++) cts[i] = S + i * ct1;
        if ((rc = run_merge(c, cts, d->d_out, l1, (const u64*)d_merge_mask, merge_keys, g_merge, U, ar.rest(), st))) return rc;
    }
    // 3. layout: block j moves left by mod_idx = (j % base)*delta, then by base_idx = (j / base)*base*delta
    u64* out = (u64*)d_out;
    {
        std::vector<const u64*> masks((size_t)n_hi * n_lo, nullptr);
        for (u32 j = 0; j < d->batch; j++) masks[(size_t)(j / base) * n_lo + j % base] = (const u64*)d_place_masks + (size_t)j * (l2 + 1) * N;
        const u64* u_in = U;
        if ((rc = run_relayout(c, l2, 1, &u_in, n_lo, lo_keys, g_lo.data(), n_hi, hi_keys, g_hi.data(), masks.data(), &out, ar.rest(), st)))
            return rc;
    }
    // 4. bias on component 0
    HIP_TRY(launch_add_plain(c, l3, (const u64*)d_bias, out, st));
    return CKKS_OK;
}

int he_poly_act_deg7(const ckks_ctx* c, const uint64_t* const* h_d_x, uint32_t n_ct, uint32_t level, const int64_t* h_k,
                     const ckks_key* rlk, int merged_division, uint64_t* const* h_d_out, void* d_ws, size_t ws_bytes, void* stream) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (!h_d_x || !h_k || !h_d_out || n_ct == 0) return set_err(c, CKKS_ERR_INVALID_ARG, "null pointer or no ciphertexts");
    if (!c->dnum) return set_err(c, CKKS_ERR_UNSUPPORTED_PARAMS, "context has no key-switching digits");
    if (!rlk) return set_err(c, CKKS_ERR_NO_KEY, "no relinearisation key");
    if (rlk->galois_elt != 0) return set_err(c, CKKS_ERR_NO_KEY, "key is a rotation key, not the relinearisation key");
    if (!level_ok(c, level) || level < 4) return set_err(c, CKKS_ERR_LEVEL_MISMATCH, "activation needs 4 <= level < num_q");
    for (u32 i = 0; i < n_ct; i++)
        if (!h_d_x[i] || !h_d_out[i]) return set_err(c, CKKS_ERR_INVALID_ARG, "null ciphertext pointer");
    const size_t N = c->N;
    const u32 l1 = level - 1, l2 = level - 2, l3 = level - 3;
    const size_t xs = (size_t)(level + 1) * N;  // component stride of x
    const size_t x2s = (size_t)(l1 + 1) * N, x3s = (size_t)(l2 + 1) * N, Bs = (size_t)(l3 + 1) * N;
    // Batches of channels are independent: with room for two sets of scratch, every other batch goes to the library's side
    // stream (fork after the caller's earlier work, join before the call returns to the caller's stream).
    // (In a small call up to sixteen go together instead: see act_batch.)
    u32 most = merged_division ? act_batch(c, level, n_ct) : CT_BATCH;
    if (most > CT_BATCH && ws_bytes < ws_poly_act(c, level, n_ct)) most = CT_BATCH;  // in a smaller workspace
    const u32 nb_max = n_ct < most ? n_ct : most;
    const bool want_pairs = merged_division && act_pairs(c, nb_max);
    const u32 want_lanes = n_ct > most && c->side_stream() ? 2 : 1;
    const bool pairs = want_pairs && ws_bytes >= want_lanes * ws_poly_act_in(c, level, nb_max, true);  // else in what one product at a time needs
    const size_t lane_bytes = ws_poly_act_in(c, level, nb_max, pairs);
    const u32 n_lanes = (want_lanes == 2 && ws_bytes >= 2 * lane_bytes) ? 2 : 1;
    if (ws_bytes < lane_bytes || !d_ws) return set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for the activation");
    hipStream_t st0 = (hipStream_t)stream;
    auto residues = [&](int64_t k, u32 lv, u64* out) {
        for (u32 i = 0; i <= lv; i++) {
            const u64 q = c->mod[i];
            out[i] = k >= 0 ? (u64)k % q : (q - ((u64)(-k) % q)) % q;
        }
    };
    u64 ka[CKKS_MAX_MODULI], kb[CKKS_MAX_MODULI];
    if (n_lanes == 2) {
        HIP_TRY(hipEventRecord(c->ev_fork, st0));
        HIP_TRY(hipStreamWaitEvent(c->side, c->ev_fork, 0));
    }
    auto join = [&](int rc) -> int {  // also on the error paths: the caller's stream never runs ahead of the side stream
        if (n_lanes == 2) {
            hipError_t e = hipEventRecord(c->ev_join, c->side);
            if (e == hipSuccess) e = hipStreamWaitEvent(st0, c->ev_join, 0);
            if (e != hipSuccess && rc == CKKS_OK) {
                c->err = std::string("joining the side stream: ") + hipGetErrorString(e);
                return CKKS_ERR_HIP;
            }
        }
        return rc;
    };

    for (u32 i0 = 0, batch_no = 0; i0 < n_ct; i0 += most, batch_no++) {
        const u32 n = n_ct - i0 < most ? n_ct - i0 : most;
        const u32 lane = n_lanes == 2 ? (batch_no & 1) : 0;
        hipStream_t st = lane ? c->side : st0;
        Arena ar((char*)d_ws + (size_t)lane * lane_bytes, lane_bytes);
        u64* x2 = ar.take(nb_max * 2 * x2s);        // level-1
        u64* x3 = ar.take(nb_max * 2 * x3s);        // level-2
        u64* x4 = ar.take(nb_max * 2 * x3s);        // level-2
        u64* B = ar.take(nb_max * 2 * Bs);          // level-3
        u64* tmp = ar.take(nb_max * 2 * xs);        // un-rescaled products
        if (!ar.ok()) return join(set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for the activation"));
        // pointer lists of this batch: inputs, and the per-item slices of the intermediates
        const u64 *px[KS_MAX_BATCH], *px2[KS_MAX_BATCH], *px3[KS_MAX_BATCH], *px4[KS_MAX_BATCH], *pB[KS_MAX_BATCH], *ptmp[KS_MAX_BATCH];
        u64 *ox2[KS_MAX_BATCH], *ox3[KS_MAX_BATCH], *ox4[KS_MAX_BATCH], *oB[KS_MAX_BATCH], *otmp[KS_MAX_BATCH], *oout[KS_MAX_BATCH];
        for (u32 b = 0; b < n; b++) {
            px[b] = (const u64*)h_d_x[i0 + b];
            px2[b] = ox2[b] = x2 + b * 2 * x2s;
            px3[b] = ox3[b] = x3 + b * 2 * x3s;
            px4[b] = ox4[b] = x4 + b * 2 * x3s;
            pB[b] = oB[b] = B + b * 2 * Bs;
            oout[b] = (u64*)h_d_out[i0 + b];
        }
        auto tmp_at = [&](size_t cstride) {  // un-rescaled results, compact at the level that produced them
            for (u32 b = 0; b < n; b++) ptmp[b] = otmp[b] = tmp + b * 2 * cstride;
        };
        int rc;
        if (merged_division) {  // every relinearise-then-rescale pair as one division by P*q_level
            if ((rc = run_ctct_merged(c, level, px, xs, px, xs, nullptr, 0, rlk->d_key, ox2, n, ar.rest(), st))) return join(rc);
            if (pairs) {  // the products by x and by x^2 side by side: operands with two component strides
                const u64 *pa[KS_MAX_BATCH], *pb0[KS_MAX_BATCH], *pb1[KS_MAX_BATCH];
                u64* po[KS_MAX_BATCH];
                for (u32 b = 0; b < n; b++) {
                    pa[b] = pa[n + b] = px2[b];
                    pb0[b] = px[b], pb1[b] = px[b] + xs, po[b] = ox3[b];
                    pb0[n + b] = px2[b], pb1[n + b] = px2[b] + x2s, po[n + b] = ox4[b];
                }
                KsWs ws;
                Arena sub = ar.rest();
                if (!carve_ks(c, l1, 2 * n, 2 * n, sub, ws)) return join(set_err(c, CKKS_ERR_WORKSPACE_TOO_SMALL, "workspace too small for the activation"));
                if ((rc = run_product(c, l1, pa, x2s, pb0, pb1, rlk->d_key, po, 2 * n, ws, st, true))) return join(rc);
            } else {
                if ((rc = run_ctct_merged(c, l1, px2, x2s, px, xs, nullptr, 0, rlk->d_key, ox3, n, ar.rest(), st))) return join(rc);
                if ((rc = run_ctct_merged(c, l1, px2, x2s, px2, x2s, nullptr, 0, rlk->d_key, ox4, n, ar.rest(), st))) return join(rc);
            }
            residues(h_k[2], l2, ka);
            residues(h_k[3], l2, kb);
            if (ntt_has_modup(c)) {  // B = Rescale(k5 * x + k7 * x3) without storing the linear combination
                for (u32 b0 = 0; b0 < n; b0 += CT_BATCH)
                    if ((rc = run_rescale_lin(c, l2, px + b0, xs, ka, px3 + b0, x3s, kb, oB + b0, n - b0 < CT_BATCH ? n - b0 : CT_BATCH, ar.rest(), st))) return join(rc);
            } else {
                tmp_at(x3s);
                if (hipError_t he_ = (launch_lincomb2(c, l2, ptr_list(px, n), xs, ka, ptr_list(px3, n), x3s, kb, nullptr, 0, tmp, 2 * x3s, n, st)); he_ != hipSuccess) return join(set_hip_err(c, he_));
                if ((rc = run_rescale(c, l2, ptmp, x3s, oB, n, ar.rest(), st))) return join(rc);
            }
            // y = Rescale(x4 * B + (k1 * x + k3 * x3)): the linear part rides along as the product's addend
            residues(h_k[0], l3, ka);
            residues(h_k[1], l3, kb);
            if (ntt_has_modup(c)) {  // the linear part is formed inside the product's fused inner product
                const LinAddend lin = {px, xs, ka, px3, x3s, kb};
                if ((rc = run_ctct_merged(c, l3, px4, x3s, pB, Bs, nullptr, 0, rlk->d_key, oout, n, ar.rest(), st, &lin))) return join(rc);
                continue;
            }
            if (hipError_t he_ = (launch_lincomb2(c, l3, ptr_list(px, n), xs, ka, ptr_list(px3, n), x3s, kb, nullptr, 0, tmp, 2 * Bs, n, st)); he_ != hipSuccess) return join(set_hip_err(c, he_));
            if ((rc = run_ctct_merged(c, l3, px4, x3s, pB, Bs, tmp, 2 * Bs, rlk->d_key, oout, n, ar.rest(), st))) return join(rc);
            continue;
        }
        // x2 = Rescale(x * x)                                  level -> level-1
        tmp_at(xs);
        if ((rc = run_ctct(c, level, px, xs, px, xs, rlk->d_key, otmp, n, ar.rest(), st))) return join(rc);
        if ((rc = run_rescale(c, level, ptmp, xs, ox2, n, ar.rest(), st))) return join(rc);
        // x3 = Rescale(x2 * x), x4 = Rescale(x2 * x2)           level-1 -> level-2
        tmp_at(x2s);
        if ((rc = run_ctct(c, l1, px2, x2s, px, xs, rlk->d_key, otmp, n, ar.rest(), st))) return join(rc);
        if ((rc = run_rescale(c, l1, ptmp, x2s, ox3, n, ar.rest(), st))) return join(rc);
        if ((rc = run_ctct(c, l1, px2, x2s, px2, x2s, rlk->d_key, otmp, n, ar.rest(), st))) return join(rc);
        if ((rc = run_rescale(c, l1, ptmp, x2s, ox4, n, ar.rest(), st))) return join(rc);
        // B = Rescale(k5 * x + k7 * x3)                         level-2 -> level-3
        residues(h_k[2], l2, ka);
        residues(h_k[3], l2, kb);
        tmp_at(x3s);
        if (hipError_t he_ = (launch_lincomb2(c, l2, ptr_list(px, n), xs, ka, ptr_list(px3, n), x3s, kb, nullptr, 0, tmp, 2 * x3s, n, st)); he_ != hipSuccess) return join(set_hip_err(c, he_));
        if ((rc = run_rescale(c, l2, ptmp, x3s, oB, n, ar.rest(), st))) return join(rc);
        // y = Rescale((k1 * x + k3 * x3) + x4 * B)              level-3 -> level-4
        u64* prod = x2;  // x2 is no longer needed; n * [2][l3+1][N] fits in it
        u64* oprod[CT_BATCH];
        for (u32 b = 0; b < n; b++) oprod[b] = prod + b * 2 * Bs;
        if ((rc = run_ctct(c, l3, px4, x3s, pB, Bs, rlk->d_key, oprod, n, ar.rest(), st))) return join(rc);
        residues(h_k[0], l3, ka);
        residues(h_k[1], l3, kb);
        tmp_at(Bs);
        if (hipError_t he_ = (launch_lincomb2(c, l3, ptr_list(px, n), xs, ka, ptr_list(px3, n), x3s, kb, prod, 2 * Bs, tmp, 2 * Bs, n, st)); he_ != hipSuccess) return join(set_hip_err(c, he_));
        if ((rc = run_rescale(c, l3, ptmp, Bs, oout, n, ar.rest(), st))) return join(rc);
    }
    return join(CKKS_OK);
}

// ---- optional per-kernel timing -------------------------------------------------------------------
static const char* const kKernelNames[K_COUNT] = {
    "ntt_fwd_hi", "ntt_fwd_lo", "ntt_inv_lo", "ntt_inv_hi", "modup_conv", "key_inner", "moddown_conv", "moddown_final",
    "automorph", "copy", "ptct_mac", "rescale_conv", "rescale_final", "tensor", "mask_mul", "weighted_sum", "lincomb2"};

uint32_t ckks_prof_kernel_count(void) { return K_COUNT; }
const char* ckks_prof_kernel_name(uint32_t id) { return id < K_COUNT ? kKernelNames[id] : ""; }

int ckks_prof_begin(ckks_ctx* c, uint32_t kernel_mask, uint32_t max_launches) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    if (c->prof) return set_err(c, CKKS_ERR_INVALID_ARG, "profiling already on");
    if (max_launches == 0) return set_err(c, CKKS_ERR_INVALID_ARG, "max_launches must be positive");
    ProfState* p = new (std::nothrow) ProfState;
    if (!p) return set_err(c, CKKS_ERR_INVALID_ARG, "out of host memory");
    p->mask = kernel_mask;
    p->events.resize(2 * (size_t)max_launches);
    p->kernel_of_pair.resize(max_launches);
    for (size_t i = 0; i < p->events.size(); i++) {
        hipError_t e = hipEventCreate(&p->events[i]);
        if (e != hipSuccess) {
            for (size_t j = 0; j < i; j++) (void)hipEventDestroy(p->events[j]);
            delete p;
            c->err = std::string("hipEventCreate: ") + hipGetErrorString(e);
            return CKKS_ERR_HIP;
        }
    }
    c->prof = p;
    return CKKS_OK;
}

int ckks_prof_end(ckks_ctx* c, double* h_ms, uint64_t* h_launches, double* h_bytes, double* h_ops, uint64_t* h_dropped) {
    if (!c) return CKKS_ERR_INVALID_ARG;
    ProfState* p = c->prof;
    if (!p) return set_err(c, CKKS_ERR_INVALID_ARG, "profiling is not on");
    c->prof = nullptr;
    int rc = CKKS_OK;
    for (u32 k = 0; k < K_COUNT; k++) {
        if (h_ms) h_ms[k] = 0.0;
        if (h_launches) h_launches[k] = 0;
        if (h_bytes) h_bytes[k] = p->bytes[k];
        if (h_ops) h_ops[k] = p->ops[k];
    }
    for (size_t i = 0; i < p->used_pairs && rc == CKKS_OK; i++) {
        hipError_t e = hipEventSynchronize(p->events[2 * i + 1]);
        float ms = 0.f;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, p->events[2 * i], p->events[2 * i + 1]);
        if (e != hipSuccess) {
            c->err = std::string("profiling events: ") + hipGetErrorString(e);
            rc = CKKS_ERR_HIP;
            break;
        }
        if (h_ms) h_ms[p->kernel_of_pair[i]] += ms;
        if (h_launches) h_launches[p->kernel_of_pair[i]]++;
    }
    if (h_dropped) *h_dropped = p->dropped;
    for (hipEvent_t ev : p->events) (void)hipEventDestroy(ev);
    delete p;
    return rc;
}

}  // extern "C"
