// Hybrid (digit-decomposed) key switching for gfx950: the arithmetic behind every Rot and every
// relinearisation (Background, "Rotations and Key Switching"; Experiments, "HE Security
// Parameters": key switching with digits).
//
//   ModUp      digit j's limbs (coefficient form) -> all live q-limbs and the special primes:
//              y_a = [c_a * (Q_j/q_a)^-1] mod q_a  taken centred in [-(q_a-1)/2, (q_a-1)/2],
//              d_j[t] = sum_a y_a * [Q_j/q_a]_t  mod t          (plain sum, no correction term).
//              Computed on the unsigned residues plus  (#negative y_a) * (-Q_j mod t), which is
//              the same integer modulo t because q_a * (Q_j/q_a) = Q_j.
//   inner      v_comp[t] = sum_j sigma_g(d_j)[t] * key[j][comp][t]   (sigma_g = gather, g = 1: none)
//   ModDown    z_a = [v_{p_a} * (P/p_a)^-1] mod p_a centred,  w[i] = sum_a z_a * [P/p_a]_{q_i}
//              (coefficient form, same negative-count trick with -P mod q_i), then in NTT form
//              u[i] = (v[q_i] - w[i]) * P^-1  (+ an optional addend)
// Sums of products are accumulated unreduced in 128 bits and reduced once.
#include "ctx.h"
#include "f64mod.h"
#include "galois.h"

#define KS_THREADS 256
#define KS_MAX_DIGIT 16  // limbs per digit / special primes handled in registers

// row [N] of (batch item b, digit j, extended-basis position e): see DigitSrc
__device__ __forceinline__ const u64* digit_row(const DigitSrc& D, u32 b, u32 j, u32 e, u32 E, u32 N, u32 level) {
    if (e <= level && e / D.alpha == j) return D.own.p[b] + (size_t)e * N;
    return D.digits + b * D.bstride + ((size_t)j * E + e) * N;
}

// ---- ModUp: basis extension of one digit --------------------------------------------------------
// y     [nd][N]      digit limbs in coefficient form (canonical)
// digit [E][N]       out: every limb but the digit's own, in coefficient form (the own limbs stay where they are: DigitSrc)
// This one takes digits j0 .. j0 + nj - 1 of every polynomial: y [level+1][N], digit [beta][E][N], tab the table of digit j0,
// the next digit's tab_stride on; size: limbs per digit (the last may have fewer).
__global__ __launch_bounds__(KS_THREADS) void modup_conv_kernel(const u64* __restrict__ y, size_t y_bstride,
                                                                u64* __restrict__ digit, size_t digit_bstride,
                                                                const u64* __restrict__ tab, size_t tab_stride, const ModConst* __restrict__ mc, u32 N,
                                                                u32 level, u32 num_q, u32 size, u32 j0, u32 nj, u32 alpha, u32 M, u32 E, u32 lpb) {
    const u32 x = blockIdx.x * KS_THREADS + threadIdx.x;
    if (x >= N) return;
    const u32 b = blockIdx.z / nj, dj = blockIdx.z - b * nj, lo = (j0 + dj) * size, nd = min(size, level + 1 - lo);
    y += b * y_bstride + (size_t)lo * N;
    digit += b * digit_bstride + (size_t)(j0 + dj) * E * N;
    tab += dj * tab_stride;
    u64 yv[KS_MAX_DIGIT];
    u64 n_neg = 0;
#pragma unroll
    for (u32 a = 0; a < KS_MAX_DIGIT; a++)
        if (a < nd) {
            const u64 qa = mc[lo + a].q;
            yv[a] = mul_shoup(y[(size_t)a * N + x], tab[a], tab[alpha + a], qa);
            n_neg += yv[a] > (qa >> 1) ? 1 : 0;
        }
    const u64* negq = tab + (size_t)alpha * (2 + M);  // alpha = padded row length here
    const u32 e0 = blockIdx.y * lpb;
    for (u32 e = e0; e < e0 + lpb && e < E; e++) {
        const u32 t = e <= level ? e : num_q + (e - level - 1);
        if (t >= lo && t < lo + nd) continue;  // the digit's own limbs are read from the polynomial itself (DigitSrc)
        U128 acc = {0, 0};
#pragma unroll
        for (u32 a = 0; a < KS_MAX_DIGIT; a++)
            if (a < nd) acc_wide(acc, yv[a], tab[2 * alpha + (size_t)e * alpha + a]);
        acc_wide(acc, n_neg, negq[e]);
        digit[(size_t)e * N + x] = barrett_reduce(acc, mc[t]);
    }
}

// ModUp for moduli below 2^50: carry-free 25-bit-split accumulation (three multiply-adds per term).
// AP = padded digit size: the AP constants of a target limb are one aligned run (wide scalar load).
template <int AP>
__global__ __launch_bounds__(KS_THREADS) void modup_conv50_kernel(const u64* __restrict__ y, size_t y_bstride,
                                                                  u64* __restrict__ digit, size_t digit_bstride,
                                                                  const u64* __restrict__ tab, const ModConst* __restrict__ mc, u32 N,
                                                                  u32 level, u32 num_q, u32 lo, u32 nd, u32 M, u32 E, u32 lpb) {
    const u32 x = blockIdx.x * KS_THREADS + threadIdx.x;
    if (x >= N) return;
    y += blockIdx.z * y_bstride;
    digit += blockIdx.z * digit_bstride;
    Split50 yv[AP];
    u32 n_neg = 0;
#pragma unroll
    for (u32 a = 0; a < AP; a++) {
        yv[a] = {0, 0, 0};
        if (a < nd) {
            const u64 qa = mc[lo + a].q;
            const u64 v = mul_shoup(y[(size_t)a * N + x], tab[a], tab[AP + a], qa);
            n_neg += v > (qa >> 1) ? 1 : 0;
            yv[a] = split50(v);
        }
    }
    const u64* conv = (const u64*)__builtin_assume_aligned(tab + 2 * AP, 8 * AP);
    const u64* negq = tab + (size_t)AP * (2 + M);
    const u32 e0 = blockIdx.y * lpb;
    for (u32 e = e0; e < e0 + lpb && e < E; e++) {
        const u32 t = e <= level ? e : num_q + (e - level - 1);
        if (t >= lo && t < lo + nd) continue;  // the digit's own limbs are read from the polynomial itself (DigitSrc)
        const u64* ce = (const u64*)__builtin_assume_aligned(conv + (size_t)e * AP, 8 * AP);
        u64 cv[AP];
#pragma unroll
        for (u32 a = 0; a < AP; a++) cv[a] = ce[a];
        Acc50 acc = {0, 0, 0};
#pragma unroll
        for (u32 a = 0; a < AP; a++) acc50_mad(acc, yv[a], split50(cv[a]));
        U128 v = acc50_value(acc);
        acc_wide(v, n_neg, negq[e]);
        digit[(size_t)e * N + x] = barrett_reduce(v, mc[t]);
    }
}

// ModUp for moduli below 2^50 in double precision (the ring of 2^11 points): the centred residues of the digit as doubles, summed
// in chains of fused multiply-adds of up to eight terms, each chain reduced once (f64m_dot).  No correction for the negative
// terms is needed, their representatives are negative doubles.  convf: [E][AP] (centred constant, its quotient, not read).
template <int AP>
__global__ __launch_bounds__(KS_THREADS) void modup_conv_f64_kernel(const u64* __restrict__ y, size_t y_bstride,
                                                                    u64* __restrict__ digit, size_t digit_bstride,
                                                                    const u64* __restrict__ tab, const TwF* __restrict__ convf,
                                                                    const ModConst* __restrict__ mc, const ModConstF* __restrict__ mcf,
                                                                    u32 N, u32 level, u32 num_q, u32 lo, u32 nd, u32 E, u32 lpb) {
    const u32 x = blockIdx.x * KS_THREADS + threadIdx.x;
    if (x >= N) return;
    y += blockIdx.z * y_bstride;
    digit += blockIdx.z * digit_bstride;
    double yd[AP];
#pragma unroll
    for (u32 a = 0; a < AP; a++) {
        yd[a] = 0.0;
        if (a < nd) {
            const u64 qa = mc[lo + a].q;
            const u64 v = mul_shoup(y[(size_t)a * N + x], tab[a], tab[AP + a], qa);
            yd[a] = v > (qa >> 1) ? -f64m_from_u64(qa - v) : f64m_from_u64(v);
        }
    }
    const u32 e0 = blockIdx.y * lpb;
    for (u32 e = e0; e < e0 + lpb && e < E; e++) {
        const u32 t = e <= level ? e : num_q + (e - level - 1);
        if (t >= lo && t < lo + nd) continue;  // the digit's own limbs are read from the polynomial itself (DigitSrc)
        const TwF* ce = (const TwF*)__builtin_assume_aligned(convf + (size_t)e * AP, 16 * AP);
        const double q = mcf[t].q, qinv = mcf[t].qinv;
        digit[(size_t)e * N + x] = f64m_canonical(f64m_dot<AP>(yd, ce, q, qinv), q);
    }
}

// Digits j .. j + nj - 1 of n <= KS_MAX_BATCH polynomials at once (nj > 1 only with moduli of 2^50 and above): item b reads
// y + b*y_bstride ([level+1][N]), writes digits + b*digit_bstride ([beta][E][N])
hipError_t launch_modup_conv(const ckks_ctx* c, u32 level, u32 j, u32 nj, const u64* y, size_t y_bstride, u64* digits,
                             size_t digit_bstride, u32 n, hipStream_t st) {
    const u32 E = c->ext_limbs(level), lo = c->digit_lo(j), nd = c->digit_hi(j, level) - lo;
    if (nj == 0 || j + nj > c->live_digits(level) || (nj > 1 && c->small_q)) return hipErrorInvalidValue;
    u64* digit = digits + (size_t)j * E * c->N;
    const u64* y_all = y;
    y += (size_t)lo * c->N;
    // target limbs per thread: the digit's prepared residues are reused for all of them, but a small batch needs the
    // limbs spread over more workgroups to fill the chip
    const u32 x_wgs = (c->N + KS_THREADS - 1) / KS_THREADS;
    const u32 lpb = x_wgs * n * nj >= 1024 ? 32 : (x_wgs * n * nj >= 512 ? 8 : 4);
    dim3 grid(x_wgs, (E + lpb - 1) / lpb, n * nj);
    const u64* tab = c->modup_table(level, j);
    ProfScope ps__(c, K_MODUP_CONV, st, 8.0 * n * nj * c->N * (2.0 * nd + E), (double)n * nj * c->N * nd * (1.0 + E - nd));
    if (c->ntt_f64 && c->d_modup_f) {
        const TwF* tf = c->modup_table_f(level, j);
        if (c->alpha_pad == 4)
            hipLaunchKernelGGL(modup_conv_f64_kernel<4>, grid, dim3(KS_THREADS), 0, st, y, y_bstride, digit, digit_bstride, tab, tf, c->d_mc, c->d_mcf, c->N, level, c->num_q, lo, nd, E, lpb);
        else if (c->alpha_pad == 8)
            hipLaunchKernelGGL(modup_conv_f64_kernel<8>, grid, dim3(KS_THREADS), 0, st, y, y_bstride, digit, digit_bstride, tab, tf, c->d_mc, c->d_mcf, c->N, level, c->num_q, lo, nd, E, lpb);
        else
            hipLaunchKernelGGL(modup_conv_f64_kernel<16>, grid, dim3(KS_THREADS), 0, st, y, y_bstride, digit, digit_bstride, tab, tf, c->d_mc, c->d_mcf, c->N, level, c->num_q, lo, nd, E, lpb);
    } else if (c->small_q) {
        if (c->alpha_pad == 4)
            hipLaunchKernelGGL(modup_conv50_kernel<4>, grid, dim3(KS_THREADS), 0, st, y, y_bstride, digit, digit_bstride, tab, c->d_mc, c->N, level, c->num_q, lo, nd, c->M, E, lpb);
        else if (c->alpha_pad == 8)
            hipLaunchKernelGGL(modup_conv50_kernel<8>, grid, dim3(KS_THREADS), 0, st, y, y_bstride, digit, digit_bstride, tab, c->d_mc, c->N, level, c->num_q, lo, nd, c->M, E, lpb);
        else
            hipLaunchKernelGGL(modup_conv50_kernel<16>, grid, dim3(KS_THREADS), 0, st, y, y_bstride, digit, digit_bstride, tab, c->d_mc, c->N, level, c->num_q, lo, nd, c->M, E, lpb);
    } else {
        hipLaunchKernelGGL(modup_conv_kernel, grid, dim3(KS_THREADS), 0, st, y_all, y_bstride, digits, digit_bstride, tab, c->modup_digit_stride(),
                           c->d_mc, c->N, level, c->num_q, c->alpha, j, nj, c->alpha_pad, c->M, E, lpb);
    }
    return hipGetLastError();
}

// ---- inner product with the switching key ------------------------------------------------------
// Of n <= CT_BATCH key switches in one launch: item b has its digits ([beta][E][N], see DigitSrc), key ([dnum][2][M][N]) and
// Galois element; results v + b*v_bstride: [2][E][N].  blockIdx.z = a run of neighbouring items with the same key (the channels
// of a layer share their rotation and relinearisation keys): every thread keeps its key words while it walks the run, so the key
// streams from HBM once per run.  add0 (optional, [level+1][N]): P sigma_g(add0) joins component 0 on the live q-limbs, which
// makes the division by P that follows the whole rotation, with no gather left in it.
// F64 (every modulus below 2^50, at most four digits): the sums as chains of fused multiply-adds on centred doubles
// (f64m_dot_w), as in the fused taps; otherwise 128-bit integer sums.
// (As a launch per key, rotations of 9 to 11 extended limbs at N = 2^16 were 8 us each; up to eight now take 27 us together.)
struct KeyItems {
    const u64* key[CT_BATCH];
    const u64* add0[CT_BATCH];
    u32 g[CT_BATCH];
    u32 first[CT_BATCH + 1];  // run r: items first[r] .. first[r + 1] - 1
};
template <bool F64, bool ADD>
__global__ __launch_bounds__(KS_THREADS) void key_inner_items_kernel(DigitSrc digits, KeyItems K, u64* __restrict__ v, size_t v_bstride,
                                                                     const u64* __restrict__ negp, const ModConst* __restrict__ mc, u32 log_n,
                                                                     u32 level, u32 num_q, u32 M, u32 E, u32 beta,
                                                                     const ModConstF* __restrict__ mcf) {
    const u32 N = 1u << log_n;
    const u32 x = blockIdx.x * KS_THREADS + threadIdx.x;
    if (x >= N) return;
    const u32 e = blockIdx.y, b0 = K.first[blockIdx.z], b1 = K.first[blockIdx.z + 1];
    const u32 t = e <= level ? e : num_q + (e - level - 1);
    const u32 g = K.g[b0];
    const u64* __restrict__ key = K.key[b0];
    const u32 xs = g == 1 ? x : galois_gather_index(x, g, log_n);
    const ModConst m = mc[t];
    const bool has_add = ADD && e <= level;
    const u64 pres = has_add ? m.q - negp[e] : 0;  // P mod q_e
    if constexpr (F64) {  // beta <= 4: entries past the last digit are zero on both sides
        const double qd = mcf[t].q, qinv = mcf[t].qinv, halfq = 0.5 * qd;
        auto centred = [&](u64 w) {
            const double d = f64m_from_u64(w);
            return d > halfq ? d - qd : d;
        };
        double w0[5], w1[4];
#pragma unroll
        for (u32 j = 0; j < 4; j++) {
            w0[j] = j < beta ? centred(key[(((size_t)j * 2 + 0) * M + t) * N + x]) : 0.0;
            w1[j] = j < beta ? centred(key[(((size_t)j * 2 + 1) * M + t) * N + x]) : 0.0;
        }
        w0[4] = centred(pres);
        for (u32 b = b0; b < b1; b++) {
            double y[5];
#pragma unroll
            for (u32 j = 0; j < 4; j++) y[j] = j < beta ? centred(digit_row(digits, b, j, e, E, N, level)[xs]) : 0.0;
            y[4] = has_add ? centred(K.add0[b][(size_t)e * N + xs]) : 0.0;
            u64* vb = v + b * v_bstride;
            vb[((size_t)0 * E + e) * N + x] = f64m_canonical(f64m_dot_w<ADD ? 5 : 4>(y, w0, qd, qinv), qd);
            vb[((size_t)1 * E + e) * N + x] = f64m_canonical(f64m_dot_w<4>(y, w1, qd, qinv), qd);
        }
        return;
    }
    u64 k0[4], k1[4];  // beta <= 4: the thread's key words stay in registers for the whole run
    if (beta <= 4) {
#pragma unroll
        for (u32 j = 0; j < 4; j++) {
            k0[j] = j < beta ? key[(((size_t)j * 2 + 0) * M + t) * N + x] : 0;
            k1[j] = j < beta ? key[(((size_t)j * 2 + 1) * M + t) * N + x] : 0;
        }
    }
    for (u32 b = b0; b < b1; b++) {
        U128 acc0 = {0, 0}, acc1 = {0, 0};
        if (has_add) acc_wide(acc0, K.add0[b][(size_t)e * N + xs], pres);
        if (beta <= 4) {
#pragma unroll
            for (u32 j = 0; j < 4; j++) {
                const u64 dv = j < beta ? digit_row(digits, b, j, e, E, N, level)[xs] : 0;
                acc_wide(acc0, dv, k0[j]);
                acc_wide(acc1, dv, k1[j]);
            }
        } else {
            for (u32 j = 0; j < beta; j++) {
                const u64 dv = digit_row(digits, b, j, e, E, N, level)[xs];
                acc_wide(acc0, dv, key[(((size_t)j * 2 + 0) * M + t) * N + x]);
                acc_wide(acc1, dv, key[(((size_t)j * 2 + 1) * M + t) * N + x]);
                if ((j & 15) == 15) {  // keep the unreduced sums inside the Barrett input range
                    acc0.lo = barrett_reduce(acc0, m); acc0.hi = 0;
                    acc1.lo = barrett_reduce(acc1, m); acc1.hi = 0;
                }
            }
        }
        u64* vb = v + b * v_bstride;
        vb[((size_t)0 * E + e) * N + x] = barrett_reduce(acc0, m);
        vb[((size_t)1 * E + e) * N + x] = barrett_reduce(acc1, m);
    }
}

// keys / gs / add0s (or null): host arrays of n entries
hipError_t launch_key_inner_items(const ckks_ctx* c, u32 level, const DigitSrc& digits, const u64* const* keys, const u32* gs,
                                  const u64* const* add0s, u64* v, size_t v_bstride, u32 n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    if (n > CT_BATCH) return hipErrorInvalidValue;
    const u32 E = c->ext_limbs(level), beta = c->live_digits(level);
    KeyItems K = {};
    u32 runs = 0;
    for (u32 b = 0; b < n; b++) {
        K.key[b] = keys[b];
        K.g[b] = gs[b];
        K.add0[b] = add0s ? add0s[b] : nullptr;
        if (!keys[b] || (add0s && !add0s[b])) return hipErrorInvalidValue;
        if (b == 0 || keys[b] != keys[b - 1] || gs[b] != gs[b - 1]) K.first[runs++] = b;
    }
    K.first[runs] = n;
    const u64* negp = c->d_moddown + 2 * c->k_pad + (size_t)c->k_pad * c->num_q + 2 * c->num_q;
    dim3 grid((c->N + KS_THREADS - 1) / KS_THREADS, E, runs);
    ProfScope ps__(c, K_KEY_INNER, st, 8.0 * c->N * (E * (2.0 * beta * runs + n * (beta + 2.0)) + (add0s ? n * (level + 1.0) : 0.0)), 2.0 * n * c->N * E * beta);
#define KI_ITEMS(F64_, ADD_) hipLaunchKernelGGL((key_inner_items_kernel<F64_, ADD_>), grid, dim3(KS_THREADS), 0, st, digits, K, v, v_bstride, negp, c->d_mc, c->log_n, level, c->num_q, c->M, E, beta, c->d_mcf)
    const bool f64 = c->small_q && beta <= 4;
    if (f64 && add0s) KI_ITEMS(true, true);
    else if (f64) KI_ITEMS(true, false);
    else if (add0s) KI_ITEMS(false, true);
    else KI_ITEMS(false, false);
#undef KI_ITEMS
    return hipGetLastError();
}

// The inner product of a batch, finished for an operation that divides by P later (the convolution that
// takes one ModDown per output channel after its sum; the ciphertext product whose ModDown is merged with
// the rescale): on all E limbs of the extended basis,
//   out_b[comp][e][x] = mask[e][x] * ( v_b[comp][e][x] + (e <= level ? [P]_{q_e} * add_comp,b[e][sigma_g x] : 0) )
// add0 / add1 [level+1][N] (optional) are what the result of the key switch would have been added to
// (Rot: c0; relinearisation: d0, d1); P times them vanishes on the special primes and joins the
// unreduced 128-bit sum as one more term.  mask [E][N] (optional): a plaintext on the extended basis.
struct ExtItems {
    const u64* add0[KS_MAX_BATCH];
    const u64* add1[KS_MAX_BATCH];
    u64* out[KS_MAX_BATCH];
};

__global__ __launch_bounds__(KS_THREADS) void key_inner_ext_kernel(DigitSrc digits, const u64* __restrict__ key, ExtItems items,
                                                                   const u64* __restrict__ mask, const u64* __restrict__ negp,
                                                                   const ModConst* __restrict__ mc, u32 log_n, u32 level, u32 num_q,
                                                                   u32 M, u32 E, u32 beta, u32 g, u32 n) {
    const u32 N = 1u << log_n;
    const u32 x = blockIdx.x * KS_THREADS + threadIdx.x;
    if (x >= N) return;
    const u32 e = blockIdx.y;
    const u32 t = e <= level ? e : num_q + (e - level - 1);
    const u32 xs = g == 1 ? x : galois_gather_index(x, g, log_n);
    const ModConst m = mc[t];
    const bool has_mask = mask != nullptr;
    const u64 mk = has_mask ? mask[(size_t)e * N + x] : 0;
    const bool has_add = e <= level;
    const u64 pres = has_add ? m.q - negp[e] : 0;  // P mod q_e
    u64 k0[4], k1[4];  // beta <= 4: the thread's key words stay in registers for the whole batch
    if (beta <= 4) {
#pragma unroll
        for (u32 j = 0; j < 4; j++) {
            k0[j] = j < beta ? key[(((size_t)j * 2 + 0) * M + t) * N + x] : 0;
            k1[j] = j < beta ? key[(((size_t)j * 2 + 1) * M + t) * N + x] : 0;
        }
    }
    for (u32 b = 0; b < n; b++) {
        U128 acc0 = {0, 0}, acc1 = {0, 0};
        if (beta <= 4) {
#pragma unroll
            for (u32 j = 0; j < 4; j++) {
                const u64 dv = j < beta ? digit_row(digits, b, j, e, E, N, level)[xs] : 0;
                acc_wide(acc0, dv, k0[j]);
                acc_wide(acc1, dv, k1[j]);
            }
        } else {
            for (u32 j = 0; j < beta; j++) {
                const u64 dv = digit_row(digits, b, j, e, E, N, level)[xs];
                acc_wide(acc0, dv, key[(((size_t)j * 2 + 0) * M + t) * N + x]);
                acc_wide(acc1, dv, key[(((size_t)j * 2 + 1) * M + t) * N + x]);
                if ((j & 15) == 15) {
                    acc0.lo = barrett_reduce(acc0, m); acc0.hi = 0;
                    acc1.lo = barrett_reduce(acc1, m); acc1.hi = 0;
                }
            }
        }
        if (has_add && items.add0[b]) acc_wide(acc0, items.add0[b][(size_t)e * N + xs], pres);
        if (has_add && items.add1[b]) acc_wide(acc1, items.add1[b][(size_t)e * N + xs], pres);
        u64 r0 = barrett_reduce(acc0, m), r1 = barrett_reduce(acc1, m);
        if (has_mask) {
            r0 = mulmod_barrett(r0, mk, m);
            r1 = mulmod_barrett(r1, mk, m);
        }
        u64* ob = items.out[b];
        ob[((size_t)0 * E + e) * N + x] = r0;
        ob[((size_t)1 * E + e) * N + x] = r1;
    }
}

// add0s / add1s / outs: host arrays of n <= KS_MAX_BATCH device pointers ([level+1][N], [level+1][N], [2][E][N]);
// add0s, add1s or single entries of them may be null
hipError_t launch_key_inner_ext(const ckks_ctx* c, u32 level, const DigitSrc& digits, const u64* key, u32 g,
                                const u64* const* add0s, const u64* const* add1s, const u64* mask, u64* const* outs, u32 n,
                                hipStream_t st) {
    const u32 E = c->ext_limbs(level), beta = c->live_digits(level);
    ExtItems items;
    double n_add = 0.0;
    for (u32 b = 0; b < KS_MAX_BATCH; b++) {
        items.add0[b] = (b < n && add0s) ? add0s[b] : nullptr;
        items.add1[b] = (b < n && add1s) ? add1s[b] : nullptr;
        items.out[b] = b < n ? outs[b] : nullptr;
        n_add += (items.add0[b] ? 1.0 : 0.0) + (items.add1[b] ? 1.0 : 0.0);
    }
    const u64* negp = c->d_moddown + 2 * c->k_pad + (size_t)c->k_pad * c->num_q + 2 * c->num_q;
    dim3 grid((c->N + KS_THREADS - 1) / KS_THREADS, E);
    ProfScope ps__(c, K_KEY_INNER, st, 8.0 * c->N * (E * (2.0 * beta + (mask ? 1.0 : 0.0) + n * (beta + 2.0)) + n_add * (level + 1.0)),
                   2.0 * n * c->N * E * (beta + 1.0));
    hipLaunchKernelGGL(key_inner_ext_kernel, grid, dim3(KS_THREADS), 0, st, digits, key, items, mask, negp, c->d_mc,
                       c->log_n, level, c->num_q, c->M, E, beta, g, n);
    return hipGetLastError();
}

// All the taps of a convolution for a batch of input channels in one launch: the same arithmetic as
// key_inner_ext_kernel (P * sigma_g(c0) added, tap mask multiplied in) for up to 8 (key, Galois element,
// mask) triples, organised by SOURCE point: a thread loads the digits and c0 of one evaluation point of
// every batch item once (coalesced) and, for each tap, sends them to the point sigma_g^-1 maps it to,
// where it reads the key and the mask and writes the result.  sigma_g maps every aligned run of 2^m
// points onto an aligned run of 2^m points, so a wavefront's 64 destinations are one 512-byte run,
// permuted inside: key reads and result writes are as coalesced as unpermuted ones.  The digits stream
// from HBM once per batch instead of once per tap, with no reliance on a cache.
// result of (item b, tap i): term k0 + b * k_bstride + tap[i] of xs in layout xl
struct TapSet {
    const u64* key[8];
    const u64* mask[8];
    u32 ginv[8];  // inverse Galois elements: the destination of source point x under sigma_g is gather(x, g^-1)
    u32 tap[8];
    u32 n_taps;
    const u64* centre_mask;  // the tap without a rotation (P * ct times this mask), or null
    u32 centre_tap;
};

// F64: every modulus below 2^50: the sums of BETA + 1 products as chains of fused multiply-adds on centred doubles (f64m_dot_w:
// four full-rate operations per term where a split integer sum takes three quarter-rate 64-bit multiply-adds and the splits:
// 117 registers instead of 232, 776 us instead of 904 for eight ciphertexts and nine taps at N = 2^16); the digits and the
// ciphertext's words are centred once per thread, a tap's key words once per tap.  Otherwise 128-bit integer sums.
// NB: most ciphertexts of the launch (their digits are held in registers; hoisted 56-bit rotations, one ciphertext: 10.9e3 per second
// with eight, 11.5e3 with one).
// MASKED: every result is multiplied by its tap's mask word (one product per result; folding the masks into copies of the keys
// beforehand, as this kernel did while its sums were integers, writes and reads the eight keys once more per call, 329 of 16600 us for 64
// channels at N = 2^16 and 10.8 of 73 us for three at 2^13; the eight-channel launch takes 780 us instead of 770).
template <int BETA, bool F64, int NB, bool MASKED>
__global__ __launch_bounds__(KS_THREADS) void key_inner_taps_kernel(DigitSrc digits, TapSet T, PtrList8 c0s, u64* __restrict__ xs, XLayout xl,
                                                                    u32 k0base, u32 k_bstride, const ModConst* __restrict__ mc, u32 log_n,
                                                                    u32 level, u32 num_q, u32 E, u32 n, u32 M, const u64* __restrict__ negp,
                                                                    const ModConstF* __restrict__ mcf, u32 taps_per_wg) {
    // blockIdx.z: which taps_per_wg of the taps
    const u32 N = 1u << log_n;
    const u32 xsrc = blockIdx.x * KS_THREADS + threadIdx.x;
    if (xsrc >= N) return;
    const u32 e = blockIdx.y;
    const u32 t = e <= level ? e : num_q + (e - level - 1);
    const ModConst m = mc[t];
    const bool has_add = e <= level;
    const u64 pres = has_add ? m.q - negp[e] : 0;  // P mod q_e
    u64 dv[NB][BETA], cv[NB];
#pragma unroll
    for (u32 b = 0; b < NB; b++) {
        const bool on = b < n;
        cv[b] = (on && has_add) ? c0s.p[b][(size_t)e * N + xsrc] : 0;
#pragma unroll
        for (u32 j = 0; j < BETA; j++) dv[b][j] = on ? digit_row(digits, b, j, e, E, N, level)[xsrc] : 0;
    }
    // F64: the centred representative of a residue as a double
    const double qd = F64 ? mcf[t].q : 0.0, qinv = F64 ? mcf[t].qinv : 0.0, halfq = 0.5 * qd;
    auto centred = [&](u64 v) {
        const double d = f64m_from_u64(v);
        return d > halfq ? d - qd : d;
    };
    double yd[NB][BETA + 1];  // F64: digits and the ciphertext's word of every batch item
    if (F64) {
#pragma unroll
        for (u32 b = 0; b < NB; b++) {
#pragma unroll
            for (u32 j = 0; j < BETA; j++) yd[b][j] = centred(dv[b][j]);
            yd[b][BETA] = centred(cv[b]);
        }
    }
    const u32 i0 = blockIdx.z * taps_per_wg, i1 = min(T.n_taps, i0 + taps_per_wg);
    for (u32 i = i0; i < i1; i++) {
        const u32 x = galois_gather_index(xsrc, T.ginv[i], log_n);  // destination point
        u64 k0[BETA], k1[BETA];
#pragma unroll
        for (u32 j = 0; j < BETA; j++) {
            const u64* kb = T.key[i] + (((size_t)j * 2) * M + t) * N + x;
            k0[j] = kb[0];
            k1[j] = kb[(size_t)M * N];
        }
        const u64 mk = MASKED ? T.mask[i][(size_t)e * N + x] : 0;
        u64* ot = xs + xl.at(k0base + T.tap[i], 0, e, x);
        if (F64) {
            double w0[BETA + 1], w1[BETA];
#pragma unroll
            for (u32 j = 0; j < BETA; j++) { w0[j] = centred(k0[j]); w1[j] = centred(k1[j]); }
            w0[BETA] = centred(pres);  // zero on the special primes
            const double md = f64m_from_u64(mk);
#pragma unroll
            for (u32 b = 0; b < NB; b++) {
                if (b < n) {
                    u64* ob = ot + (size_t)b * k_bstride * xl.s_k;
                    double r0 = f64m_dot_w<BETA + 1>(yd[b], w0, qd, qinv), r1 = f64m_dot_w<BETA>(yd[b], w1, qd, qinv);
                    if (MASKED) r0 = f64m_mulmod_any(r0, md, qd, qinv), r1 = f64m_mulmod_any(r1, md, qd, qinv);
                    ob[0] = f64m_canonical(r0, qd);
                    ob[xl.s_comp] = f64m_canonical(r1, qd);
                }
            }
        } else {
#pragma unroll
            for (u32 b = 0; b < NB; b++) {
                if (b < n) {
                    U128 acc0 = {0, 0}, acc1 = {0, 0};
#pragma unroll
                    for (u32 j = 0; j < BETA; j++) {
                        acc_wide(acc0, dv[b][j], k0[j]);
                        acc_wide(acc1, dv[b][j], k1[j]);
                    }
                    acc_wide(acc0, cv[b], pres);
                    u64* ob = ot + (size_t)b * k_bstride * xl.s_k;
                    u64 r0 = barrett_reduce(acc0, m), r1 = barrett_reduce(acc1, m);
                    if (MASKED) r0 = mulmod_barrett(r0, mk, m), r1 = mulmod_barrett(r1, mk, m);
                    ob[0] = r0;
                    ob[xl.s_comp] = r1;
                }
            }
        }
    }
    if (T.centre_mask && blockIdx.z == 0) {  // no rotation: mask * P * ct on the live limbs, zero on the special primes
        const u64 kp = has_add ? mulmod_barrett(T.centre_mask[(size_t)e * N + xsrc], pres, m) : 0;
        u64* ot = xs + xl.at(k0base + T.centre_tap, 0, e, xsrc);
#pragma unroll
        for (u32 b = 0; b < NB; b++) {
            if (b < n) {
                const u64 c1 = has_add ? c0s.p[b][((size_t)(level + 1) + e) * N + xsrc] : 0;
                u64* ob = ot + (size_t)b * k_bstride * xl.s_k;
                ob[0] = has_add ? mulmod_barrett(cv[b], kp, m) : 0;
                ob[xl.s_comp] = has_add ? mulmod_barrett(c1, kp, m) : 0;
            }
        }
    }
}

// keys / gs / masks / taps: n_taps <= 8 entries (taps[i] = position of tap i in the output's tap stride); masks: null, or one
// [E][N] plaintext per tap; c0s: n <= CT_BATCH device pointers [2][level+1][N].
// Needs beta <= 4 (returns hipErrorNotSupported otherwise: the caller then falls back to one launch per tap).
hipError_t launch_key_inner_taps(const ckks_ctx* c, u32 level, const DigitSrc& digits, const u64* const* keys,
                                 const u32* gs, const u64* const* masks, const u32* taps, u32 n_taps, const u64* const* c0s,
                                 u64* xs, XLayout xl, u32 k0, u32 k_bstride, u32 n, hipStream_t st, const u64* centre_mask, u32 centre_tap) {
    if ((n_taps == 0 && !centre_mask) || n == 0) return hipSuccess;
    if (n_taps > 8 || n > CT_BATCH) return hipErrorInvalidValue;
    for (u32 i = 0; i < n_taps; i++)
        if (!keys[i] || (masks && !masks[i])) return hipErrorInvalidValue;
    const u32 E = c->ext_limbs(level), beta = c->live_digits(level);
    if (beta > 4) return hipErrorNotSupported;
    TapSet T;
    const u64 two_n = 2ull * c->N;
    for (u32 i = 0; i < 8; i++) {
        T.key[i] = i < n_taps ? keys[i] : nullptr;
        T.mask[i] = (i < n_taps && masks) ? masks[i] : nullptr;
        T.tap[i] = i < n_taps ? taps[i] : 0;
        u64 inv = 1;
        if (i < n_taps) {  // g^-1 mod 2N: g is odd, the group has exponent N/2
            u64 base = gs[i] % two_n;
            for (u64 ex = c->N / 2 - 1; ex; ex >>= 1) {
                if (ex & 1) inv = inv * base % two_n;
                base = base * base % two_n;
            }
        }
        T.ginv[i] = (u32)inv;
    }
    T.n_taps = n_taps;
    T.centre_mask = centre_mask;
    T.centre_tap = centre_tap;
    PtrList8 cl;
    for (u32 b = 0; b < KS_MAX_BATCH; b++) cl.p[b] = b < n ? c0s[b] : nullptr;
    const u32 nxb = (c->N + KS_THREADS - 1) / KS_THREADS;
    const u64* negp = c->d_moddown + 2 * c->k_pad + (size_t)c->k_pad * c->num_q + 2 * c->num_q;
    // Taps per workgroup: all, so that the digits are read once for them; in a launch that does not give every CU four workgroups
    // the taps one after the other are a serial chain next to idle CUs, and what is read again comes from cache: fewer per
    // workgroup (one channel, eight taps, 6 limbs at N = 2^12: 10.2 us with eight, 7.1 with one)
    u32 taps_per_wg = 8;
    while (taps_per_wg > 1 && nxb * E * ((n_taps + taps_per_wg - 1) / taps_per_wg) < 1024) taps_per_wg >>= 1;
    const u32 groups = (n_taps + taps_per_wg - 1) / taps_per_wg;
    dim3 grid(nxb, E, groups ? groups : 1);
    // digits and c0 once per batch, per tap one key, one mask and the outputs
    ProfScope ps__(c, K_KEY_INNER, st, 8.0 * c->N * (E * (n * (double)beta + n_taps * (2.0 * beta + (masks ? 1.0 : 0.0) + 2.0 * n)) + n * (level + 1.0)),
                   2.0 * n_taps * n * c->N * E * (beta + 1.0 + (masks ? 1.0 : 0.0)));
#define KI_TAPS_LAUNCH(B_, F_, NB_, M_)                                                                                              \
    hipLaunchKernelGGL((key_inner_taps_kernel<B_, F_, NB_, M_>), grid, dim3(KS_THREADS), 0, st, digits, T, cl, xs, xl, k0, k_bstride, \
                       c->d_mc, c->log_n, level, c->num_q, E, n, c->M, negp, c->d_mcf, taps_per_wg)
#define KI_TAPS_NB(B_, M_)                                                                                                           \
    do {                                                                                                                             \
        if (!c->small_q && n == 1) KI_TAPS_LAUNCH(B_, false, 1, M_);                                                                 \
        else if (!c->small_q) KI_TAPS_LAUNCH(B_, false, CT_BATCH, M_);                                                               \
        else if (n == 1) KI_TAPS_LAUNCH(B_, true, 1, M_);                                                                            \
        else if (n <= 4) KI_TAPS_LAUNCH(B_, true, 4, M_);                                                                            \
        else KI_TAPS_LAUNCH(B_, true, CT_BATCH, M_);                                                                                 \
    } while (0)
#define KI_TAPS(B_)                                                                                                                  \
    do {                                                                                                                             \
        if (masks) KI_TAPS_NB(B_, true);                                                                                             \
        else KI_TAPS_NB(B_, false);                                                                                                  \
    } while (0)
    if (beta == 1) KI_TAPS(1);
    else if (beta == 2) KI_TAPS(2);
    else if (beta == 3) KI_TAPS(3);
    else KI_TAPS(4);
#undef KI_TAPS
#undef KI_TAPS_NB
#undef KI_TAPS_LAUNCH
    return hipGetLastError();
}

// The deferred convolution's inner products, masks and weighted sum in one kernel, for few output channels: the aligned copies are not stored.
//   acc[o][comp][e][x] (+)= sum_t mask_t[x] * sum_b w[o][b][t] * ( <digits_b[s_t x], key_t[x]> + P c0_b[s_t x] )
// organised by DESTINATION point, so that a thread holds the sums of its point: digits and c0 are gathered through the tap's automorphism s_t
// (a wavefront's 64 points are one aligned run of 512 bytes), once per tap, from cache after the first.  What a copy costs otherwise, two words
// written and read again per (channel, tap), was most of the time of the two launches that this one replaces.  A workgroup is 64 points
// times TW wavefronts that take 9 / TW taps each and add up their sums in LDS; the operands of the next NB
// channels, or of the next tap's first, are requested while the current ones are multiplied.  A tap without a rotation has no key:
// P times the ciphertext itself, whose component 1 comes in place of the first digit.  Three channels, two outputs, 5 + 2 limbs at N = 2^13: 16.4 us
// with the workgroups of a limb on all dies, 13 with them on one (25 in two launches, 25 MB of copies written and read); 16 channels, four
// outputs, 24 + 8 limbs at 2^16: a layer takes 2.5 ms instead of 3.3, bound by the double-precision units.
struct SumTaps {
    const u64* key[9];  // null: no rotation
    u32 g[9];
};
#define KSUM_MAX_CH KS_MAX_BATCH
template <int BETA, int OT, int NB, int TW>
__global__ __launch_bounds__(64 * TW) void key_inner_sum_kernel(DigitSrc digits, SumTaps T, PtrList8 cts, const u64* __restrict__ masks,
                                                                const u64* __restrict__ w_res, u64* __restrict__ acc, const u64* __restrict__ negp,
                                                                const ModConstF* __restrict__ mcf, u32 log_n, u32 level, u32 num_q, u32 M, u32 E, u32 n,
                                                                u32 ch0, u32 n_ch, u32 c_out) {
    constexpr u32 TPW = 9 / TW;
    __shared__ double lw[9 * KSUM_MAX_CH * OT];  // [tap][channel][output], centred; zero beyond the last channel or output
    __shared__ double ls[TW > 1 ? TW - 1 : 1][2][OT][64];
    const u32 N = 1u << log_n, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroups are dealt to the eight dies in turn: each die takes a contiguous eighth of the (limb, points) list, so that what its taps
    // gather stays in its own L2 cache
    const u32 log_xw = log_n - 6, list = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3), e = list >> log_xw, o0 = blockIdx.y * OT;
    if (e >= E) return;  // whole workgroup
    const u32 x = (list & ((1u << log_xw) - 1)) * 64 + lane;
    const u32 t_mod = e <= level ? e : num_q + (e - level - 1), el = e <= level ? e : level;
    const u32 own = e <= level ? e / digits.alpha : 0xffffffffu;
    const double q = mcf[t_mod].q, qinv = mcf[t_mod].qinv, halfq = 0.5 * q;
    auto centred = [&](u64 v) {
        const double d = f64m_from_u64(v);
        return d > halfq ? d - q : d;
    };
    // up to four products of a residue as it is, below 2^50, with a centred word, below 2^49, keep a chain's sum below 2^101 (f64m_dot_w): nothing to
    // centre
    auto plain = [&](u64 v) { return BETA < 4 ? f64m_from_u64(v) : centred(v); };
    const double pres = e <= level ? centred((u64)q - negp[el]) : 0.0;  // P mod q_e; nothing is added on the special primes
    const u32 groups = (n + NB - 1) / NB;
    u64 dv[NB][BETA], cv[NB], k0[BETA], k1[BETA], mk;
    auto load = [&](u32 t, u32 grp) {  // the operands of tap t, channels grp * NB ..
        const u64* key = T.key[t];
        const u32 xs = galois_gather_index(x, T.g[t], log_n);
        if (grp == 0) {
            // without a key any address that can be read: the words meet zero weights
            const u64* kp = (key ? key + (size_t)t_mod * N : masks) + x;
            const size_t kstride = key ? (size_t)M * N : 0;
#pragma unroll
            for (int j = 0; j < BETA; j++) k0[j] = kp[2 * j * kstride], k1[j] = kp[(2 * j + 1) * kstride];
            mk = masks[((size_t)t * E + e) * N + x];
        }
#pragma unroll
        for (int i = 0; i < NB; i++) {
            const u32 b = min(grp * NB + i, n - 1);
            const u64* ct = cts.p[b] + (size_t)el * N;
#pragma unroll
            for (int j = 0; j < BETA; j++) {
                const u64* row = own == (u32)j ? digits.own.p[b] + (size_t)e * N : digits.digits + b * digits.bstride + ((size_t)j * E + e) * N;
                if (j == 0 && !key) row = ct + (size_t)(level + 1) * N;
                dv[i][j] = row[xs];
            }
            cv[i] = ct[xs];
        }
    };
    const u32 t0 = wave * TPW;
    load(t0, 0);
    for (u32 i = tid; i < 9 * KSUM_MAX_CH * OT; i += 64 * TW) {
        const u32 o = o0 + i % OT, b = i / OT % KSUM_MAX_CH, t = i / (OT * KSUM_MAX_CH);
        lw[i] = (b < n && o < c_out) ? centred(w_res[(((size_t)o * n_ch + ch0 + b) * 9 + t) * E + e]) : 0.0;
    }
    __syncthreads();
    double s[2][OT];
#pragma unroll
    for (int o = 0; o < OT; o++) s[0][o] = s[1][o] = 0.0;
    for (u32 t = t0; t < t0 + TPW; t++) {
        const bool rot = T.key[t] != nullptr;
        double w0[BETA + 1], w1[BETA], st[2][OT], ct_[2][OT], cl[2][OT];
        const double md = f64m_from_u64(mk);
#pragma unroll
        for (int j = 0; j < BETA; j++) {
            w0[j] = rot ? centred(k0[j]) : 0.0;
            w1[j] = rot ? centred(k1[j]) : (j == 0 ? pres : 0.0);
        }
        w0[BETA] = pres;
        auto chain_begin = [&]() {
#pragma unroll
            for (int o = 0; o < OT; o++) ct_[0][o] = ct_[1][o] = F64M_DOT_BASE, cl[0][o] = cl[1][o] = 0.0;
        };
        chain_begin();
        bool first = true;
        for (u32 grp = 0; grp < groups; grp++) {
            double X[2][NB];
#pragma unroll
            for (int i = 0; i < NB; i++) {
                double y[BETA + 1];
#pragma unroll
                for (int j = 0; j < BETA; j++) y[j] = plain(dv[i][j]);
                y[BETA] = plain(cv[i]);
                X[0][i] = f64m_dot_w<BETA + 1>(y, w0, q, qinv);
                X[1][i] = f64m_dot_w<BETA>(y, w1, q, qinv);
            }
            const bool last = grp + 1 == groups;
            if (!last || t + 1 < t0 + TPW) load(last ? t + 1 : t, last ? 0 : grp + 1);
            const double* lwt = lw + ((size_t)t * KSUM_MAX_CH + grp * NB) * OT;
#pragma unroll
            for (int o = 0; o < OT; o++)
#pragma unroll
                for (int i = 0; i < NB; i++) {
                    const double wo = lwt[i * OT + o];
#pragma unroll
                    for (int c = 0; c < 2; c++) f64m_chain_add(ct_[c][o], cl[c][o], X[c][i], wo);
                }
            if (last || (grp + 1) % (8 / NB) == 0) {  // a chain takes eight terms
#pragma unroll
                for (int c = 0; c < 2; c++)
#pragma unroll
                    for (int o = 0; o < OT; o++) {
                        const double r = f64m_chain_join(ct_[c][o], cl[c][o], q, qinv);
                        st[c][o] = first ? r : f64m_reduce(st[c][o] + r, q, qinv);
                    }
                first = false;
                if (!last) chain_begin();
            }
        }
        // nine products below 0.63 q in all
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int o = 0; o < OT; o++) s[c][o] += f64m_mulmod_any(st[c][o], md, q, qinv);
    }
    if (TW > 1) {
        if (wave)
#pragma unroll
            for (int c = 0; c < 2; c++)
#pragma unroll
                for (int o = 0; o < OT; o++) ls[wave - 1][c][o][lane] = s[c][o];
        __syncthreads();
        if (wave) return;
    }
#pragma unroll
    for (int c = 0; c < 2; c++)
#pragma unroll
        for (int o = 0; o < OT; o++) {
            double r = s[c][o];
#pragma unroll
            for (int i = 0; i < TW - 1; i++) r += ls[i][c][o][lane];
            if (o0 + o < c_out) {
                u64* a = acc + (((size_t)(o0 + o) * 2 + c) * E + e) * N + x;
                if (ch0) r += f64m_from_u64(*a);
                *a = f64m_canonical(f64m_reduce(r, q, qinv), q);
            }
        }
}

// Channels ch0 .. ch0 + n - 1 of n_ch (n <= KSUM_MAX_CH, their digits and ciphertexts; the sums of the channels before are in acc), keys[t] null and gs[t] = 1 for a
// tap without a rotation, masks [9][E][N], w_res [c_out][n_ch][9][E], acc [c_out][2][E][N]
hipError_t launch_key_inner_sum(const ckks_ctx* c, u32 level, const DigitSrc& digits, const u64* const* keys, const u32* gs, const u64* masks,
                                const u64* const* cts, u32 n, const u64* w_res, u32 ch0, u32 n_ch, u32 c_out, u64* acc, hipStream_t st) {
    const u32 E = c->ext_limbs(level), beta = c->live_digits(level);
    if (n == 0 || n > KSUM_MAX_CH || ch0 + n > n_ch || c_out == 0 || c_out > 8 || beta > 4 || !c->small_q || c->N % 64) return hipErrorInvalidValue;
    SumTaps T;
    double n_keys = 0.0;
    for (u32 t = 0; t < 9; t++) {
        if (keys[t]) n_keys += 1.0;
        if ((gs[t] == 1) != (keys[t] == nullptr)) return hipErrorInvalidValue;
        T.key[t] = keys[t];
        T.g[t] = gs[t];
    }
    // TW: three taps per wavefront and a sum in LDS; one wavefront for all nine only where a chip full of workgroups makes the sum of several
    // outputs the dearer part.  Whole convolutions, TW = 1 / 3 in us: N = 2^12, 5 + 2 limbs, 4 -> 4 56.3 / 44.4, 2^14, 12 + 4 132.9 / 132.9, 2^15, 9 + 3 182.5 / 186.0,
    // 2^16, 24 + 8, 1 -> 4 510 / 553, 16 -> 1 2079 / 2017.
    const u32 xw = c->N / 64, ot = c_out <= 4 ? c_out : (c_out + 1) / 2, tw = ot > 1 && xw * E >= 5120 ? 1 : 3;
    // NB: three channels at once where they come out even, else pairs (four: 2 % faster on rings of 2^12, 15 % slower on large ones, 188 registers for four
    // outputs).  But not where three take more than the 168 registers that leave three waves per SIMD and pairs do not: four outputs with one digit (170 / 164),
    // and with three and one wavefront for all taps (170 / 158); four digits are at two waves either way.  Three channels, which leave a pair half empty, stay
    // together there too.  Pairs / three, us: 3 -> 3 channels at 2^16, 8 + 8 limbs in one digit 264 / 241, 16 + 8 in two 434 / 393, 24 + 8 in three 690 / 638, 24 + 6 in
    // four 772 / 710, 3 -> 4 294 / 297, 504 / 459, 764 / 743, 884 / 806; 6 -> 4 357 / 380, 657 / 644, 1035 / 1092, 1243 / 1231; at 2^12, 5 + 5 in one 6 -> 4 49.0 / 50.9,
    // 15 -> 4 70.1 / 74.0, 5 + 2 in three 73.2 / 71.8, 15 -> 1 65.8 / 63.5
    const bool short_of_registers = ot == 4 && (beta == 1 || (beta == 3 && tw == 1));
    const u32 nb = n == 1 ? 1 : (n % 3 == 0 && (n == 3 || !short_of_registers) ? 3 : 2);
    const u64* negp = c->d_moddown + 2 * c->k_pad + (size_t)c->k_pad * c->num_q + 2 * c->num_q;
    const dim3 grid((xw * E + 7) / 8 * 8, (c_out + ot - 1) / ot);
    // in: the digits with their own limbs, c0, the keys, nine masks, the weights, the sums so far; out: the sums
    ProfScope ps__(c, K_KEY_INNER, st, 8.0 * c->N * (E * (n * (double)beta + n_keys * 2.0 * beta + 9.0 + (ch0 ? 4.0 : 2.0) * c_out) + n * (level + 1.0)) + 72.0 * n * c_out * E,
                   2.0 * c->N * E * n * (9 * (beta + 1.0) + 9.0 * c_out));
    PtrList8 ptrs;
    for (u32 b = 0; b < KS_MAX_BATCH; b++) ptrs.p[b] = b < n ? cts[b] : nullptr;
#define KS_SUM(B_, O_, NB_, TW_)                                                                                                       \
    if (beta == B_ && ot == O_ && nb == NB_ && tw == TW_) {                                                                            \
        hipLaunchKernelGGL((key_inner_sum_kernel<B_, O_, NB_, TW_>), grid, dim3(64 * TW_), 0, st, digits, T, ptrs, masks, w_res, acc, negp, c->d_mcf, c->log_n, level, c->num_q, c->M, E, n, ch0, n_ch, c_out); \
        return hipGetLastError();                                                                                                      \
    }
#define KS_SUM_O(B_, NB_)                                                                                                              \
    KS_SUM(B_, 1, NB_, 3) KS_SUM(B_, 2, NB_, 3) KS_SUM(B_, 3, NB_, 3) KS_SUM(B_, 4, NB_, 3)                                            \
    KS_SUM(B_, 2, NB_, 1) KS_SUM(B_, 3, NB_, 1) KS_SUM(B_, 4, NB_, 1)
#define KS_SUM_N(B_) KS_SUM_O(B_, 1) KS_SUM_O(B_, 2) KS_SUM_O(B_, 3)
    KS_SUM_N(1) KS_SUM_N(2) KS_SUM_N(3) KS_SUM_N(4)
#undef KS_SUM_N
#undef KS_SUM_O
#undef KS_SUM
    return hipErrorInvalidValue;
}

// ---- ModDown, conversion of the P-part ----------------------------------------------------------
// v [2][E][N]: limbs level+1.. hold the P-part in coefficient form.  w [2][level+1][N] (coefficients)
// Dropped limbs: positions first..first+k-1 of v's E limbs; their moduli: `merged` ? (q_level, p_0, ...) : (p_0, ...).
// Results on limbs 0..n_out-1 (n_out = level+1, or level when merged).
__device__ __forceinline__ u32 dropped_modulus(u32 a, u32 level, u32 num_q, bool merged) {
    return merged ? (a == 0 ? level : num_q + a - 1) : num_q + a;
}

__global__ __launch_bounds__(KS_THREADS) void moddown_conv_kernel(const u64* __restrict__ v, u64* __restrict__ w,
                                                                  const u64* __restrict__ tab, const ModConst* __restrict__ mc,
                                                                  u32 N, u32 level, u32 num_q, u32 k, u32 kp, u32 E, u32 first,
                                                                  u32 n_out, bool merged, u32 lpb) {
    const u32 x = blockIdx.x * KS_THREADS + threadIdx.x;
    if (x >= N) return;
    const u32 comp = blockIdx.z;
    u64 z[KS_MAX_DIGIT];
    u64 n_neg = 0;
#pragma unroll
    for (u32 a = 0; a < KS_MAX_DIGIT; a++)
        if (a < k) {
            const u64 pa = mc[dropped_modulus(a, level, num_q, merged)].q;
            z[a] = mul_shoup(v[((size_t)comp * E + first + a) * N + x], tab[a], tab[kp + a], pa);
            n_neg += z[a] > (pa >> 1) ? 1 : 0;
        }
    const u64* phat_q = tab + 2 * kp;  // [num_q][kp]
    const u64* negp = tab + 2 * kp + (size_t)kp * num_q + 2 * num_q;
    const u32 i0 = blockIdx.y * lpb;
    for (u32 i = i0; i < i0 + lpb && i < n_out; i++) {
        U128 acc = {0, 0};
#pragma unroll
        for (u32 a = 0; a < KS_MAX_DIGIT; a++)
            if (a < k) acc_wide(acc, z[a], phat_q[(size_t)i * kp + a]);
        acc_wide(acc, n_neg, negp[i]);
        w[((size_t)comp * n_out + i) * N + x] = barrett_reduce(acc, mc[i]);
    }
}

// KP: padded row length of the tables; KR: how many of the row's entries are real (the rest are zeros that need no arithmetic)
template <int KP, int KR = KP>
__global__ __launch_bounds__(KS_THREADS) void moddown_conv50_kernel(const u64* __restrict__ v, u64* __restrict__ w,
                                                                    const u64* __restrict__ tab, const ModConst* __restrict__ mc,
                                                                    u32 N, u32 level, u32 num_q, u32 k, u32 E, u32 first, u32 n_out,
                                                                    bool merged, u32 lpb) {
    const u32 x = blockIdx.x * KS_THREADS + threadIdx.x;
    if (x >= N) return;
    const u32 comp = blockIdx.z;
    Split50 z[KR];
    u32 n_neg = 0;
#pragma unroll
    for (u32 a = 0; a < KR; a++) {
        z[a] = {0, 0, 0};
        if (a < k) {
            const u64 pa = mc[dropped_modulus(a, level, num_q, merged)].q;
            const u64 zv = mul_shoup(v[((size_t)comp * E + first + a) * N + x], tab[a], tab[KP + a], pa);
            n_neg += zv > (pa >> 1) ? 1 : 0;
            z[a] = split50(zv);
        }
    }
    constexpr int ROW_ALIGN = (KP & (KP - 1)) == 0 ? 8 * KP : 32;  // rows of 12 words are 32-byte aligned
    const u64* phat_q = (const u64*)__builtin_assume_aligned(tab + 2 * KP, ROW_ALIGN);  // [num_q][KP]
    const u64* negp = tab + 2 * KP + (size_t)KP * num_q + 2 * num_q;
    const u32 i0 = blockIdx.y * lpb;
    for (u32 i = i0; i < i0 + lpb && i < n_out; i++) {
        const u64* pe = (const u64*)__builtin_assume_aligned(phat_q + (size_t)i * KP, ROW_ALIGN);
        u64 cv[KP];
#pragma unroll
        for (u32 a = 0; a < KP; a++) cv[a] = pe[a];
        Acc50 acc = {0, 0, 0};
#pragma unroll
        for (u32 a = 0; a < KR; a++) acc50_mad(acc, z[a], split50(cv[a]));
        U128 s = acc50_value(acc);
        acc_wide(s, n_neg, negp[i]);
        w[((size_t)comp * n_out + i) * N + x] = barrett_reduce(s, mc[i]);
    }
}

// The same conversion in double precision (see modup_conv_f64_kernel).  phf: [num_q][KP] (constant, constant / q_i).
template <int KP, int KR = KP>
__global__ __launch_bounds__(KS_THREADS) void moddown_conv_f64_kernel(const u64* __restrict__ v, u64* __restrict__ w,
                                                                      const u64* __restrict__ tab, const TwF* __restrict__ phf,
                                                                      const ModConst* __restrict__ mc, const ModConstF* __restrict__ mcf,
                                                                      u32 N, u32 level, u32 num_q, u32 k, u32 E, u32 first, u32 n_out,
                                                                      bool merged, u32 lpb) {
    const u32 x = blockIdx.x * KS_THREADS + threadIdx.x;
    if (x >= N) return;
    const u32 comp = blockIdx.z;
    double z[KR];
#pragma unroll
    for (u32 a = 0; a < KR; a++) {
        z[a] = 0.0;
        if (a < k) {
            const u64 pa = mc[dropped_modulus(a, level, num_q, merged)].q;
            const u64 zv = mul_shoup(v[((size_t)comp * E + first + a) * N + x], tab[a], tab[KP + a], pa);
            z[a] = zv > (pa >> 1) ? -f64m_from_u64(pa - zv) : f64m_from_u64(zv);
        }
    }
    const u32 i0 = blockIdx.y * lpb;
    for (u32 i = i0; i < i0 + lpb && i < n_out; i++) {
        const TwF* pe = phf + (size_t)i * KP;
        const double q = mcf[i].q, qinv = mcf[i].qinv;
        w[((size_t)comp * n_out + i) * N + x] = f64m_canonical(f64m_dot<KR>(z, pe, q, qinv), q);
    }
}

hipError_t launch_moddown_conv(const ckks_ctx* c, u32 level, bool merged, const u64* v, u64* w, u32 batch, hipStream_t st) {
    const u32 n_out = merged ? level : level + 1, k = merged ? c->num_p + 1 : c->num_p, kp = merged ? c->k2_pad : c->k_pad;
    const u32 first = merged ? level : level + 1, E = c->ext_limbs(level);
    const u64* tab = merged ? c->moddown_rs_table(level) : c->d_moddown;
    const u32 x_wgs = (c->N + KS_THREADS - 1) / KS_THREADS;
    const u32 lpb = x_wgs * batch >= 2048 ? 12 : 6;  // as in launch_modup_conv
    dim3 grid(x_wgs, (n_out + lpb - 1) / lpb, batch);
    ProfScope ps__(c, K_MODDOWN_CONV, st, 8.0 * batch * c->N * (k + n_out), 1.0 * batch * c->N * k * (n_out + 1.0));
    if (c->ntt_f64 && c->d_moddown_f) {
        const TwF* pf = merged ? c->moddown_rs_table_f(level) : c->d_moddown_f;
#define MD_F64(KP_, KR_) hipLaunchKernelGGL((moddown_conv_f64_kernel<KP_, KR_>), grid, dim3(KS_THREADS), 0, st, v, w, tab, pf, c->d_mc, c->d_mcf, c->N, level, c->num_q, k, E, first, n_out, merged, lpb)
        if (kp == 4) MD_F64(4, 4);
        else if (kp == 8) MD_F64(8, 8);
        else if (kp == 12 && k == 9) MD_F64(12, 9);
        else if (kp == 12) MD_F64(12, 12);
        else MD_F64(16, 16);
#undef MD_F64
        return hipGetLastError();
    }
    if (c->small_q) {
        if (kp == 4)
            hipLaunchKernelGGL(moddown_conv50_kernel<4>, grid, dim3(KS_THREADS), 0, st, v, w, tab, c->d_mc, c->N, level, c->num_q, k, E, first, n_out, merged, lpb);
        else if (kp == 8)
            hipLaunchKernelGGL(moddown_conv50_kernel<8>, grid, dim3(KS_THREADS), 0, st, v, w, tab, c->d_mc, c->N, level, c->num_q, k, E, first, n_out, merged, lpb);
        else if (kp == 12 && k == 9)
            hipLaunchKernelGGL((moddown_conv50_kernel<12, 9>), grid, dim3(KS_THREADS), 0, st, v, w, tab, c->d_mc, c->N, level, c->num_q, k, E, first, n_out, merged, lpb);
        else if (kp == 12)
            hipLaunchKernelGGL(moddown_conv50_kernel<12>, grid, dim3(KS_THREADS), 0, st, v, w, tab, c->d_mc, c->N, level, c->num_q, k, E, first, n_out, merged, lpb);
        else
            hipLaunchKernelGGL(moddown_conv50_kernel<16>, grid, dim3(KS_THREADS), 0, st, v, w, tab, c->d_mc, c->N, level, c->num_q, k, E, first, n_out, merged, lpb);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(moddown_conv_kernel, grid, dim3(KS_THREADS), 0, st, v, w, tab, c->d_mc, c->N, level, c->num_q, k, kp, E, first, n_out, merged, lpb);
    return hipGetLastError();
}

// ---- ModDown, last step, for a batch of key switches -------------------------------------------
// out_r[comp][i] = ((v_r[comp][i] - w_r[comp][i]) * P^-1 + addend) * mask, r < n (grid.z = 2n).
// add0 / add1: optional polynomials [level+1][N] added to component 0 / 1; when g != 1 the addend is
// read through the sigma_g gather (Rot: c0' = sigma_g(c0) + u0).  mask: optional plaintext
// [level+1][N] multiplied into both components (the tap's validity mask of the convolution).
__global__ __launch_bounds__(KS_THREADS) void moddown_final_kernel(const u64* __restrict__ v, const u64* __restrict__ w,
                                                                   FinalBatch B, const u64* __restrict__ tab,
                                                                   const ModConst* __restrict__ mc, u32 log_n, u32 n_out,
                                                                   u32 num_q, u32 kp, u32 E) {
    const u32 N = 1u << log_n;
    const u32 x = blockIdx.x * KS_THREADS + threadIdx.x;
    if (x >= N) return;
    const u32 i = blockIdx.y, b = blockIdx.z, comp = b & 1;
    const FinalItem it = B.it[b >> 1];
    const ModConst m = mc[i];
    const u64* pinv = tab + 2 * kp + (size_t)kp * num_q;
    u64 d = sub_mod(v[((size_t)b * E + i) * N + x], w[((size_t)b * n_out + i) * N + x], m.q);
    u64 r = mul_shoup(d, pinv[i], pinv[num_q + i], m.q);
    const u64* add = comp == 0 ? it.add0 : it.add1;
    if (add) {
        const u32 xs = it.g == 1 ? x : galois_gather_index(x, it.g, log_n);
        r = add_mod(r, add[(size_t)i * N + xs], m.q);
    }
    if (it.mask) r = mulmod_barrett(r, it.mask[(size_t)i * N + x], m);
    if (it.acc) r = add_mod(r, it.acc[((size_t)comp * n_out + i) * N + x], m.q);
    it.out[((size_t)comp * n_out + i) * N + x] = r;
}

// merged: division by P*q_level (results on limbs 0..level-1; addends and masks, if any, are [level][N])
hipError_t launch_moddown_final(const ckks_ctx* c, u32 level, bool merged, const u64* v, const u64* w, const FinalItem* items, u32 n,
                                hipStream_t st) {
    FinalBatch B;
    double extra = 0.0;
    for (u32 r = 0; r < KS_MAX_BATCH; r++) {
        if (r < n) {
            B.it[r] = items[r];
            extra += (items[r].add0 ? 1.0 : 0.0) + (items[r].add1 ? 1.0 : 0.0) + (items[r].mask ? 1.0 : 0.0) + (items[r].acc ? 2.0 : 0.0);
        } else {
            B.it[r] = FinalItem{nullptr, nullptr, nullptr, nullptr, 1, 0, nullptr};
        }
    }
    const u32 n_out = merged ? level : level + 1;
    dim3 grid((c->N + KS_THREADS - 1) / KS_THREADS, n_out, 2 * n);
    ProfScope ps__(c, K_MODDOWN_FINAL, st, 8.0 * c->N * n_out * (6.0 * n + extra), 2.0 * c->N * n_out * n);
    hipLaunchKernelGGL(moddown_final_kernel, grid, dim3(KS_THREADS), 0, st, v, w, B, merged ? c->moddown_rs_table(level) : c->d_moddown,
                       c->d_mc, c->log_n, n_out, c->num_q, merged ? c->k2_pad : c->k_pad, c->ext_limbs(level));
    return hipGetLastError();
}
