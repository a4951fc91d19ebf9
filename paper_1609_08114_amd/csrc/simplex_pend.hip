// Streaming simplex kernel with pending pivots: one LP per workgroup, the
// condensed tableau in a per-workgroup workspace slot in HBM, and the rank-1
// updates of Step 3 (Sec. 4.3) collected and applied KP at a time.
//
// Streaming the tableau once per pivot (simplex_gm.hip) moves 16 bytes per
// entry and pivot, and that traffic is all of its time.  But a pivot reads
// only one column of the tableau (Step 2) and one row (Step 3); the objective
// rows and the rhs column are kept current in registers.  So the last s
// pivots' columns (negated, F) and pivot rows (Q) stay in LDS, and just the
// entering column and the leaving row are brought up to date when they are
// read, with the s pending FMAs in pivot order: exactly the operations the
// eager update makes, bit for bit.  After KP pivots the flush brings the
// whole tableau up to date, KP FMAs per entry and one trip through memory.
//
// The flush is a product, T += F^T Q with KP terms per entry, and runs on the
// matrix cores: v_mfma_f64_16x16x4_f64 adds its four terms to the accumulator
// as four FMAs, each rounded to nearest, in increasing k (checked on gfx950
// against fma() on normal, cancelling, denormal and signed-zero operands), so
// it too gives the eager update's bits.
//
// Thread t owns row t (rhs, basis) and the slots t and t + NT (reduced costs,
// variables).  A pivot has two barriers: after every wave's best entering slot
// is published, and after every wave's best leaving row is.
//
// Pivot (l, e) at pending index s: row l becomes the pivot row p, so its older
// pending factors count for nothing and its factor is 1 on an entry of 0
// (fma(1, p, 0) = p); slot e becomes the leaving variable's column, on an
// entry of 0 likewise.  Each row and slot keeps the index at which that last
// happened since the flush (`rbirth`, `sbirth`; its tableau entries count as
// 0 and its terms start there).  In the flush the terms before a birth are
// zeroed factors, which change nothing while the other factor is finite: a
// pivot with a non-finite entry is flushed before the next one, so that all
// older terms are finite.
//
// What bounds it: the flush's trips through the last-level cache (a 200 x 200
// type-2 tableau of ~480 KB, 20 pivots per flush), then the two dependent
// memory reads and two barriers of a pivot; two workgroups per CU overlap
// them.  1,000 type-2 LPs of 200 x 200 (2,055 pivots each): 203 ms streaming at
// every pivot, 38.4 ms here; 2,000 mixed LPs of 5..300 rows and columns: 253
// and 39.9 ms.
//
// Layout of a slot: strips of four rows, in a strip blocks of 4 x 4 entries
// (the last one 4 x (slots mod 4)), in a block row-major: element (i, j) at
// (i / 4) 4 ns + (j / 4) 16 + (i mod 4) w + j mod 4, w the block's width.  One
// 128-byte line then serves four rows of a column read and four slots of a
// row read, and the 16 x 4 part of a matrix-core tile that one register holds
// is 512 consecutive bytes.
#include "aux_kernels.hpp"
#include "blp_kernels.hpp"
#include "simplex_blk.hpp"
#include "simplex_common.hpp"

namespace blp {

typedef double acc4 __attribute__((ext_vector_type(4)));

// a wave's candidate: key (as wave_argmax_i64), packed (id, pos), and what
// goes with the winner
struct alignas(16) PendRec {
    int hi;
    unsigned lo;
    int pk;
    int aux;
    double v0, v1, v2;
    int nonfinite, pad;
};

// The best of NW <= 8 records (in lanes 0..NW-1 after the read), under the
// order of wave_argmax_i64; returns its packed (id, pos), its record index
// and whether any record's non-finite flag is set.  Every wave computes it.
template <int NW>
__device__ __forceinline__ int pend_best(const PendRec* rec, int lane, int& hi, unsigned& lo, int& idx,
                                         bool& nonfinite) {
    static_assert(NW <= 8, "one row of eight lanes");
    const PendRec& r = rec[lane & 7 & (NW - 1)];
    const bool in = lane < NW;
    const int h = in ? r.hi : (int)0x80000000;
    const unsigned l = r.lo;
    const int pk = r.pk;
    nonfinite = __ballot(in && r.nonfinite) != 0;
    int v = h;
    v = max(v, dpp_src<0xB1, 0xF>(v));
    v = max(v, dpp_src<0x4E, 0xF>(v));
    v = max(v, dpp_src<0x141, 0xF>(v));
    hi = __builtin_amdgcn_readlane(v, 0);
    uint64_t mk = __ballot(in && h == hi);
    if (__popcll(mk) > 1) {  // equal high words: the low word, then the smallest id
        unsigned best = 0;
        for (uint64_t q = mk; q; q &= q - 1)
            best = max(best, (unsigned)__builtin_amdgcn_readlane((int)l, __ffsll((long long)q) - 1));
        mk = __ballot(in && h == hi && l == best);
        int win = 0, wpk = PACK_NONE;
        bool any = false;
        for (uint64_t q = mk; q; q &= q - 1) {
            const int c = __ffsll((long long)q) - 1, p = __builtin_amdgcn_readlane(pk, c);
            if (!any || p < wpk) {
                any = true;
                wpk = p;
                win = c;
            }
        }
        idx = win;
        lo = best;
        return wpk;
    }
    idx = __builtin_amdgcn_readfirstlane(__ffsll((long long)mk) - 1);
    lo = (unsigned)__builtin_amdgcn_readlane((int)l, idx);
    return __builtin_amdgcn_readlane(pk, idx);
}

template <int NW>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(4, 4)))
simplex_pend_kernel(KParams P) {
    constexpr int NT = NW * 64;
    extern __shared__ __align__(16) double s_mem[];  // F (KP x ldf), then Q (KP x ldq)
    __shared__ PendRec rec1[NW], rec2[NW];
    __shared__ int s_art[NT];  // artificial rows in row order
    __shared__ unsigned long long s_mask[NW];
    __shared__ unsigned short s_rowmask[NT / 16], s_slotmask[2 * NT / 16];
    __shared__ int s_ctl[2][2];

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    BLP_TDECL;
    double* const T = P.ws + (int64_t)blockIdx.x * P.ws_slot;
    const int64_t len = work_len(P);
    bool first = true;
    int par = 0;
    for (;;) {
        par ^= 1;
        if (t == 0) {
            int64_t q;
            if (P.direct)
                q = first ? P.direct_first + (int64_t)blockIdx.x : len;
            else
                q = pop_position(P, len, first);
            s_ctl[par][0] = q < len ? (int)work_item(P, q) : -1;
            s_ctl[par][1] = 0;
        }
        first = false;
        __syncthreads();
        const int k = __builtin_amdgcn_readfirstlane(s_ctl[par][0]);
        if (k < 0) break;
        BLP_T(t_load0);
        const LpRef L = lp_ref(P, k);
        const LpRef Lin = lp_in(P, L);  // constraint reads
        const int m = L.m, n = L.n;
        if (!pend_shape(m, n)) continue;  // the other streaming kernel's (uniform over the workgroup)

        // ------------------------------------------------------------ load
        const bool rowt = t < m;
        int bad = 0;
        double bR = 0.0;
        int bs = ID_NONE;
        bool art = false, neg = false;
        if (rowt) {
            const double bi = P.b[Lin.row_off + t];
            const bool ge = P.sense[Lin.row_off + t] != 0;
            const double ble = ge ? -bi : bi;
            art = ble < 0.0;
            neg = ge != art;  // the row's sign is -1
            bR = art ? -ble : ble;
            bad = !isfinite(bi);
        }
        // artificial rows in row order: each wave's ballot, then a prefix
        const unsigned long long mart = __ballot(art);
        const unsigned long long mneg = __ballot(neg);
        if (lane == 0) {
            s_mask[wave] = mart;
            rec1[wave].hi = (int)(unsigned)mneg;
            rec1[wave].lo = (unsigned)(mneg >> 32);
        }
        __syncthreads();
        int nart = 0, rank = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const unsigned long long mw = s_mask[w];
            if (w < wave) rank += __popcll(mw);
            nart += __popcll(mw);
        }
        nart = __builtin_amdgcn_readfirstlane(nart);
        if (art) s_art[rank + __popcll(mart & ((1ull << lane) - 1ull))] = t;
        bs = rowt ? (art ? n + m + t : n + t) : ID_NONE;
        __syncthreads();
        const int ns = n + nart;  // column slots; the rhs is not one of them
        // this LP's pending factors: KP pivots of ldf + ldq entries
        const int ldf = (m + 15) & ~15, ldq = (ns + 15) & ~15;
        const int KP = min(32, (P.ws_lds / (ldf + ldq)) & ~3);
        double* const F = s_mem;
        double* const Q = s_mem + KP * ldf;
        if (KP < 4 || (int64_t)((m + 3) & ~3) * ns > P.ws_slot) {  // never launched so
            write_numerical<NT>(P, L, k, t, ST_INTERNAL);
            continue;
        }
        const int ns4 = ns >> 2, nrem = ns & 3;
        auto at = [&](int i, int j) __attribute__((always_inline)) -> int {
            return (i >> 2) * (4 * ns) + (j >> 2) * 16 + (i & 3) * ((j >> 2) == ns4 ? nrem : 4) + (j & 3);
        };
        const unsigned tbytes = (unsigned)((m + 3) & ~3) * (unsigned)ns * 8u;
        const __amdgpu_buffer_rsrc_t wsr = __builtin_amdgcn_make_buffer_rsrc(T, (short)0, (int)tbytes, 0x00020000);
        // byte offset of tile column j in strip `st4`, this lane's row of the strip
        const int lr = lane >> 4, lc = lane & 15;
        // constraint rows into the slot, a strip of four rows by 16 slots per
        // wave and step, eight steps' loads in flight
        {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<double*>(P.A + Lin.a_off), (short)0, m * n * (int)sizeof(double), 0x00020000);
            const int strips = (m + 3) >> 2, cols = (ns + 15) >> 4;
            for (int g = wave; g < strips; g += NW) {
                const int i = 4 * g + lr;
                const unsigned lo = (unsigned)rec1[(i >> 6) & (NW - 1)].hi, hi = rec1[(i >> 6) & (NW - 1)].lo;
                const unsigned long long mw = ((unsigned long long)hi << 32) | lo;
                const bool flip = (mw >> (i & 63)) & 1ull;
                for (int c0 = 0; c0 < cols; c0 += 8) {
                    double v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int j = (c0 + u) * 16 + lc;
                        const unsigned o = i < m && j < n ? (unsigned)(i * n + j) * 8u : 0x80000000u;
                        v[u] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)o, 0, 0));
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int j = (c0 + u) * 16 + lc;
                        bad |= !isfinite(v[u]);
                        double w = flip ? -v[u] : v[u];
                        if (j >= n && j < ns) w = s_art[j - n] == i ? -1.0 : 0.0;
                        if (j < ns && i < m) T[at(i, j)] = w;
                    }
                }
            }
        }
        double dO[2], dW[2];
        int cv[2];
        double w0 = 0.0;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int j = t + c * NT;
            dO[c] = dW[c] = 0.0;
            cv[c] = j < n ? j : (j < ns ? n + s_art[j - n] : ID_NONE);
            if (j < n) {
                dO[c] = P.c[L.col_off + j];
                bad |= !isfinite(dO[c]);
                // phase-1 row: the artificial rows (signs applied) summed in row order
                double acc = 0.0;
                for (int q0 = 0; q0 < nart; q0 += 8) {
                    double v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        v[u] = P.A[Lin.a_off + (int64_t)s_art[q0 + u < nart ? q0 + u : q0] * n + j];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (q0 + u < nart) {
                            const int i = s_art[q0 + u];
                            const unsigned long long mw =
                                ((unsigned long long)rec1[i >> 6].lo << 32) | (unsigned)rec1[i >> 6].hi;
                            acc = acc + ((mw >> (i & 63)) & 1ull ? -v[u] : v[u]);
                        }
                }
                dW[c] = acc;
            } else if (j < ns) {
                dW[c] = -1.0;
            }
        }
        for (int q = 0; q < nart; ++q) {
            const double bi = P.b[Lin.row_off + s_art[q]];
            w0 = w0 + fabs(bi);  // an artificial row's normalised rhs is |b|
        }
        if (bad) atomicOr(&s_ctl[par][1], 1);
        __syncthreads();
        if (s_ctl[par][1]) {
            write_numerical<NT>(P, L, k, t, ST_NUMERICAL);
            continue;
        }
        double zO = 0.0, zW = w0;
        bool dead = false;
        int mode = nart > 0 ? 1 : 2;
        const int max_iter = P.max_iter > 0 ? P.max_iter : 50 * (m + n);
        const int bland_after = P.bland_after > 0 ? P.bland_after : (m > n ? m : n);
        const int id_lim = n + m;
        int iters = 0, degen = 0, st = -1, drive_r = 0;
        int s = 0;                      // pending pivots
        int rbirth = -1;                // row t replaced at this pending index
        int sbirth[2] = {-1, -1};       // slots likewise
        bool nf = false;                // this thread saw a non-finite pivot entry
        bool nf_any = false;

        // pending terms k0..s-1 on v: factors a[k * lda] (this thread's) and
        // b[k * ldb] (the same for the whole workgroup)
        auto pending = [&](double v, int k0, const double* a, int lda, const double* b,
                           int ldb) __attribute__((always_inline)) -> double {
            for (int kb = 0; kb < s; kb += 8) {
                double fa[8], fb[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int kk = min(kb + u, s - 1);
                    fa[u] = a[kk * lda];
                    fb[u] = b[kk * ldb];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const double w = __builtin_fma(fa[u], fb[u], v);
                    v = kb + u >= k0 && kb + u < s ? w : v;
                }
            }
            return v;
        };
        // value of (row r, slot t + c NT) now
        auto row_value = [&](int r, int rb, double (&x)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int j = t + c * NT;
                x[c] = 0.0;
                if (c == 0 || ns > NT) {
                    const bool in = j < ns, born = rb >= 0 || sbirth[c] >= 0;
                    double v = 0.0;
                    if (in && !born) v = T[at(r, j)];
                    v = pending(v, max(rb, sbirth[c]), Q + (in ? j : 0), ldq, F + r, ldf);
                    x[c] = in ? v : 0.0;
                }
            }
        };
        // bring the tableau up to date
        auto flush = [&]() __attribute__((always_inline)) {
            const int s4 = (s + 3) & ~3;
            // terms before a birth are zeroed; the tail of the last group of
            // four adds -0 (+0 times -0), which leaves every accumulator as it is
            if (t < ldf) {
                for (int q = 0; q < rbirth; ++q) F[q * ldf + t] = 0.0;
                for (int q = s; q < s4; ++q) F[q * ldf + t] = 0.0;
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int j = t + c * NT;
                if (j < ldq) {
                    for (int q = 0; q < sbirth[c]; ++q) Q[q * ldq + j] = 0.0;
                    for (int q = s; q < s4; ++q) Q[q * ldq + j] = -0.0;
                }
                const unsigned long long ms = __ballot(sbirth[c] >= 0);
                if ((lane & 15) == 0) s_slotmask[(j >> 4)] = (unsigned short)(ms >> (lane & 48));
            }
            const unsigned long long mr = __ballot(rbirth >= 0);
            if ((lane & 15) == 0) s_rowmask[t >> 4] = (unsigned short)(mr >> (lane & 48));
            __syncthreads();
            const int nr = ldf >> 4, ncg = (ldq + 63) >> 6;
            for (int u = wave; u < nr * ncg; u += NW) {
                const int R = u % nr, cg = u / nr;
                const unsigned rm = s_rowmask[R];
                acc4 d[4];
                unsigned o[4][4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int j = cg * 64 + c * 16 + lc;
                    const int w = (j >> 2) == ns4 ? nrem : 4;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int off = (4 * R + r) * (4 * ns) + (j >> 2) * 16 + lr * w + (j & 3);
                        o[c][r] = j < ns ? (unsigned)off * 8u : 0x80000000u;
                        d[c][r] = __builtin_bit_cast(
                            double, __builtin_amdgcn_raw_buffer_load_b64(wsr, (int)o[c][r], 0, 0));
                    }
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int jt = cg * 4 + c;  // slot tile
                    const bool cb = jt * 16 < ldq && ((s_slotmask[jt] >> lc) & 1);
#pragma unroll
                    for (int r = 0; r < 4; ++r) d[c][r] = cb || ((rm >> (4 * r + lr)) & 1) ? 0.0 : d[c][r];
                }
                const double* fa = F + lr * ldf + R * 16 + lc;
                for (int g = 0; g < s4; g += 4) {
                    const double a = fa[g * ldf];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int j = min(cg * 64 + c * 16, ldq - 16) + lc;
                        const double b = Q[(g + lr) * ldq + j];
                        d[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, d[c], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const double w = d[c][r];
                        __builtin_amdgcn_raw_buffer_store_b64(
                            __builtin_bit_cast(unsigned int __attribute__((ext_vector_type(2))), w), wsr, (int)o[c][r], 0,
                            0);
                    }
            }
            __syncthreads();
            s = 0;
            rbirth = sbirth[0] = sbirth[1] = -1;
        };
        BLP_T(t_load1);
        BLP_TACC(TM_LOAD, t_load0, t_load1);

        // ------------------------------------------------------ pivot loop
        // mode 1 = phase 1, 2 = phase 2, 3 = driving the remaining basic
        // artificials out after a feasible phase 1
        for (;;) {
            BLP_T(t_p0);
            int e, e_id, l = -1, lv = ID_NONE, idx, th;
            unsigned tl;
            if (mode == 3) {
                // the first row still holding an artificial variable
                const unsigned long long mk = __ballot(rowt && t >= drive_r && bs >= id_lim && !dead);
                if (lane == 0) {
                    rec1[wave].hi = mk ? -(wave * 64 + __ffsll((long long)mk) - 1) : -NT;
                    rec1[wave].lo = 0;
                    rec1[wave].pk = 0;
                    rec1[wave].nonfinite = __ballot(nf) != 0;
                }
                nf = false;
                __syncthreads();
                bool any;
                pend_best<NW>(rec1, lane, th, tl, idx, any);
                nf_any |= any;
                const int r0 = -th;
                __syncthreads();  // rec1 is written again below
                if (r0 >= NT) {
                    mode = 2;
                    degen = 0;
                    continue;
                }
                if (s == KP || nf_any) {
                    flush();
                    nf_any = false;
                }
                drive_r = r0 + 1;
                if (t == r0) {
                    rec2[0].aux = rbirth;
                    rec2[0].pk = bs;
                }
                __syncthreads();
                const int rb = __builtin_amdgcn_readfirstlane(rec2[0].aux);
                lv = __builtin_amdgcn_readfirstlane(rec2[0].pk);
                // the lowest-id non-artificial column with a usable entry enters
                double x[2];
                row_value(r0, rb, x);
                int pk = PACK_NONE;
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    if (t + c * NT < ns && cv[c] < id_lim && fabs(x[c]) > P.eps_piv)
                        pk = min(pk, pack_id(cv[c], t + c * NT));
                pk = wave_min_i32(pk);
                const int pos = unpack_pos(pk);
                if (lane == 0) {
                    rec1[wave].hi = pk == PACK_NONE ? (int)0x80000001 : -(pk >> 16);
                    rec1[wave].lo = 0;
                    rec1[wave].pk = pk;
                    rec1[wave].nonfinite = 0;
                }
                if (pk != PACK_NONE && lane == (pos & 63)) {
                    const int c = pos >= NT;
                    rec1[wave].v0 = c ? dO[1] : dO[0];
                    rec1[wave].v1 = c ? dW[1] : dW[0];
                    rec1[wave].aux = c ? sbirth[1] : sbirth[0];
                }
                __syncthreads();
                pk = pend_best<NW>(rec1, lane, th, tl, idx, any);
                if (pk == PACK_NONE) {  // redundant row
                    if (t == r0) dead = true;
                    __syncthreads();
                    continue;
                }
                l = r0;
                e = unpack_pos(pk);
                e_id = unpack_id(pk);
            } else {
                // Step 1: this wave's best slot
                double bk = -__builtin_inf();
                int bid = ID_NONE, bpos = -1;
                const bool rpc = P.pivot_rule == 1 && degen < bland_after;
                const bool bland = degen >= bland_after;
                int elig = 0;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int j = t + c * NT;
                    const double d = mode == 1 ? dW[c] : dO[c];
                    const bool ok = j < ns && cv[c] < id_lim && d > P.eps_price;
                    const double key = bland ? 0.0 : d;
                    const bool take = ok & ((key > bk) | ((key == bk) & (cv[c] < bid)));
                    bk = take ? key : bk;
                    bid = take ? cv[c] : bid;
                    bpos = take ? j : bpos;
                    elig |= ok ? 1 << c : 0;
                }
                if (rpc) {
                    // Sec. 4.2's random positive coefficient: the eligible
                    // slots are counted in slot order (slots of chunk 0 of all
                    // waves, then chunk 1)
                    __syncthreads();  // the previous pivot's reads of rec2 are done
                    const unsigned long long m0 = __ballot(elig & 1), m1 = __ballot(elig & 2);
                    if (lane == 0) {
                        rec2[wave].hi = __popcll(m0);
                        rec2[wave].aux = __popcll(m1);
                    }
                    __syncthreads();
                    int total = 0, before0 = 0, before1 = 0, all0 = 0;
                    for (int w = 0; w < NW; ++w) {
                        const int c0 = rec2[w].hi, c1 = rec2[w].aux;
                        if (w < wave) {
                            before0 += c0;
                            before1 += c1;
                        }
                        all0 += c0;
                        total += c0 + c1;
                    }
                    bk = -__builtin_inf();
                    bid = ID_NONE;
                    if (total > 0) {
                        uint32_t c4[4] = {(uint32_t)iters, (uint32_t)k, 0x52504321u, 0u};
                        philox4x32_10(c4, (uint32_t)P.seed, (uint32_t)(P.seed >> 32));
                        const double u01 = (double)((uint64_t)(c4[0] >> 5) * 67108864ull + (c4[1] >> 6)) *
                                           (1.0 / 9007199254740992.0);
                        int target = (int)(u01 * total);
                        if (target >= total) target = total - 1;
                        const unsigned long long below = (1ull << lane) - 1ull;
                        const int r0 = before0 + __popcll(m0 & below), r1 = all0 + before1 + __popcll(m1 & below);
                        const bool h0 = (elig & 1) && r0 == target, h1 = (elig & 2) && r1 == target;
                        if (h0 || h1) {
                            bk = 1.0;
                            bid = h1 ? cv[1] : cv[0];
                            bpos = h1 ? t + NT : t;
                        }
                    }
                    __syncthreads();  // rec2 is written again by Step 2
                }
                const long long kb = __double_as_longlong(bk);
                int wh;
                unsigned wl;
                const int wpk = wave_argmax_i64((int)(kb >> 32), (unsigned)kb, pack_id(bid, bpos), wh, wl);
                const unsigned long long wnf = __ballot(nf);
                nf = false;
                if (lane == (wpk == PACK_NONE ? 0 : unpack_pos(wpk) & 63)) {
                    const bool c1 = wpk != PACK_NONE && unpack_pos(wpk) >= NT;
                    PendRec& r = rec1[wave];
                    r.hi = wh;
                    r.lo = wl;
                    r.pk = wpk;
                    r.aux = c1 ? sbirth[1] : sbirth[0];
                    r.v0 = c1 ? dO[1] : dO[0];
                    r.v1 = c1 ? dW[1] : dW[0];
                    r.nonfinite = wnf != 0;
                }
                lds_barrier();
                bool any;
                const int pk = pend_best<NW>(rec1, lane, th, tl, idx, any);
                nf_any |= any;
                if (pk == PACK_NONE) {
                    if (mode == 2) {
                        st = ST_OPTIMAL;
                        break;
                    }
                    if (zW > P.eps_feas * (1.0 + w0)) {
                        st = ST_INFEASIBLE;
                        break;
                    }
                    mode = 3;
                    drive_r = 0;
                    __syncthreads();  // rec1 is written again
                    continue;
                }
                if (iters >= max_iter) {
                    st = ST_ITER_LIMIT;
                    break;
                }
                e = unpack_pos(pk);
                e_id = unpack_id(pk);
            }
            const double fO = rec1[idx].v0, fW = rec1[idx].v1;
            int sbe = __builtin_amdgcn_readfirstlane(rec1[idx].aux);
            if (mode != 3 && (s == KP || nf_any)) {
                flush();
                nf_any = false;
                sbe = -1;
            }
            // entering column: this thread's row
            BLP_T(t_p1);
            double f = 0.0;
            {
                double v = 0.0;
                if (rowt && rbirth < 0 && sbe < 0) v = T[at(t, e)];
                v = pending(v, max(rbirth, sbe), F + (rowt ? t : 0), ldf, Q + e, ldq);
                f = rowt ? v : 0.0;
            }
            nf |= !isfinite(f);
            BLP_T(t_p2);
            // Step 2: one IEEE reciprocal y = 1 / f gives the ratio (rhs / f by
            // the corrected product of div_rn_fast) and, for the winner, the
            // reciprocal that divides the pivot row
            double rmin = 1.0, pe, y, pr;
            if (mode != 3) {
                const bool cand = rowt & !dead & (f > P.eps_piv);
                const double a = cand ? f : 1.0;
                double yv = 1.0 / a;
                __asm__("" : "+v"(yv));
                bool ok;
                double qt = div_rn_fast(bR, a, yv, (a >= 0x1p-500) & (a <= 0x1p500), ok);
                if (__ballot(cand & !ok)) qt = bR / a;
                const double ratio = bR <= 0.0 ? 0.0 : qt;
                const bool take = cand & (ratio <= __builtin_inf());  // (a NaN ratio is no candidate)
                const long long kb = __double_as_longlong(take ? ratio : __builtin_inf());
                int wh;
                unsigned wl;
                const int wpk =
                    wave_argmax_i64(~(int)(kb >> 32), ~(unsigned)kb, take ? pack_id(bs, t) : PACK_NONE, wh, wl);
                if (lane == (wpk == PACK_NONE ? 0 : unpack_pos(wpk) & 63)) {
                    PendRec& r = rec2[wave];
                    r.hi = wh;
                    r.lo = wl;
                    r.pk = wpk;
                    r.aux = rbirth;
                    r.v0 = f;
                    r.v1 = yv;
                    r.v2 = qt;
                    r.nonfinite = 0;
                }
                lds_barrier();
                bool any;
                const int pk = pend_best<NW>(rec2, lane, th, tl, idx, any);
                if (pk == PACK_NONE) {
                    st = mode == 2 ? ST_UNBOUNDED : ST_NUMERICAL;
                    break;
                }
                rmin = __longlong_as_double((long long)(((unsigned long long)(unsigned)~th << 32) | (unsigned)~tl));
                l = unpack_pos(pk);
                lv = unpack_id(pk);
                pe = rec2[idx].v0;
                y = rec2[idx].v1;
                pr = rec2[idx].v2;
            } else {
                __syncthreads();  // rec2[0] has been read by everyone
                if (t == l) {
                    rec2[0].v0 = f;
                    rec2[0].v1 = 1.0 / f;
                    rec2[0].v2 = bR / f;
                    rec2[0].aux = rbirth;
                }
                idx = 0;
                __syncthreads();
                pe = rec2[0].v0;
                y = rec2[0].v1;
                pr = rec2[0].v2;
            }
            const int rbl = __builtin_amdgcn_readfirstlane(rec2[idx].aux);
            BLP_T(t_p3);
            // Step 3: the new pivot row, the mirrors, and the pending factors
            double x[2];
            row_value(l, rbl, x);
            const double ape = fabs(pe);
            const bool pe_ok = ape >= 0x1p-500 && ape <= 0x1p500;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if (c == 1 && ns <= NT) break;
                const int j = t + c * NT;
                const bool ent = j == e;
                const double xv = ent ? 1.0 : x[c];
                bool ok;
                double p = div_rn_fast(xv, pe, y, pe_ok, ok);
                if (__ballot(!ok)) p = ok ? p : xv / pe;
                dO[c] = __builtin_fma(-fO, p, ent ? 0.0 : dO[c]);
                if (mode != 2) dW[c] = __builtin_fma(-fW, p, ent ? 0.0 : dW[c]);
                cv[c] = ent ? lv : cv[c];
                sbirth[c] = ent ? s : sbirth[c];
                nf |= !isfinite(p);
                if (j < ldq) Q[s * ldq + j] = p;
            }
            zO = __builtin_fma(-fO, pr, zO);
            zW = __builtin_fma(-fW, pr, zW);
            const bool piv = t == l;
            bR = piv ? pr : __builtin_fma(-f, pr, bR);
            bs = piv ? e_id : bs;
            rbirth = piv ? s : rbirth;
            if (t < ldf) F[s * ldf + t] = piv ? 1.0 : (rowt ? -f : 0.0);
            ++s;
            ++iters;
            if (mode != 3)
                degen = rmin == 0.0 ? degen + 1 : 0;
            else
                __syncthreads();  // rec1 and rec2 are written again
            BLP_T(t_p4);
            BLP_TACC(TM_PRICE, t_p0, t_p1);
            BLP_TACC(TM_PUBCOL, t_p1, t_p2);
            BLP_TACC(TM_RATIO, t_p2, t_p3);
            BLP_TACC(TM_PIVOT, t_p3, t_p4);
        }

        // ------------------------------------------------------ extraction
        // every structural and logical variable sits in one row (basic: x =
        // rhs, dual 0) or one slot (nonbasic: x = 0, dual from the objective
        // row); the duals take the row's sense
        BLP_T(t_x0);
        const double z = -zO;
        const int sto = st == ST_OPTIMAL && !isfinite(z) ? ST_NUMERICAL : st;
        const bool nan_out = sto == ST_NUMERICAL;
        const double qnan = __builtin_nan("");
        auto put_y = [&](int i, double d) __attribute__((always_inline)) {
            P.y[L.row_off + i] = nan_out ? qnan : (P.sense[Lin.row_off + i] != 0 ? d : -d);
        };
        if (rowt) {
            if (bs < n)
                P.x[L.col_off + bs] = nan_out ? qnan : bR;
            else if (bs < n + m)
                put_y(bs - n, 0.0);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int j = t + c * NT;
            if (j < ns) {
                if (cv[c] < n)
                    P.x[L.col_off + cv[c]] = nan_out ? qnan : 0.0;
                else if (cv[c] < n + m)
                    put_y(cv[c] - n, dO[c]);
            }
        }
        if (t == 0) {
            P.status[k] = sto;
            P.iters[k] = iters;
            P.obj[k] = (sto == ST_OPTIMAL || sto == ST_ITER_LIMIT) ? z
                       : sto == ST_UNBOUNDED                      ? __builtin_inf()
                       : sto == ST_INFEASIBLE                     ? -__builtin_inf()
                                                                  : qnan;
        }
        BLP_T(t_x1);
        BLP_TACC(TM_EXTRACT, t_x0, t_x1);
        BLP_TCOUNT(TM_PIVOTS, (unsigned long long)iters);
        BLP_TCOUNT(TM_LPS, 1ull);
    }
    BLP_TFLUSH();
}

constexpr int kPendWaves = 8;
static_assert(kPendRows == kPendWaves * 64 && kPendSlots == 2 * kPendWaves * 64, "one row and two slots per thread");
hipError_t launch_pend(const KParams& P, int grid, size_t lds_bytes, hipStream_t s) {
    hipLaunchKernelGGL(simplex_pend_kernel<kPendWaves>, dim3(grid), dim3(kPendWaves * 64), lds_bytes, s, P);
    return hipGetLastError();
}
const void* pend_kernel_ptr() { return reinterpret_cast<const void*>(&simplex_pend_kernel<kPendWaves>); }
int pend_threads() { return kPendWaves * 64; }

}  // namespace blp
