// Simplex kernel with pending pivots: one LP per workgroup, the condensed
// tableau in a per-workgroup workspace slot in HBM, and the rank-1 updates of
// Step 3 (Sec. 4.3) collected and applied KP at a time.  Until the first of
// these flushes the tableau is the caller's A.
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
// Each thread owns RT rows (rhs, basis) and CT slots (reduced costs,
// variables).  A pivot has two barriers: after every wave's best entering slot
// is published, and after every wave's best leaving row is; LPs that one wave
// holds have none.
//
// Pivot (l, e) at pending index s: row l becomes the pivot row p, so its older
// pending factors count for nothing and its factor is 1 on an entry of 0
// (fma(1, p, 0) = p); slot e becomes the leaving variable's column, on an
// entry of 0 likewise.  A bit per row and slot (`rb`, `sb`) says that its
// tableau entries count as 0, and its older factors are zeroed, which changes
// nothing while the other factor is finite: a pivot with a non-finite entry is
// flushed before the next one, so that all older terms are finite.
//
// What bounds it: for large LPs the flush's trips through the last-level cache
// (a 200 x 200 type-2 tableau of ~480 KB, 16 pivots per flush), then the two
// dependent memory reads and the reductions of a pivot, which several
// workgroups per CU overlap.  Slots that an artificial variable left behind are
// dropped at each flush (a third of a type-2 tableau in the end).  Measured
// against the kernels that took these LPs before: 1,000 two-phase LPs 200 x
// 200 (2,055 pivots each) 203 ms streaming at every pivot, 23.3 ms here; 4,000
// of 100 x 100 22.0 ms in the 160 x 160 block tile, 10.4 here; 4,001 of 47 x 61
// 3.51 ms in the 112 x 112 block tile, 1.59 here; 50,000 one-phase LPs 100 x 100
// 3.67 ms in the block tile, 2.96 here (most of them end before the first
// flush, and their tableau is never written).
//
// Layout of a slot: strips of four rows, in a strip blocks of 4 x 4 entries
// (the last one 4 x (slots mod 4)), in a block row-major: element (i, j) at
// (i / 4) 4 ns + (j / 4) 16 + (i mod 4) w + j mod 4, w the block's width.  One
// 128-byte line then serves four rows of a column read and four slots of a
// row read, and the 16 x 4 part of a matrix-core tile that one register holds
// is 512 consecutive bytes.
#include <utility>

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

// v, opaque to the compiler: what is computed from it is computed here, not
// ahead of the pivot loop and then spilled across it
__device__ __forceinline__ int here(int v) {
    __asm__ volatile("" : "+v"(v));
    return v;
}

// The best of the NW waves' records, under the order of wave_argmax_i64, and
// whether any record's non-finite flag is set; every wave computes it.
// Returns the packed (id, pos); idx is the record.
template <int NW>
__device__ __forceinline__ int pend_best(const PendRec* rec, int lane, int& hi, unsigned& lo, int& idx,
                                         bool& nonfinite) {
    static_assert(NW <= 8, "one row of eight lanes");
    const PendRec& r = rec[lane & (NW - 1)];
    const bool in = lane < NW;
    const int h = in ? r.hi : (int)0x80000000;
    const unsigned l = r.lo;
    const int pk = r.pk;
    nonfinite = __ballot(in && r.nonfinite) != 0;
    int v = h;
    v = max(v, dpp_src<0xB1, 0xF>(v));
    if (NW > 2) v = max(v, dpp_src<0x4E, 0xF>(v));
    if (NW > 4) v = max(v, dpp_src<0x141, 0xF>(v));
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

// NW waves; thread t owns the rows t + q NT (q < RT) and the slots t + c NT
// (c < CT), NT = 64 NW; a wave flushes TC slot tiles at a time.
template <int NW, int RT, int CT, int TC, int WPE>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
simplex_pend_kernel(KParams) {
    constexpr int NT = NW * 64;
    extern __shared__ __align__(16) double s_mem[];  // F (ldf x KS), then Q (ldq x KS)
    __shared__ PendRec rec1[NW], rec2[NW];
    __shared__ unsigned short s_art[RT * NT];  // artificial rows in row order
    __shared__ unsigned long long s_mask[RT * NW], s_neg[RT * NW];  // artificial rows, negated rows (bit per row)
    __shared__ unsigned long long s_dead[CT * NW];
    __shared__ unsigned short s_rowmask[RT * NT / 16], s_slotmask[CT * NT / 16];
    __shared__ int s_ctl[2][2];

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    BLP_TDECL;
    bool first = true;
    int par = 0;
    for (;;) {
        par ^= 1;
        const KParams P = kparams();
        if (t == 0) {
            const int64_t len = work_len(P);
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
        if (m > RT * NT || n + m > CT * NT) continue;  // another streaming kernel's (uniform over the workgroup)

        // ------------------------------------------------------------ load
        double* const T = P.ws + (int64_t)blockIdx.x * P.ws_slot;
        const double* const A = P.A + Lin.a_off;
        const double eps_price = P.eps_price, eps_piv = P.eps_piv;
        const int rule = P.pivot_rule;
        int bad = 0;
        double bR[RT];
        int bs[RT];
        unsigned neg = 0;  // bit q: this thread's row q is negated
        bool art[RT];
#pragma unroll
        for (int q = 0; q < RT; ++q) {
            const int i = t + q * NT;
            bR[q] = 0.0;
            bs[q] = ID_NONE;
            art[q] = false;
            if (i < m) {
                const double bi = P.b[Lin.row_off + i];
                const bool ge = P.sense[Lin.row_off + i] != 0;
                const double ble = ge ? -bi : bi;
                art[q] = ble < 0.0;
                neg |= (ge != art[q] ? 1u : 0u) << q;
                bR[q] = art[q] ? -ble : ble;
                bs[q] = art[q] ? n + m + i : n + i;
                bad |= !isfinite(bi);
            }
            const unsigned long long mart = __ballot(art[q]), mneg = __ballot((neg >> q) & 1u);
            if (lane == 0) {
                s_mask[q * NW + wave] = mart;
                s_neg[q * NW + wave] = mneg;
            }
        }
        __syncthreads();
        // artificial rows in row order: the masks before this thread's, then its own
        int nart = 0;
#pragma unroll
        for (int w = 0; w < RT * NW; ++w) {
            const unsigned long long mw = s_mask[w];
            if (art[w / NW] && (w & (NW - 1)) == wave)
                s_art[nart + __popcll(mw & ((1ull << lane) - 1ull))] = (unsigned short)(t + w / NW * NT);
            nart += __popcll(mw);
        }
        nart = __builtin_amdgcn_readfirstlane(nart);
        __syncthreads();
        const int ns0 = n + nart;  // column slots; the rhs is not one of them
        int ns = ns0;              // slots still in use (the flush drops those of artificial variables)
        // this LP's pending factors: KP pivots of ldf + ldq entries
        const int ldf = (m + 15) & ~15, ldq = (ns0 + 15) & ~15;
        // (a row's or slot's factors lie together, KS = KP + 2 apart: KS / 2
        // is odd, so 16-byte reads of consecutive rows spread over the banks)
        const int KP = min(32, (P.ws_lds / (ldf + ldq) - 2) & ~3);
        const int KS = KP + 2;
        double* const F = s_mem;
        double* const Q = s_mem + KS * ldf;
        if (KP < 4 || (int64_t)((m + 3) & ~3) * ns0 > P.ws_slot) {  // never launched so
            write_numerical<NT>(P, L, k, t, ST_INTERNAL);
            continue;
        }
        const int ns4 = ns0 >> 2, nrem = ns0 & 3;
        auto at = [&](int i, int j) __attribute__((always_inline)) -> int {
            return (i >> 2) * (4 * ns0) + (j >> 2) * 16 + (i & 3) * ((j >> 2) == ns4 ? nrem : 4) + (j & 3);
        };
        const unsigned tbytes = (unsigned)((m + 3) & ~3) * (unsigned)ns0 * 8u;
        const __amdgpu_buffer_rsrc_t wsr = __builtin_amdgcn_make_buffer_rsrc(T, (short)0, (int)tbytes, 0x00020000);
        // this LP's constraints; until the first flush they are the tableau
        const __amdgpu_buffer_rsrc_t asr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<double*>(A), (short)0, m * n * (int)sizeof(double), 0x00020000);
        {
            // every entry is checked once: 16-byte loads (dword-aligned is
            // enough for them), U of them in flight per lane
            constexpr int U = 12;
            const int pairs = (m * n) >> 1;
            for (int x0 = t; x0 < pairs; x0 += U * NT) {
                double v[U][2];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int x = x0 + u * NT;
                    typedef unsigned int quad __attribute__((ext_vector_type(4)));
                    typedef double two __attribute__((ext_vector_type(2)));
                    const two w = __builtin_bit_cast(
                        two, (quad)__builtin_amdgcn_raw_buffer_load_b128(asr, x < pairs ? x * 16 : (int)0x80000000, 0, 0));
                    v[u][0] = w[0];
                    v[u][1] = w[1];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) bad |= !isfinite(v[u][0]) | !isfinite(v[u][1]);
            }
            if ((m * n) & 1) bad |= !isfinite(A[m * n - 1]);
        }
#pragma unroll
        for (int q = 0; q < RT; ++q)
            if (t + q * NT < ldf)
                for (int u = 0; u < KP; ++u) F[(t + q * NT) * KS + u] = 0.0;
#pragma unroll
        for (int c = 0; c < CT; ++c)
            if (t + c * NT < ldq)
                for (int u = 0; u < KP; ++u) Q[(t + c * NT) * KS + u] = -0.0;
        double dO[CT], dW[CT];
        int cv[CT];
        double w0 = 0.0;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int j = t + c * NT;
            dO[c] = dW[c] = 0.0;
            cv[c] = j < n ? j : (j < ns ? n + (int)s_art[j - n] : ID_NONE);
            if (j < n) {
                dO[c] = P.c[L.col_off + j];
                bad |= !isfinite(dO[c]);
                // phase-1 row: the artificial rows (signs applied) summed in row order
                double acc = 0.0;
                for (int q0 = 0; q0 < nart; q0 += 8) {
                    double v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[u] = A[(int)s_art[q0 + u < nart ? q0 + u : q0] * n + j];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (q0 + u < nart) {
                            const int i = s_art[q0 + u];
                            acc = acc + ((s_neg[i >> 6] >> (i & 63)) & 1ull ? -v[u] : v[u]);
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
        unsigned dead = 0;  // bit q: this thread's row q is redundant
        int mode = nart > 0 ? 1 : 2;
        const int max_iter = P.max_iter > 0 ? P.max_iter : 50 * (m + n);
        const int bland_after = P.bland_after > 0 ? P.bland_after : (m > n ? m : n);
        const int id_lim = n + m;
        int iters = 0, degen = 0, st = -1, drive_r = 0;
        int s = 0;               // pending pivots
        unsigned rb = 0, sb = 0;  // bit q: this thread's row / slot q was replaced since the last flush
        bool nf = false;         // this thread saw a non-finite pivot entry
        bool nf_any = false;
        bool from_a = true;  // no flush yet: the tableau is A with the row signs, and the surplus columns
        int zl = -1;         // row whose older factors are still to be zeroed

        // row r's sign (uniform r): set when the row is negated
        auto row_neg = [&](int r) __attribute__((always_inline)) {
            return (bool)((s_neg[r >> 6] >> (r & 63)) & 1ull);
        };
        // The pending terms.  The entries past s are +0 in F and -0 in Q: their
        // products, -0, leave every value as it is.
        // Current column of slot e (col_new: replaced since the flush).
        auto column = [&](int e, bool col_new, double (&f)[RT]) __attribute__((always_inline)) {
            const int th = here(t);
#pragma unroll
            for (int q = 0; q < RT; ++q) {
                const int i = th + q * NT;
                f[q] = 0.0;
                if (i < m && !((rb >> q) & 1u) && !col_new) {
                    if (!from_a)
                        f[q] = T[at(i, e)];
                    else if (e >= n)
                        f[q] = s_art[e - n] == i ? -1.0 : 0.0;
                    else
                        f[q] = (neg >> q) & 1u ? -A[i * n + e] : A[i * n + e];
                }
            }
            // the last pivot row's older factors: nobody else reads them now
            if (zl >= 0 && wave == ((zl >> 6) & (NW - 1)) && lane < s - 1) F[zl * KS + lane] = 0.0;
            zl = -1;
            const double* const fb = Q + e * KS;
            const double* const fa = F + th * KS;
            for (int kb = 0; kb < s; kb += 4) {
                double b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) b[u] = fb[kb + u];
#pragma unroll
                for (int q = 0; q < RT; ++q)
                    if (q == 0 || m > q * NT) {
                        const double* const a = fa + (th + q * NT < ldf ? q * NT * KS : 0) + kb;
#pragma unroll
                        for (int u = 0; u < 4; ++u) f[q] = __builtin_fma(a[u], b[u], f[q]);
                    }
            }
#pragma unroll
            for (int q = 0; q < RT; ++q) f[q] = th + q * NT < m ? f[q] : 0.0;
        };
        // Current values of row r at this thread's slots.
        auto row_value = [&](int r, bool row_new, double (&x)[CT]) __attribute__((always_inline)) {
            const bool flip = from_a && row_neg(r);
            const int th = here(t);
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const int j = th + c * NT;
                x[c] = 0.0;
                if (j < ns && !row_new && !((sb >> c) & 1u)) {
                    if (!from_a)
                        x[c] = T[at(r, j)];
                    else if (j >= n)
                        x[c] = s_art[j - n] == r ? -1.0 : 0.0;
                    else
                        x[c] = flip ? -A[r * n + j] : A[r * n + j];
                }
            }
            const double* const fa = F + r * KS;
            const double* const fq = Q + th * KS;
            for (int kb = 0; kb < s; kb += 4) {
                double a[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) a[u] = fa[kb + u];
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    if (c == 0 || ns > c * NT) {
                        const double* const b = fq + (th + c * NT < ldq ? c * NT * KS : 0) + kb;
#pragma unroll
                        for (int u = 0; u < 4; ++u) x[c] = __builtin_fma(a[u], b[u], x[c]);
                    }
            }
        };
        // Bring the tableau up to date.
        auto flush = [&]() __attribute__((always_inline)) {
            lds_barrier();  // the last pivot's factors have been read
            const int lh = here(lane), lr = lh >> 4, lc = lh & 15;  // row of a strip, column of a slot tile
            if (zl >= 0 && wave == ((zl >> 6) & (NW - 1)) && lane < s - 1) F[zl * KS + lane] = 0.0;
            zl = -1;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const unsigned long long ms = __ballot((sb >> c) & 1u);
                if (lc == 0) s_slotmask[(c * NT + wave * 64 + lh) >> 4] = (unsigned short)(ms >> lh);
            }
#pragma unroll
            for (int q = 0; q < RT; ++q) {
                const unsigned long long mr = __ballot((rb >> q) & 1u);
                if (lc == 0) s_rowmask[(q * NT + wave * 64 + lh) >> 4] = (unsigned short)(mr >> lh);
            }
            __syncthreads();
            // A unit is a row tile by TC slot tiles; a wave takes every NW-th.
            // (Loading the next unit's entries meanwhile changed nothing: the
            // workgroups of a CU already overlap each other's loads.)
            const int nr = ldf >> 4, ncg = (ns + 16 * TC - 1) / (16 * TC);
            int R = wave, cg = 0;
            while (R >= nr) {
                R -= nr;
                ++cg;
            }
            while (cg < ncg) {
                acc4 d[TC];
                int o[TC];  // byte offset of register 0; the next strips follow 32 ns0 bytes apart
#pragma unroll
                for (int c = 0; c < TC; ++c) {
                    const int j = (cg * TC + c) * 16 + lc;
                    const int w = (j >> 2) == ns4 ? nrem : 4;
                    o[c] = j < ns ? (16 * R * ns0 + (j >> 2) * 16 + lr * w + (j & 3)) * 8 : (int)0x80000000;
                }
                if (!from_a) {
#pragma unroll
                    for (int c = 0; c < TC; ++c)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            d[c][r] = __builtin_bit_cast(
                                double, __builtin_amdgcn_raw_buffer_load_b64(wsr, o[c], r * (32 * ns0), 0));
                } else {  // with the row signs and the surplus columns
                    const unsigned long long mw = s_neg[R >> 2] >> ((R & 3) * 16);
#pragma unroll
                    for (int c = 0; c < TC; ++c) {
                        const int j = (cg * TC + c) * 16 + lc;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int i = 16 * R + 4 * r + lr;
                            const int off = i < m && j < n ? (i * n + j) * 8 : (int)0x80000000;
                            d[c][r] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(asr, off, 0, 0));
                        }
                    }
#pragma unroll
                    for (int c = 0; c < TC; ++c) {
                        const int j = (cg * TC + c) * 16 + lc;
#pragma unroll
                        for (int r = 0; r < 4; ++r) d[c][r] = (mw >> (4 * r + lr)) & 1 ? -d[c][r] : d[c][r];
                        if (j >= n && j < ns) {
                            const int ar = s_art[j - n];
#pragma unroll
                            for (int r = 0; r < 4; ++r) d[c][r] = 16 * R + 4 * r + lr == ar ? -1.0 : 0.0;
                        }
                    }
                }
                const unsigned rm = s_rowmask[R];
                bool rz[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) rz[r] = (rm >> (4 * r + lr)) & 1;
#pragma unroll
                for (int c = 0; c < TC; ++c) {
                    const int jt = cg * TC + c;  // slot tile
                    const unsigned sm = jt * 16 < ldq ? s_slotmask[jt] : 0u;
                    if (__builtin_amdgcn_readfirstlane((int)(sm | rm))) {
                        const bool cb = (sm >> lc) & 1;
#pragma unroll
                        for (int r = 0; r < 4; ++r) d[c][r] = cb | rz[r] ? 0.0 : d[c][r];
                    }
                }
                // four terms per step; the next step's factors are read ahead
                const double* fa = F + (R * 16 + lc) * KS + lr;
                const double* qb[TC];
#pragma unroll
                for (int c = 0; c < TC; ++c) qb[c] = Q + (min((cg * TC + c) * 16, ldq - 16) + lc) * KS + lr;
                double a = fa[0], b[TC];
#pragma unroll
                for (int c = 0; c < TC; ++c) b[c] = qb[c][0];
                for (int g = 0; g < s; g += 4) {
                    const int gn = min(g + 4, KP - 4);
                    const double an = fa[gn];
                    double bn[TC];
#pragma unroll
                    for (int c = 0; c < TC; ++c) bn[c] = qb[c][gn];
#pragma unroll
                    for (int c = 0; c < TC; ++c) d[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[c], d[c], 0, 0, 0);
                    a = an;
#pragma unroll
                    for (int c = 0; c < TC; ++c) b[c] = bn[c];
                }
#pragma unroll
                for (int c = 0; c < TC; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const double w = d[c][r];
                        __builtin_amdgcn_raw_buffer_store_b64(
                            __builtin_bit_cast(unsigned int __attribute__((ext_vector_type(2))), w), wsr, o[c],
                            r * (32 * ns0), 0);
                    }
                R += NW;
                while (R >= nr) {
                    R -= nr;
                    ++cg;
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < RT; ++q)
                if (t + q * NT < ldf)
                    for (int u = 0; u < s; ++u) F[(t + q * NT) * KS + u] = 0.0;
#pragma unroll
            for (int c = 0; c < CT; ++c)
                if (t + c * NT < ldq)
                    for (int u = 0; u < s; ++u) Q[(t + c * NT) * KS + u] = -0.0;
            s = 0;
            rb = sb = 0;
            from_a = false;
            lds_barrier();  // the factors are reset (others read them)
            // A slot that holds an artificial variable never enters again and
            // feeds no output: the last slot takes its place.  (The random
            // rule ranks the slots in slot order, so it keeps them.)
            while (rule != 1 && ns > n) {
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const unsigned long long dm = __ballot(t + c * NT < ns && cv[c] >= id_lim);
                    if (lane == 0) s_dead[c * NW + wave] = dm;
                }
                lds_barrier();
                int to = -1;
#pragma unroll
                for (int w = CT * NW - 1; w >= 0; --w) {
                    const unsigned long long mk = s_dead[w];
                    if (mk) to = w * 64 + __ffsll((long long)mk) - 1;
                }
                to = __builtin_amdgcn_readfirstlane(to);
                if (to < 0) break;
                const int from = ns - 1;
                const bool gone = (s_dead[from >> 6] >> (from & 63)) & 1ull;
                if (!gone) {
#pragma unroll
                    for (int q = 0; q < RT; ++q)
                        if (t + q * NT < m) T[at(t + q * NT, to)] = T[at(t + q * NT, from)];
#pragma unroll
                    for (int c = 0; c < CT; ++c)
                        if (t + c * NT == from) {
                            rec1[0].v0 = dO[c];
                            rec1[0].v1 = dW[c];
                            rec1[0].aux = cv[c];
                        }
                }
                __syncthreads();
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    if (!gone && t + c * NT == to) {
                        dO[c] = rec1[0].v0;
                        dW[c] = rec1[0].v1;
                        cv[c] = rec1[0].aux;
                    }
                    cv[c] = t + c * NT == from ? ID_NONE : cv[c];
                }
                --ns;
                lds_barrier();  // rec1 and s_dead are written again
            }
            lds_barrier();
        };
        BLP_T(t_load1);
        BLP_TACC(TM_LOAD, t_load0, t_load1);

        // ------------------------------------------------------ pivot loop
        // mode 1 = phase 1, 2 = phase 2, 3 = driving the remaining basic
        // artificials out after a feasible phase 1
        for (;;) {
            BLP_T(t_p0);
            if (s == KP || nf_any) {
                flush();
                nf_any = false;
            }
            BLP_T(t_p0b);
            BLP_TACC(TM_RTEST, t_p0, t_p0b);
            int e, e_id, l = -1, lv = ID_NONE, idx, th;
            unsigned tl;
            double fO, fW;
            bool col_new;
            if (mode == 3) {
                // the first row still holding an artificial variable
                int mine = RT * NT;
#pragma unroll
                for (int q = RT - 1; q >= 0; --q)
                    if (t + q * NT < m && t + q * NT >= drive_r && bs[q] >= id_lim && !((dead >> q) & 1u))
                        mine = t + q * NT;
                mine = wave_min_i32(mine);
                if (lane == 0) rec1[wave].hi = -mine;
                if (__ballot(nf)) nf_any = true;
                nf = false;
                if (lane == 0) {
                    rec1[wave].lo = 0;
                    rec1[wave].pk = 0;
                    rec1[wave].nonfinite = nf_any;
                }
                __syncthreads();
                bool any;
                pend_best<NW>(rec1, lane, th, tl, idx, any);
                const int r0 = -th;
                __syncthreads();  // rec1 is written again below
                nf_any = any;
                if (any) continue;  // flush first
                if (r0 >= RT * NT) {
                    mode = 2;
                    degen = 0;
                    continue;
                }
                drive_r = r0 + 1;
#pragma unroll
                for (int q = 0; q < RT; ++q)
                    if (t + q * NT == r0) {
                        rec2[0].aux = (rb >> q) & 1u;
                        rec2[0].pk = bs[q];
                    }
                __syncthreads();
                const bool row_new = __builtin_amdgcn_readfirstlane(rec2[0].aux) != 0;
                lv = __builtin_amdgcn_readfirstlane(rec2[0].pk);
                // the lowest-id non-artificial column with a usable entry enters
                double x[CT];
                row_value(r0, row_new, x);
                int pk = PACK_NONE;
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    if (t + c * NT < ns && cv[c] < id_lim && fabs(x[c]) > eps_piv) pk = min(pk, pack_id(cv[c], t + c * NT));
                pk = wave_min_i32(pk);
                if (lane == 0) {
                    rec1[wave].hi = pk == PACK_NONE ? (int)0x80000001 : -(pk >> 16);
                    rec1[wave].lo = 0;
                    rec1[wave].pk = pk;
                    rec1[wave].nonfinite = 0;
                }
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    if (pk != PACK_NONE && t + c * NT == unpack_pos(pk)) {
                        rec1[wave].v0 = dO[c];
                        rec1[wave].v1 = dW[c];
                        rec1[wave].aux = (sb >> c) & 1u;
                    }
                __syncthreads();
                pk = pend_best<NW>(rec1, lane, th, tl, idx, any);
                if (pk == PACK_NONE) {  // redundant row
#pragma unroll
                    for (int q = 0; q < RT; ++q) dead |= (t + q * NT == r0 ? 1u : 0u) << q;
                    __syncthreads();
                    continue;
                }
                l = r0;
                e = unpack_pos(pk);
                e_id = unpack_id(pk);
                fO = rec1[idx].v0;
                fW = rec1[idx].v1;
                col_new = __builtin_amdgcn_readfirstlane(rec1[idx].aux) != 0;
            } else {
                // Step 1: this wave's best slot
                double bk = -__builtin_inf();
                int bid = ID_NONE, bpos = -1;
                const bool rpc = rule == 1 && degen < bland_after;
                const bool bland = degen >= bland_after;
                unsigned elig = 0;
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const int j = t + c * NT;
                    const double d = mode == 1 ? dW[c] : dO[c];
                    const bool ok = (j < ns) & (cv[c] < id_lim) & (d > eps_price);
                    const double key = bland ? 0.0 : d;
                    const bool take = ok & ((key > bk) | ((key == bk) & (cv[c] < bid)));
                    bk = take ? key : bk;
                    bid = take ? cv[c] : bid;
                    bpos = take ? j : bpos;
                    elig |= (ok ? 1u : 0u) << c;
                }
                if (rpc) {
                    // Sec. 4.2's random positive coefficient: the target-th
                    // eligible slot in slot order
                    __syncthreads();  // s_dead is free
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
                        const unsigned long long em = __ballot((elig >> c) & 1u);
                        if (lane == 0) s_dead[c * NW + wave] = em;
                    }
                    __syncthreads();
                    int total = 0, rank[CT];
#pragma unroll
                    for (int w = 0; w < CT * NW; ++w) {
                        const unsigned long long em = s_dead[w];
                        if ((w & (NW - 1)) == wave) rank[w / NW] = total + __popcll(em & ((1ull << lane) - 1ull));
                        total += __popcll(em);
                    }
                    bk = -__builtin_inf();
                    bid = ID_NONE;
                    if (total > 0) {
                        uint32_t c4[4] = {(uint32_t)iters, (uint32_t)k, 0x52504321u, 0u};
                        const uint64_t seed = kparams().seed;
                        philox4x32_10(c4, (uint32_t)seed, (uint32_t)(seed >> 32));
                        const double u01 = (double)((uint64_t)(c4[0] >> 5) * 67108864ull + (c4[1] >> 6)) *
                                           (1.0 / 9007199254740992.0);
                        int target = (int)(u01 * total);
                        if (target >= total) target = total - 1;
#pragma unroll
                        for (int c = 0; c < CT; ++c)
                            if (((elig >> c) & 1u) && rank[c] == target) {
                                bk = 1.0;
                                bid = cv[c];
                                bpos = t + c * NT;
                            }
                    }
                }
                const long long kb = __double_as_longlong(bk);
                int wh;
                unsigned wl;
                int pk = wave_argmax_i64((int)(kb >> 32), (unsigned)kb, pack_id(bid, bpos), wh, wl);
                bool any = __ballot(nf) != 0;
                nf = false;
                if constexpr (NW > 1) {
                    PendRec& r = rec1[wave];
                    if (lane == 0) {
                        r.hi = wh;
                        r.lo = wl;
                        r.pk = pk;
                        r.nonfinite = any;
                    }
                    const int pos = unpack_pos(pk);
#pragma unroll
                    for (int c = 0; c < CT; ++c)
                        if (t + c * NT == pos) {
                            r.aux = (sb >> c) & 1u;
                            r.v0 = dO[c];
                            r.v1 = dW[c];
                        }
                    lds_barrier();
                    pk = pend_best<NW>(rec1, lane, th, tl, idx, any);
                }
                if (any) {  // a non-finite pivot entry: flush first, then price again
                    nf_any = true;
                    if (NW > 1) __syncthreads();  // rec1 is written again
                    continue;
                }
                if (pk == PACK_NONE) {
                    if (mode == 2) {
                        st = ST_OPTIMAL;
                        break;
                    }
                    if (zW > kparams().eps_feas * (1.0 + w0)) {
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
                if constexpr (NW > 1) {
                    fO = rec1[idx].v0;
                    fW = rec1[idx].v1;
                    col_new = __builtin_amdgcn_readfirstlane(rec1[idx].aux) != 0;
                } else {
                    fO = mirror_at(dO, e);
                    fW = mirror_at(dW, e);
                    col_new = ((unsigned)__builtin_amdgcn_readlane((int)sb, e & 63) >> (e >> 6)) & 1u;
                }
            }
            // entering column
            BLP_T(t_p1);
            double f[RT];
            column(e, col_new, f);
#pragma unroll
            for (int q = 0; q < RT; ++q) nf |= !isfinite(f[q]);
            BLP_T(t_p2);
            // Step 2: one IEEE reciprocal y = 1 / f per row gives the ratio
            // (rhs / f by the corrected product of div_rn_fast) and, for the
            // winner, the reciprocal that divides the pivot row
            double rmin = 1.0, pe, y, pr;
            bool row_new;
            if (mode != 3) {
                double yv[RT], qt[RT];
                bool cand[RT], slow = false;
#pragma unroll
                for (int q = 0; q < RT; ++q) {
                    cand[q] = (t + q * NT < m) & !((dead >> q) & 1u) & (f[q] > eps_piv);
                    const double a = cand[q] ? f[q] : 1.0;
                    yv[q] = 1.0 / a;
                    __asm__("" : "+v"(yv[q]));
                    bool ok;
                    qt[q] = div_rn_fast(bR[q], a, yv[q], (a >= 0x1p-500) & (a <= 0x1p500), ok);
                    slow |= cand[q] & !ok;
                }
                if (__ballot(slow)) {
#pragma unroll
                    for (int q = 0; q < RT; ++q) qt[q] = bR[q] / (cand[q] ? f[q] : 1.0);
                }
                double bk = -__builtin_inf();
                int bid = ID_NONE, bpos = -1;
#pragma unroll
                for (int q = 0; q < RT; ++q) {
                    const double key = bR[q] <= 0.0 ? -0.0 : -qt[q];
                    const bool take = cand[q] & ((key > bk) | ((key == bk) & (bs[q] < bid)));
                    bk = take ? key : bk;
                    bid = take ? bs[q] : bid;
                    bpos = take ? t + q * NT : bpos;
                }
                const long long kb = __double_as_longlong(-bk);
                int wh;
                unsigned wl;
                int pk = wave_argmax_i64(~(int)(kb >> 32), ~(unsigned)kb, pack_id(bid, bpos), wh, wl);
                if constexpr (NW > 1) {
                    PendRec& r = rec2[wave];
                    if (lane == 0) {
                        r.hi = wh;
                        r.lo = wl;
                        r.pk = pk;
                        r.nonfinite = 0;
                    }
                    const int pos = unpack_pos(pk);
#pragma unroll
                    for (int q = 0; q < RT; ++q)
                        if (t + q * NT == pos) {
                            r.aux = (rb >> q) & 1u;
                            r.v0 = f[q];
                            r.v1 = yv[q];
                            r.v2 = qt[q];
                        }
                    lds_barrier();
                    bool any;
                    pk = pend_best<NW>(rec2, lane, wh, wl, idx, any);
                }
                if (pk == PACK_NONE) {
                    st = mode == 2 ? ST_UNBOUNDED : ST_NUMERICAL;
                    break;
                }
                rmin = __longlong_as_double((long long)(((unsigned long long)(unsigned)~wh << 32) | (unsigned)~wl));
                l = unpack_pos(pk);
                lv = unpack_id(pk);
                if constexpr (NW > 1) {
                    pe = rec2[idx].v0;
                    y = rec2[idx].v1;
                    pr = rec2[idx].v2;
                    row_new = __builtin_amdgcn_readfirstlane(rec2[idx].aux) != 0;
                } else {
                    pe = mirror_at(f, l);
                    y = mirror_at(yv, l);
                    pr = mirror_at(qt, l);
                    row_new = ((unsigned)__builtin_amdgcn_readlane((int)rb, l & 63) >> (l >> 6)) & 1u;
                }
            } else {
                __syncthreads();  // rec2[0] has been read by everyone
#pragma unroll
                for (int q = 0; q < RT; ++q)
                    if (t + q * NT == l) {
                        rec2[0].v0 = f[q];
                        rec2[0].v1 = 1.0 / f[q];
                        rec2[0].v2 = bR[q] / f[q];
                        rec2[0].aux = (rb >> q) & 1u;
                    }
                __syncthreads();
                pe = rec2[0].v0;
                y = rec2[0].v1;
                pr = rec2[0].v2;
                row_new = __builtin_amdgcn_readfirstlane(rec2[0].aux) != 0;
            }
            BLP_T(t_p3);
            // Step 3: the new pivot row, the mirrors, and the pending factors
            double x[CT];
            row_value(l, row_new, x);
            const double ape = fabs(pe);
            const bool pe_ok = ape >= 0x1p-500 && ape <= 0x1p500;
            // slot e's older factors (its column has been read by everyone)
            if (wave == ((e >> 6) & (NW - 1)) && lane < s) Q[e * KS + lane] = -0.0;
            double p[CT];
            bool slow = false;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                x[c] = t + c * NT == e ? 1.0 : x[c];
                bool ok;
                p[c] = div_rn_fast(x[c], pe, y, pe_ok, ok);
                slow |= !ok;
            }
            if (__ballot(slow)) {  // extreme magnitudes only: the plain division
#pragma unroll
                for (int c = 0; c < CT; ++c) p[c] = x[c] / pe;
            }
            const int th2 = here(t);
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                if (c > 0 && ns <= c * NT) break;
                const int j = th2 + c * NT;
                const bool ent = j == e;
                dO[c] = __builtin_fma(-fO, p[c], ent ? 0.0 : dO[c]);
                if (mode != 2) dW[c] = __builtin_fma(-fW, p[c], ent ? 0.0 : dW[c]);
                cv[c] = ent ? lv : cv[c];
                sb |= (ent ? 1u : 0u) << c;
                nf |= !isfinite(p[c]);
                if (j < ldq) Q[j * KS + s] = p[c];
            }
            zO = __builtin_fma(-fO, pr, zO);
            zW = __builtin_fma(-fW, pr, zW);
#pragma unroll
            for (int q = 0; q < RT; ++q) {
                const int i = th2 + q * NT;
                const bool piv = i == l;
                bR[q] = piv ? pr : __builtin_fma(-f[q], pr, bR[q]);
                bs[q] = piv ? e_id : bs[q];
                rb |= (piv ? 1u : 0u) << q;
                if (i < ldf) F[i * KS + s] = piv ? 1.0 : (i < m ? -f[q] : 0.0);
            }
            zl = l;
            ++s;
            ++iters;
            if (mode != 3)
                degen = rmin == 0.0 ? degen + 1 : 0;
            else
                __syncthreads();  // rec1 and rec2 are written again
            BLP_T(t_p4);
            BLP_TACC(TM_PRICE, t_p0b, t_p1);
            BLP_TACC(TM_PUBCOL, t_p1, t_p2);
            BLP_TACC(TM_RATIO, t_p2, t_p3);
            BLP_TACC(TM_PIVOT, t_p3, t_p4);
        }

        // ------------------------------------------------------ extraction
        // every structural and logical variable sits in one row (basic: x =
        // rhs, dual 0) or one slot (nonbasic: x = 0, dual from the objective
        // row); the duals take the row's sense
        BLP_T(t_x0);
        const KParams PX = kparams();
        const LpRef LX = lp_ref(PX, k);
        const int64_t sense_off = lp_in(PX, LX).row_off;
        const double z = -zO;
        const int sto = st == ST_OPTIMAL && !isfinite(z) ? ST_NUMERICAL : st;
        const bool nan_out = sto == ST_NUMERICAL;
        const double qnan = __builtin_nan("");
        auto put_y = [&](int i, double d) __attribute__((always_inline)) {
            PX.y[LX.row_off + i] = nan_out ? qnan : (PX.sense[sense_off + i] != 0 ? d : -d);
        };
#pragma unroll
        for (int q = 0; q < RT; ++q)
            if (t + q * NT < m) {
                if (bs[q] < n)
                    PX.x[LX.col_off + bs[q]] = nan_out ? qnan : bR[q];
                else if (bs[q] < n + m)
                    put_y(bs[q] - n, 0.0);
            }
#pragma unroll
        for (int c = 0; c < CT; ++c)
            if (t + c * NT < ns) {
                if (cv[c] < n)
                    PX.x[LX.col_off + cv[c]] = nan_out ? qnan : 0.0;
                else if (cv[c] < n + m)
                    put_y(cv[c] - n, dO[c]);
            }
        if (t == 0) {
            PX.status[k] = sto;
            PX.iters[k] = iters;
            PX.obj[k] = (sto == ST_OPTIMAL || sto == ST_ITER_LIMIT) ? z
                        : sto == ST_UNBOUNDED                      ? __builtin_inf()
                        : sto == ST_INFEASIBLE                     ? -__builtin_inf()
                                                                   : qnan;
        }
        BLP_T(t_x1);
        BLP_TACC(TM_EXTRACT, t_x0, t_x1);
        BLP_TCOUNT(TM_PIVOTS, (unsigned long long)iters);
        BLP_TCOUNT(TM_LPS, 1ull);
    }
    const KParams P = kparams();  // (the phase timers' counters)
    (void)P;
    BLP_TFLUSH();
}

// The instantiations, smallest first (aux_kernels.hpp: kPendTiles).
template <int I>
static hipError_t launch_pend_i(const KParams& P, int grid, size_t lds_bytes, hipStream_t s) {
    constexpr PendTile T = kPendTiles[I];
    hipLaunchKernelGGL((simplex_pend_kernel<T.waves, T.rows_per, T.slots_per, T.tiles, T.wpe>), dim3(grid), dim3(T.waves * 64), lds_bytes,
                       s, P);
    return hipGetLastError();
}
template <int I>
static const void* pend_ptr_i() {
    constexpr PendTile T = kPendTiles[I];
    return reinterpret_cast<const void*>(&simplex_pend_kernel<T.waves, T.rows_per, T.slots_per, T.tiles, T.wpe>);
}
static_assert(kPendRows == kPendTiles[kPendTileCount - 1].rows() && kPendSlots == kPendTiles[kPendTileCount - 1].slots(),
              "pend_shape() is what the largest tile holds");
template <int... I>
static hipError_t launch_pend_any(std::integer_sequence<int, I...>, const KParams& P, int tile, int grid, size_t lds,
                                  hipStream_t s) {
    hipError_t e = hipErrorInvalidValue;
    (void)((tile == I && ((e = launch_pend_i<I>(P, grid, lds, s)), true)) || ...);
    return e;
}
template <int... I>
static const void* pend_ptr_any(std::integer_sequence<int, I...>, int tile) {
    const void* p = nullptr;
    (void)((tile == I && ((p = pend_ptr_i<I>()), true)) || ...);
    return p;
}
using PendIndex = std::make_integer_sequence<int, kPendTileCount>;
hipError_t launch_pend(const KParams& P, int tile, int grid, size_t lds_bytes, hipStream_t s) {
    return launch_pend_any(PendIndex{}, P, tile, grid, lds_bytes, s);
}
const void* pend_kernel_ptr(int tile) { return pend_ptr_any(PendIndex{}, tile); }

}  // namespace blp
