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
// Each thread owns a row (rhs, basis) and two slots (reduced costs,
// variables).  A pivot has two barriers: after every wave's best entering slot
// is published, and after every wave's best leaving row is; LPs that one wave
// holds have none.
//
// Pivot (l, e) at pending index s: row l becomes the pivot row p, so its older
// pending factors count for nothing and its factor is 1 on an entry of 0
// (fma(1, p, 0) = p; a -0 becomes +0, as in the kernels that update at every
// pivot); slot e becomes the leaving variable's column, on an entry of 0
// likewise.  A bit per row and slot (`rb`, `sb`) says that its
// tableau entries count as 0, and its older factors are zeroed, which changes
// nothing while the other factor is finite: a pivot with a non-finite entry is
// flushed before the next one, so that all older terms are finite.
//
// What bounds it: a pivot's chain of dependent steps (two memory reads, two
// reductions over the LP, the pending FMAs), which several workgroups per CU
// overlap, and the flush's trips through the last-level cache; for one-phase
// LPs the column reads from the row-major A.  So what counts is workgroups in
// flight, against the pending pivots that the LDS then leaves each.  Slots that
// an artificial variable left behind are dropped at each flush (a third of a
// type-2 tableau in the end), and the LDS that frees takes more pivots.
// Everything that steers a pivot is in scalar registers: with a value that the
// compiler takes for a per-lane one among them, its branches cost a sixth of
// the time.
// Measured against the kernels that took these LPs before: 1,000 two-phase LPs
// 200 x 200 (2,055 pivots each) 204 ms streaming at every pivot, 20.9 ms here;
// 4,000 of 100 x 100 22.0 ms in the 160 x 160 block tile, 7.8 here; 4,001 of 47 x
// 61 3.53 ms in the 112 x 112 block tile, 1.40 here; 50,000 one-phase LPs 100 x
// 100 3.67 ms in the block tile, 2.36 here (most of them end before the first
// flush, and their tableau is never written).
//
// Layout of a workspace slot: strips of four rows, in a strip blocks of 4 x 4
// entries, in a block row-major: an entry's offset is its row's part plus its
// slot's part.  One 128-byte line then serves four rows of a column read and
// four slots of a row read, and the 16 x 4 part of a matrix-core tile that one
// register holds is 512 consecutive bytes.  A strip is an odd number of lines
// (and so is a slot, one line longer than its strips), or columns and
// workgroups would meet in the same cache channels: 8,000 one-phase LPs 150 x
// 150 take 2.1 ms without that, 1.25 with it.
#include <type_traits>
#include <utility>

#include "aux_kernels.hpp"
#include "blp_kernels.hpp"
#include "simplex_blk.hpp"
#include "simplex_common.hpp"

namespace blp {

typedef double acc4 __attribute__((ext_vector_type(4)));

// a byte offset past any tableau: a buffer load there reads 0, a store is dropped
constexpr unsigned kPendOob = 0x80000000u;

// A wave's candidate: key (as wave_argmax_i64), packed (id, pos), flags (bit 0:
// the slot or row was replaced since the flush; bit 1: the wave saw a
// non-finite pivot entry), and what goes with the winner.
struct alignas(16) PendRec {
    int hi;
    unsigned lo;
    int pk, flags;
    double v0, v1, v2, pad;
};

// v's value in lane `src` (wave-uniform)
__device__ __forceinline__ double lane_f64(double v, int src) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), src),
                            __builtin_amdgcn_readlane(__double2loint(v), src));
}

// x + a0 b0, and so on over the four terms, one rounding each
__device__ __forceinline__ double fma4(double2 a0, double2 a1, double2 b0, double2 b1, double x) {
    x = __builtin_fma(a0.x, b0.x, x);
    x = __builtin_fma(a0.y, b0.y, x);
    x = __builtin_fma(a1.x, b1.x, x);
    return __builtin_fma(a1.y, b1.y, x);
}

// a value that is the same in every lane, in scalar registers
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <class T>
__device__ __forceinline__ T* uniform(T* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<T*>((uint64_t)(unsigned)uniform((int)v) |
                                (uint64_t)(unsigned)uniform((int)(v >> 32)) << 32);
}

// x / b, kept in its branch: the compiler would rather always make both quotients
__device__ __forceinline__ double plain_div(double x, double b) {
    __asm__ volatile("" : "+v"(x));
    return x / b;
}

// v, opaque to the compiler: what is computed from it is computed here, not
// ahead of the pivot loop and then spilled across it
__device__ __forceinline__ int here(int v) {
    __asm__ volatile("" : "+v"(v));
    return v;
}

// The best of the NW waves' records, under the order of wave_argmax_i64; every
// wave computes it.  (hi, lo, pk): this wave's own.  Returns the packed (id,
// pos); flags are the winner's bit 0 and bit 1 of any wave.  The winner's wave
// follows from its position.
template <int NW>
__device__ __forceinline__ int pend_best(const PendRec* rec, int lane, int wave, int hi, unsigned lo, int pk,
                                         unsigned& flags) {
    if constexpr (NW == 2) {  // against the other wave's, in scalar registers
        const PendRec& r = rec[wave ^ 1];
        const int ohi = __builtin_amdgcn_readfirstlane(r.hi), opk = __builtin_amdgcn_readfirstlane(r.pk);
        const unsigned olo = (unsigned)__builtin_amdgcn_readfirstlane((int)r.lo);
        const unsigned of = (unsigned)__builtin_amdgcn_readfirstlane(r.flags);
        const bool other = ohi > hi || (ohi == hi && (olo > lo || (olo == lo && opk < pk)));
        flags = (other ? of : flags) | ((flags | of) & 2u);
        return other ? opk : pk;
    } else {
        static_assert(NW == 4 || NW == 8, "one row of eight lanes");
        const PendRec& r = rec[lane & (NW - 1)];
        const bool in = lane < NW;
        const int h = in ? r.hi : (int)0x80000000;
        const unsigned l = r.lo;
        const int k = r.pk, f = r.flags;
        int v = h;
        v = max(v, dpp_src<0xB1, 0xF>(v));
        v = max(v, dpp_src<0x4E, 0xF>(v));
        if (NW > 4) v = max(v, dpp_src<0x141, 0xF>(v));
        const int top = __builtin_amdgcn_readlane(v, 0);
        const uint64_t nonfin = __ballot(in && (f & 2));
        uint64_t mk = __ballot(in && h == top);
        int idx = __ffsll((long long)mk) - 1;
        if (__popcll(mk) > 1) {  // equal high words: the low word, then the smallest id
            unsigned best = 0;
            for (uint64_t q = mk; q; q &= q - 1)
                best = max(best, (unsigned)__builtin_amdgcn_readlane((int)l, __ffsll((long long)q) - 1));
            mk = __ballot(in && h == top && l == best);
            idx = __ffsll((long long)mk) - 1;
            int wpk = __builtin_amdgcn_readlane(k, idx);
            for (uint64_t q = mk & (mk - 1); q; q &= q - 1) {
                const int c = __ffsll((long long)q) - 1, p = __builtin_amdgcn_readlane(k, c);
                idx = p < wpk ? c : idx;
                wpk = p < wpk ? p : wpk;
            }
        }
        idx = __builtin_amdgcn_readfirstlane(idx);
        flags = ((unsigned)__builtin_amdgcn_readlane(f, idx) & 1u) | (nonfin ? 2u : 0u);
        return __builtin_amdgcn_readlane(k, idx);
    }
}

// NW waves; thread t owns row t and the slots t and t + NT, NT = 64 NW; a wave
// flushes TC slot tiles at a time.
template <int NW, int TC, int WPE>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
simplex_pend_kernel(KParams) {
    constexpr int NT = NW * 64, CT = 2;
    extern __shared__ __align__(16) double s_mem[];  // pending factors: F of the rows, then Q of the slots
    __shared__ PendRec rec1[NW], rec2[NW];
    __shared__ unsigned short s_art[NT];  // artificial rows in row order
    __shared__ unsigned long long s_mask[NW], s_neg[NW];  // artificial rows, negated rows (bit per row)
    __shared__ unsigned long long s_dead[CT * NW];
    __shared__ unsigned short s_rowmask[NT / 16], s_slotmask[CT * NT / 16];
    __shared__ int s_ctl[2][2];

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    BLP_TDECL;
    bool first = true;
    int shard = 0;  // (thread 0)
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
                q = pop_position(P, len, first, shard);
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
        const int m = uniform(L.m), n = uniform(L.n);
        if (m > NT || n + m > CT * NT) continue;  // another streaming kernel's (uniform over the workgroup)

        // ------------------------------------------------------------ load
        double* const T = uniform(P.ws + (int64_t)blockIdx.x * P.ws_slot);
        const double* const A = uniform(P.A + Lin.a_off);
        const double eps_price = P.eps_price, eps_piv = P.eps_piv;
        const int rule = P.pivot_rule, lds = P.ws_lds;
        const bool rowt = t < m;
        int bad = 0;
        double bR = 0.0;
        int bs = ID_NONE;
        bool art = false;
        unsigned neg = 0;  // sign bit of the row's factor
        if (rowt) {
            const double bi = P.b[Lin.row_off + t];
            const bool ge = P.sense[Lin.row_off + t] != 0;
            const double ble = ge ? -bi : bi;
            art = ble < 0.0;
            neg = ge != art ? 0x80000000u : 0u;
            bR = art ? -ble : ble;
            bs = art ? n + m + t : n + t;
            bad = !isfinite(bi);
        }
        const unsigned long long mart = __ballot(art), mneg = __ballot(neg != 0);
        if (lane == 0) {
            s_mask[wave] = mart;
            s_neg[wave] = mneg;
        }
        __syncthreads();
        // artificial rows in row order: the masks before this wave's, then its own
        int nart = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            if (w == wave && art) s_art[nart + __popcll(mart & ((1ull << lane) - 1ull))] = (unsigned short)t;
            nart += __popcll(s_mask[w]);
        }
        nart = __builtin_amdgcn_readfirstlane(nart);
        __syncthreads();
        const int ns0 = n + nart;  // column slots; the rhs is not one of them
        int ns = ns0;              // slots still in use (the flush drops those of artificial variables)
        const int nsp = ((ns0 + 3) & ~3) | 4;  // slots of the workspace tableau: an odd number of blocks
        // Pending factors: KP pivots of m + ns entries, in groups of four
        // pivots: a group holds its four factors of row (slot) i in 32 bytes.
        // Their two halves change places with every fourth i, so that 16-byte
        // reads of consecutive rows spread over the LDS banks.
        int KP, qbase;  // qbase: byte offset of Q
        auto layout = [&]() {
            KP = min(32, (lds / (m + ns)) & ~3);
            qbase = KP * m * 8;
        };
        layout();
        // byte offset of row (slot) i's first pair within a group of F (Q); the
        // other pair is at this ^ 16
        auto f_off = [](int i) __attribute__((always_inline)) { return i * 32 + ((i >> 2) & 1) * 16; };
        auto pair = [](int off) __attribute__((always_inline)) -> double2 {
            return *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(s_mem) + off);
        };
        // factor u of row i of an array with `len` rows at byte offset `base`
        auto cell = [](int base, int len, int i, int u) __attribute__((always_inline)) -> double& {
            return *reinterpret_cast<double*>(reinterpret_cast<char*>(s_mem) + base + ((u >> 2) * len + i) * 32 +
                                              ((((u >> 1) ^ (i >> 2)) & 1) * 16 + (u & 1) * 8));
        };
        if (KP < 4 || (int64_t)((m + 15) & ~15) * nsp > P.ws_slot) {  // never launched so
            write_numerical<NT>(P, L, k, t, ST_INTERNAL);
            continue;
        }
        // byte offset of (i, j) in the tableau: the row's part plus the slot's
        auto row_part = [&](int i) __attribute__((always_inline)) { return ((i >> 2) * nsp + (i & 3)) * 32; };
        auto slot_part = [](int j) __attribute__((always_inline)) { return (j >> 2) * 128 + (j & 3) * 8; };
        const unsigned tbytes = (unsigned)((m + 3) & ~3) * (unsigned)nsp * 8u;
        const __amdgpu_buffer_rsrc_t wsr = __builtin_amdgcn_make_buffer_rsrc(T, (short)0, (int)tbytes, 0x00020000);
        // this LP's constraints; until the first flush they are the tableau
        const __amdgpu_buffer_rsrc_t asr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<double*>(A), (short)0, m * n * (int)sizeof(double), 0x00020000);
        auto buf = [](__amdgpu_buffer_rsrc_t r, unsigned vo, int so) __attribute__((always_inline)) {
            return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)vo, so, 0));
        };
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
                        two, (quad)__builtin_amdgcn_raw_buffer_load_b128(asr, x < pairs ? x * 16 : (int)kPendOob, 0, 0));
                    v[u][0] = w[0];
                    v[u][1] = w[1];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) bad |= !isfinite(v[u][0]) | !isfinite(v[u][1]);
            }
            if ((m * n) & 1) bad |= !isfinite(A[m * n - 1]);
        }
        // every factor +0 in F and -0 in Q: the products, -0, leave every value as it is
        auto clear_factors = [&](int pivots) __attribute__((always_inline)) {
            typedef double two __attribute__((ext_vector_type(2)));
            auto fill = [&](int off, int len, double v) __attribute__((always_inline)) {
                for (int u = 0; u < pivots; u += 4, off += len * 32) {
                    two* const w = reinterpret_cast<two*>(reinterpret_cast<char*>(s_mem) + off);
                    w[0] = w[1] = two{v, v};
                }
            };
            if (rowt) fill(t * 32, m, 0.0);
#pragma unroll
            for (int c = 0; c < CT; ++c)
                if (t + c * NT < ns) fill(qbase + (t + c * NT) * 32, ns, -0.0);
        };
        clear_factors(KP);
        // dP: the objective row that prices (the phase-1 row first, then the
        // objective); dS: the objective during phase 1.  A slot that cannot
        // enter (an artificial variable's, or none) holds -inf.
        double dP[CT], dS[CT];
        int cv[CT];
        double w0 = 0.0;
        const double ninf = -__builtin_inf();
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int j = t + c * NT;
            dP[c] = dS[c] = ninf;
            cv[c] = j < n ? j : (j < ns ? n + (int)s_art[j - n] : ID_NONE);
            if (j < n) {
                const double cj = P.c[L.col_off + j];
                bad |= !isfinite(cj);
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
                dP[c] = nart > 0 ? acc : cj;
                dS[c] = cj;
            } else if (j < ns) {
                dP[c] = -1.0;
                dS[c] = 0.0;
            }
        }
        for (int q = 0; q < nart; ++q) {
            const double bi = P.b[Lin.row_off + s_art[q]];
            w0 = w0 + fabs(bi);  // an artificial row's normalised rhs is |b|
        }
        if (bad) atomicOr(&s_ctl[par][1], 1);
        __syncthreads();
        if (uniform(s_ctl[par][1])) {
            write_numerical<NT>(P, L, k, t, ST_NUMERICAL);
            continue;
        }
        double zP = nart > 0 ? w0 : 0.0, zS = 0.0;  // rhs cells of the objective rows
        bool live = rowt;                           // not a redundant row
        int mode = nart > 0 ? 1 : 2;
        const int max_iter = P.max_iter > 0 ? P.max_iter : 50 * (m + n);
        const int bland_after = P.bland_after > 0 ? P.bland_after : (m > n ? m : n);
        const int id_lim = n + m;
        int iters = 0, degen = 0, st = -1, drive_r = 0;
        int s = 0;                   // pending pivots
        bool rb = false;             // this thread's row was replaced since the last flush
        unsigned sb = 0;             // bit c: its slot c likewise
        unsigned long long nfm = 0;  // lanes of this wave that saw a non-finite pivot entry
        bool nf_any = false;
        bool from_a = true;  // no flush yet: the tableau is A with the row signs, and the surplus columns
        int zl = -1;         // row whose older factors are still to be zeroed
        // byte offsets of this thread's row and slots in the tableau (or in A):
        // out of range where the entries count as 0
        unsigned ro = rowt ? (unsigned)t * (unsigned)n * 8u : kPendOob;
        unsigned so[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) so[c] = t + c * NT < n ? (unsigned)(t + c * NT) * 8u : kPendOob;
        // byte offsets of its factors (clamped into the arrays)
        const int fad = f_off(min(t, m - 1));
        int qad[CT];
        auto slot_factors = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < CT; ++c) qad[c] = qbase + f_off(min(t + c * NT, ns - 1));
        };
        slot_factors();

        // Current values of row r at this thread's slots (row_new: its entries count as 0).
        auto row_value = [&](int r, bool row_new, double (&x)[CT]) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < CT; ++c) x[c] = 0.0;
            if (!row_new) {
                if (!from_a) {
                    const int lp = row_part(r);
                    x[0] = buf(wsr, so[0], lp);
                    if (ns > NT) x[1] = buf(wsr, so[1], lp);
                } else {
                    const bool flip = (s_neg[r >> 6] >> (r & 63)) & 1ull;
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
                        const double v = buf(asr, so[c], r * n * 8);
                        x[c] = flip && so[c] != kPendOob ? -v : v;
                        const int j = t + c * NT;
                        if (j >= n && j < ns && !((sb >> c) & 1u)) x[c] = s_art[j - n] == r ? -1.0 : 0.0;
                    }
                }
            }
            int fa = f_off(r), q0 = qad[0], q1 = qad[1];
            if (ns > NT) {
                for (int kb = 0; kb < s; kb += 4, fa += m * 32, q0 += ns * 32, q1 += ns * 32) {
                    const double2 a0 = pair(fa), a1 = pair(fa ^ 16), b0 = pair(q0), b1 = pair(q0 ^ 16), c0 = pair(q1),
                                  c1 = pair(q1 ^ 16);
                    x[0] = fma4(a0, a1, b0, b1, x[0]);
                    x[1] = fma4(a0, a1, c0, c1, x[1]);
                }
            } else {
                for (int kb = 0; kb < s; kb += 4, fa += m * 32, q0 += ns * 32)
                    x[0] = fma4(pair(fa), pair(fa ^ 16), pair(q0), pair(q0 ^ 16), x[0]);
            }
        };
        // Bring the tableau up to date.
        auto flush = [&]() __attribute__((always_inline)) {
            lds_barrier();  // the last pivot's factors have been read
            const int lh = here(lane), lr = lh >> 4, lc = lh & 15;  // row of a strip, column of a slot tile
            if (zl >= 0 && wave == zl >> 6 && lane < s - 1) cell(0, m, zl, lane) = 0.0;
            zl = -1;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const unsigned long long ms = __ballot((sb >> c) & 1u);
                if (lc == 0) s_slotmask[(c * NT + wave * 64 + lh) >> 4] = (unsigned short)(ms >> lh);
            }
            const unsigned long long mr = __ballot(rb);
            if (lc == 0) s_rowmask[(wave * 64 + lh) >> 4] = (unsigned short)(mr >> lh);
            __syncthreads();
            // A unit is a row tile by TC slot tiles; a wave takes every NW-th.
            // (Loading the next unit's entries meanwhile changed nothing: the
            // workgroups of a CU already overlap each other's loads.)
            const int nr = (m + 15) >> 4, ncg = (ns + 16 * TC - 1) / (16 * TC);
            int R = wave, cg = 0;
            while (R >= nr) {
                R -= nr;
                ++cg;
            }
            while (cg < ncg) {
                acc4 d[TC];
                unsigned o[TC];  // byte offset of register 0; the next strips follow 32 nsp bytes apart
                int sr[4];       // (cut at the end, which the range check subtracts it from)
#pragma unroll
                for (int r = 0; r < 4; ++r) sr[r] = min(r * (32 * nsp), (int)tbytes);
#pragma unroll
                for (int c = 0; c < TC; ++c) {
                    const int j = (cg * TC + c) * 16 + lc;
                    o[c] = j < ns ? (unsigned)(row_part(16 * R + lr) + slot_part(j)) : kPendOob;
                }
                if (!from_a) {
#pragma unroll
                    for (int c = 0; c < TC; ++c)
#pragma unroll
                        for (int r = 0; r < 4; ++r) d[c][r] = buf(wsr, o[c], sr[r]);
                } else {  // with the row signs and the surplus columns
                    const unsigned long long mw = s_neg[R >> 2] >> ((R & 3) * 16);
#pragma unroll
                    for (int c = 0; c < TC; ++c) {
                        const int j = (cg * TC + c) * 16 + lc;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int i = 16 * R + 4 * r + lr;
                            d[c][r] = buf(asr, i < m && j < n ? (unsigned)(i * n + j) * 8u : kPendOob, 0);
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
                    const unsigned sm = jt * 16 < ns ? s_slotmask[jt] : 0u;
                    if (__builtin_amdgcn_readfirstlane((int)(sm | rm))) {
                        const bool cb = (sm >> lc) & 1;
#pragma unroll
                        for (int r = 0; r < 4; ++r) d[c][r] = cb | rz[r] ? 0.0 : d[c][r];
                    }
                }
                // four terms per step; the next step's factors are read ahead
                // (the rows and slots past the end use the last one's)
                auto term = [&](int off) __attribute__((always_inline)) {
                    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(s_mem) + off);
                };
                const int half = (lr >> 1) * 16, odd = (lr & 1) * 8;
                int fa = (f_off(min(R * 16 + lc, m - 1)) ^ half) + odd, qb[TC];
#pragma unroll
                for (int c = 0; c < TC; ++c)
                    qb[c] = qbase + (f_off(min((cg * TC + c) * 16 + lc, ns - 1)) ^ half) + odd;
                double a = term(fa), b[TC];
#pragma unroll
                for (int c = 0; c < TC; ++c) b[c] = term(qb[c]);
                for (int g = 0; g < s; g += 4) {
                    const bool more = g + 4 < s;
                    fa += more ? m * 32 : 0;
                    const double an = term(fa);
                    double bn[TC];
#pragma unroll
                    for (int c = 0; c < TC; ++c) {
                        qb[c] += more ? ns * 32 : 0;
                        bn[c] = term(qb[c]);
                    }
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
                            __builtin_bit_cast(unsigned int __attribute__((ext_vector_type(2))), w), wsr, (int)o[c],
                            sr[r], 0);
                    }
                R += NW;
                while (R >= nr) {
                    R -= nr;
                    ++cg;
                }
            }
            __syncthreads();
            // A slot that holds an artificial variable never enters again and
            // feeds no output: the last slot takes its place.  (The random
            // rule ranks the slots in slot order, so it keeps them.)
            const int ns_was = ns;
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
                    if (rowt) T[(row_part(t) + slot_part(to)) >> 3] = T[(row_part(t) + slot_part(from)) >> 3];
#pragma unroll
                    for (int c = 0; c < CT; ++c)
                        if (t + c * NT == from) {
                            rec1[0].v0 = dP[c];
                            rec1[0].v1 = dS[c];
                            rec1[0].pk = cv[c];
                        }
                }
                __syncthreads();
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    if (!gone && t + c * NT == to) {
                        dP[c] = rec1[0].v0;
                        dS[c] = rec1[0].v1;
                        cv[c] = rec1[0].pk;
                    }
                    if (t + c * NT == from) {
                        dP[c] = dS[c] = ninf;
                        cv[c] = ID_NONE;
                    }
                }
                --ns;
                lds_barrier();  // rec1 and s_dead are written again
            }
            // clean factors; with fewer slots, room for more pivots
            if (ns != ns_was) layout();
            clear_factors(ns != ns_was ? KP : s);
            s = 0;
            rb = false;
            sb = 0;
            from_a = false;
            ro = rowt ? (unsigned)row_part(t) : kPendOob;
            slot_factors();
#pragma unroll
            for (int c = 0; c < CT; ++c) so[c] = t + c * NT < ns ? (unsigned)slot_part(t + c * NT) : kPendOob;
            lds_barrier();  // the factors are clean before anyone reads them
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
            int e, e_id, l, lv;
            double fP, fS;
            bool col_new;
            if (mode == 3) {
                // the first row still holding an artificial variable
                const int mine = wave_min_i32(live && t >= drive_r && bs >= id_lim ? t : NT);
                if (lane == 0) rec1[wave] = {-mine, 0u, 0, nfm ? 2 : 0};
                __syncthreads();
                int r0 = NT;
                bool any = false;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    r0 = min(r0, -rec1[w].hi);
                    any |= (rec1[w].flags & 2) != 0;
                }
                r0 = __builtin_amdgcn_readfirstlane(r0);
                nf_any = __builtin_amdgcn_readfirstlane((int)any) != 0;
                nfm = 0;
                __syncthreads();  // rec1 is written again below
                if (nf_any) continue;  // flush first
                if (r0 >= NT) {  // phase 2: the objective prices
                    mode = 2;
                    degen = 0;
                    zP = zS;
#pragma unroll
                    for (int c = 0; c < CT; ++c) dP[c] = dS[c];
                    continue;
                }
                drive_r = r0 + 1;
                if (t == r0) rec2[0] = {0, 0u, bs, rb ? 1 : 0};
                __syncthreads();
                const bool row_new = __builtin_amdgcn_readfirstlane(rec2[0].flags) != 0;
                lv = __builtin_amdgcn_readfirstlane(rec2[0].pk);
                // the lowest-id non-artificial column with a usable entry enters
                double x[CT];
                row_value(r0, row_new, x);
                int pk = PACK_NONE;
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    if (t + c * NT < ns && cv[c] < id_lim && fabs(x[c]) > eps_piv) pk = min(pk, pack_id(cv[c], t + c * NT));
                pk = wave_min_i32(pk);
                if (lane == 0) rec1[wave] = {0, 0u, pk, 0};
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    if (pk != PACK_NONE && t + c * NT == unpack_pos(pk)) {
                        rec1[wave].flags = (sb >> c) & 1u;
                        rec1[wave].v0 = dP[c];
                        rec1[wave].v1 = dS[c];
                    }
                __syncthreads();
#pragma unroll
                for (int w = 0; w < NW; ++w) pk = min(pk, rec1[w].pk);
                pk = __builtin_amdgcn_readfirstlane(pk);
                if (pk == PACK_NONE) {  // redundant row
                    live = live && t != r0;
                    __syncthreads();
                    continue;
                }
                l = r0;
                e = unpack_pos(pk);
                e_id = unpack_id(pk);
                const PendRec& r = rec1[(e >> 6) & (NW - 1)];
                fP = r.v0;
                fS = r.v1;
                col_new = __builtin_amdgcn_readfirstlane(r.flags) != 0;
            } else {
                // Step 1: this wave's best slot
                double key = dP[0], ds = dS[0];
                int pk;
                unsigned bit = sb & 1u;
                bool ok = key > eps_price;
                const bool bland = degen >= bland_after;
                if (ns > NT) {
                    const double d1 = dP[1];
                    const bool ok1 = d1 > eps_price;
                    const bool less = bland ? cv[0] < cv[1] : (key > d1) | ((key == d1) & (cv[0] < cv[1]));
                    const bool take = ok1 & !(ok & less);
                    key = take ? d1 : key;
                    ds = take ? dS[1] : ds;
                    bit = take ? (sb >> 1) & 1u : bit;
                    ok |= ok1;
                    pk = take ? (cv[1] << 16) | (t + NT) : (cv[0] << 16) | t;
                } else {
                    pk = (cv[0] << 16) | t;
                }
                double ck = ok ? (bland ? 0.0 : key) : ninf;
                pk = ok ? pk : PACK_NONE;
                if (rule == 1 && !bland) {
                    // Sec. 4.2's random positive coefficient: the target-th
                    // eligible slot in slot order
                    __syncthreads();  // s_dead is free
                    unsigned long long em[CT];
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
                        em[c] = __ballot(t + c * NT < ns && cv[c] < id_lim && dP[c] > eps_price);
                        if (lane == 0) s_dead[c * NW + wave] = em[c];
                    }
                    __syncthreads();
                    int total = 0, rank[CT];
#pragma unroll
                    for (int w = 0; w < CT * NW; ++w) {
                        if ((w & (NW - 1)) == wave) rank[w / NW] = total + __popcll(em[w / NW] & ((1ull << lane) - 1ull));
                        total += __popcll(s_dead[w]);
                    }
                    ck = ninf;
                    pk = PACK_NONE;
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
                            if (((em[c] >> lane) & 1ull) && rank[c] == target) {
                                ck = 1.0;
                                pk = pack_id(cv[c], t + c * NT);
                                key = dP[c];
                                ds = dS[c];
                                bit = (sb >> c) & 1u;
                            }
                    }
                }
                const long long kb = __double_as_longlong(ck);
                int wh;
                unsigned wl;
                pk = wave_argmax_i64((int)(kb >> 32), (unsigned)kb, pk, wh, wl);
                unsigned flags = nfm ? 2u : 0u;
                nfm = 0;
                if constexpr (NW > 1) {
                    if (lane == (pk == PACK_NONE ? 0 : pk & 63)) {
                        PendRec& r = rec1[wave];
                        *reinterpret_cast<int4*>(&r) = make_int4(wh, (int)wl, pk, (int)(flags | bit));
                        r.v0 = key;
                        r.v1 = ds;
                    }
                    if (NW == 2)
                        flags = (flags & 2u) | ((unsigned)__builtin_amdgcn_readlane((int)bit, pk & 63) & 1u);
                    lds_barrier();
                    pk = pend_best<NW>(rec1, lane, wave, wh, wl, pk, flags);
                }
                if (flags & 2u) {  // a non-finite pivot entry: flush first, then price again
                    nf_any = true;
                    if (NW > 1) __syncthreads();  // rec1 is written again
                    continue;
                }
                if (pk == PACK_NONE) {
                    if (mode == 2) {
                        st = ST_OPTIMAL;
                        break;
                    }
                    if (zP > kparams().eps_feas * (1.0 + w0)) {
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
                    const PendRec& r = rec1[(e >> 6) & (NW - 1)];
                    fP = r.v0;
                    fS = r.v1;
                    col_new = flags & 1u;
                } else {
                    fP = lane_f64(key, e & 63);
                    fS = lane_f64(ds, e & 63);
                    col_new = __builtin_amdgcn_readlane((int)bit, e & 63) & 1;
                }
            }
            // entering column: this thread's row
            BLP_T(t_p1);
            double f = 0.0;
            if (!col_new) {
                if (!from_a) {
                    f = buf(wsr, ro, slot_part(e));
                } else if (e < n) {
                    f = buf(asr, ro, e * 8);
                    f = __hiloint2double(__double2hiint(f) ^ (int)neg, __double2loint(f));
                } else {
                    f = s_art[e - n] == t && !rb ? -1.0 : 0.0;
                }
            }
            // the last pivot row's older factors: nobody else reads them now
            if (zl >= 0 && wave == zl >> 6 && lane < s - 1) cell(0, m, zl, lane) = 0.0;
            int fb = qbase + f_off(e), fa = fad;
            for (int kb = 0; kb < s; kb += 4, fa += m * 32, fb += ns * 32)
                f = fma4(pair(fa), pair(fa ^ 16), pair(fb), pair(fb ^ 16), f);
            f = rowt ? f : 0.0;
            nfm |= __ballot(!isfinite(f));
            BLP_T(t_p2);
            // Step 2: one IEEE reciprocal y = 1 / f gives the ratio (rhs / f by
            // the corrected product of div_rn_fast) and, for the winner, the
            // reciprocal that divides the pivot row
            double pe, y, pr;
            bool row_new;
            if (mode != 3) {
                const bool cand = live & (f > eps_piv);
                const double a = cand ? f : 1.0;
                double yv = 1.0 / a;
                __asm__("" : "+v"(yv));
                bool ok;
                double qt = div_rn_fast(bR, a, yv, (a >= 0x1p-500) & (a <= 0x1p500), ok);
                if (__ballot(cand & !ok)) qt = plain_div(bR, a);
                const double ratio = bR <= 0.0 ? 0.0 : qt;
                const bool take = cand & (ratio <= __builtin_inf());  // (a NaN ratio is no candidate)
                const long long kb = __double_as_longlong(take ? ratio : __builtin_inf());
                int wh;
                unsigned wl;
                int pk =
                    wave_argmax_i64(~(int)(kb >> 32), ~(unsigned)kb, take ? (bs << 16) | t : PACK_NONE, wh, wl);
                unsigned flags = 0;
                if constexpr (NW > 1) {
                    if (lane == (pk == PACK_NONE ? 0 : pk & 63)) {
                        PendRec& r = rec2[wave];
                        *reinterpret_cast<int4*>(&r) = make_int4(wh, (int)wl, pk, rb ? 1 : 0);
                        r.v0 = f;
                        r.v1 = yv;
                        r.v2 = qt;
                    }
                    if (NW == 2) flags = (__ballot(rb) >> (pk & 63)) & 1ull;
                    lds_barrier();
                    pk = pend_best<NW>(rec2, lane, wave, wh, wl, pk, flags);
                }
                if (pk == PACK_NONE) {
                    st = mode == 2 ? ST_UNBOUNDED : ST_NUMERICAL;
                    break;
                }
                l = unpack_pos(pk);
                lv = unpack_id(pk);
                if constexpr (NW > 1) {
                    const PendRec& r = rec2[l >> 6];
                    pe = r.v0;
                    y = r.v1;
                    pr = r.v2;
                    row_new = flags & 1u;
                } else {
                    pe = lane_f64(f, l);
                    y = lane_f64(yv, l);
                    pr = lane_f64(qt, l);
                    row_new = (__ballot(rb) >> l) & 1ull;
                }
                degen = pr <= 0.0 ? degen + 1 : 0;  // a zero step
            } else {
                __syncthreads();  // rec2[0] has been read by everyone
                if (t == l) {
                    rec2[0].flags = rb ? 1 : 0;
                    rec2[0].v0 = f;
                    rec2[0].v1 = 1.0 / f;
                    rec2[0].v2 = bR / f;
                }
                __syncthreads();
                pe = rec2[0].v0;
                y = rec2[0].v1;
                pr = rec2[0].v2;
                row_new = __builtin_amdgcn_readfirstlane(rec2[0].flags) != 0;
            }
            BLP_T(t_p3);
            // Step 3: the new pivot row, the mirrors, and the pending factors
            double x[CT];
            row_value(l, row_new, x);
            const double ape = fabs(pe);
            const bool pe_ok = ape >= 0x1p-500 && ape <= 0x1p500;
            // slot e's older factors (its column has been read by everyone)
            if (wave == ((e >> 6) & (NW - 1)) && lane < s) cell(qbase, ns, e, lane) = -0.0;
            auto new_slot = [&](auto cc) __attribute__((always_inline)) {
                constexpr int c = decltype(cc)::value;
                const int j = t + c * NT;
                const bool ent = j == e;
                const double xv = ent ? 1.0 : x[c];
                bool ok;
                double p = div_rn_fast(xv, pe, y, pe_ok, ok);
                if (__ballot(!ok)) p = plain_div(xv, pe);  // extreme magnitudes only: the plain division
                dP[c] = __builtin_fma(-fP, p, ent ? 0.0 : dP[c]);
                if (mode != 2) dS[c] = __builtin_fma(-fS, p, ent ? 0.0 : dS[c]);
                cv[c] = ent ? lv : cv[c];
                so[c] = ent ? kPendOob : so[c];
                sb |= ent ? 1u << c : 0u;
                if (lv >= id_lim) {  // an artificial variable never enters again
                    dP[c] = ent ? ninf : dP[c];
                    dS[c] = ent ? ninf : dS[c];
                }
                nfm |= __ballot(!isfinite(p));
                if (j < ns) cell(qbase, ns, j, s) = p;
            };
            new_slot(std::integral_constant<int, 0>{});
            if (ns > NT) new_slot(std::integral_constant<int, 1>{});
            zP = __builtin_fma(-fP, pr, zP);
            zS = __builtin_fma(-fS, pr, zS);
            const bool piv = t == l;
            bR = piv ? pr : __builtin_fma(-f, pr, bR);
            bs = piv ? e_id : bs;
            ro = piv ? kPendOob : ro;
            neg = piv ? 0u : neg;
            rb |= piv;
            if (rowt) cell(0, m, t, s) = piv ? 1.0 : -f;
            zl = l;
            ++s;
            ++iters;
            if (mode == 3) __syncthreads();  // rec1 and rec2 are written again
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
        const double z = mode == 2 ? -zP : -zS;
        const int sto = st == ST_OPTIMAL && !isfinite(z) ? ST_NUMERICAL : st;
        const bool nan_out = sto == ST_NUMERICAL;
        const double qnan = __builtin_nan("");
        auto put_y = [&](int i, double d) __attribute__((always_inline)) {
            PX.y[LX.row_off + i] = nan_out ? qnan : (PX.sense[sense_off + i] != 0 ? d : -d);
        };
        if (rowt) {
            if (bs < n)
                PX.x[LX.col_off + bs] = nan_out ? qnan : bR;
            else if (bs < n + m)
                put_y(bs - n, 0.0);
        }
#pragma unroll
        for (int c = 0; c < CT; ++c)
            if (t + c * NT < ns) {
                if (cv[c] < n)
                    PX.x[LX.col_off + cv[c]] = nan_out ? qnan : 0.0;
                else if (cv[c] < n + m)
                    put_y(cv[c] - n, mode == 2 ? dP[c] : dS[c]);
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
    hipLaunchKernelGGL((simplex_pend_kernel<T.waves, T.tiles, T.wpe>), dim3(grid), dim3(T.waves * 64), lds_bytes,
                       s, P);
    return hipGetLastError();
}
template <int I>
static const void* pend_ptr_i() {
    constexpr PendTile T = kPendTiles[I];
    return reinterpret_cast<const void*>(&simplex_pend_kernel<T.waves, T.tiles, T.wpe>);
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
