// Device kernels of the numerical setup, phase (b) of the paper's solver
// structure (Sec. V-A): local matrix values, local factorisations, the
// energy-minimising extension of eq. (2), the coarse matrix A_0 = Phi^T A Phi
// and its inverse.
#pragma once

#include "kernels_dense.hpp"

namespace gdsw {

// out[dst[p]] = val[src[p]] * (scale ? scale[row[src[p]]] * scale[col[src[p]]] : 1)
// (dst == nullptr: out[p]; src[p] < 0: a fill entry, 0).  Used to gather the
// local matrices A_i and A_{I_i I_i} from A, optionally symmetrically
// diagonally scaled.
__global__ void k_gather_vals(const double *__restrict__ val, const int64_t *__restrict__ src,
                              const int64_t *__restrict__ dst, double *__restrict__ out, int64_t cnt,
                              const double *__restrict__ scale, const int32_t *__restrict__ arow,
                              const int32_t *__restrict__ acol) {
    for (int64_t p = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; p < cnt;
         p += int64_t(gridDim.x) * blockDim.x) {
        const int64_t s = src[p];
        double v = 0.0;
        if (s >= 0) {
            v = val[s];
            if (scale) v *= scale[arow[s]] * scale[acol[s]];
        }
        out[dst ? dst[p] : p] = v;
    }
}

// ---------------------------------------------------------------------------
// FastILU (Sec. V-B, iterative variant of the incomplete factorisation):
// the entries of L (unit lower, strictly lower part stored) and U on the
// local patterns are fixed points of
//     l_ij = (a_ij - sum_{m<j} l_im u_mj) / u_jj   (i > j)
//     u_ij =  a_ij - sum_{m<i} l_im u_mj           (i <= j)
// and a sweep evaluates every entry from the previous sweep's values (one
// thread per entry, product pairs precomputed in ascending m).  Start:
// l_ij = a_ij / a_jj, u_ij = a_ij.
__global__ void k_fastilu_start(const double *__restrict__ a, const int32_t *__restrict__ dpos,
                                double *__restrict__ v, int64_t ne) {
    const int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (e >= ne) return;
    const int32_t d = dpos[e];
    v[e] = d >= 0 ? a[e] / a[d] : a[e];
}

__global__ void k_fastilu_sweep(const double *__restrict__ a, const int64_t *__restrict__ fptr,
                                const int32_t *__restrict__ pairs, const int32_t *__restrict__ dpos,
                                const double *__restrict__ vold, double *__restrict__ vnew, int64_t ne) {
    const int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (e >= ne) return;
    double acc = a[e];
    for (int64_t q = fptr[e]; q < fptr[e + 1]; ++q) acc -= vold[pairs[2 * q]] * vold[pairs[2 * q + 1]];
    const int32_t d = dpos[e];
    vnew[e] = d >= 0 ? acc / vold[d] : acc;
}

// status[i] = 1 + a local row of subdomain i whose pivot is zero or not
// finite (after FastILU sweeps); 0 if there is none
__global__ void k_ilu_pivot_check(const int64_t *__restrict__ ov_ptr, const int64_t *__restrict__ lrowptr,
                                  const int32_t *__restrict__ ldiag, const double *__restrict__ v,
                                  int *__restrict__ status) {
    const int i = blockIdx.x;
    const int64_t o = ov_ptr[i], ni = ov_ptr[i + 1] - o;
    for (int64_t l = threadIdx.x; l < ni; l += blockDim.x) {
        const double u = v[lrowptr[o + l] + ldiag[o + l]];
        if (u == 0.0 || !isfinite(u)) atomicCAS(status + i, 0, int(1 + l));
    }
}

// scale[d] = 1 / sqrt(A[d,d])
__global__ void k_diag_scale(const double *__restrict__ val, const int64_t *__restrict__ adiag,
                             double *__restrict__ scale, int64_t n) {
    int64_t d = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (d < n) scale[d] = 1.0 / sqrt(val[adiag[d]]);
}

__global__ void k_fill_i32(int *__restrict__ x, int v, int n) {
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < n; p += gridDim.x * blockDim.x) x[p] = v;
}

__global__ void k_fill(double *__restrict__ x, double v, int64_t n) {
    for (int64_t p = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; p < n;
         p += int64_t(gridDim.x) * blockDim.x)
        x[p] = v;
}

// ---------------------------------------------------------------------------
// ILU(0) of every A_i in its natural (ascending global dof) order, in place on
// the local CSR values; one workgroup per subdomain, rows of one level of the
// dependency DAG in parallel (level-set scheduling, Sec. V-B "Incomplete
// Local Solver").  Row-by-row form: for each k < l in row l (ascending),
// l_lk = a_lk / u_kk and a_lj -= l_lk u_kj for the j > k in both rows.
// status[i] = 1 + local row of a zero pivot.
__global__ void k_ilu0_factor(const int64_t *__restrict__ ov_ptr, const int64_t *__restrict__ lrowptr,
                              const int32_t *__restrict__ lcol, const int32_t *__restrict__ ldiag,
                              const int64_t *__restrict__ lvl_base, const int32_t *__restrict__ lvl_ptr,
                              const int32_t *__restrict__ lvl_rows, double *__restrict__ lval,
                              int *__restrict__ status) {
    const int i = blockIdx.x;
    const int64_t o = ov_ptr[i];
    const int64_t lb = lvl_base[i];
    const int nlev = int(lvl_base[i + 1] - lb) - 1;
    for (int L = 0; L < nlev; ++L) {
        const int beg = lvl_ptr[lb + L], end = lvl_ptr[lb + L + 1];
        for (int q = beg + threadIdx.x; q < end; q += blockDim.x) {
            const int l = lvl_rows[o + q];
            const int64_t p = o + l;
            const int64_t rs = lrowptr[p], re = lrowptr[p + 1];
            for (int64_t e = rs; e < re; ++e) {
                const int k = lcol[e];
                if (k >= l) break;
                const int64_t pk = o + k;
                const int64_t dk = lrowptr[pk] + ldiag[pk];
                const double lik = lval[e] / lval[dk];
                lval[e] = lik;
                int64_t a = dk + 1, f = e + 1;
                const int64_t ke = lrowptr[pk + 1];
                while (a < ke && f < re) {
                    const int ca = lcol[a], cf = lcol[f];
                    if (ca == cf) {
                        lval[f] -= lik * lval[a];
                        ++a;
                        ++f;
                    } else if (ca < cf) {
                        ++a;
                    } else {
                        ++f;
                    }
                }
            }
            if (lval[rs + ldiag[p]] == 0.0) atomicCAS(status + i, 0, 1 + l);
        }
        __syncthreads();
    }
}

// Packs the ILU(0) factors into the padded slot-major layout of the Jacobi
// sweeps: for row p of subdomain i (padded row R = ell_off[i] + l) slot s of
// the strictly lower part L at [s * ell_rows + R], of the strictly upper part
// scaled by the pivot (U_lj / U_ll) likewise, and 1 / U_ll.  Unused slots
// hold 0 with column 0.
// Slots of the register-resident ILU(0) sweeps: three L and three U entries
// per row; their local columns packed two per 32-bit word.
constexpr int ILU_KL = 3, ILU_KU = 3, ILU_CW = (ILU_KL + ILU_KU + 1) / 2;
// slot counts of the register-resident sweeps with phased L and U loads
// (ILU(k) with fill)
constexpr int ILU_KL2 = 6, ILU_KU2 = 6, ILU_CW2 = (ILU_KL2 + ILU_KU2 + 1) / 2;
// zeroed factor rows past the last subdomain's (the phased sweeps read up
// to workgroup size x rows per thread rows from a subdomain's first)
constexpr int64_t ILU_PAD_ROWS = 8192;

template <typename VT>
__global__ void k_ilu_pack(const int64_t *__restrict__ ov_ptr, const int64_t *__restrict__ ell_off,
                           const int64_t *__restrict__ lrowptr, const int32_t *__restrict__ lcol,
                           const int32_t *__restrict__ ldiag, const double *__restrict__ lval,
                           int64_t ell_rows, int KL, int KU, VT *__restrict__ Lv,
                           uint16_t *__restrict__ Lc, VT *__restrict__ Uv, uint16_t *__restrict__ Uc,
                           VT *__restrict__ dinv, uint32_t *__restrict__ Cp, int64_t cp_stride) {
    const int i = blockIdx.y;
    const int64_t o = ov_ptr[i], ni = ov_ptr[i + 1] - o;
    const int64_t npad = ell_off[i + 1] - ell_off[i];
    const int64_t l = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (l >= npad) return;
    const int64_t R = ell_off[i] + l;
    int sl = 0, su = 0;
    if (l < ni) {
        const int64_t p = o + l;
        const int64_t rs = lrowptr[p], re = lrowptr[p + 1];
        const double piv = lval[rs + ldiag[p]];
        for (int64_t e = rs; e < re; ++e) {
            const int c = lcol[e];
            if (c < l) {
                Lv[sl * ell_rows + R] = from_double<VT>(lval[e]);
                Lc[sl * ell_rows + R] = uint16_t(c);
                ++sl;
            } else if (c > l) {
                Uv[su * ell_rows + R] = from_double<VT>(lval[e] / piv);
                Uc[su * ell_rows + R] = uint16_t(c);
                ++su;
            }
        }
        dinv[R] = from_double<VT>(1.0 / piv);
    } else {
        dinv[R] = from_double<VT>(0.0);
    }
    // padding: a zero in the row's own column, so that whichever rows of an
    // iterate a kernel keeps at hand the padding reads one of them, and an
    // infinity reaches no row that does not couple to it (rows past the
    // subdomain: column 0)
    const uint16_t own = l < ni ? uint16_t(l) : uint16_t(0);
    const int nl = sl, nu = su;
    for (; sl < KL; ++sl) {
        Lv[sl * ell_rows + R] = from_double<VT>(0.0);
        Lc[sl * ell_rows + R] = own;
    }
    for (; su < KU; ++su) {
        Uv[su * ell_rows + R] = from_double<VT>(0.0);
        Uc[su * ell_rows + R] = own;
    }
    // Cp != nullptr: the row's L then U columns again, two per 32-bit word
    // (low half first), (KL + KU + 1) / 2 words per row, for the
    // register-resident sweeps: the words of a row together (cp_stride 0),
    // or word w of every row at w * cp_stride (each phase of the phased
    // sweeps then reads only its own words); padding in column 0, which these
    // sweeps keep (every row)
    if (Cp) {
        const int cw = (KL + KU + 1) / 2;
        for (int w = 0; w < cw; ++w) {
            uint32_t v = 0;
            for (int h = 0; h < 2; ++h) {
                const int k = 2 * w + h;
                const uint32_t c = k < nl ? Lc[k * ell_rows + R]
                                   : k >= KL && k < KL + nu ? Uc[(k - KL) * ell_rows + R] : 0u;
                v |= c << (16 * h);
            }
            Cp[cp_stride ? w * cp_stride + R : R * cw + w] = v;
        }
    }
}

// ---------------------------------------------------------------------------
// Banded Cholesky A = L L^T of one symmetric positive definite matrix per
// workgroup, in place in FP64.  Row-major band storage: row r holds columns
// r-b .. r at band[r*(b+1) + (c - r + b)]; the diagonal slot holds 1/L_rr.
// The arithmetic is that of a right-looking loop over panels of 16 columns,
// bit for bit: per earlier panel an entry loses one sum of 16 products formed
// on its own in ascending order, then its own panel's elimination.  The order
// of the work is left-looking, since each value is then written once
// (right-looking rewrites the whole b x b window per panel), by panels of 32
// columns (two of the 16), since the earlier columns are read once per panel,
// and by blocks of 32 rows.  Per panel:
//   (1) the diagonal block's sums, the earlier panels dealt to the wavefronts,
//       and their ordered subtraction through LDS;
//   (2) wavefront 0 eliminates that block (elim16, a row per lane) while each
//       other wavefront forms one block below it, C = A - sums, by matrix
//       instructions, transposed in registers;
//   (3) the rows of C eliminated with the block's rows (subst16), then the
//       blocks past the first ones, sums and elimination together.
// Each wavefront brings its operands (32 panel rows and 32 block rows of 16
// columns) in by whole 128-byte row segments, eight lanes to a row, and turns
// them through LDS of its own, the next ones' loads in flight meanwhile:
// operands loaded straight from the band (16 lanes on 16 rows) are bound by
// the cache lines touched per load.  The fill of a banded Cholesky factor
// stays inside the band; slots left of the band (the neighbouring row's) are
// masked in the chunks that meet its edge.  Bound by the chain of one panel
// (about 45,000 clocks at band 225: sums 15,000, the diagonal block's 32 pivots
// 18,000 beside the first blocks' 33,000, elimination of the rows 12,000), one
// workgroup per compute unit.  Against a right-looking loop with scalar
// multiply-adds and window updates through memory: 512 matrices of 3,375 rows
// and band 225 33.1 -> 8.0 ms, 27 of 3,000 and 335 28.2 -> 3.6 ms (45 of the 256
// registers a lane spill).  status[i] = 1 + row of the first non-positive pivot.
constexpr int DB = 32, DB_LD = DB + 1;   // panel width, padded LDS row stride (bank spread)
constexpr int CH_ST = 64 * 16;           // a wavefront's chunk: 64 rows of 16 columns

typedef double dbl2 __attribute__((ext_vector_type(2)));
typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));   // (rows start at any 8-byte address)

// LDS place of column c of a chunk's row r: a lane's four operands (columns
// g, g + 4, g + 8, g + 12) together, in 16-byte units permuted by the row, so
// that eight rows' reads of one unit cover all banks
__device__ __forceinline__ int chunk_unit(int r, int u) { return r * 16 + 2 * (u ^ (r & 7)); }
__device__ __forceinline__ int chunk_at(int r, int c) {
    return chunk_unit(r, 2 * (c & 3) + (c >> 3)) + ((c >> 2) & 1);
}

// this lane's operand of row r (columns j + g + 4 q); EDGE: columns below cmin
// (left of the band) count as zero
template <bool EDGE>
__device__ __forceinline__ dbl4 chunk_operand(const double *st, int r, int lg, int j, int cmin) {
    const dbl2 lo = *reinterpret_cast<const dbl2 *>(st + chunk_unit(r, 2 * lg));
    const dbl2 hi = *reinterpret_cast<const dbl2 *>(st + chunk_unit(r, 2 * lg + 1));
    dbl4 v = {lo[0], lo[1], hi[0], hi[1]};
    if constexpr (EDGE) {
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = j + lg + 4 * q >= cmin ? v[q] : 0.0;
    }
    return v;
}

// 32 rows of a chunk on their way to LDS: row 8 q + lane / 8, columns 2 (lane %
// 8) + {0, 1} of the chunk at j, row q at p + d[q].  Slots left of the band
// are read all the same: L(r, c) with c >= 0 lies at r b + b + c >= 0 of the
// subdomain's array.
__device__ __forceinline__ void chunk_load(dbl2 (&v)[4], const double *p, const int (&d)[4], int j) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const dbl2u *>(p + d[q] + j);
}
__device__ __forceinline__ void chunk_store(const dbl2 (&v)[4], double *st, int lane) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h) st[chunk_at(8 * q + (lane >> 3), 2 * (lane & 7) + h)] = v[q][h];
}

template <int NT>
__global__ __launch_bounds__(NT) void k_band_chol(double *__restrict__ band, const int64_t *__restrict__ off,
                                                  const int32_t *__restrict__ bwid,
                                                  const int64_t *__restrict__ rptr, int *__restrict__ status) {
    constexpr int NW = NT / 64;
    static_assert(NW == 8 && DB * DB_LD <= 2 * CH_ST, "eight wavefronts; a block's rows fit a wavefront's chunks");
    __shared__ __align__(16) double sC[NW][2 * CH_ST];   // the wavefronts' chunks
    __shared__ double sX[DB * DB_LD];                    // the diagonal block, then its factor's rows
    __shared__ __align__(16) double sd[2 * DB];          // sqrt(pivot) and reciprocal
    __shared__ __align__(16) double sT[2][EB * EB];      // the factor's two 16x16 triangles by columns
    const int i = blockIdx.x;
    if (off[i + 1] == off[i]) return;   // no band (empty, or a supernodal subdomain)
    const int n = int(rptr[i + 1] - rptr[i]);
    const int b = bwid[i];
    const int64_t w = b + 1;
    double *L = band + off[i];
    // (wv in a scalar register)
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    int li = lane & 15, lg = lane >> 4;
    double *st = sC[wv];
    // the block a wavefront forms in (2): the first block has the most columns
    // and goes to the wavefront beside the diagonal block's (wavefronts wv and
    // wv + 4 share a SIMD, whose matrix unit (2) leaves idle), the others pair
    // a long one with a short one
    const int t1 = wv < 4 ? wv + 1 : wv == 4 ? 1 : 12 - wv;
    auto row_at = [&](int r) { return L + (int64_t(r) * w + (b - r)); };   // &L(r, 0)
    // this lane's rows of a chunk of rows r0 .. r0 + 31 (past the matrix: its last row)
    auto chunk_rows = [&](int r0, int (&d)[4]) {
        const int r = min(r0 + (lane >> 3), n - 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) d[q] = (min(r0 + 8 * q + (lane >> 3), n - 1) - r) * b;
        return row_at(r) + 2 * (lane & 7);
    };
    for (int k0 = 0; k0 < n; k0 += DB) {
        const int kb = min(DB, n - k0);
        const int rend = min(n, k0 + kb + b);
        const int nblk = (rend - k0 + DB - 1) / DB;
        asm volatile("" : "+v"(li), "+v"(lg));   // (their addresses and masks are not to be kept across panels)
        int dp[4];
        const double *pp = chunk_rows(k0, dp);   // the panel's rows
        // ---- (1) two earlier panels of 16 per wavefront and round: the lower
        // tiles t of each sum at 768 slot + 256 t (value v of lane l at 64 v + l),
        // then A - sums in panel order
        const int j0 = max(0, k0 - b) & ~15;
        for (int jr = j0; jr == j0 || jr < k0; jr += 32 * NW) {
            const int c0 = min(k0 + li, n - 1) - b, c1 = min(k0 + 16 + li, n - 1) - b;
            dbl2 v[2][4];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int j = jr + 16 * (NW * u + wv);
                if (j < k0) chunk_load(v[u], pp, dp, j);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int j = jr + 16 * (NW * u + wv);
                if (j < k0) {
                    double *ck = st + 2 * 768;   // (past the sums)
                    wave_lds_fence();
                    chunk_store(v[u], ck, lane);
                    wave_lds_fence();
                    const dbl4 a0 = chunk_operand<true>(ck, li, lg, j, c0);
                    const dbl4 a1 = chunk_operand<true>(ck, 16 + li, lg, j, c1);
                    const dbl4 zero = {0.0, 0.0, 0.0, 0.0};
                    const dbl4 s0 = mfma_k16(a0, a0, zero), s1 = mfma_k16(a1, a0, zero), s2 = mfma_k16(a1, a1, zero);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        st[768 * u + 64 * q + lane] = s0[q];
                        st[768 * u + 256 + 64 * q + lane] = s1[q];
                        st[768 * u + 512 + 64 * q + lane] = s2[q];
                    }
                }
            }
            __syncthreads();
            const int np = min(2 * NW, (k0 - jr + 15) / 16);   // panels of this round
            for (int e = threadIdx.x; e < 3 * 256; e += NT) {
                const int t = e >> 8, q = (e >> 6) & 3, l = e & 63;
                const int r = 16 * (t > 0) + (l >> 4) + 4 * q, c = 16 * (t > 1) + (l & 15);
                double d;
                if (jr == j0) {
                    const int rr = min(k0 + r, n - 1);
                    d = row_at(rr)[max(min(k0 + c, rr), rr - b)];
                    d = r < kb && c <= r && r - c <= b ? d : (r >= kb && r == c ? 1.0 : 0.0);   // (identity past the matrix)
                } else {
                    d = sX[r * DB_LD + c];
                }
                if (r < kb && c <= r) {
#pragma unroll 4
                    for (int u = 0; u < np; ++u) d -= sC[u % NW][768 * (u / NW) + e];
                }
                if (c <= r) {   // (mirrored above the diagonal)
                    sX[r * DB_LD + c] = d;
                    sX[c * DB_LD + r] = d;
                }
            }
            __syncthreads();
        }
        // ---- (2)
        // C^T of block t (rows k0 + 32 t ..): cc[p][q], panel columns 16 p .., rows 16 q ..
        dbl4 cc[2][2];
        auto block_sum = [&](int t) __attribute__((always_inline)) {
            const int r0 = k0 + DB * t;
            int db[4];
            const double *pb = chunk_rows(r0, db);
            const int ib0 = min(r0 + li, n - 1), ib1 = min(r0 + 16 + li, n - 1);
            int j = max(0, r0 - b) & ~15;
            dbl2 va[4], vb[4];
            if (j < k0) {
                chunk_load(va, pp, dp, j);
                chunk_load(vb, pb, db, j);
            }
            {
                const double *rb0 = row_at(ib0) + k0, *rb1 = row_at(ib1) + k0;
                const int m0 = ib0 - b - k0, m1 = ib1 - b - k0;
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int c = 16 * p + lg + 4 * v;
                        cc[p][0][v] = rb0[max(c, m0)];
                        cc[p][1][v] = rb1[max(c, m1)];
                    }
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int c = 16 * p + lg + 4 * v;
                        cc[p][0][v] = c >= m0 ? cc[p][0][v] : 0.0;
                        cc[p][1][v] = c >= m1 ? cc[p][1][v] : 0.0;
                    }
            }
            // one chunk in use, the next one in LDS, the one after loading
            dbl4 f[4];
            auto to_lds = [&](int buf) __attribute__((always_inline)) {
                chunk_store(va, st + buf * CH_ST, lane);
                chunk_store(vb, st + buf * CH_ST + CH_ST / 2, lane);
            };
            auto operands = [&](int buf, int jj, dbl4 (&g)[4]) __attribute__((always_inline)) {
                const double *sb = st + buf * CH_ST;
                // (uniform: does the chunk meet the band's left edge?)
                if (jj < r0 + DB - 1 - b) {
                    g[0] = chunk_operand<true>(sb, li, lg, jj, k0 + li - b);
                    g[1] = chunk_operand<true>(sb, 16 + li, lg, jj, k0 + 16 + li - b);
                    g[2] = chunk_operand<true>(sb, 32 + li, lg, jj, ib0 - b);
                    g[3] = chunk_operand<true>(sb, 48 + li, lg, jj, ib1 - b);
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) g[u] = chunk_operand<false>(sb, 16 * u + li, lg, jj, 0);
                }
            };
            auto load = [&](int jj) __attribute__((always_inline)) {
                if (jj < k0) {
                    chunk_load(va, pp, dp, jj);
                    chunk_load(vb, pb, db, jj);
                }
            };
            if (j < k0) {
                to_lds(0);
                load(j + 16);
                for (int buf = 0; j < k0; j += 16, buf ^= 1) {
                    wave_lds_fence();
                    operands(buf, j, f);
                    if (j + 16 < k0) {
                        to_lds(buf ^ 1);
                        load(j + 32);
                    }
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        dbl4 s0 = {0.0, 0.0, 0.0, 0.0}, s1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            s0 = __builtin_amdgcn_mfma_f64_16x16x4f64(f[p][q], f[2][q], s0, 0, 0, 0);
                            s1 = __builtin_amdgcn_mfma_f64_16x16x4f64(f[p][q], f[3][q], s1, 0, 0, 0);
                        }
                        cc[p][0] -= s0;
                        cc[p][1] -= s1;
                    }
                }
                wave_lds_fence();
            }
        };
        if (wv == 0) {
            int r = lane & 31;
            asm volatile("" : "+v"(r));   // (no addresses kept across panels)
            double a[EB], ds, dy;
            int bad = 0;
            // columns 0..15: rows 0..15, and rows 16..31 in lanes 16..31
            static_for<EB>([&](auto c) { a[c] = sX[r * DB_LD + c]; });
            elim16(a, lane, 0, bad, ds, dy);
            wave_lds_fence();
            if (lane < 32) {
                static_for<EB>([&](auto c) { sX[r * DB_LD + c] = a[c]; });
                if (lane < EB) {
                    static_for<EB>([&](auto c) { sT[0][EB * c + r] = a[c]; });
                    sd[2 * lane] = ds, sd[2 * lane + 1] = dy;
                }
            }
            wave_lds_fence();
            // rows and columns 16..31 lose L10 L10^T
            {
                dbl4 f, s = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int q = 0; q < 4; ++q) f[q] = sX[(16 + li) * DB_LD + lg + 4 * q];
                s = mfma_k16(f, f, s);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    double *x = &sX[(16 + lg + 4 * v) * DB_LD + 16 + li];
                    // (rows past the matrix keep the identity)
                    if (max(lg + 4 * v, li) + 16 < kb) *x -= s[v];
                }
            }
            wave_lds_fence();
            static_for<EB>([&](auto c) { a[c] = sX[(16 + (r & 15)) * DB_LD + 16 + c]; });
            elim16(a, lane, 16, bad, ds, dy);
            wave_lds_fence();
            if (lane < EB) {
                static_for<EB>([&](auto c) {
                    sX[(16 + r) * DB_LD + 16 + c] = a[c];
                    sT[1][EB * c + r] = a[c];
                });
                sd[2 * (16 + lane)] = ds, sd[2 * (16 + lane) + 1] = dy;
            }
            if (bad && lane == 0) atomicCAS(status + i, 0, k0 + bad);
        } else if (t1 < nblk) {
            block_sum(t1);
        }
        __syncthreads();
        // ---- (3)
        auto block_finish = [&](int t) __attribute__((always_inline)) {
            const int r0 = k0 + DB * t;
            // C by rows of 33 in this wavefront's chunks
            wave_lds_fence();
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v) st[(16 * u + li) * DB_LD + 16 * p + lg + 4 * v] = cc[p][u][v];
            wave_lds_fence();
            double *row = st + (lane & 31) * DB_LD;
            double a[EB];
            static_for<EB>([&](auto c) { a[c] = row[c]; });
            subst16(a, sT[0], sd);
            if (lane < 32) static_for<EB>([&](auto c) { row[c] = a[c]; });
            wave_lds_fence();
            // columns 16..31 lose L(rows, 0..15) L10^T
            {
                dbl4 x, f0, f1;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    x[q] = sX[(16 + li) * DB_LD + lg + 4 * q];
                    f0[q] = st[li * DB_LD + lg + 4 * q];
                    f1[q] = st[(16 + li) * DB_LD + lg + 4 * q];
                }
                dbl4 s0 = {0.0, 0.0, 0.0, 0.0}, s1 = {0.0, 0.0, 0.0, 0.0};
                s0 = mfma_k16(x, f0, s0);
                s1 = mfma_k16(x, f1, s1);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    st[li * DB_LD + 16 + lg + 4 * v] = cc[1][0][v] - s0[v];
                    st[(16 + li) * DB_LD + 16 + lg + 4 * v] = cc[1][1][v] - s1[v];
                }
            }
            wave_lds_fence();
            static_for<EB>([&](auto c) { a[c] = row[16 + c]; });
            subst16(a, sT[1], sd + 2 * EB);
            wave_lds_fence();
            if (lane < 32) static_for<EB>([&](auto c) { row[16 + c] = a[c]; });
            wave_lds_fence();
#pragma unroll 4
            for (int q = 0; q < DB / 2; ++q) {
                const int rr = 2 * q + (lane >> 5), c = lane & 31, r = r0 + rr;
                if (r < rend && k0 + c >= r - b) row_at(r)[k0 + c] = st[rr * DB_LD + c];
            }
        };
        if (wv == 0) {
            for (int e = lane; e < kb * DB; e += 64) {
                const int r = e / DB, c = e % DB;
                const double v = r == c ? sd[2 * r + 1] : sX[r * DB_LD + c];
                if (c <= r && r - c <= b) row_at(k0 + r)[k0 + c] = v;
            }
        } else if (t1 < nblk) {
            block_finish(t1);
        }
#pragma unroll 1
        for (int t = NW + wv; t < nblk; t += NW) {
            block_sum(t);
            block_finish(t);
        }
        __syncthreads();
    }
}

// The same factor, bit for bit, for many narrow bands: the right-looking loop
// itself, panels of 16 columns, multiply-adds, the window below a panel updated
// in memory.  k_band_chol's 141 KB of LDS hold one workgroup per compute unit,
// whatever the band; here sixteen of 128 threads fit one, and a band of a few
// panels has no long chain to hide.  LDS: band_chol_small_lds(largest band).
// Per launch against k_band_chol: 4,096 bands of 160 rows (bandwidth 32) 537
// against 1,029 us, 8,000 of 81 (21) 420 against 1,162, 1,000 of 275 (45) 422
// against 473; 512 of 275 374 against 247, 1,000 of 432 (60) 806 against 757.
constexpr int CH_NB = 16;
constexpr int CH_LD = CH_NB + 1;   // padded LDS row stride (bank spread)
__host__ __device__ constexpr size_t band_chol_small_lds(int b) {
    return sizeof(double) * (CH_NB * CH_LD + CH_NB + size_t(b < 1 ? 1 : b) * CH_LD);
}

template <int NT>
__global__ __launch_bounds__(NT) void k_band_chol_small(double *__restrict__ band, const int64_t *__restrict__ off,
                                                        const int32_t *__restrict__ bwid,
                                                        const int64_t *__restrict__ rptr, int *__restrict__ status) {
    extern __shared__ double smem[];
    const int i = blockIdx.x;
    if (off[i + 1] == off[i]) return;   // no band (empty, or a supernodal subdomain)
    const int n = int(rptr[i + 1] - rptr[i]);
    const int b = bwid[i];
    const int64_t w = b + 1;
    double *L = band + off[i];
    double *sD = smem;                 // CH_NB x CH_LD
    double *sdg = sD + CH_NB * CH_LD;  // CH_NB
    double *sP = sdg + CH_NB;          // b x CH_LD
    const int tid = threadIdx.x;
    for (int k0 = 0; k0 < n; k0 += CH_NB) {
        const int kb = min(CH_NB, n - k0);
        // (a) diagonal block, left-looking by columns
        for (int e = tid; e < CH_NB * CH_NB; e += NT) {
            const int t = e / CH_NB, s = e % CH_NB;
            double v = 0.0;
            if (t < kb && s <= t && t - s <= b) v = L[int64_t(k0 + t) * w + (s - t + b)];
            sD[t * CH_LD + s] = v;
        }
        __syncthreads();
        for (int j = 0; j < kb; ++j) {
            const int t = j + tid;
            if (t < kb) {
                double v = sD[t * CH_LD + j];
                for (int s = 0; s < j; ++s) v -= sD[t * CH_LD + s] * sD[j * CH_LD + s];
                if (t == j) {
                    if (!(v > 0.0)) {
                        atomicCAS(status + i, 0, 1 + k0 + j);
                        v = 1.0;
                    }
                    sdg[j] = sqrt(v);
                } else {
                    sD[t * CH_LD + j] = v;
                }
            }
            __syncthreads();
            if (t > j && t < kb) sD[t * CH_LD + j] /= sdg[j];
            __syncthreads();
        }
        for (int e = tid; e < kb * kb; e += NT) {
            const int t = e / kb, s = e % kb;
            if (s <= t && t - s <= b)
                L[int64_t(k0 + t) * w + (s - t + b)] = (s == t) ? 1.0 / sdg[t] : sD[t * CH_LD + s];
        }
        // (b) rows below the diagonal block: P <- P L_D^{-T}
        const int rbeg = k0 + kb;
        const int rend = min(n, k0 + kb + b);
        const int m = max(0, rend - rbeg);
        for (int q = tid; q < m; q += NT) {
            const int r = rbeg + q;
            const int s0 = max(0, r - b - k0);
            double x[CH_NB];
#pragma unroll
            for (int s = 0; s < CH_NB; ++s) {
                double v = 0.0;
                if (s >= s0 && s < kb) {
                    v = L[int64_t(r) * w + (k0 + s - r + b)];
                    for (int t = 0; t < s; ++t) v -= x[t] * sD[s * CH_LD + t];   // x[t] = 0 for t < s0
                    v /= sdg[s];
                }
                x[s] = v;
            }
#pragma unroll
            for (int s = 0; s < CH_NB; ++s) {
                sP[q * CH_LD + s] = x[s];
                if (s >= s0 && s < kb) L[int64_t(r) * w + (k0 + s - r + b)] = x[s];
            }
        }
        __syncthreads();
        // (c) trailing window: A(r, c) -= P(r,:) . P(c,:), c <= r
        for (int e = tid; e < m * m; e += NT) {
            const int rq = e / m, cq = e % m;
            if (cq > rq) continue;
            double acc = 0.0;
#pragma unroll
            for (int s = 0; s < CH_NB; ++s) acc += sP[rq * CH_LD + s] * sP[cq * CH_LD + s];
            const int r = rbeg + rq, c = rbeg + cq;
            L[int64_t(r) * w + (c - r + b)] -= acc;
        }
        __syncthreads();
    }
}

// Partitioned inverse of the diagonal blocks of a band Cholesky factor
// (FP64, before any cast): the 64x64 diagonal block L_kk of rows k0 ..
// k0+kb-1 is replaced in place by X = L_kk^{-1} (lower triangular; its
// diagonal, 1/L_tt, is what the band already holds there), so that the
// triangle solves of the block become products with X.  Only for bands of
// at least BS_NB - 1, where the whole triangle lies inside the band.  One
// wavefront per diagonal block (block q of subdomain i with blk_ptr[i] <= q <
// blk_ptr[i+1]).  With L = [L0; M L1]: the inverses of the two 32x32 triangles
// at once, a column per lane of either half, in registers (x_j = x_j / L_jj,
// then x_r -= L(r, j) x_j for r > j: independent multiply-adds with broadcast
// LDS reads), the sums M X0 by matrix instructions, then the lower left quarter
// the same way from those sums.  Every value is the forward substitution's, bit
// for bit: -(1/L_tt) sum_{c <= s < t} L(t, s) X(s, c) in ascending s.  (Both
// triangles and the inverse in LDS, one value at a time per lane, held two
// wavefronts per compute unit: 4.07 ms for 27,136 blocks; now 1.3 ms.)
constexpr int BS_NB_INV = 64;

// forward substitution with a 32x32 triangle (T: column j at LD j, reciprocal
// diagonal), one right-hand side per lane
template <int LD>
__device__ __forceinline__ void subst_columns(double (&x)[DB], const double *T) {
    static_for<DB>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        x[j] *= T[j * LD + j];
        static_for<DB - 1 - j>([&](auto u) {
            constexpr int r = j + 1 + decltype(u)::value;
            x[r] = __builtin_fma(-T[j * LD + r], x[j], x[r]);
        });
        // (one column at a time: neither the LDS reads of later columns nor
        // the multiply-adds of this one are to be moved past here)
        static_for<DB - 1 - j>([&](auto u) { pin(x[j + 1 + decltype(u)::value]); });
    });
}

__global__ __launch_bounds__(64) void k_band_invert_diag(double *__restrict__ band, const int64_t *__restrict__ off,
                                                         const int32_t *__restrict__ bwid,
                                                         const int64_t *__restrict__ rptr,
                                                         const int64_t *__restrict__ blk_ptr, int np) {
    constexpr int NB = BS_NB_INV, LD = DB + 2;   // (even: 16-byte aligned columns)
    // the triangles transposed (column j at j LD), M by rows, later M X0 by
    // rows, X0 by rows
    __shared__ __align__(16) double sT[2][DB * LD], sM[DB * LD], sX[DB * LD];
    const int64_t q = blockIdx.x;
    int lo = 0, hi = np;   // subdomain with blk_ptr[i] <= q < blk_ptr[i+1]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (blk_ptr[mid] <= q) lo = mid; else hi = mid;
    }
    const int i = lo;
    const int b = bwid[i];
    if (b < NB - 1) return;   // (the host gives narrow bands no blocks)
    const int n = int(rptr[i + 1] - rptr[i]);
    const int k0 = int(q - blk_ptr[i]) * NB;
    const int kb = min(NB, n - k0);
    const int64_t w = b + 1;
    double *L = band + off[i];
    const int lane = threadIdx.x, half = lane >> 5, c = lane & 31, li = lane & 15, lg = lane >> 4;
    // (rows past the last one: those of the identity)
#pragma unroll 8
    for (int t = 0; t < NB; ++t) {
        const double v = t < kb && lane <= t ? L[int64_t(k0 + t) * w + (lane - t + b)] : (t == lane ? 1.0 : 0.0);
        if (t < DB) {
            if (half == 0) sT[0][c * LD + t] = v;
        } else if (half == 0) {
            sM[(t - DB) * LD + c] = v;
        } else {
            sT[1][c * LD + (t - DB)] = v;
        }
    }
    __syncthreads();
    double x[DB];
    static_for<DB>([&](auto t) { x[t] = t == c ? 1.0 : 0.0; });
    subst_columns<LD>(x, sT[half]);
    static_for<DB>([&](auto t) {
        if (half == 0) sX[t * LD + c] = x[t];
        const int r = half * DB + t;
        if (r < kb && c < t) L[int64_t(k0 + r) * w + (c - t + b)] = x[t];
    });
    if (kb <= DB) return;
    __syncthreads();
    // M X0: tiles of 16x16, ascending k (rows of X0 above its diagonal are zero)
    dbl4 p[2][2] = {};
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
        dbl4 a[2], f[2];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = 16 * kt + 4 * u + lg;
            a[0][u] = sM[li * LD + k];
            a[1][u] = sM[(16 + li) * LD + k];
            f[0][u] = sX[k * LD + li];
            f[1][u] = sX[k * LD + 16 + li];
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int s = 0; s < 2; ++s) p[r][s] = mfma_k16(a[r], f[s], p[r][s]);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int v = 0; v < 4; ++v) sM[(16 * r + lg + 4 * v) * LD + 16 * s + li] = p[r][s][v];
    __syncthreads();
    static_for<DB>([&](auto t) { x[t] = -sM[t * LD + c]; });
    subst_columns<LD>(x, sT[1]);
    static_for<DB>([&](auto t) {
        if (half == 0 && DB + t < kb) L[int64_t(k0 + DB + t) * w + (c - DB - t + b)] = x[t];
    });
}

// Casts a band (FP64) into the storage precision of the local factors.
template <typename VT>
__global__ void k_cast(const double *__restrict__ src, VT *__restrict__ dst, int64_t cnt) {
    for (int64_t p = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; p < cnt;
         p += int64_t(gridDim.x) * blockDim.x)
        dst[p] = from_double<VT>(src[p]);
}

// ---------------------------------------------------------------------------
// Band triangular solves with one LDS vector: y <- (L L^T)^{-1} y, L in the
// band layout above (reciprocal diagonal).  Blocks of 64 rows, two barriers
// per block:
//   forward, step of block k: block k's contribution is subtracted from the
//   rows below it, 16 lanes per row reading the row's 64-value band segment
//   side by side, and the workgroup stages block k+1's triangle in LDS; then
//   wavefront 0 solves block k+1 (lane t = row t), broadcasting each solved
//   value with a lane read;
//   backward (L^T z = y) is the mirror image by columns: the entries above
//   block k get its contribution (column j of the block's rows: consecutive
//   threads, consecutive addresses), and wavefront 0 solves block k-1's
//   transposed triangle (lane t = column t).
constexpr int BS_NB = 64;
static_assert(BS_NB == BS_NB_INV, "the inverted diagonal blocks are the solve's blocks");

// Loads of band entries: non-temporal for 8-byte entries (each band is
// streamed once per pass in whole cache lines); 4- and 2-byte entries use
// plain loads, since a row's 64-entry segment then fills only part of a
// line and the rest of the line is read by the next load.
template <typename VT>
__device__ __forceinline__ VT band_ld(const VT *p) {
    if constexpr (sizeof(VT) == 8)
        return ld_once(p);
    else
        return *p;
}

// A band of width b holds whole 64x64 triangles, and so gets its diagonal
// blocks inverted (k_band_invert_diag), when b >= 63.  The choice depends
// on the subdomain alone, so a problem's results do not depend on what it
// is packed with; the solve kernels come in one instance per choice, each
// leaving the other kind's subdomains alone.
__host__ __device__ constexpr bool band_inverted(int b) { return b >= BS_NB - 1; }
constexpr int BS_LD = BS_NB + 1;


// sT(t, s) = L(k0+t, k0+s) for s < t, 1/L(k0+t, k0+t) for s = t (all threads)
template <typename VT, typename AT, int NT>
__device__ __forceinline__ void band_stage_triangle(const VT *__restrict__ L, int64_t w, int b, int k0, int kb,
                                                    AT *sT) {
#pragma unroll 4
    for (int e = threadIdx.x; e < BS_NB * BS_NB; e += NT) {
        const int t = e / BS_NB, s = e % BS_NB;
        AT v = 0;
        if (t < kb && s <= t && t - s <= b) v = to_acc(band_ld(&L[int64_t(k0 + t) * w + (s - t + b)]));
        sT[t * BS_LD + s] = v;
    }
}

// The same block solves with the inverted diagonal block staged (bands of at
// least BS_NB - 1): lane t forms row t of X y (forward) or of X^T y
// (backward) in one pass of products; entries outside the triangle are zero
// in the staging, and the clamp keeps the reads inside the block.
// For a whole block (kb = 64, every block but a subdomain's last) the
// vector entries sit at fixed offsets from a 16-byte aligned address (the
// solve's LDS vector starts 16-byte aligned and blocks start at multiples of
// 64 entries), so their broadcast reads merge into wide LDS reads.
template <typename AT>
__device__ __forceinline__ const AT *band_block_vec(const AT *y, int k0) {
    return static_cast<const AT *>(__builtin_assume_aligned(y + k0, 16));
}

template <typename AT>
__device__ __forceinline__ void band_block_fwd_inv(const AT *sT, AT *y, int k0, int kb, int lane) {
    const AT *row = sT + lane * BS_LD;
    AT acc = 0;
    if (kb == BS_NB) {
        const AT *yb = band_block_vec(y, k0);
#pragma unroll 8
        for (int s = 0; s < BS_NB; ++s) acc += row[s] * yb[s];
    } else {
#pragma unroll 8
        for (int s = 0; s < BS_NB; ++s) acc += row[s] * y[k0 + min(s, kb - 1)];
    }
    if (lane < kb) y[k0 + lane] = acc;
}

template <typename AT>
__device__ __forceinline__ void band_block_bwd_inv(const AT *sT, AT *y, int k0, int kb, int lane) {
    AT acc = 0;
    if (kb == BS_NB) {
        const AT *yb = band_block_vec(y, k0);
#pragma unroll 8
        for (int s = 0; s < BS_NB; ++s) acc += sT[s * BS_LD + lane] * yb[s];
    } else {
#pragma unroll 8
        for (int s = 0; s < BS_NB; ++s) acc += sT[s * BS_LD + lane] * y[k0 + min(s, kb - 1)];
    }
    if (lane < kb) y[k0 + lane] = acc;
}

// The staged triangle is zero in rows kb..63 (pivot included), so the steps
// s >= kb leave the lanes below kb unchanged: no per-step test, which lets
// the unrolled steps read their LDS entries eight at a time ahead of the
// dependent arithmetic.
template <typename AT>
__device__ __forceinline__ void band_block_fwd(const AT *sT, AT *y, int k0, int kb, int lane) {
    AT yt = lane < kb ? y[k0 + lane] : AT(0);
    const AT *row = sT + lane * BS_LD;
#pragma unroll 8
    for (int s = 0; s < BS_NB; ++s) {
        const AT l = row[s];
        if (lane == s) yt *= l;
        const AT ys = lane_read(yt, s);
        if (lane > s) yt -= l * ys;
    }
    if (lane < kb) y[k0 + lane] = yt;
}

template <typename AT>
__device__ __forceinline__ void band_block_bwd(const AT *sT, AT *y, int k0, int kb, int lane) {
    AT yt = lane < kb ? y[k0 + lane] : AT(0);
#pragma unroll 8
    for (int s = BS_NB - 1; s >= 0; --s) {
        const AT l = sT[s * BS_LD + lane];   // L(k0+s, k0+lane), or the reciprocal pivot at s = lane
        if (lane == s) yt *= l;
        const AT zs = lane_read(yt, s);
        if (lane < s) yt -= l * zs;
    }
    if (lane < kb) y[k0 + lane] = yt;
}

// The staging split in two, for the register budgets that allow it: the
// triangle's loads into registers, issued with the row or column updates of
// the same step so that both are in flight together, and the store into
// LDS after the updates.
template <int NT>
constexpr int tri_per_thread() { return (BS_NB * BS_NB + NT - 1) / NT; }

template <typename VT, typename AT, int NT>
__device__ __forceinline__ void band_load_triangle(const VT *__restrict__ L, int64_t w, int b, int k0, int kb,
                                                   AT (&tv)[tri_per_thread<NT>()]) {
#pragma unroll
    for (int c = 0; c < tri_per_thread<NT>(); ++c) {
        const int e = int(threadIdx.x) + c * NT;
        const int t = e / BS_NB, s = e % BS_NB;
        tv[c] = (e < BS_NB * BS_NB && t < kb && s <= t && t - s <= b) ? to_acc(band_ld(&L[int64_t(k0 + t) * w + (s - t + b)]))
                                                                      : AT(0);
    }
}

template <typename AT, int NT>
__device__ __forceinline__ void band_store_triangle(const AT (&tv)[tri_per_thread<NT>()], AT *sT) {
#pragma unroll
    for (int c = 0; c < tri_per_thread<NT>(); ++c) {
        const int e = int(threadIdx.x) + c * NT;
        if (e < BS_NB * BS_NB) sT[(e / BS_NB) * BS_LD + e % BS_NB] = tv[c];
    }
}

// Band entries from `base` on by buffer loads: an offset (bytes) past the
// last entry reads as zero, which is how entries outside the band are left
// out (offset BAND_NONE) without a branch around each load, and an offset
// fixed over the steps needs no arithmetic in them.  base: uniform over the
// workgroup; left: the entries from it to the end of the subdomain's band.
// Offsets used with it stay under 2^31 - 4,096: 448 rows of a band at most.
constexpr int BAND_NONE = int(0x80000000u);

template <typename VT>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t band_window(const VT *base, int64_t left) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(a)), hi = __builtin_amdgcn_readfirstlane(uint32_t(a >> 32));
    const int bytes = __builtin_amdgcn_readfirstlane(int(min(max(left, int64_t(0)) * int64_t(sizeof(VT)), int64_t(0x7fffffff))));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(uint64_t(hi) << 32 | lo), 0, bytes, 0x00020000);
}

template <typename VT>
__device__ __forceinline__ auto band_window_ld(__amdgpu_buffer_rsrc_t win, int at) {
    if constexpr (sizeof(VT) == 8)   // (non-temporal, as band_ld)
        return to_acc(__builtin_bit_cast(VT, __builtin_amdgcn_raw_buffer_load_b64(win, at, 0, 2)));
    else if constexpr (sizeof(VT) == 4)
        return to_acc(__builtin_bit_cast(VT, __builtin_amdgcn_raw_buffer_load_b32(win, at, 0, 0)));
    else
        return to_acc(__builtin_bit_cast(VT, __builtin_amdgcn_raw_buffer_load_b16(win, at, 0, 0)));
}

// The solve with its band loads one block step ahead (1024 threads).  A
// step first uses the entries loaded during the step before (the rows below
// the solved block, forward; the thread's column above it, backward),
// then issues the next step's entries and triangle into the same registers,
// so that those loads are in flight across the triangle solve and its two
// barriers instead of being waited for at the start of the next step.  Rows
// (columns) past the held ones are loaded in the step itself.  Every sum is
// formed in the same order as in the plain form below, so both give the
// same bits.  Bound by the instructions of a step's critical path: with a
// test and a 64-bit address per load and a branch around it, the loads of a
// step took longer to issue than to arrive; through the window (band_window)
// the forward step issues its 28 with a handful of scalar instructions: 365
// -> 268 us per launch on 216 subdomains of 2,700 rows FP32, 331 -> 226 on 27
// of elasticity, 389 -> 319 on 48^3 elasticity, 154 -> 139 on 8 of 1,331 rows
// FP64.
template <typename VT, typename AT, int NT, bool INV>
__device__ void band_llt_solve_ahead(const VT *__restrict__ L, int n, int b, AT *y, AT *sT) {
    constexpr bool F64 = sizeof(AT) == 8;
    constexpr int LPR = 16, RPI = NT / LPR, QN = BS_NB / LPR;
    static_assert(LPR == 16, "the row sums use rows of 16 lanes");
    constexpr int PF = F64 ? 4 : 6;      // forward: row groups of RPI rows held per step
    constexpr int RB = F64 ? 2 : 4;      // forward: row groups per pass past the held ones
    // backward: rows of the thread's first column held (FP32 all 64 of a block:
    // 375 -> 365 us on 216 subdomains of 2,700 rows against 32, 400 -> 389 on
    // 48^3 elasticity; FP64 32, 154 -> 139 on 8 of 1,331 rows against 16: three
    // or four registers past what 1,024 threads have, which spill)
    constexpr int BPF = F64 ? 32 : 64;
    constexpr int G = F64 ? 8 : 32;      // backward: loads per group past the held rows
    const int64_t w = b + 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int sub = tid & (LPR - 1), rg = tid / LPR;
    const int nblk = (n + BS_NB - 1) / BS_NB;
    AT tv[tri_per_thread<NT>()];
    // ---- forward
    // v[it][q] = L(r, k0 + sub + 16 q) for the row r = k0 + 64 + it RPI + rg
    // below the block at k0 (zero outside the band and past the subdomain)
    AT v[PF][QN];
    constexpr int VS = sizeof(VT);
    const int64_t len = int64_t(n) * w;
    // entry (k0 + i, k0 + c) lies i b + c entries after entry (k0, k0), so a
    // lane's offsets are the same in every step; rows past the subdomain are
    // past the window
    auto load_rows = [&](int k0) __attribute__((always_inline)) {
        const int64_t at0 = int64_t(k0) * w + b;
        const __amdgpu_buffer_rsrc_t win = band_window(L + at0, len - at0);
#pragma unroll
        for (int it = 0; it < PF; ++it) {
            const int i = BS_NB + it * RPI + rg;
            const int at = (i * b + sub) * VS;
#pragma unroll
            for (int q = 0; q < QN; ++q)
                v[it][q] = band_window_ld<VT>(win, sub + q * LPR >= i - b ? at + q * LPR * VS : BAND_NONE);
        }
    };
    auto load_triangle = [&](int k0) __attribute__((always_inline)) {
        const int64_t at0 = int64_t(k0) * w + b;
        const __amdgpu_buffer_rsrc_t win = band_window(L + at0, len - at0);
#pragma unroll
        for (int c = 0; c < tri_per_thread<NT>(); ++c) {
            const int e = tid + c * NT, t = e / BS_NB, q = e % BS_NB;
            tv[c] = band_window_ld<VT>(win, e < BS_NB * BS_NB && q <= t && t - q <= b ? (t * b + q) * VS : BAND_NONE);
        }
    };
    band_stage_triangle<VT, AT, NT>(L, w, b, 0, min(BS_NB, n), sT);
    __syncthreads();
    if (tid < 64) {
        if constexpr (INV) band_block_fwd_inv(sT, y, 0, min(BS_NB, n), lane);
        else band_block_fwd(sT, y, 0, min(BS_NB, n), lane);
    }
    if (nblk > 1) {
        load_rows(0);
        load_triangle(BS_NB);
    }
    __syncthreads();
    for (int blk = 0; blk + 1 < nblk; ++blk) {
        const int k0 = blk * BS_NB, k1 = k0 + BS_NB, kb1 = min(BS_NB, n - k1);
        const int rend = min(n, k1 + b);
        AT yq[QN];
#pragma unroll
        for (int q = 0; q < QN; ++q) yq[q] = y[k0 + sub + q * LPR];
#pragma unroll
        for (int it = 0; it < PF; ++it) {
            const int r = k1 + it * RPI + rg;
            AT acc = 0;
#pragma unroll
            for (int q = 0; q < QN; ++q) acc += v[it][q] * yq[q];
            acc = row16_sum(acc);
            if (r < rend && sub == 0) y[r] -= acc;
        }
        for (int r0 = k1 + PF * RPI; r0 < rend; r0 += RB * RPI) {
            AT u[RB][QN];
#pragma unroll
            for (int it = 0; it < RB; ++it) {
                const int r = r0 + it * RPI + rg;
                const int s0 = max(0, r - b - k0);
                const VT *row = L + int64_t(r) * w + (k0 - r + b);
#pragma unroll
                for (int q = 0; q < QN; ++q) {
                    const int s = sub + q * LPR;
                    u[it][q] = (r < rend && s >= s0) ? to_acc(band_ld(&row[s])) : AT(0);
                }
            }
#pragma unroll
            for (int it = 0; it < RB; ++it) {
                const int r = r0 + it * RPI + rg;
                AT acc = 0;
#pragma unroll
                for (int q = 0; q < QN; ++q) acc += u[it][q] * yq[q];
                acc = row16_sum(acc);
                if (r < rend && sub == 0) y[r] -= acc;
            }
        }
        band_store_triangle<AT, NT>(tv, sT);
        if (blk + 2 < nblk) {   // the next step's rows and triangle
            load_rows(k1);
            load_triangle(k1 + BS_NB);
        }
        __syncthreads();
        if (tid < 64) {
            if constexpr (INV) band_block_fwd_inv(sT, y, k1, kb1, lane);
            else band_block_fwd(sT, y, k1, kb1, lane);
        }
        __syncthreads();
    }
    // ---- backward
    // cv[s] = L(k0 + s, j) for the thread's first column j = max(0, k0 - b) + tid
    // above the block at k0 (zero outside the band)
    AT cv[BPF];
    // entry (k0 + s, j) lies s b + j - (k0 - b) entries after row k0's first;
    // only the first wavefront's columns end inside the block's rows
    auto load_col = [&](int k0) __attribute__((always_inline)) {
        const int64_t at0 = int64_t(k0) * w;
        const __amdgpu_buffer_rsrc_t win = band_window(L + at0, len - at0);
        const int wv = __builtin_amdgcn_readfirstlane(tid / 64);
        int jj = tid + max(0, b - k0);   // j - (k0 - b)
        int at = jj < b ? jj * VS : BAND_NONE, step = b * VS;
        // (tests and offsets are formed one by one as the loads go out: no
        // registers hold them)
        asm volatile("" : "+v"(jj), "+v"(at), "+s"(step));
        if (wv == 0) {
#pragma unroll
            for (int s = 0; s < BPF; ++s, at += step) {
                cv[s] = band_window_ld<VT>(win, s <= jj ? at : BAND_NONE);
                asm volatile("" : "+v"(at), "+v"(jj) : : "memory");
            }
        } else if (wv * 64 < min(b, k0)) {
#pragma unroll
            for (int s = 0; s < BPF; ++s, at += step) {
                cv[s] = band_window_ld<VT>(win, at);
                asm volatile("" : "+v"(at) : : "memory");
            }
        }
    };
    {
        const int k0 = (nblk - 1) * BS_NB, kb = n - k0;
        band_stage_triangle<VT, AT, NT>(L, w, b, k0, kb, sT);
        __syncthreads();
        if (tid < 64) {
            if constexpr (INV) band_block_bwd_inv(sT, y, k0, kb, lane);
            else band_block_bwd(sT, y, k0, kb, lane);
        }
        if (nblk > 1) {
            load_col(k0);
            load_triangle(k0 - BS_NB);
        }
        __syncthreads();
    }
    for (int blk = nblk - 1; blk > 0; --blk) {
        const int k0 = blk * BS_NB, kb = min(BS_NB, n - k0);
        const int p0 = k0 - BS_NB;
        const int jbeg = max(0, k0 - b);
        {
            const int j = jbeg + tid;
            if (j < k0) {
                const int64_t at0 = int64_t(k0) * w;
                const __amdgpu_buffer_rsrc_t win = band_window(L + at0, len - at0);
                const int jj = j - (k0 - b);
                // (the block's vector entries: at fixed offsets for a whole
                // block, clamped to the last row for the last one)
                auto col_sum = [&](auto yat) {
                    AT acc = 0;
#pragma unroll
                    for (int s = 0; s < BPF; ++s) acc += cv[s] * yat(s);
#pragma unroll 1
                    for (int g = BPF; g < BS_NB; g += G) {
                        AT u[G];
#pragma unroll
                        for (int q = 0; q < G; ++q)
                            u[q] = band_window_ld<VT>(win, g + q <= jj ? (jj + (g + q) * b) * VS : BAND_NONE);
#pragma unroll
                        for (int q = 0; q < G; ++q) acc += u[q] * yat(g + q);
                    }
                    return acc;
                };
                const AT *yb = band_block_vec(y, k0);
                y[j] -= kb == BS_NB ? col_sum([&](int s) { return yb[s]; })
                                    : col_sum([&](int s) { return y[k0 + min(s, kb - 1)]; });
            }
        }
        // columns past the first NT (bands wider than the workgroup)
        for (int j = jbeg + tid + NT; j < k0; j += NT) {
            const int smax = min(kb, j + b - k0 + 1);
            const VT *col = L + int64_t(k0) * w + (j - k0 + b);
            AT acc = 0;
#pragma unroll 1
            for (int g = 0; g < BS_NB; g += G) {
                AT u[G];
#pragma unroll
                for (int q = 0; q < G; ++q)
                    u[q] = (g + q < smax) ? to_acc(band_ld(&col[int64_t(g + q) * (w - 1)])) : AT(0);
#pragma unroll
                for (int q = 0; q < G; ++q) acc += u[q] * y[k0 + min(g + q, kb - 1)];
            }
            y[j] -= acc;
        }
        band_store_triangle<AT, NT>(tv, sT);
        if (blk > 1) {   // the next step's column and triangle
            load_col(p0);
            load_triangle(p0 - BS_NB);
        }
        __syncthreads();
        if (tid < 64) {
            if constexpr (INV) band_block_bwd_inv(sT, y, p0, BS_NB, lane);
            else band_block_bwd(sT, y, p0, BS_NB, lane);
        }
        __syncthreads();
    }
}

// INV: the diagonal blocks hold their inverses (band_inverted(b)), so each
// triangle solve is one product with the staged block.
// AHEAD: the form with the loads one step ahead (1024 threads: that
// register budget holds the extra entries without spills).
template <typename VT, typename AT, int NT, bool INV, bool AHEAD = false>
__device__ void band_llt_solve(const VT *__restrict__ L, int n, int b, AT *y, AT *sT) {
    if (n <= 0) return;   // an empty subdomain or interior (uniform over the workgroup)
    constexpr bool F64 = sizeof(AT) == 8;
    constexpr bool inv = INV;
    constexpr int G = F64 ? 8 : 32;   // loads in flight per thread and group (backward)
    // triangle loads overlapped with the updates where the register budget
    // holds the extra values (FP32 accumulation from 512 threads, FP64 at 1024)
    constexpr bool PREF = F64 ? NT >= 1024 : NT >= 512;
    if constexpr (AHEAD && PREF && NT >= 1024) {
        band_llt_solve_ahead<VT, AT, NT, INV>(L, n, b, y, sT);
        return;
    }
    const int64_t w = b + 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int nblk = (n + BS_NB - 1) / BS_NB;
    // ---- forward
    band_stage_triangle<VT, AT, NT>(L, w, b, 0, min(BS_NB, n), sT);
    __syncthreads();
    if (tid < 64) {
        if constexpr (inv) band_block_fwd_inv(sT, y, 0, min(BS_NB, n), lane);
        else band_block_fwd(sT, y, 0, min(BS_NB, n), lane);
    }
    __syncthreads();
    // rows below a solved block: 16 lanes per row, lane q takes the block's
    // columns q, q+16, q+32, q+48 (consecutive lanes, consecutive addresses)
    // and the 16 partial products are summed across the lanes
    constexpr int LPR = 16, RPI = NT / LPR;
    static_assert(LPR == 16, "the row sums use rows of 16 lanes");
    const int sub = tid & (LPR - 1), rg = tid / LPR;
    for (int blk = 0; blk + 1 < nblk; ++blk) {
        const int k0 = blk * BS_NB;
        const int k1 = k0 + BS_NB, kb1 = min(BS_NB, n - k1);
        const int rend = min(n, k1 + b);
        AT tv[tri_per_thread<NT>()];
        if constexpr (PREF) band_load_triangle<VT, AT, NT>(L, w, b, k1, kb1, tv);   // block k+1's triangle
        AT yq[BS_NB / LPR];
#pragma unroll
        for (int q = 0; q < BS_NB / LPR; ++q) yq[q] = y[k0 + sub + q * LPR];
        // RB row groups per pass: all their loads are issued before the sums
        constexpr int RB = sizeof(AT) == 8 ? 2 : 4;
        for (int r0 = k1; r0 < rend; r0 += RB * RPI) {
            AT v[RB][BS_NB / LPR];
#pragma unroll
            for (int it = 0; it < RB; ++it) {
                const int r = r0 + it * RPI + rg;
                const int s0 = max(0, r - b - k0);
                const VT *row = L + int64_t(r) * w + (k0 - r + b);
#pragma unroll
                for (int q = 0; q < BS_NB / LPR; ++q) {
                    const int s = sub + q * LPR;
                    v[it][q] = (r < rend && s >= s0) ? to_acc(band_ld(&row[s])) : AT(0);
                }
            }
#pragma unroll
            for (int it = 0; it < RB; ++it) {
                const int r = r0 + it * RPI + rg;
                AT acc = 0;
#pragma unroll
                for (int q = 0; q < BS_NB / LPR; ++q) acc += v[it][q] * yq[q];
                acc = row16_sum(acc);   // (LPR = 16 lanes per row)
                if (r < rend && sub == 0) y[r] -= acc;
            }
        }
        if constexpr (PREF) band_store_triangle<AT, NT>(tv, sT);
        else band_stage_triangle<VT, AT, NT>(L, w, b, k1, kb1, sT);
        __syncthreads();
        if (tid < 64) {
            if constexpr (inv) band_block_fwd_inv(sT, y, k1, kb1, lane);
            else band_block_fwd(sT, y, k1, kb1, lane);
        }
        __syncthreads();
    }
    // ---- backward
    {
        const int k0 = (nblk - 1) * BS_NB, kb = n - k0;
        band_stage_triangle<VT, AT, NT>(L, w, b, k0, kb, sT);
        __syncthreads();
        if (tid < 64) {
            if constexpr (inv) band_block_bwd_inv(sT, y, k0, kb, lane);
            else band_block_bwd(sT, y, k0, kb, lane);
        }
        __syncthreads();
    }
    for (int blk = nblk - 1; blk > 0; --blk) {
        const int k0 = blk * BS_NB, kb = min(BS_NB, n - k0);
        const int p0 = k0 - BS_NB;
        const int jbeg = max(0, k0 - b);
        AT tv[tri_per_thread<NT>()];
        if constexpr (PREF) band_load_triangle<VT, AT, NT>(L, w, b, p0, BS_NB, tv);   // block k-1's triangle
        for (int j = jbeg + tid; j < k0; j += NT) {
            const int smax = min(kb, j + b - k0 + 1);
            const VT *col = L + int64_t(k0) * w + (j - k0 + b);   // entry s at col[s * (w - 1)]
            AT acc = 0;
#pragma unroll 1
            for (int g = 0; g < BS_NB; g += G) {
                AT v[G];
#pragma unroll
                for (int q = 0; q < G; ++q) v[q] = (g + q < smax) ? to_acc(band_ld(&col[int64_t(g + q) * (w - 1)])) : AT(0);
#pragma unroll
                for (int q = 0; q < G; ++q) acc += v[q] * y[k0 + min(g + q, kb - 1)];
            }
            y[j] -= acc;
        }
        if constexpr (PREF) band_store_triangle<AT, NT>(tv, sT);
        else band_stage_triangle<VT, AT, NT>(L, w, b, p0, BS_NB, sT);
        __syncthreads();
        if (tid < 64) {
            if constexpr (inv) band_block_bwd_inv(sT, y, p0, BS_NB, lane);
            else band_block_bwd(sT, y, p0, BS_NB, lane);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Extension, eq. (2).  E_i = A_{I_i Gamma} Phi_Gamma(:, cols_i) is assembled
// one thread per interior row (couplings in CSR order), column-major
// n_Ii x k_i per subdomain at ext_off[i].
__global__ void k_ext_rhs(const double *__restrict__ Aval, const int64_t *__restrict__ int_ptr, int np,
                          const int64_t *__restrict__ ext_off, const int64_t *__restrict__ cpl_ptr,
                          const int64_t *__restrict__ cpl_apos, const int64_t *__restrict__ cpl_phi,
                          const int32_t *__restrict__ cpl_stride, const int32_t *__restrict__ cpl_rank,
                          const int32_t *__restrict__ cpl_slot, const int32_t *__restrict__ slotmap,
                          const double *__restrict__ phig, double *__restrict__ E, int64_t nint) {
    const int64_t q = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (q >= nint) return;
    int lo = 0, hi = np;   // subdomain with int_ptr[i] <= q < int_ptr[i+1]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (int_ptr[mid] <= q) lo = mid; else hi = mid;
    }
    const int i = lo;
    const int64_t nr = int_ptr[i + 1] - int_ptr[i];
    const int64_t l = q - int_ptr[i];
    double *Ei = E + ext_off[i];
    for (int64_t e = cpl_ptr[q]; e < cpl_ptr[q + 1]; ++e) {
        const double a = Aval[cpl_apos[e]];
        const double *ph = phig + cpl_phi[e];
        const int st = cpl_stride[e], rk = cpl_rank[e], sl = cpl_slot[e];
        for (int j = 0; j < rk; ++j) Ei[int64_t(slotmap[sl + j]) * nr + l] += a * ph[int64_t(j) * st];
    }
}

// Phi_{I_i} = -A_{I_i I_i}^{-1} E_i, one workgroup per subdomain, one right
// hand side at a time through LDS, written into the subdomain's interior
// block of Phi: for bands without inverted diagonal blocks (interiors of a few
// hundred rows) and for bands too wide for k_ext_solve_mm's LDS.
template <int NT, bool INV>
__global__ __launch_bounds__(1024) void k_ext_solve(const double *__restrict__ iband,
                                                  const int64_t *__restrict__ iband_off,
                                                  const int32_t *__restrict__ ibw,
                                                  const int64_t *__restrict__ int_ptr,
                                                  const int64_t *__restrict__ scol_ptr,
                                                  const int64_t *__restrict__ ext_off,
                                                  const double *__restrict__ E,
                                                  const int32_t *__restrict__ sub_blk,
                                                  const int64_t *__restrict__ blk_val_off,
                                                  double *__restrict__ phi) {
    extern __shared__ __align__(16) double sxs[];   // (16-byte aligned: the band solve's block reads)
    double *smem = sxs;
    const int i = blockIdx.x;
    const int n = int(int_ptr[i + 1] - int_ptr[i]);
    const int k = int(scol_ptr[i + 1] - scol_ptr[i]);
    const int g = sub_blk[i];
    if (n == 0 || k == 0 || g < 0 || band_inverted(ibw[i]) != INV) return;
    double *y = smem;
    double *sT = smem + n;
    const double *L = iband + iband_off[i];
    for (int s = 0; s < k; ++s) {
        const double *e = E + ext_off[i] + int64_t(s) * n;
        for (int l = threadIdx.x; l < n; l += NT) y[l] = e[l];
        __syncthreads();
        band_llt_solve<double, double, NT, INV>(L, n, ibw[i], y, sT);
        double *out = phi + blk_val_off[g] + int64_t(s) * n;
        for (int l = threadIdx.x; l < n; l += NT) out[l] = -y[l];
        __syncthreads();
    }
}

// The same solve for 16 right-hand sides per workgroup (grid: subdomains x
// groups of 16), for bands whose diagonal blocks are inverted: the band is
// read once per pass for all 16 instead of once per right-hand side, and the
// products are matrix instructions.  Blocks of 64 rows, 16 rows per wavefront,
// right-hand sides transposed (D(i, j): right-hand side i, row j, so that a
// column's rows are consecutive in memory).  Left-looking: a block takes the
// contributions of the blocks before it (forward) or after it (backward) in
// band_llt_solve's order, so that every value has that solve's bits: forward,
// a row's 64 products per block are 16 chains of four (columns s, s + 16, s +
// 32, s + 48: one matrix instruction each) added by the tree of row16_sum;
// backward and in the triangles one ascending chain of 64.  The solved blocks
// within reach are kept in LDS (a ring of nring = ceil(b / 64) + 1 blocks);
// the forward pass turns its band rows (512-byte row segments) through LDS,
// the backward pass reads operands in place (16 lanes on one row).  LDS:
// ext_mm_lds(nring).  Against one right-hand side at a time: 24^3 elasticity
// (27 interiors, 180 right-hand sides) 52.7 -> 0.50 ms, 128^3 Poisson (512
// interiors of 3,375 rows, 6 right-hand sides padded to 16; bound by reading
// the band twice) 9.0 -> 2.07 ms.
constexpr int XS_R = 16;   // right-hand sides per workgroup
__host__ __device__ constexpr int ext_mm_ring(int b) { return (b + BS_NB - 1) / BS_NB + 1; }
__host__ __device__ constexpr size_t ext_mm_lds(int nring) {
    return sizeof(double) * (size_t(nring) + 1 + 4) * (XS_R * BS_NB);
}

__global__ __launch_bounds__(256) void k_ext_solve_mm(const double *__restrict__ iband,
                                                      const int64_t *__restrict__ iband_off,
                                                      const int32_t *__restrict__ ibw,
                                                      const int64_t *__restrict__ int_ptr,
                                                      const int64_t *__restrict__ scol_ptr,
                                                      const int64_t *__restrict__ ext_off,
                                                      const double *__restrict__ E,
                                                      const int32_t *__restrict__ sub_blk,
                                                      const int64_t *__restrict__ blk_val_off,
                                                      double *__restrict__ phi, int nring) {
    extern __shared__ __align__(16) double sxs[];
    const int i = blockIdx.x, c0 = XS_R * blockIdx.y;
    const int n = int(int_ptr[i + 1] - int_ptr[i]);
    const int k = int(scol_ptr[i + 1] - scol_ptr[i]);
    const int g = sub_blk[i], b = ibw[i];
    if (n == 0 || k <= c0 || g < 0 || !band_inverted(b)) return;
    constexpr int BLK = XS_R * BS_NB;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int li = lane & 15, lg = lane >> 4;
    double *ring = sxs;                  // solved blocks, right-hand side i, row s at 64 i + (s ^ i)
    double *sR = sxs + nring * BLK;      // the block's right-hand sides before its triangle
    double *st = sR + BLK + wv * BLK;    // this wavefront's band rows, in 16-byte units permuted by the row
    const int64_t w = b + 1;
    const double *L = iband + iband_off[i];
    auto row_at = [&](int r) { return L + (int64_t(r) * w + (b - r)); };   // &L(r, 0)
    const int nblk = (n + BS_NB - 1) / BS_NB;
    const double *Ei = E + ext_off[i] + int64_t(c0) * n;
    double *X = phi + blk_val_off[g] + int64_t(c0) * n;
    const int nc = min(XS_R, k - c0);
    // band rows r0 .. r0 + 15, columns k0 .. k0 + 63: two rows per load, 32
    // lanes to a row (rows past the matrix: its last one; slots left of the
    // band are read, L(r, c) with c >= 0 lies at r b + b + c >= 0; columns
    // right of the diagonal, in a block's own triangle, at most up to the
    // array's last value)
    const int64_t last = int64_t(n) * w - 1;
    dbl2 v[8];
    auto load_rows = [&](int r0, int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int r = min(r0 + 2 * q + (lane >> 5), n - 1);
            const int64_t at = int64_t(r) * b + b + k0 + 2 * (lane & 31);
            if (k0 + BS_NB <= r0)
                v[q] = *reinterpret_cast<const dbl2u *>(L + at);
            else
                v[q] = dbl2{L[min(at, last)], L[min(at + 1, last)]};
        }
    };
    auto rows_to_lds = [&]() __attribute__((always_inline)) {
        wave_lds_fence();
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int r = 2 * q + (lane >> 5);
            *reinterpret_cast<dbl2 *>(st + r * BS_NB + 2 * ((lane & 31) ^ (r & 7))) = v[q];
        }
        wave_lds_fence();
    };
    // ---- forward
    for (int blk = 0; blk < nblk; ++blk) {
        const int r0 = blk * BS_NB + 16 * wv, r = r0 + li, rr = min(r, n - 1);
        dbl4 y;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s = lg + 4 * u;
            y[u] = s < nc && r < n ? Ei[int64_t(s) * n + r] : 0.0;
        }
        const int kf = max(0, r0 - b) / BS_NB;   // (earlier blocks are out of the band's reach)
        load_rows(r0, (kf < blk ? kf : blk) * BS_NB);
        for (int kk = kf; kk < blk; ++kk) {
            const int k0 = kk * BS_NB;
            rows_to_lds();
            load_rows(r0, k0 + BS_NB);   // (the next block's, at last the triangle's)
            const double *yk = ring + (kk % nring) * BLK + li * BS_NB;
            const int cmin = rr - b - k0 - 16 * lg;
            // chains s and s + 1 of the tree's leaves, pairs, quads, ...
            dbl4 q4[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                dbl4 p[4];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int s = 4 * m + 2 * h;
                    const dbl2 f = *reinterpret_cast<const dbl2 *>(st + li * BS_NB + 2 * ((8 * lg + s / 2) ^ (li & 7)));
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const dbl4 zero = {0.0, 0.0, 0.0, 0.0};
                        p[2 * h + u] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            yk[(16 * lg + s + u) ^ li], s + u >= cmin ? f[u] : 0.0, zero, 0, 0, 0);
                    }
                }
                q4[m] = (p[0] + p[1]) + (p[2] + p[3]);
            }
            y -= (q4[0] + q4[1]) + (q4[2] + q4[3]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s = lg + 4 * u;
            sR[s * BS_NB + ((16 * wv + li) ^ s)] = y[u];
        }
        rows_to_lds();
        __syncthreads();
        // the triangle: rows 16 wv + li of the inverse, columns up to the row
        y = dbl4{0.0, 0.0, 0.0, 0.0};
        for (int q = 0; q < 4 * (wv + 1); ++q) {
            const int s = 4 * q + lg;
            const double f = st[li * BS_NB + 2 * ((s >> 1) ^ (li & 7)) + (s & 1)];
            y = __builtin_amdgcn_mfma_f64_16x16x4f64(sR[li * BS_NB + (s ^ li)], s <= 16 * wv + li ? f : 0.0, y, 0, 0, 0);
        }
        double *yb = ring + (blk % nring) * BLK;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s = lg + 4 * u;
            if (r >= n) y[u] = 0.0;
            yb[s * BS_NB + ((16 * wv + li) ^ s)] = y[u];
            if (s < nc && r < n) X[int64_t(s) * n + r] = y[u];
        }
        __syncthreads();
    }
    // ---- backward (a lane reads back the values it wrote)
    for (int blk = nblk - 1; blk >= 0; --blk) {
        const int c = blk * BS_NB + 16 * wv + li;   // the column (c < n where it is stored)
        const int cc = min(c, n - 1);
        dbl4 y;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s = lg + 4 * u;
            y[u] = s < nc && c < n ? X[int64_t(s) * n + c] : 0.0;
        }
        const int kl = min(nblk - 1, (blk * BS_NB + 16 * wv + 15 + b) / BS_NB);
        for (int kk = kl; kk > blk; --kk) {
            const int k0 = kk * BS_NB;
            const double *zk = ring + (kk % nring) * BLK + li * BS_NB;
            double f[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int r = min(k0 + 4 * q + lg, n - 1);
                f[q] = row_at(r)[cc];
            }
            dbl4 a = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int r = k0 + 4 * q + lg;
                a = __builtin_amdgcn_mfma_f64_16x16x4f64(zk[(4 * q + lg) ^ li], r < n && c >= r - b ? f[q] : 0.0, a, 0, 0, 0);
            }
            y -= a;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s = lg + 4 * u;
            sR[s * BS_NB + ((16 * wv + li) ^ s)] = y[u];
        }
        __syncthreads();
        y = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int q = 4 * wv; q < 16; ++q) {
            const int s = 4 * q + lg, r = blk * BS_NB + s;
            const double f = r < n && s >= 16 * wv + li ? row_at(min(r, n - 1))[min(c, min(r, n - 1))] : 0.0;
            y = __builtin_amdgcn_mfma_f64_16x16x4f64(sR[li * BS_NB + (s ^ li)], f, y, 0, 0, 0);
        }
        double *zb = ring + (blk % nring) * BLK;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s = lg + 4 * u;
            if (c >= n) y[u] = 0.0;
            zb[s * BS_NB + ((16 * wv + li) ^ s)] = y[u];
            if (s < nc && c < n) X[int64_t(s) * n + c] = -y[u];
        }
        __syncthreads();
    }
}

// T1_i = E_i^T Phi_{I_i} (k_i x k_i), one wavefront per 16x16 tile of one
// subdomain, the rows of I_i in ascending order through matrix instructions
// (each value is one ascending chain over the rows; 128^3 Poisson 0.88 -> 0.18 ms
// and 24^3 elasticity 1.52 -> 0.09 ms against a thread per value).  Four
// instructions' operands are loaded at a time, the next four's beside them.
__global__ __launch_bounds__(64) void k_t1(const int64_t *__restrict__ int_ptr, const int64_t *__restrict__ scol_ptr,
                                           const int64_t *__restrict__ ext_off, const double *__restrict__ E,
                                           const int32_t *__restrict__ sub_blk,
                                           const int64_t *__restrict__ blk_val_off, const double *__restrict__ phi,
                                           const int64_t *__restrict__ t1_off, double *__restrict__ T1, int tiles) {
    const int i = blockIdx.y;
    const int n = int(int_ptr[i + 1] - int_ptr[i]);
    const int k = int(scol_ptr[i + 1] - scol_ptr[i]);
    const int g = sub_blk[i];
    const int ta = 16 * (blockIdx.x / tiles), tb = 16 * (blockIdx.x % tiles);
    if (n == 0 || ta >= k || tb >= k || g < 0) return;
    const int lane = threadIdx.x, li = lane & 15, lg = lane >> 4;
    const double *Ea = E + ext_off[i] + int64_t(min(ta + li, k - 1)) * n;
    const double *Xb = phi + blk_val_off[g] + int64_t(min(tb + li, k - 1)) * n;
    constexpr int U = 4;
    dbl4 acc = {0.0, 0.0, 0.0, 0.0};
    double a[U], x[U];
    auto load = [&](int l0, double (&aa)[U], double (&xx)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int l = l0 + 4 * u + lg;
            aa[u] = Ea[min(l, n - 1)];
            xx[u] = l < n ? Xb[l] : 0.0;   // (rows past the last add nothing)
        }
    };
    load(0, a, x);
    for (int l0 = 0; l0 < n; l0 += 4 * U) {
        double a2[U], x2[U];
        load(l0 + 4 * U, a2, x2);
#pragma unroll
        for (int u = 0; u < U; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], x[u], acc, 0, 0, 0);
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = a2[u], x[u] = x2[u];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int ra = ta + lg + 4 * v, cb = tb + li;
        if (ra < k && cb < k) T1[t1_off[i] + int64_t(ra) * k + cb] = acc[v];
    }
}

// Interface-interface part of A_0: for every component pair (c, d) with
// couplings in A, the entries of Phi_Gc^T A_{cd} Phi_Gd, couplings in a fixed
// order, into T2 (added into A_0 by target, k_a0_segments: components may share
// coarse columns).  One wavefront per pair and 64 entries, an entry per lane:
// the lanes bring 64 couplings' indices and values in together, through LDS;
// the entries' own values are read 16 couplings at a time before the 16
// dependent additions.  (An entry per thread with its own pair's loads: every
// lane on lines of its own, 128^3 Poisson 0.80 ms, 24^3 elasticity 0.83; now
// 0.28 and 0.32.)
__global__ __launch_bounds__(64) void k_t2(const double *__restrict__ Aval, const int32_t *__restrict__ pair_c,
                     const int32_t *__restrict__ pair_d, const int64_t *__restrict__ pair_off,
                     const int64_t *__restrict__ pair_eptr, const int64_t *__restrict__ pair_apos,
                     const int32_t *__restrict__ pair_lr_c, const int32_t *__restrict__ pair_lr_d,
                     const int32_t *__restrict__ comp_rank, const int64_t *__restrict__ phig_off,
                     const double *__restrict__ phig, double *__restrict__ T2) {
    __shared__ double sA[64];
    __shared__ int32_t sC[64], sD[64];
    const int q = blockIdx.x, lane = threadIdx.x;
    const int64_t loc = int64_t(blockIdx.y) * 64 + lane, cnt = pair_off[q + 1] - pair_off[q];
    if (int64_t(blockIdx.y) * 64 >= cnt) return;
    const int c = pair_c[q], d = pair_d[q];
    const int rd = comp_rank[d];
    // (lanes past the pair's entries repeat its last one)
    const int64_t mine = min(loc, cnt - 1);
    const int a = int(mine / rd), bb = int(mine % rd);
    const int64_t nrc = (phig_off[c + 1] - phig_off[c]) / comp_rank[c];
    const int64_t nrd = (phig_off[d + 1] - phig_off[d]) / rd;
    const double *pc = phig + phig_off[c] + a * nrc;
    const double *pd = phig + phig_off[d] + bb * nrd;
    const int64_t e1 = pair_eptr[q + 1];
    double acc = 0.0;
    for (int64_t e = pair_eptr[q]; e < e1; e += 64) {
        const int64_t f = min(e + lane, e1 - 1);
        wave_lds_fence();
        sC[lane] = pair_lr_c[f];
        sD[lane] = pair_lr_d[f];
        sA[lane] = Aval[pair_apos[f]];
        wave_lds_fence();
        const int m = int(min<int64_t>(64, e1 - e));
        constexpr int U = 16;
        for (int u0 = 0; u0 < m; u0 += U) {
            double x[U], y[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = pc[sC[u0 + u]], y[u] = pd[sD[u0 + u]];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u0 + u < m) acc += x[u] * sA[u0 + u] * y[u];
        }
    }
    if (loc < cnt) T2[pair_off[q] + loc] = acc;
}

// A0[tgt] += sum of the subdomain contributions of the segment, ascending
// subdomain order
__global__ void k_a0_segments(const int64_t *__restrict__ seg_tgt, const int64_t *__restrict__ seg_ptr,
                              const int64_t *__restrict__ seg_src, const double *__restrict__ T1,
                              double *__restrict__ A0, int64_t nseg) {
    const int64_t s = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (s >= nseg) return;
    double acc = 0.0;
    for (int64_t e = seg_ptr[s]; e < seg_ptr[s + 1]; ++e) acc += T1[seg_src[e]];
    A0[seg_tgt[s]] += acc;
}

// B = (A + A^T) / 2
__global__ void k_symmetrize(const double *__restrict__ A, double *__restrict__ B, int n) {
    const int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (t >= int64_t(n) * n) return;
    const int r = int(t / n), c = int(t % n);
    B[t] = 0.5 * (A[t] + A[int64_t(c) * n + r]);
}

// ---------------------------------------------------------------------------
// Inverse of the SPD coarse matrix by blocked Gauss-Jordan sweeps without
// pivoting (the pivots are Schur complements of an SPD matrix).  Sweeping
// block K of a symmetric matrix with P = A_KK^{-1}:
//   A_KK <- -P,  A_iK <- A_iK P,  A_Kj <- P A_Kj,  A_ij <- A_ij - A_iK P A_Kj;
// after all blocks the matrix holds -A^{-1}.
constexpr int GJ_NB = 32;
constexpr int GJ_LD = GJ_NB + 1;

// Two launches per block K (a separate pivot kernel of one workgroup and
// separate kernels for W and for storing it took 56, 48 and 16 us per block at
// n = 2,863 beside the update's 48; now 23 + 31 us).  KR = false: a handle with a
// memory cap and no room for the rows A(K, :), which the update then reads in
// place, and k_gj_fix stores the block's rows and columns after it.

// P = A_KK^{-1} by scalar sweeps, in every workgroup (one launch less, and no
// workgroup waits for another's), then for 64 rows i per workgroup: W(i, :) =
// A(i, K) P (rows in K get 0) and Kr(:, i) = A(K, i) as the update needs
// them, and the block's new values A(i, K) = W(i, :), A(K, i) = W(i, :)^T for i
// outside K.  A_KK itself is left for the update to replace (other workgroups
// read it here).  Each sweep writes the other of two LDS copies, one barrier per
// pivot; W is one ascending chain of products per value, by matrix instructions.
template <bool KR>
__global__ __launch_bounds__(256) void k_gj_panel(double *__restrict__ A, int n, int k0, int kb,
                                                  double *__restrict__ Pout, double *__restrict__ W,
                                                  double *__restrict__ Kr, int64_t ldk, int *__restrict__ status) {
    __shared__ double S[2][GJ_NB * GJ_LD];
    __shared__ double sW[64 * GJ_LD];
    const int tid = threadIdx.x, i0 = blockIdx.x * 64;
    const int pr = tid >> 5, pc = tid & 31;   // this thread's values (pr + 8 q, pc)
    const int wv = tid >> 6, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    // A(i, K) of this wavefront's 16 rows as operands, A(K, i) of the 64 columns
    const int ir = min(i0 + 16 * wv + li, n - 1);
    double a[8], kr[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int t = 4 * q + lg;
        a[q] = t < kb ? A[int64_t(ir) * n + k0 + t] : 0.0;
        kr[q] = A[int64_t(k0 + min(wv + 4 * q, kb - 1)) * n + min(i0 + lane, n - 1)];
    }
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = pr + 8 * q;
        v[q] = r < kb && pc < kb ? A[int64_t(k0 + r) * n + (k0 + pc)] : 0.0;
        S[0][r * GJ_LD + pc] = v[q];
    }
    __syncthreads();
    for (int j = 0; j < kb; ++j) {
        const double *T = S[j & 1];
        const double piv = T[j * GJ_LD + j];
        if (!(piv > 0.0)) {
            if (tid == 0) atomicCAS(status, 0, 1 + k0 + j);
            return;
        }
        const double p = 1.0 / piv, ajk = T[j * GJ_LD + pc];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = pr + 8 * q;
            const double aij = T[r * GJ_LD + j];
            if (r == j && pc == j) v[q] = -p;
            else if (pc == j) v[q] = aij * p;
            else if (r == j) v[q] = p * ajk;
            else v[q] = v[q] - aij * p * ajk;
            S[(j & 1) ^ 1][r * GJ_LD + pc] = v[q];
        }
        __syncthreads();
    }
    const double *T = S[kb & 1];   // -P
    if (blockIdx.x == 0)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (pr + 8 * q < kb && pc < kb) Pout[(pr + 8 * q) * kb + pc] = -v[q];
    // W, 16 rows per wavefront
    dbl4 w0 = {0.0, 0.0, 0.0, 0.0}, w1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int t = 4 * q + lg;   // (rows of P past kb: zeros, a is zero there too)
        w0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], t < kb ? -T[t * GJ_LD + li] : 0.0, w0, 0, 0, 0);
        w1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], t < kb ? -T[t * GJ_LD + 16 + li] : 0.0, w1, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int r = 16 * wv + lg + 4 * u, i = i0 + r;
        const bool inK = i >= k0 && i < k0 + kb;
        sW[r * GJ_LD + li] = inK || li >= kb ? 0.0 : w0[u];
        sW[r * GJ_LD + 16 + li] = inK || 16 + li >= kb ? 0.0 : w1[u];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {   // rows of W: two per pass and wavefront
        const int r = 2 * (wv + 4 * q) + (lane >> 5), t = lane & 31, i = i0 + r;
        if (i >= n) continue;
        const double x = sW[r * GJ_LD + t];
        W[int64_t(i) * GJ_NB + t] = x;
        if (KR && t < kb && !(i >= k0 && i < k0 + kb)) A[int64_t(i) * n + k0 + t] = x;
    }
    const int i = i0 + lane;
    if (KR && i < n) {
        const bool inK = i >= k0 && i < k0 + kb;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int t = wv + 4 * q;
            if (t < kb) {
                Kr[t * ldk + i] = kr[q];
                if (!inK) A[int64_t(k0 + t) * n + i] = sW[lane * GJ_LD + t];
            }
        }
    }
}

// A(i, j) -= W(i, :) . Kr(:, j) for i, j outside K, A_KK = -P; 64x64 tiles, 16
// rows per wavefront, by matrix instructions (one ascending chain per value,
// subtracted once).  Bound by reading and writing A.
template <bool KR>
__global__ __launch_bounds__(256) void k_gj_update(double *A, int n, int k0, int kb,
                                                   const double *__restrict__ W, const double *__restrict__ Kr,
                                                   int64_t ldk, const double *__restrict__ P) {
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
    const int i0 = blockIdx.y * 64 + 16 * wv, j0 = blockIdx.x * 64;
    const int ir = min(i0 + li, n - 1);
    double old[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            old[u][v] = A[int64_t(min(i0 + lg + 4 * v, n - 1)) * n + min(j0 + 16 * u + li, n - 1)];
    dbl4 acc[4] = {};
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int t = 4 * q + lg;
        const double a = W[int64_t(ir) * GJ_NB + t];   // (zero past kb)
        const double *row = KR ? Kr + min(t, kb - 1) * ldk : A + int64_t(k0 + min(t, kb - 1)) * n;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, row[min(j0 + 16 * u + li, n - 1)], acc[u], 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = i0 + lg + 4 * v;
        if (i >= n) continue;
        const bool iK = i >= k0 && i < k0 + kb;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = j0 + 16 * u + li;
            if (j >= n) continue;
            const bool jK = j >= k0 && j < k0 + kb;
            if (KR && iK && jK) A[int64_t(i) * n + j] = -P[(i - k0) * kb + (j - k0)];
            else if (!iK && !jK) A[int64_t(i) * n + j] = old[u][v] - acc[u][v];
        }
    }
}

// A(i, K) = W(i, :), A(K, i) = W(i, :)^T (i outside K), A_KK = -P
__global__ __launch_bounds__(256) void k_gj_fix(double *__restrict__ A, int n, int k0, int kb,
                                                const double *__restrict__ W, const double *__restrict__ P) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const bool inK = i >= k0 && i < k0 + kb;
    for (int t = 0; t < kb; ++t) {
        const double x = inK ? -P[(i - k0) * kb + t] : W[int64_t(i) * GJ_NB + t];
        A[int64_t(i) * n + k0 + t] = x;
        if (!inK) A[int64_t(k0 + t) * n + i] = x;
    }
}

__global__ void k_negate(double *__restrict__ A, int64_t cnt) {
    for (int64_t p = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; p < cnt;
         p += int64_t(gridDim.x) * blockDim.x)
        A[p] = -A[p];
}

}  // namespace gdsw
