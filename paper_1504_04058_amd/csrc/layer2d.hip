// 2D auxiliary problems H^M_q, H^R_p, H^L_p (Section 3.1): factorization
// (Algorithm 1), batched solves (the G~ operators of Algorithm 2) and the
// dense boundary-to-boundary maps used by the sweeps.
//
// Each 2D auxiliary problem lives on the n x L grid (i1 = 1..n, L sweep lines).
// Grouping the unknowns with the sweep axis fastest (Section 3.1: the quasi-1D
// subproblems reordered into a banded system) makes H block tridiagonal in i1
// with L x L blocks:
//   D_k      tridiagonal: the sweep-axis couplings s(lo+j+1/2)/(s1(k) h^2) and the diagonal,
//   E_k      diagonal coupling of block k to k+1: s1(k+1/2) / (s(lo+j) h^2),
// in the symmetric form.  The banded LU of the paper in block form, S_k = D_k -
// E_{k-1} S_{k-1}^-1 E_{k-1}, runs from both ends towards the middle block; the
// factor keeps the inverse of every block.  A solve is the forward sweep of both
// halves, y_k = S_k^-1 (g_k - E_{k-1} y_{k-1}), the middle block, and the
// backward sweep outwards, v_k = y_k - S_k^-1 E_k v_{k+1}.
#include <algorithm>

#include "asp_internal.h"
#include "mfma.h"

namespace {

// at most 256 registers per lane (two wavefronts per SIMD): the accumulators of
// the matrix instructions then live in ordinary registers.  With a larger
// budget the compiler puts them in the accumulation registers and copies them
// out and back around every scalar use (150 copies per pivot pair of the
// factorization).
#define ASP_PLAIN_ACC(...) __attribute__((amdgpu_waves_per_eu(__VA_ARGS__)))

// raw buffer stores: dword 3 of the resource (32-bit data format) and an
// offset past any range, whose writes the hardware drops
constexpr int BUF_DW3 = 0x00020000;
constexpr unsigned BUF_OOB = 0x80000000u;
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// off past the range drops the write, soff (uniform, < 2^31) is added to it.
// A 16-byte store adds soff to the lane's offset and gives the instruction none:
// the compiler separates a store of more than 8 bytes from a following write of
// its data registers only when the instruction has no scalar offset, and with
// one the last lanes' data were overwritten before the store had read them
// (measured: low-order bits of FP64 forward results, lanes 60 - 63).
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned soff, zd v) {
    u32x4 d;
    __builtin_memcpy(&d, &v, sizeof(d));
    __builtin_amdgcn_raw_buffer_store_b128(d, r, off + soff, 0, 0);
}
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned soff, zf v) {
    u32x2 d;
    __builtin_memcpy(&d, &v, sizeof(d));
    __builtin_amdgcn_raw_buffer_store_b64(d, r, off, soff, 0);
}

// ----------------------------------------------------------------------------
// Twisted order of the blocks: the block recurrence runs from both ends towards
// the middle block p = mid_block(n),
//   S_k = D_k - E_{k-1} S_{k-1}^-1 E_{k-1}   for k = 1 .. p-1,
//   R_k = D_k - E_k R_{k+1}^-1 E_k           for k = n .. p+1,
//   M_p = D_p - E_{p-1} S_{p-1}^-1 E_{p-1} - E_p R_{p+1}^-1 E_p,
// so that every chain of dependent blocks (the factorization, each pass of a
// solve, the boundary maps) is half as long as with one direction and the two
// halves run at the same time.  Half `dir` (0: blocks 1 .. p-1, 1: blocks n ..
// p+1) counts its blocks s = 1 .. np from its end; s = np + 1 is block p.
// ----------------------------------------------------------------------------
struct Half {
    int n, dir, np;
    __device__ __forceinline__ Half(int n_, int dir_)
        : n(n_), dir(dir_), np(dir_ ? n_ - mid_block(n_) : mid_block(n_) - 1) {}
    __device__ __forceinline__ int blk(int s) const { return dir ? n + 1 - s : s; }
    // the half line between blocks s and s + 1 of this half (index into AxisTables::sh)
    __device__ __forceinline__ int half_line(int s) const { return dir ? n - s : s; }
};

// orders the LDS accesses of one wavefront among its lanes (LDS operations of
// a wavefront complete in order; this keeps the compiler from moving them)
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// ----------------------------------------------------------------------------
// factorization: each half of a problem is a chain of np blocks, one 16-row
// strip of the current block per wavefront, held in the accumulator layout of
// the FP64 matrix instructions (lane l: column l % 16 of each 16-wide tile,
// rows l / 16 + 4 v).  S_k is formed from S_{k-1}^-1 in place and inverted by
// Gauss-Jordan elimination without pivoting, two pivots at a time: the two
// pivot rows pass through LDS (one exchange per pair), every wavefront inverts
// the 2 x 2 pivot block itself, and the rank-2 complex update of a tile is one
// FP64 matrix instruction for the real and one for the imaginary plane (K = 4:
// re and im of both pivots).  S_k is complex symmetric, and an in-place
// elimination keeps A[i][k] = -A[k][i] between eliminated and remaining rows
// and A[i][k] = A[k][i] otherwise, so the pivot columns are read from the pivot
// rows.  A zero or non-finite pivot is reported as a breakdown.  Arithmetic in
// double; the stored factor is rounded to TS.
// What bounds it: the chain pivot rows -> LDS -> 2 x 2 inverse (two dependent
// FP64 reciprocals) -> update, once per pair and block, about 1500 cycles; hence
// two pivots per exchange, both halves at once and few instructions per pair
// (n = 255, layers of 8 lines, FP64: 2.66 ms with one direction, one pivot per
// exchange and vector arithmetic, 0.99 ms now; n = 1023: 11.9 -> 4.7 ms).
// ----------------------------------------------------------------------------
// 1 / p, q = |p|^2: the hardware reciprocal estimate with two Newton steps
// (full precision) instead of an IEEE division, half the latency
__device__ __forceinline__ zd cinv_fast(zd p, double q) {
    double r = __builtin_amdgcn_rcp(q);
    r = fma(fma(-q, r, 1.0), r, r);
    r = fma(fma(-q, r, 1.0), r, r);
    return mk(p.x * r, -p.y * r);
}

template <typename TS, int LR>
__device__ __forceinline__ void factor2d_body(const SubDesc& d, bool live, int npair, int wl, AxisTables ax,
                                              const zd* __restrict__ subtab,
                                              const double* __restrict__ ksq, int n,
                                              cplx<TS>* __restrict__ fac, int* __restrict__ flag,
                                              zd* __restrict__ rowbuf_, zd* __restrict__ xch) {
    constexpr int NW = LR / 16, CT = LR / 16;   // strips per half, tiles per strip
    using D = Mfma<double>;
    const Half H(n, wl / NW);
    const int rt = wl % NW;
    const int L = d.L;
    const int l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
    zd* rowbuf = rowbuf_ + H.dir * (4 * LR + 8);   // [parity]: two rows of LR, a 2 x 2 block
    const zd* tab = subtab + d.tab_off;
    const zd* ssh = tab;                // s at half lines lo-1/2 .. hi+1/2
    const zd* sinv2 = tab + L + 1;      // 1/(s h^2) on lines lo..hi
    const zd* sinv = tab + 2 * L + 1;   // 1/s on lines lo..hi
    const zd zero = mk(0.0, 0.0);
    zd srow[4], scol[CT];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = 16 * rt + lk + 4 * v;
        srow[v] = csel(i < L, sinv2[min(i, L - 1)], zero);
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) scol[ct] = csel(16 * ct + li < L, sinv2[min(16 * ct + li, L - 1)], zero);
    // D_k: this lane holds at most one entry of the tridiagonal in its diagonal
    // tile (column jd, row jd + od), of value kq is1 cd + (s1 terms) cs + cn / (s1 h^2);
    // tiles next to the diagonal one hold one corner entry each, cn / (s1 h^2)
    const int jd = 16 * rt + li, jc = min(jd, L - 1);
    const int od = ((lk - li + 1) & 3) - 1;                 // -1, 0, 1 (2: none)
    const int vd = (li + od - lk) >> 2;                     // its register, 0..3 if inside
    const bool has = od < 2 && li + od >= 0 && li + od < 16 && jd < L && jd + od < L;
    const bool ond = has && od == 0;
    const zd cd_ = csel(ond, sinv[jc], zero);
    const zd cs_ = csel(ond, -sinv2[jc], zero);
    const zd cn_ = csel(ond, -(ssh[jc + 1] + ssh[jc]), csel(has, ssh[max(jc, min(jd + od, L))], zero));
    const bool padd = od == 0 && li + od >= 0 && jd >= L;   // identity padding
    // corner of tile rt - 1 (row 16 rt, column 16 rt - 1) and rt + 1
    const bool clo = lk == 0 && li == 15 && rt > 0 && 16 * rt < L;
    const bool chi = lk == 3 && li == 0 && 16 * rt + 16 < L;
    const zd cnlo = csel(clo, ssh[min(16 * rt, L)], zero);
    const zd cnhi = csel(chi, ssh[min(16 * rt + 16, L)], zero);
    const double* ksq_j = ksq + (long long)n * (d.lo + jc - 1);
    // S_k^-1 column-major with leading dimension LR through a buffer resource,
    // stored as its transpose (it is symmetric): 16 lanes write one line
    const __amdgpu_buffer_rsrc_t rf =
        __builtin_amdgcn_make_buffer_rsrc(fac + d.fac_off, 0, 0x7fffffff, BUF_DW3);
    unsigned foff[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = 16 * rt + lk + 4 * v;
        foff[v] = live && i < L ? (unsigned)((i * LR + li) * sizeof(cplx<TS>)) : BUF_OOB;
    }
    const unsigned fstep = (unsigned)(L * LR * sizeof(cplx<TS>));
    bool bad = false;
    f64x4 re[CT], im[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int v = 0; v < 4; ++v) re[ct][v] = im[ct][v] = 0.0;

    // V <- D_k - c1 V c1 (c1 the couplings to the previous block), from the
    // tables of block k; sm + sp: s1 at the half lines around it
    auto form = [&](zd c1, zd ssum, zd is2, zd is, double kq) {
        const zd addd = (kq * is) * cd_ + ssum * cs_ + is2 * cn_;
        const zd alo = is2 * cnlo, ahi = is2 * cnhi;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const zd cc = c1 * scol[ct];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                zd x = -((c1 * srow[v]) * mk(re[ct][v], im[ct][v]) * cc);
                if (ct == rt) {
                    x = x + csel(v == vd && has, addd, zero);
                    if (v == vd && padd) x = mk(1.0, 0.0);
                }
                if (ct + 1 == rt && v == 0) x = x + alo;
                if (ct == rt + 1 && v == 3) x = x + ahi;
                re[ct][v] = x.x;
                im[ct][v] = x.y;
            }
        }
    };
    int par = 0;
    auto invert = [&]() {
        for (int tb = 0; tb < CT; ++tb) {
            const bool strip = rt == tb;   // this wavefront holds the pivot rows
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (8 * tb + q >= npair) break;
                const int kk = 16 * tb + 2 * q;
                const int vk = q >> 1;
                zd* R0 = rowbuf + par * (2 * LR + 4);   // rows kk, kk + 1, then the pivot block
                zd* const PB = R0 + 2 * LR;
                par ^= 1;
                const bool mine = strip && (lk >> 1) == (q & 1);   // lanes holding the pivot rows
                const bool ep = (li >> 1) == q;                    // ... the pivot columns of tile tb
                if (mine) {
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        zd x = mk(re[ct][vk], im[ct][vk]);
                        if (ct == tb) {
                            // the pivot block apart; in its place the identity, whose product
                            // with the inverse gives the pivot columns
                            if (ep) PB[2 * (lk & 1) + (li & 1)] = x;
                            x = csel(ep, mk((li & 1) == (lk & 1) ? 1.0 : 0.0, 0.0), x);
                        }
                        R0[(lk & 1) * LR + 16 * ct + li] = x;
                    }
                }
                if constexpr (NW == 1)
                    wave_lds_fence();
                else
                    __syncthreads();
                const zd a = PB[0], b = PB[1], dd = PB[3];
                zd r0[CT], r1[CT];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    r0[ct] = R0[16 * ct + li];
                    r1[ct] = R0[LR + 16 * ct + li];
                }
                // row i = 16 rt + li of -[A[i][kk] A[i][kk+1]], this lane's K entry of
                // the real and the imaginary plane; the pivot rows take the rows of
                // the inverse times the rows themselves (unit entries)
                const zd ci = R0[(lk >> 1) * LR + 16 * rt + li];
                const double sg = 16 * rt + li < kk ? 1.0 : -1.0;
                const bool odd = lk & 1;
                double are = sg * (odd ? -ci.y : ci.x);
                double aim = sg * (odd ? ci.x : ci.y);
                // pivot columns and rows start from zero
                if (strip) {
                    are = ep ? (lk == 2 * (li & 1) ? 1.0 : 0.0) : are;
                    aim = ep ? (lk == 2 * (li & 1) + 1 ? 1.0 : 0.0) : aim;
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        re[ct][vk] = mine ? 0.0 : re[ct][vk];
                        im[ct][vk] = mine ? 0.0 : im[ct][vk];
                    }
                }
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
                    if (ct == tb)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            re[ct][v] = ep ? 0.0 : re[ct][v];
                            im[ct][v] = ep ? 0.0 : im[ct][v];
                        }
                // the inverse of the 2 x 2 pivot block [a b; b d], eliminated in order
                const double pa = abs2(a);
                const zd i1 = cinv_fast(a, pa);
                const zd m = b * i1;
                const zd p2 = dd - m * b;
                const double pb = abs2(p2);
                const zd i2 = cinv_fast(p2, pb);
                const zd p01 = -(m * i2);
                const zd p00 = i1 - m * p01;
                if (!(pa > 1e-300) || !(pb > 1e-300) || !isfinite(pa) || !isfinite(pb)) bad = true;
                // this lane's K entry of the inverse times the rows: re / im of row
                // kk (lk = 0, 1) or kk + 1 (lk = 2, 3)
                const zd c0 = csel(lk < 2, p00, p01), c1 = csel(lk < 2, p01, i2);
                const double f0 = odd ? c0.y : c0.x, f1 = odd ? c0.x : -c0.y;
                const double f2 = odd ? c1.y : c1.x, f3 = odd ? c1.x : -c1.y;
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const double bk = fma(f0, r0[ct].x, fma(f1, r0[ct].y, fma(f2, r1[ct].x, f3 * r1[ct].y)));
                    re[ct] = D::mac(are, bk, re[ct]);
                    im[ct] = D::mac(aim, bk, im[ct]);
                }
            }
        }
    };
    auto store = [&](int k, bool on) {
        const unsigned base = (unsigned)(k - 1) * fstep;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const zd x = csel(16 * ct + li < L, mk(re[ct][v], im[ct][v]), zero);
                buf_store(rf, on ? foff[v] + (unsigned)(16 * ct * sizeof(cplx<TS>)) : BUF_OOB, base, ccast<TS>(x));
            }
    };
    // the tables of block k: couplings s1 at k -+ 1/2, 1/(s1 h^2), 1/s1 and
    // omega^2/c^2 on this lane's column, fetched one block ahead
    struct Step {
        zd sh_m, sh_p, is2, is;
        double kq;
    };
    auto fetch = [&](Step& S, int k) {
        S.sh_m = ax.sh[k - 1];
        S.sh_p = ax.sh[k];
        S.is2 = ax.inv_sh2[k - 1];
        S.is = ax.inv_s[k - 1];
        S.kq = ksq_j[k - 1];
    };
    // both halves take smax steps together (shared barriers): the shorter one
    // starts late, on its first block, which it forms and inverts once unstored
    const int p = mid_block(n);
    const int smax = max(p - 1, n - p);
    Step cur, nxt;
    fetch(cur, H.blk(1));
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    for (int it = 1; it <= smax; ++it) {
        const int s = it - (smax - H.np);
        fetch(nxt, H.blk(min(max(s, 0), H.np) + 1));
        // s <= 1: no previous block (the state is finite, the coupling zero)
        const zd c1 = csel(s > 1, H.dir ? cur.sh_p : cur.sh_m, zero);
        form(c1, cur.sh_m + cur.sh_p, cur.is2, cur.is, cur.kq);
        invert();
        store(H.blk(max(s, 1)), s >= 1);
        cur = nxt;
    }
    // the middle block: half 1 hands R_{p+1}^-1 over in the accumulator layout
    if (H.dir == 1)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int v = 0; v < 4; ++v) xch[((rt * CT + ct) * 4 + v) * 64 + l] = mk(re[ct][v], im[ct][v]);
    __syncthreads();
    const bool bad_halves = bad;
    if (H.dir == 0) {
        fetch(cur, p);
        f64x4 xr[CT], xi[CT];
        const zd cp = csel(n > p, cur.sh_p, zero);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const zd x = xch[((rt * CT + ct) * 4 + v) * 64 + l];
                const zd t = (cp * srow[v]) * x * (cp * scol[ct]);
                xr[ct][v] = t.x;
                xi[ct][v] = t.y;
            }
        form(csel(p > 1, cur.sh_m, zero), cur.sh_m + cur.sh_p, cur.is2, cur.is, cur.kq);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                re[ct][v] -= xr[ct][v];
                im[ct][v] -= xi[ct][v];
            }
    }
    invert();
    if (H.dir == 1) bad = bad_halves;
    store(p, H.dir == 0);
    if (bad && live) *flag = 1;
}

// Workgroups of 2 LX / 16 wavefronts, LX the larger row count of the plan: a
// problem of LR rows takes 2 LR / 16 of them (one strip per wavefront and
// half), so LX / LR problems share a workgroup.  The M problems come first,
// then the R and L problems.
struct FactorClass {
    int first, count, LR, npair;   // problems desc[first ..), pivot pairs (the widest problem's)
    int blocks;
};
template <typename TS, int LX>
__global__ __launch_bounds__(8 * LX) ASP_PLAIN_ACC(2) void factor2d_kernel(const SubDesc* __restrict__ desc,
                                                         FactorClass cm, FactorClass cr, AxisTables ax,
                                                         const zd* __restrict__ subtab,
                                                         const double* __restrict__ ksq, int n,
                                                         cplx<TS>* __restrict__ fac,
                                                         int* __restrict__ flag) {
    __shared__ zd rows[8 * LX + 16 * (LX / 16)];   // pivot rows of every problem
    __shared__ zd xch[LX * LX];      // R_{p+1}^-1 of every problem
    const bool ism = (int)blockIdx.x < cm.blocks;
    const FactorClass c = ism ? cm : cr;
    const int g = ism ? blockIdx.x : blockIdx.x - cm.blocks;
    const int w = threadIdx.x >> 6;
    const int per = LX / c.LR, wpp = c.LR / 8;
    const int slot = w / wpp;
    const int idx = g * per + slot;
    const bool live = idx < c.count;
    const SubDesc d = desc[c.first + min(idx, c.count - 1)];
    zd* rb = rows + slot * (8 * c.LR + 16);
    zd* xc = xch + slot * c.LR * c.LR;
    const int wl = w % wpp;
    if (LX == 16 || c.LR == 16)
        factor2d_body<TS, 16>(d, live, c.npair, wl, ax, subtab, ksq, n, fac, flag, rb, xc);
    else if (LX == 32 || c.LR == 32)
        factor2d_body<TS, (LX < 32 ? 16 : 32)>(d, live, c.npair, wl, ax, subtab, ksq, n, fac, flag, rb, xc);
    else
        factor2d_body<TS, LX>(d, live, c.npair, wl, ax, subtab, ksq, n, fac, flag, rb, xc);
}

// ----------------------------------------------------------------------------
// The diagonal blocks G_k of H^-1 of a map problem (R_p or L_p, 1 < p < m),
// from the stored inverses: G = M_p^-1 at the middle block and, outwards in
// each half (S_k^-1 standing for R_k^-1 in the second, s counted from its end),
//   G_s = S_s^-1 + S_s^-1 E_s G_{s+1} E_s S_s^-1,
// E_s the diagonal coupling of blocks s and s + 1 (H, S_k^-1 and G_k are complex
// symmetric).  The boundary maps then start from two columns of every G_k
// (IN_TWIST solves).  One 256-thread workgroup per problem and half; thread
// (j, g) holds rows g RPL .. of column j of G in double, the two products of a
// step go through LDS.  Columns grow and jout of each G_k are stored (type TS)
// at the problem's g_off in the map buffer, [k][2][LR].  Bound by the latency
// of the step chain.
// ----------------------------------------------------------------------------
constexpr int FB = 256;   // threads per workgroup

template <typename TS, int LR>
__device__ __forceinline__ void rgf2d_body(const SubDesc& d, AxisTables ax, const zd* __restrict__ subtab,
                                           int n, int dir, const cplx<TS>* __restrict__ fac,
                                           cplx<TS>* __restrict__ tbuf, zd (*A)[LR + 1], zd (*Bm)[LR + 1]) {
    constexpr int G = FB / LR, RPL = LR / G;
    const Half H(n, dir);
    const int L = d.L;
    const int t = threadIdx.x, j = t % LR, g = t / LR;
    const zd* sinv2 = subtab + d.tab_off + L + 1;        // 1/(s h^2) on lines lo..hi
    const zd ecol = j < L ? sinv2[min(j, L - 1)] : mk(0.0, 0.0);
    zd erow[RPL];
#pragma unroll
    for (int q = 0; q < RPL; ++q) {
        const int r = g * RPL + q;
        erow[q] = r < L ? sinv2[min(r, L - 1)] : mk(0.0, 0.0);
    }
    const int grow = (d.kind == ASP_SUB_R) ? 0 : L - 1;
    const int jout = (d.kind == ASP_SUB_R) ? (d.xe - d.lo) : (d.xs - d.lo);
    const cplx<TS>* F = fac + d.fac_off;
    cplx<TS>* Gout = tbuf + d.g_off;
    zd Gv[RPL], sv[RPL];
    for (int s = H.np + 1; s >= 1; --s) {
        const int k = H.blk(s);
        // S_k^-1 (block k - 1, column-major, rows past L zero): column j
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
            const int r = g * RPL + q;
            sv[q] = (j < L && r < L) ? ccast<double>(F[(long long)(k - 1) * L * LR + (long long)j * LR + r])
                                     : mk(0.0, 0.0);
        }
        if (s == H.np + 1) {
#pragma unroll
            for (int q = 0; q < RPL; ++q) Gv[q] = sv[q];
        } else {
            const zd sh = ax.sh[H.half_line(s)];               // s1 between blocks s and s + 1
            // A = G_{s+1} E_s, Bm = S_s^-1
#pragma unroll
            for (int q = 0; q < RPL; ++q) {
                const int r = g * RPL + q;
                A[r][j] = Gv[q] * (sh * ecol);
                Bm[r][j] = sv[q];
            }
            __syncthreads();
            // X = E_s (A Bm) = E_s G_{s+1} E_s S_s^-1
            zd xv[RPL];
#pragma unroll
            for (int q = 0; q < RPL; ++q) {
                const int r = g * RPL + q;
                zd acc = mk(0.0, 0.0);
                for (int l = 0; l < L; ++l) acc = cfma(A[r][l], Bm[l][j], acc);
                xv[q] = (sh * erow[q]) * acc;
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < RPL; ++q) A[g * RPL + q][j] = xv[q];
            __syncthreads();
            // G_s = S_s^-1 + S_s^-1 X, with (S_s^-1)[r][l] = Bm[l][r] (symmetric)
#pragma unroll
            for (int q = 0; q < RPL; ++q) {
                const int r = g * RPL + q;
                zd acc = mk(0.0, 0.0);
                for (int l = 0; l < L; ++l) acc = cfma(Bm[l][r], A[l][j], acc);
                Gv[q] = sv[q] + acc;
            }
            __syncthreads();   // A and Bm are written again at the next step
        }
        if (s == H.np + 1 && dir) continue;   // the middle block is written by half 0
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
            const int r = g * RPL + q;
            if (r < L && j == grow) Gout[(long long)(k - 1) * 2 * LR + r] = ccast<TS>(Gv[q]);
            if (r < L && j == jout) Gout[(long long)(k - 1) * 2 * LR + LR + r] = ccast<TS>(Gv[q]);
        }
    }
}

template <typename TS, int LR>
__global__ __launch_bounds__(FB) void rgf2d_kernel(const SubDesc* __restrict__ desc,
                                                  const int* __restrict__ jobs0,
                                                  const int* __restrict__ jobs1, AxisTables ax,
                                                  const zd* __restrict__ subtab, int n,
                                                  const cplx<TS>* __restrict__ fac,
                                                  cplx<TS>* __restrict__ tbuf) {
    __shared__ zd A[LR][LR + 1];
    __shared__ zd Bm[LR][LR + 1];
    // blockIdx.y picks one of two job lists (the map problems of the two sweeps), z the half
    const SubDesc d = desc[(blockIdx.y ? jobs1 : jobs0)[blockIdx.x]];
    rgf2d_body<TS, LR>(d, ax, subtab, n, blockIdx.z, fac, tbuf, A, Bm);
}

// ----------------------------------------------------------------------------
// batched solves on the matrix cores: one workgroup per (auxiliary problem,
// chunk of 16 right-hand sides, half), one, two or four wavefronts per 16-row
// tile of the step vectors.  The forward kernel runs both halves towards
// the middle block and keeps its results in scratch; the backward kernel
// solves the middle block (each half for itself) and runs outwards.  A block
// step is the product of S_k^-1 with the chunk's step vectors.  The wavefront's
// rows of S_k^-1 come straight from memory into the matrix-core operand layout,
// some steps ahead into fixed register slots (the step loops are unrolled by
// their number); columns past L lie past the buffer resource's range and read zero.
// With 16 rows a wavefront holds the whole step vector: the columns of the
// product run in the order in which the result tile holds its rows, so a
// step's result is the next step's operand without leaving its lanes (no LDS,
// no barrier).  With more rows the step vectors pass through LDS, one barrier
// per step.
// What bounds it: few right-hand sides, the latency of a step (the matrix
// instructions of one tile in sequence, the exchange, the scaling; n = 511 with 8:
// matrix cores 15 - 24% busy); many, the memory instructions (n = 1023 with 64:
// address units busy 64 - 82% of the time, matrix cores 26 - 36%), then the round
// trip of the forward results (an M-solve writes 3.1 GB of them and reads them and
// the factor, 6.4 GB, in 3.3 ms).  Two halves at once and
// 16 right-hand sides per workgroup give twice the chains of half the length
// and no work for absent right-hand sides beyond 16.
// ----------------------------------------------------------------------------
// complex 16 x 16 FP32 accumulator of the three-product (Gauss) form:
// p1 = (a_r + a_i) b_r, p2 = a_r (b_i - b_r), p3 = a_i (b_r + b_i);
// re = p1 - p3, im = p1 + p2 (three real products instead of four)
struct KTile3 {
    f32x4 p1, p2, p3;
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int v = 0; v < 4; ++v) p1[v] = p2[v] = p3[v] = 0.f;
    }
};
__device__ __forceinline__ void kmac3(KTile3& c, zf a, zf b) {
    c.p1 = Mfma<float>::mac(a.x + a.y, b.x, c.p1);
    c.p2 = Mfma<float>::mac(a.x, b.y - b.x, c.p2);
    c.p3 = Mfma<float>::mac(a.y, b.x + b.y, c.p3);
}

// Vectors inside an apply hold the right-hand sides (slots) fastest, in the
// factor precision: entry (sweep line, i1, slot) at ((line - 1) n + i1) ws +
// slot, ws the number of right-hand sides; boundary data of an R/L problem in
// double at (row n + i1) ws + slot.  A wavefront's 16 right-hand sides of a grid point
// are then one contiguous run (128 bytes in FP32), where the caller's layout
// puts each in a line of its own and a block step uses 16 bytes of it (written
// through an LDS stage and flushed every eight steps, that cost the R/L solves a
// third of their time).  n = 1023, 64 right-hand sides, FP32, ms per apply with
// the caller's layout / this one: M 4.34 / 3.84 (its copy in included), R and L
// 4.02 / 2.71, final sum 0.80 / 0.54.
struct SolveArgs {
    const SubDesc* desc;
    const int* jobs;
    int njobs, njobs0, jobs1;   // jobs[0 .. njobs0) and jobs[jobs1 .. ): njobs in all
    int nact;            // right-hand sides (columns of a map), slots of the vectors
    const void* fac;
    AxisTables ax;
    const zd* subtab;
    const void* r;       // IN_GRID: data
    const zd* W;         // IN_BOUNDARY: boundary data
    void* out;           // solutions on X_p
    void* out_L;         // ... of the L problems
    void* Tout;          // IN_TWIST: boundary-to-boundary maps
    void* y;             // forward results [problem][chunk][block][LR][16]
    int buf_ok;          // IN_TWIST: the byte offsets of a map fit the 31-bit buffer range
    int twist_kind;      // IN_TWIST: 0 both triangles of each half, 2 the propagators
    int n;
};

constexpr int RC = 16;         // right-hand sides per workgroup: one matrix-core tile

// 8 or 16 bytes through a buffer resource, zero past its range
template <typename T>
__device__ __forceinline__ cplx<T> buf_load(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned soff) {
    cplx<T> v;
    if constexpr (sizeof(T) == 4) {
        const u32x2 d = __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0);
        __builtin_memcpy(&v, &d, sizeof(v));
    } else {
        const u32x4 d = __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0);
        __builtin_memcpy(&v, &d, sizeof(v));
    }
    return v;
}

// a table entry that is the same for a whole wavefront, through the scalar cache
// (as a plain load it would take four vector registers per slot)
__device__ __forceinline__ zd uniform_load(const zd* p) {
    const auto q = (const __attribute__((address_space(4))) double*)(p);
    return mk(q[0], q[1]);
}

// One wavefront's 16-row tile of a block step, or (KW = 2, 4) its product over
// a share of the columns.  With KW = 1 a wavefront holds the rows of its result tile of
// the step vectors and reads the others' from LDS; with KW > 1 it holds those of
// its columns: every wavefront puts its product's share into LDS and forms its
// entries of the next step vector from the sum of the shares, one barrier per
// step either way.
template <typename T, int LR, bool SPL, int KW>
struct BlockTile {
    static constexpr int NW = LR / 16;
    static constexpr int KS = ((sizeof(T) == 8 && LR == 64) ? 12 : LR / 4) / KW;   // operand entries per lane
    static constexpr int NX = KW > 1 ? KS : 4;   // entries of the step vectors a lane holds
    static constexpr int TBS = RC + 1;   // padded row stride of the step vectors in LDS
    int l, li, lk, rt, kq, L;
    unsigned aoff[KS];           // byte offsets of this lane's operand entries, past the range if unused
    __amdgpu_buffer_rsrc_t rf;
    unsigned fstep;

    // the column of S^-1 that operand entry j of this lane holds
    __device__ __forceinline__ int col(int j) const {
        if constexpr (SPL) return NW == 1 ? 4 * lk + j : 32 * (j >> 3) + 8 * lk + (j & 7);
        if constexpr (KW > 1) return xrow(j);
        if constexpr (NW == 1) return Mfma<T>::row(l, j);
        return 4 * j + lk;
    }
    // the row of entry e of the step vectors: of the wavefront's result tile, or
    // of its share of the columns
    __device__ __forceinline__ int xrow(int e) const {
        if constexpr (KW > 1) {
            const int j = kq * KS + e;
            return 16 * (j >> 2) + Mfma<T>::row(l, j & 3);
        }
        return 16 * rt + Mfma<T>::row(l, e);
    }
    // KW > 1: a product's share of this wavefront into LDS, [share][tile][entry][lane]
    // (lanes in order: no bank conflicts), and the sum over the shares of the
    // entries it holds, in a fixed order
    __device__ __forceinline__ void put(cplx<T>* part, const CTile<T>& acc) const {
#pragma unroll
        for (int v = 0; v < 4; ++v) part[((kq * NW + rt) * 4 + v) * 64 + l] = mk<T>(acc.re[v], acc.im[v]);
    }
    __device__ __forceinline__ void gather(const cplx<T>* part, cplx<T> (&x)[NX]) const {
#pragma unroll
        for (int e = 0; e < NX; ++e) {
            const int j = kq * KS + e;
            x[e] = part[j * 64 + l];
#pragma unroll
            for (int q = 1; q < KW; ++q) x[e] = x[e] + part[(q * NW * 4 + j) * 64 + l];
        }
    }
    // LDS so that gather() gives x (rows of the first tile's wavefronts in share 0)
    __device__ __forceinline__ void put_sum(cplx<T>* part, const cplx<T> (&x)[NX]) const {
        if (kq > 0)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[((kq * NW + rt) * 4 + v) * 64 + l] = mk<T>(T(0), T(0));
        if (rt == 0)
#pragma unroll
            for (int e = 0; e < NX; ++e) part[(kq * KS + e) * 64 + l] = x[e];
    }
    __device__ __forceinline__ void init(const SubDesc& d, const cplx<T>* F) {
        l = threadIdx.x & 63;
        li = l & 15;
        lk = l >> 4;
        rt = (threadIdx.x >> 6) % NW;
        kq = (threadIdx.x >> 6) / NW;
        L = d.L;
        rf = __builtin_amdgcn_make_buffer_rsrc(const_cast<cplx<T>*>(F), 0, 0x7fffffff, BUF_DW3);
        fstep = (unsigned)(L * LR * sizeof(cplx<T>));
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            const int c = col(j);
            aoff[j] = c < L ? (unsigned)((c * LR + 16 * rt + li) * sizeof(cplx<T>)) : BUF_OOB;
        }
    }
    __device__ __forceinline__ void load(cplx<T> (&a)[KS], int blk) const {
#pragma unroll
        for (int j = 0; j < KS; ++j) a[j] = buf_load<T>(rf, aoff[j], (unsigned)(blk - 1) * fstep);
    }
    // the step vectors: the lane's own values u (one tile) or the LDS copy tb
    __device__ __forceinline__ void vectors(cplx<T> (&b)[KS], const cplx<T> (&u)[NX], const cplx<T> (*tb)[TBS]) const {
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            if constexpr (NW == 1 || KW > 1)
                b[j] = u[j];
            else
                b[j] = tb[col(j)][li];
        }
    }
    // S^-1 (operand a) times the step vectors
    __device__ __forceinline__ CTile<T> product(const cplx<T> (&a)[KS], const cplx<T> (&b)[KS]) const {
        CTile<T> acc;
        const int ksn = (L + 3) >> 2;   // 4-column steps in use
        if constexpr (SPL) {
            acc.zero();
#pragma unroll
            for (int h = 0; h < (KS + 7) / 8; ++h) {
                float ar[8], ai[8], br[8], bi[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bool in = 8 * h + j < KS;
                    const cplx<T> av = in ? a[(8 * h + j) % KS] : mk<T>(T(0), T(0));
                    const cplx<T> bv = in ? b[(8 * h + j) % KS] : mk<T>(T(0), T(0));
                    ar[j] = av.x;
                    ai[j] = av.y;
                    br[j] = bv.x;
                    bi[j] = bv.y;
                }
                cmac_split(acc, ar, ai, br, bi);
            }
        } else if constexpr (std::is_same<T, float>::value) {
            KTile3 k3;
            k3.zero();
#pragma unroll
            for (int j = 0; j < KS; ++j)
                if (NW == 1 || KW > 1 || j <= KS / 2 || j < ksn) kmac3(k3, a[j], b[j]);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                acc.re[v] = k3.p1[v] - k3.p3[v];
                acc.im[v] = k3.p1[v] + k3.p2[v];
            }
        } else {
            acc.zero();
#pragma unroll
            for (int j = 0; j < KS; ++j)
                if (NW == 1 || KW > 1 || j <= KS / 2 || j < ksn) cmac(acc, a[j], b[j]);
        }
        return acc;
    }
};

// the work item of a workgroup: the chunks of one (problem, half) are
// consecutive items of one XCD (they share its factor in the L2 cache)
struct SolveItem {
    int jl, ch, dir;
    bool ok;
    __device__ __forceinline__ SolveItem(int njobs, int nchunk) {
        const int B = njobs * nchunk * 2;
        const int per = (B + 7) / 8;
        const int w = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
        ok = w < B && (int)(blockIdx.x >> 3) < per;
        ch = w % nchunk;
        dir = (w / nchunk) & 1;
        jl = w / (2 * nchunk);
    }
};

// __syncthreads with the wait for this wavefront's LDS accesses spelled out: in a
// loop entered after an explicit wait for everything the compiler takes the
// barrier's own wait at the loop's head for redundant, also on the way round,
// where LDS writes are outstanding (seen in the code of the step loops: another
// wavefront then read what the step before the last had left).
__device__ __forceinline__ void step_sync() {
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __syncthreads();
}

// Register slots of a step's loads: one fewer than that many steps are in flight.
// A step of a 16-row problem in FP32 takes 0.4 us, less than half of a loaded
// HBM read, and its slots are small: three steps ahead (R and L solves at n =
// 511, ms per apply: two steps 0.353, three 0.274, five 0.276).  The other
// steps are longer and a fourth slot would spill: two ahead; the maps' chains
// have the chip full (three steps ahead: 5% slower).  Wavefronts per SIMD that
// the registers are held to: at three the slots spill.
template <typename T, int LR, int INM>
constexpr int nslot() { return LR == 16 && INM != IN_TWIST && sizeof(T) == 4 ? 4 : 3; }
template <typename T, int LR>
constexpr int solve_waves() { return LR == 64 ? 1 : 2; }

// forward pass of one half: y_s = S^-1 t_s, t_s = g_s - E y_{s-1}.  Every
// memory operation of the step loop is issued by every lane, from a valid
// address or one past the resource's range (no traffic), and the loop has no
// branch around one: the wait for a load issued some steps ahead then counts
// exactly the operations issued after it.
template <typename T, int LR, int INM, bool SPL, int KW>
__global__ __launch_bounds__(4 * LR * KW) ASP_PLAIN_ACC(solve_waves<T, LR>()) void solve2d_fwd_kernel(SolveArgs a) {
    static_assert(!SPL || std::is_same<T, float>::value, "the split products take FP32 operands");
    using Tile = BlockTile<T, LR, SPL, KW>;
    constexpr int NW = Tile::NW, KS = Tile::KS, NX = Tile::NX, NS = nslot<T, LR, INM>();
    constexpr bool TB_LDS = NW > 1 && KW == 1;
    constexpr int GO = KW > 1 ? 0 : 1;   // a slot's data: of the step's block or of the next one
    __shared__ cplx<T> tb[TB_LDS ? 2 : 1][TB_LDS ? LR : 1][Tile::TBS];
    __shared__ cplx<T> part[2][KW > 1 ? KW * LR * 16 : 1];   // KW > 1: shares of the products
    const int nchunk = (a.nact + RC - 1) / RC;
    const SolveItem it(a.njobs, nchunk);
    if (!it.ok) return;
    const SubDesc d = a.desc[a.jobs[it.jl]];
    const int n = a.n, L = d.L;
    const Half H(n, it.dir);
    if (H.np == 0) return;
    Tile M;
    M.init(d, reinterpret_cast<const cplx<T>*>(a.fac) + d.fac_off);
    const int li = M.li;
    const zd* tab = a.subtab + d.tab_off;
    const int grow = (d.kind == ASP_SUB_R) ? 0 : L - 1;          // row carrying boundary data
    const zd coupl = (d.kind == ASP_SUB_R) ? tab[0] : tab[L];    // s at lo-1/2 or hi+1/2
    // forward results through a buffer resource: rows past L are dropped
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<cplx<T>*>(a.y) + ((long long)it.jl * nchunk + it.ch) * n * LR * RC, 0, 0x7fffffff,
        BUF_DW3);
    constexpr unsigned ystep = LR * RC * sizeof(cplx<T>);
    unsigned yoff[NX];
    cplx<T> sinv2[NX];
    // step data: the rows of X (IN_GRID), or the boundary data on the carrying
    // row (IN_BOUNDARY, one entry per lane at most); rows without data and lanes
    // past the right-hand sides lie past the resource's range and read zero
    const bool valid = it.ch * RC + li < a.nact;
    constexpr int NG = INM == IN_GRID ? NX : 1;
    using TG = std::conditional_t<INM == IN_GRID, T, double>;
    const long long line_len = (long long)n * a.nact;
    const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(
        INM == IN_GRID ? static_cast<void*>(const_cast<cplx<T>*>(static_cast<const cplx<T>*>(a.r)) +
                                            (d.xs - 1) * line_len + it.ch * RC)
                       : static_cast<void*>(const_cast<zd*>(a.W) + d.wrow * line_len + it.ch * RC),
        0, 0x7fffffff, BUF_DW3);
    const unsigned gstep = (unsigned)(a.nact * sizeof(cplx<TG>));
    unsigned goff[NG];
    bool use[NX];
    if (INM != IN_GRID) goff[0] = BUF_OOB;
#pragma unroll
    for (int v = 0; v < NX; ++v) {
        const int row = M.xrow(v);
        const int line = d.lo + row;
        const bool rowv = row < L;
        yoff[v] = rowv && (KW == 1 || M.rt == 0) ? (unsigned)((row * RC + li) * sizeof(cplx<T>)) : BUF_OOB;
        sinv2[v] = rowv ? ccast<T>(tab[L + 1 + row]) : mk<T>(0, 0);
        if (INM == IN_GRID) {
            use[v] = rowv && line >= d.xs && line <= d.xe;
            goff[v % NG] = use[v] && valid ? (unsigned)(((line - d.xs) * line_len + li) * sizeof(cplx<TG>)) : BUF_OOB;
        } else {
            use[v] = rowv && row == grow;
            if (use[v] && valid) goff[0] = (unsigned)(li * sizeof(cplx<TG>));
        }
    }
    struct Slot {
        cplx<T> f[KS];   // operand of step s
        cplx<TG> g[NG];  // data of step s + 1
        zd sh, ism;      // s1 between blocks s and s + 1; 1 / (s1 h^2) at block s + 1
    };
    // data of block s + GO (the middle block past the last step: unused)
    auto fetch = [&](Slot& S, int s) {
        const int sc = min(s, H.np);
        M.load(S.f, H.blk(sc));
        const int k = H.blk(sc + GO);
#pragma unroll
        for (int e = 0; e < NG; ++e) S.g[e] = buf_load<TG>(rg, goff[e], (unsigned)(k - 1) * gstep);
    };
    auto fetch_coef = [&](Slot& S, int s) {
        const int sc = min(s, H.np);
        S.sh = uniform_load(a.ax.sh + H.half_line(sc - 1 + GO));
        if (INM != IN_GRID) S.ism = uniform_load(a.ax.inv_sh2 + H.blk(sc + GO) - 1);
    };
    cplx<T> u[NX];
    auto input = [&](const cplx<TG> (&g)[NG], zd ism, cplx<T> shc, const cplx<T> (&y)[NX], int buf) {
        cplx<T> gb;
        if constexpr (INM != IN_GRID) gb = ccast<T>(ccast<double>(g[0]) * -(coupl * ism));
#pragma unroll
        for (int v = 0; v < NX; ++v) {
            cplx<T> t;
            if constexpr (INM == IN_GRID)
                t = ccast<T>(g[v % NG]);
            else
                t = csel(use[v], gb, mk<T>(T(0), T(0)));
            u[v] = t - (shc * sinv2[v]) * y[v];
            if constexpr (TB_LDS) tb[buf][16 * M.rt + Mfma<T>::row(M.l, v)][li] = u[v];
        }
    };
    Slot sl[NS];
    {
        cplx<TG> g0[NG];
        const int k = H.blk(1);
#pragma unroll
        for (int e = 0; e < NG; ++e) g0[e] = buf_load<TG>(rg, goff[e], (unsigned)(k - 1) * gstep);
        const zd ism0 = a.ax.inv_sh2[k - 1];
#pragma unroll
        for (int q = 0; q < NS - 1; ++q) {
            fetch(sl[q], 1 + q);
            fetch_coef(sl[q], 1 + q);
        }
        cplx<T> y0[NX];
#pragma unroll
        for (int e = 0; e < NX; ++e) y0[e] = mk<T>(T(0), T(0));
        if constexpr (KW > 1) M.put_sum(part[1], y0);
        else input(g0, ism0, mk<T>(T(0), T(0)), y0, 1);
    }
    // nothing outstanding on entry: the waits in the loop count its own operations
    __builtin_amdgcn_s_waitcnt(0);
    cplx<T> y[NX];
#pragma unroll
    for (int v = 0; v < NX; ++v) y[v] = mk<T>(T(0), T(0));
    auto store = [&](int s) {
        const unsigned ys = (unsigned)(H.blk(max(s, 1)) - 1) * ystep;
#pragma unroll
        for (int v = 0; v < NX; ++v) buf_store(ry, yoff[v], ys, y[v]);
    };
    // F: the slot of step s - 1, free to take the loads of step s + NS - 1.  The
    // step's memory operations (those loads, the previous step's results; before
    // the first step zeros that its results overwrite) follow the reads of the
    // step vectors: they issue in the latency of those and under the products,
    // not between a step's result and the next barrier.
    auto step = [&](int s, Slot& S, Slot& F, auto pre) {
        if constexpr (NW > 1 || KW > 1) step_sync();
        cplx<T> b[KS];
        if constexpr (KW > 1) {
            M.gather(part[s & 1], y);
            input(S.g, S.ism, ccast<T>(S.sh), y, 0);
        }
        M.vectors(b, u, tb[TB_LDS ? s & 1 : 0]);
        __builtin_amdgcn_sched_barrier(0);
        store(s - 1);
        if constexpr (decltype(pre)::value) fetch(F, s + NS - 1);
        if constexpr (TB_LDS) __builtin_amdgcn_sched_barrier(0);
        const CTile<T> acc = M.product(S.f, b);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(pre)::value) fetch_coef(F, s + NS - 1);
        if constexpr (KW > 1) {
            M.put(part[(s + 1) & 1], acc);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) y[v] = mk<T>(acc.re[v], acc.im[v]);
            input(S.g, S.ism, ccast<T>(S.sh), y, (s + 1) & 1);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int s = 1;
    for (; s + NS - 1 <= H.np; s += NS)
#pragma unroll
        for (int q = 0; q < NS; ++q) step(s + q, sl[q], sl[(q + NS - 1) % NS], std::true_type{});
#pragma unroll
    for (int q = 0; q < NS - 1; ++q)
        if (s + q <= H.np) step(s + q, sl[q], sl[q], std::false_type{});
    if constexpr (KW > 1) {
        step_sync();
        M.gather(part[(H.np + 1) & 1], y);
    }
    store(H.np);
}

// backward pass of one half: the middle block, then x_s = y_s - S^-1 E x_{s+1}
// outwards; outputs on the lines of X.  IN_TWIST (the boundary maps): chains
// towards the end of the half that start from columns of the diagonal blocks
// of H^-1 (kind 0) or from the unit vectors at the middle block (kind 2).
template <typename T, int LR, int INM, bool SPL, int KW>
__global__ __launch_bounds__(4 * LR * KW) ASP_PLAIN_ACC(solve_waves<T, LR>()) void solve2d_bwd_kernel(SolveArgs a) {
    static_assert(!SPL || std::is_same<T, float>::value, "the split products take FP32 operands");
    using Tile = BlockTile<T, LR, SPL, KW>;
    constexpr int NW = Tile::NW, KS = Tile::KS, NX = Tile::NX, NS = nslot<T, LR, INM>();
    constexpr bool TB_LDS = NW > 1 && KW == 1;
    constexpr int YO = KW > 1 ? 1 : 0;   // a slot's y: of the step's block or of the one before
    constexpr bool TW = INM == IN_TWIST;
    __shared__ cplx<T> tb[TB_LDS ? 2 : 1][TB_LDS ? LR : 1][Tile::TBS];
    __shared__ cplx<T> part[2][KW > 1 ? KW * LR * 16 : 1];
    const int n = a.n, p = mid_block(n);
    int jl, ch, dir, nchunk;
    bool below = false;   // IN_TWIST kind 0: the triangle away from the diagonal's chains
    if constexpr (TW) {
        // kind 0: chunk ch of a half starts at step min(16 (ch + 1), columns); the
        // longest chains of every problem first, in dispatch order
        const int w = (int)blockIdx.x;
        if (a.twist_kind == 0) {
            nchunk = (p + RC - 1) / RC;
            if (w >= a.njobs * nchunk * 4) return;
            ch = nchunk - 1 - w / (4 * a.njobs);
            const int r = w % (4 * a.njobs);
            below = r & 1;
            dir = (r >> 1) & 1;
            jl = r >> 2;
            if (dir && ch * RC >= n - p) return;
        } else {
            nchunk = (a.nact + RC - 1) / RC;
            if (w >= a.njobs * nchunk * 2) return;
            ch = w % nchunk;
            dir = (w / nchunk) & 1;
            jl = w / (2 * nchunk);
        }
    } else {
        nchunk = (a.nact + RC - 1) / RC;
        const SolveItem it(a.njobs, nchunk);
        if (!it.ok) return;
        jl = it.jl;
        ch = it.ch;
        dir = it.dir;
    }
    const SubDesc d = a.desc[a.jobs[jl < a.njobs0 ? jl : a.jobs1 + jl - a.njobs0]];
    const int L = d.L;
    const Half H(n, dir);
    if (!TW && dir && H.np == 0) return;
    Tile M;
    M.init(d, reinterpret_cast<const cplx<T>*>(a.fac) + d.fac_off);
    const int li = M.li;
    const zd* tab = a.subtab + d.tab_off;
    const int slot = ch * RC + li;
    const int grow = (d.kind == ASP_SUB_R) ? 0 : L - 1;
    const int jout = (d.kind == ASP_SUB_R) ? (d.xe - d.lo) : (d.xs - d.lo);   // outgoing line
    const zd coupl = (d.kind == ASP_SUB_R) ? tab[0] : tab[L];
    int row[NX];
    bool rowv[NX];
    cplx<T> sinv2[NX];
#pragma unroll
    for (int v = 0; v < NX; ++v) {
        row[v] = M.xrow(v);
        rowv[v] = row[v] < L;
        sinv2[v] = rowv[v] ? ccast<T>(tab[L + 1 + row[v]]) : mk<T>(0, 0);
    }
    // kind 0: columns (below: rows) of this half, counted from its end, chunk by
    // chunk; the half of block p takes it too.  smax: the chain's first step
    const int ncol = TW && a.twist_kind == 0 ? H.np + (dir ? 0 : 1) : a.nact;
    const bool valid = slot < ncol;
    const int smax = TW && a.twist_kind == 0 ? min((ch + 1) * RC, ncol) : H.np + 1;

    // -- y of a step -----------------------------------------------------------
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(
        TW ? static_cast<void*>(reinterpret_cast<cplx<T>*>(a.Tout) + d.g_off)
           : static_cast<void*>(reinterpret_cast<cplx<T>*>(a.y) +
                                ((long long)jl * nchunk + ch) * n * LR * RC),
        0, 0x7fffffff, BUF_DW3);
    constexpr unsigned ystep = (TW ? 2 * LR : LR * RC) * sizeof(cplx<T>);
    unsigned yoff[NX];
#pragma unroll
    for (int v = 0; v < NX; ++v)
        yoff[v] = !rowv[v] ? BUF_OOB
                  : TW     ? (unsigned)(((below ? LR : 0) + row[v]) * sizeof(cplx<T>))
                           : (unsigned)((row[v] * RC + li) * sizeof(cplx<T>));
    // kind 0: the starting vector of the solution that starts at this lane's
    // block, zero at the others: column grow of G_k times the unit data's
    // coupling, or column jout (below); kind 2 adds nothing after the start
    const cplx<T> cin_s =
        TW && !below ? ccast<T>(-(coupl * a.ax.inv_sh2[H.blk(min(slot, n - 1) + 1) - 1])) : mk<T>(T(1), T(0));
    auto load_y = [&](int s, cplx<T> (&y)[NX]) {
        const int k = H.blk(max(s, 1));
#pragma unroll
        for (int v = 0; v < NX; ++v) y[v] = buf_load<T>(ry, yoff[v], (unsigned)(k - 1) * ystep);
    };
    auto use_y = [&](int s, cplx<T> (&y)[NX]) {
        if constexpr (TW) {
            const bool st = a.twist_kind == 0 && valid && slot == s - 1;
#pragma unroll
            for (int v = 0; v < NX; ++v) y[v] = csel(st, cin_s * y[v], mk<T>(T(0), T(0)));
        }
    };

    // -- outputs ----------------------------------------------------------------
    const bool bufo = a.buf_ok != 0;
    cplx<T>* const Tbase = reinterpret_cast<cplx<T>*>(a.Tout) + (TW ? d.tr_off : 0);
    const long long line_len = (long long)n * a.nact;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        TW ? static_cast<void*>(Tbase)
           : static_cast<void*>(static_cast<cplx<T>*>((d.kind == ASP_SUB_L) ? a.out_L : a.out) +
                                (d.xs - 1) * line_len + ch * RC),
        0, 0x7fffffff, BUF_DW3);
    const unsigned ostep = (unsigned)(a.nact * sizeof(cplx<T>));
    unsigned ooff[NX];
#pragma unroll
    for (int v = 0; v < NX; ++v) {
        const int line = d.lo + row[v];
        const bool inX = valid && rowv[v] && (KW == 1 || M.rt == 0) && line >= d.xs && line <= d.xe;
        ooff[v] = inX ? (unsigned)(((line - d.xs) * line_len + li) * sizeof(cplx<T>)) : BUF_OOB;
    }
    // IN_TWIST: the wavefront and lanes holding the row a map entry is read from
    const int jrow = below ? grow : jout;
    auto mine = [&](int r) {
        if constexpr (KW > 1)
            return M.rt == 0 && (4 * (r >> 4) + (sizeof(T) == 8 ? (r & 15) >> 2 : r & 3)) / KS == M.kq;
        return (r >> 4) == M.rt;
    };
    const bool jmine = TW && mine(jrow), gmine = TW && mine(grow), omine = TW && mine(jout);
    auto pick = [&](const cplx<T> (&x)[NX], int r, bool& hit) {
        cplx<T> y = x[0];
        hit = row[0] == r;
#pragma unroll
        for (int v = 1; v < NX; ++v) {
            y = csel(row[v] == r, x[v], y);
            hit = hit || row[v] == r;
        }
        return y;
    };
    auto emit = [&](int s, const cplx<T> (&x)[NX]) {
        const int k = H.blk(s);
        if constexpr (TW) {
            bool hit;
            if (a.twist_kind == 0) {
                if (!jmine) return;
                // boundary maps in row tiles of 16: entry (row r, column c) at
                // (r / 16) n 16 + 16 c + r % 16
                cplx<T> y = pick(x, jrow, hit);
                const int c = H.blk(slot + 1) - 1;   // this lane's column (below: row)
                const int r_ = below ? c : k - 1, c_ = below ? k - 1 : c;
                if (below) y = ccast<T>(-(coupl * a.ax.inv_sh2[k - 1])) * y;
                const bool kp = hit && valid && (below ? s - 1 < slot : s - 1 <= slot);
                const long long ti = ((long long)(r_ >> 4) * n + c_) * 16 + (r_ & 15);
                if (bufo)
                    buf_store(rs, kp ? (unsigned)(ti * sizeof(cplx<T>)) : BUF_OOB, 0u, y);
                else if (kp)
                    Tbase[ti] = y;
            } else {
                // rows grow and jout of the propagator from the middle block to k
                if (gmine) {
                    const cplx<T> y = pick(x, grow, hit);
                    buf_store(ry, hit && valid ? (unsigned)(((k - 1) * 2 * LR + slot) * sizeof(cplx<T>)) : BUF_OOB, 0u, y);
                }
                if (omine) {
                    const cplx<T> y = pick(x, jout, hit);
                    buf_store(ry, hit && valid ? (unsigned)(((k - 1) * 2 * LR + LR + slot) * sizeof(cplx<T>)) : BUF_OOB, 0u, y);
                }
            }
            return;
        }
        const bool skip = dir && s > H.np;   // the middle block is half 0's
#pragma unroll
        for (int v = 0; v < NX; ++v) buf_store(rs, skip ? BUF_OOB : ooff[v], (unsigned)(k - 1) * ostep, x[v]);
    };

    // -- start --------------------------------------------------------------------
    struct Slot {
        cplx<T> f[KS], y[NX];   // operand and y of step s
        zd sh;                 // s1 between blocks s - 1 and s
    };
    auto fetch = [&](Slot& S, int s) {
        const int sc = max(s, 1);
        M.load(S.f, H.blk(sc));
        load_y(s + YO, S.y);
    };
    auto fetch_coef = [&](Slot& S, int s) { S.sh = uniform_load(a.ax.sh + H.half_line(max(s - 1 + YO, 0))); };
    cplx<T> x[NX], u[NX], y1[NX];
    // E x_{s+1} (sh: s1 between blocks s and s + 1) for step s
    auto coupled = [&](int s, cplx<T> shc) {
#pragma unroll
        for (int v = 0; v < NX; ++v) {
            u[v] = (shc * sinv2[v]) * x[v];
            if constexpr (TB_LDS) tb[s & 1][row[v]][li] = u[v];
        }
    };
    Slot sl[NS];
#pragma unroll
    for (int q = 0; q < NS - 1; ++q) {
        fetch(sl[q], smax - 1 - q);
        fetch_coef(sl[q], smax - 1 - q);
    }
    if constexpr (TW) {
        if (a.twist_kind == 0) {
            load_y(smax, x);
            use_y(smax, x);
        } else {
#pragma unroll
            for (int v = 0; v < NX; ++v) x[v] = mk<T>(row[v] == slot ? T(1) : T(0), T(0));
        }
        if (KW == 1 && (a.twist_kind == 0 || dir == 0)) emit(smax, x);
    } else {
        // x_p = M_p^-1 (g_p - E_{p-1} y_{p-1} - E_p y_{p+1})
        cplx<T> ym[NX], yp[NX], f[KS];
        M.load(f, p);
        const cplx<T> cm = p > 1 ? ccast<T>(a.ax.sh[p - 1]) : mk<T>(T(0), T(0));
        const cplx<T> cp = p < n ? ccast<T>(a.ax.sh[p]) : mk<T>(T(0), T(0));
#pragma unroll
        for (int v = 0; v < NX; ++v) {
            ym[v] = buf_load<T>(ry, p > 1 ? yoff[v] : BUF_OOB, (unsigned)(max(p - 1, 1) - 1) * ystep);
            yp[v] = buf_load<T>(ry, p < n ? yoff[v] : BUF_OOB, (unsigned)(min(p + 1, n) - 1) * ystep);
        }
#pragma unroll
        for (int v = 0; v < NX; ++v) {
            const int line = d.lo + row[v];
            cplx<T> t = mk<T>(T(0), T(0));
            if (INM == IN_GRID && valid && rowv[v] && line >= d.xs && line <= d.xe)
                t = static_cast<const cplx<T>*>(a.r)[(line - 1) * line_len + (long long)(p - 1) * a.nact + slot];
            if (INM == IN_BOUNDARY && valid && rowv[v] && row[v] == grow)
                t = ccast<T>(a.W[d.wrow * line_len + (long long)(p - 1) * a.nact + slot] *
                             -(coupl * a.ax.inv_sh2[p - 1]));
            u[v] = (t - (cm * sinv2[v]) * ym[v]) - (cp * sinv2[v]) * yp[v];
            if constexpr (TB_LDS) tb[smax & 1][row[v]][li] = u[v];
        }
        if constexpr (TB_LDS) step_sync();
        cplx<T> b[KS];
        M.vectors(b, u, tb[TB_LDS ? smax & 1 : 0]);
        const CTile<T> acc = M.product(f, b);
        if constexpr (KW > 1) {
            M.put(part[smax & 1], acc);
            step_sync();
            M.gather(part[smax & 1], x);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) x[v] = mk<T>(acc.re[v], acc.im[v]);
        }
    }
    if constexpr (KW > 1) {
        // the first step takes x_smax as y - (sum of the shares) with y = 0
        load_y(1, y1);
        cplx<T> nx[NX];
#pragma unroll
        for (int e = 0; e < NX; ++e) {
            nx[e] = mk<T>(-x[e].x, -x[e].y);
            sl[0].y[e] = mk<T>(T(0), T(0));
            if (smax == 1) y1[e] = mk<T>(T(0), T(0));
        }
        M.put_sum(part[(smax - 1) & 1], nx);
    } else {
        if (smax > 1) coupled(smax - 1, ccast<T>(a.ax.sh[H.half_line(smax - 1)]));
    }
    __builtin_amdgcn_s_waitcnt(0);
    // the order of the forward pass's step: the loads of step s - NS + 1 and the
    // outputs of step s + 1 under the products (the maps' outputs, entries of one
    // row, stay at the step's end)
    auto step = [&](int s, Slot& S, Slot& F, auto pre) {
        if constexpr (NW > 1 || KW > 1) step_sync();
        cplx<T> b[KS];
        if constexpr (KW > 1) {
            M.gather(part[s & 1], x);
            use_y(s + 1, S.y);
#pragma unroll
            for (int v = 0; v < NX; ++v) x[v] = S.y[v] - x[v];
            coupled(s, ccast<T>(S.sh));
        }
        M.vectors(b, u, tb[TB_LDS ? s & 1 : 0]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!TW) emit(s + 1, x);
        if constexpr (decltype(pre)::value) fetch(F, s - NS + 1);
        if constexpr (TB_LDS) __builtin_amdgcn_sched_barrier(0);
        const CTile<T> acc = M.product(S.f, b);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(pre)::value) fetch_coef(F, s - NS + 1);
        if constexpr (KW > 1) {
            M.put(part[(s + 1) & 1], acc);
            if constexpr (TW)
                if (s + 1 < smax || a.twist_kind == 0 || dir == 0) emit(s + 1, x);
        } else {
            use_y(s, S.y);
#pragma unroll
            for (int v = 0; v < 4; ++v) x[v] = S.y[v] - mk<T>(acc.re[v], acc.im[v]);
            if constexpr (TW) emit(s, x);
            coupled(s - 1, ccast<T>(S.sh));
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int s = smax - 1;
    for (; s - NS + 1 >= 1; s -= NS)
#pragma unroll
        for (int q = 0; q < NS; ++q) step(s - q, sl[q], sl[(q + NS - 1) % NS], std::true_type{});
#pragma unroll
    for (int q = 0; q < NS - 1; ++q)
        if (s - q >= 1) step(s - q, sl[q], sl[q], std::false_type{});
    if constexpr (KW > 1) {
        step_sync();
        M.gather(part[0], x);
        use_y(1, y1);
#pragma unroll
        for (int v = 0; v < NX; ++v) x[v] = y1[v] - x[v];
    }
    if constexpr (!TW)
        emit(1, x);
    else if (KW > 1 && (smax > 1 || a.twist_kind == 0 || dir == 0))
        emit(1, x);
}

// ----------------------------------------------------------------------------
// The two quadrants of a boundary map across the middle block p: for r and c on
// either side of it (or one of them p),
//   T[r][c] = cin_c (row jout of Phi_r) M_p^-1 (row grow of Phi_c)^T,
// Phi_k the propagator from block p to block k (x_k = Phi_k x_p without data in
// between), whose two rows the kind-2 chains left in the column buffer: rank L.
// One wavefront per 16 columns and half of the row tiles it needs; the product
// Z = M_p^-1 (rows grow)^T first, whose result tile is the operand of the next
// product in its own lanes.  FP32 and FP64 products (also with ASP_PREC_BF16X3).
// Bound by the writes of the map entries (n^2 / 2 per problem).
// ----------------------------------------------------------------------------
template <typename T, int LR>
__global__ __launch_bounds__(256) void map_cross_kernel(SolveArgs a) {
    constexpr int JT = LR / 16;
    const int n = a.n, p = mid_block(n);
    const int ntile = (n + 15) / 16;
    const int jl = blockIdx.y;
    const int ctile = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (ctile >= ntile) return;
    const SubDesc d = a.desc[a.jobs[jl < a.njobs0 ? jl : a.jobs1 + jl - a.njobs0]];
    const int L = d.L;
    const int l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
    const zd* tab = a.subtab + d.tab_off;
    const zd coupl = (d.kind == ASP_SUB_R) ? tab[0] : tab[L];
    const cplx<T>* F = reinterpret_cast<const cplx<T>*>(a.fac) + d.fac_off + (long long)(p - 1) * L * LR;
    const cplx<T>* G = reinterpret_cast<const cplx<T>*>(a.Tout) + d.g_off;
    cplx<T>* const Tm = reinterpret_cast<cplx<T>*>(a.Tout) + d.tr_off;
    // Z[j][c], j in the accumulator order of JT tiles
    const int c = 16 * ctile + li, cc = min(c, n - 1);
    CTile<T> Z[JT];
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) Z[jt].zero();
    for (int i0 = 0; i0 < L; i0 += 4) {
        const int i = i0 + lk;
        const cplx<T> b = csel(i < L, G[(long long)cc * 2 * LR + min(i, L - 1)], mk<T>(T(0), T(0)));
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) cmac(Z[jt], F[(long long)min(i, L - 1) * LR + 16 * jt + li], b);
    }
    const cplx<T> cin = ccast<T>(-(coupl * a.ax.inv_sh2[cc]));
#pragma unroll
    for (int jt = 0; jt < JT; ++jt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const cplx<T> z = cin * mk<T>(Z[jt].re[v], Z[jt].im[v]);
            Z[jt].re[v] = z.x;
            Z[jt].im[v] = z.y;
        }
    // row tiles with rows on the other side of some column of this tile
    const bool has_left = 16 * ctile < p, has_right = min(16 * ctile + 15, n - 1) >= p;
    const int t0 = has_right ? 0 : p / 16, t1 = has_left ? ntile : (p + 15) / 16;
    for (int rtile = t0; rtile < t1; ++rtile) {
        const int r = 16 * rtile + li, rc = min(r, n - 1);
        CTile<T> D;
        D.zero();
#pragma unroll
        for (int jt = 0; jt < JT; ++jt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int j = 16 * jt + Mfma<T>::row(l, v);
                const cplx<T> b = csel(j < L, G[(long long)rc * 2 * LR + LR + min(j, L - 1)], mk<T>(T(0), T(0)));
                cmac(D, mk<T>(Z[jt].re[v], Z[jt].im[v]), b);
            }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int cq = 16 * ctile + Mfma<T>::row(l, v);
            if (r < n && cq < n && (r < p) != (cq < p))
                Tm[((long long)rtile * n + cq) * 16 + li] = mk<T>(D.re[v], D.im[v]);
        }
    }
}

// ----------------------------------------------------------------------------
// one step of the two boundary-value sweeps of Algorithm 2, with the
// boundary-to-boundary maps T (column c holds the outgoing line produced by
// unit data at i1 = c + 1):
//   right-going: W^R_{p+1} = T^R_p W^R_p + u~_{p,p} on the last line of X_p
//   left-going:  W^L_{p-1} = T^L_p W^L_p + u~_{p,p} on the first line of X_p
// ----------------------------------------------------------------------------
struct SweepArgs {
    const void* T;
    long long t_off[2];      // map of the problem stepped from (R, L)
    const void* Wt_in[2];    // W transposed: [i1][slot], row stride ws, type of the maps
    void* Wt_out[2];
    zd* W;                   // boundary data of the problems stepped into
    long long w_out[2];
    int line[2];             // line of u~_{p,p} added (last of X_p / first of X_p)
    const void* U;           // u~_{p,p}, right-hand sides fastest
    int nact;                // right-hand sides, slots of U and W
    int ws;                  // slots of Wt (multiple of SW_RT)
    int n;
};


constexpr int SW_ROWS = 16;    // output rows (i1) per block: one matrix-core tile
// One tile of right-hand sides per block while all blocks fit the CUs at once,
// else two (each column of T then serves two); four wavefronts up to 192
// columns, else eight.  A step's products take 2 x 16 x 16 columns of the FP64
// (FP32) matrix cores per batch and wavefront, so an empty or half-filled
// second tile is pure latency: per step at n = 150, 3 right-hand sides, FP64
// 8.7 -> 5.4 us (5.8 with eight wavefronts), n = 511, 8, FP32 8.3 -> 7.1 (8.6
// with four), n = 700, 24, FP64 18.4 -> 12.5; n = 1023, 64 (two tiles) 14.3.
// Four / eight wavefronts, ms of sweep per apply with one right-hand side: FP64
// n = 160 0.172 / 0.191, 192 0.242 / 0.265, 224 0.335 / 0.321, 256 0.391 / 0.376; FP32
// 192 0.183 / 0.196, 224 0.246 / 0.235, 256 0.322 / 0.295 (16 and 64: the same order).
// The number of wavefronts depends on n alone: a right-hand side's sums are the
// same in any batch.
constexpr int SW_ONE_TILE = 256, SW_FEW_COLUMNS = 192;
constexpr int SW_RT = 32;      // the slot count is a multiple of two tiles

// W_out = T W_in for 16 outputs i1 and NT tiles of 16 right-hand sides: a
// complex product on the matrix cores.  Each of NWV wavefronts takes a
// contiguous share of the columns of T in batches of 16 (four k-steps); two batches sit in two fixed
// register slots, and a slot is refilled right after its products, so one
// batch is in flight while the other is multiplied.  Every load is issued
// (columns past the wavefront's range read its last column again) and the
// columns past the range are zeroed where used: a value selected at the load
// makes the compiler wait for that load at once.  The partial tiles meet in
// LDS and are added in wavefront order (fixed, so a result does not depend on
// the other right-hand sides or on scheduling).  The two blocks of a row tile
// are 64 block ids apart and so share an XCD and its L2 copy of T.
template <typename T, bool SPL, int NT, int NWV>
__global__ __launch_bounds__(64 * NWV) ASP_PLAIN_ACC(2) void sweep_step_kernel(SweepArgs a) {
    __shared__ cplx<T> red[NWV][NT][64][4];
    const int side = blockIdx.z;
    const int n = a.n;
    const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int li = l & 15, lk = l >> 4;
    const int k0 = blockIdx.x * SW_ROWS;
    const int s0 = blockIdx.y * 16 * NT;
    if (s0 >= a.nact) return;
    const cplx<T>* __restrict__ Tm = reinterpret_cast<const cplx<T>*>(a.T) + a.t_off[side];
    const cplx<T>* __restrict__ Wi = reinterpret_cast<const cplx<T>*>(a.Wt_in[side]);
    const int ws = a.ws;
    // this block's 16 rows of T: one contiguous run of row-tile blockIdx.x (rows
    // past n are padding, their outputs are not stored)
    const cplx<T>* __restrict__ Tt = Tm + (long long)blockIdx.x * n * 16 + li;
    const int per = (n + 16 * NWV - 1) / (16 * NWV) * 16;
    const int cb = wv * per, ce = min(cb + per, n);
    // OPT outputs per thread (tile t2, lane l2, element v); their u~ values are
    // read now, ahead of the products.  Column li of tile t2 is right-hand side
    // NT li + t2, so that a lane's two right-hand sides of a column of W are
    // adjacent (one 16-byte load in FP32).
    constexpr int OPT = (256 * NT + 64 * NWV - 1) / (64 * NWV);
    struct Out {
        int t2, l2, v, k, slot;
        bool ok;
        cplx<T> u;
    } out[OPT];
#pragma unroll
    for (int o = 0; o < OPT; ++o) {
        Out& q = out[o];
        const int t = threadIdx.x + 64 * NWV * o;
        q.v = t & 3;
        q.l2 = (t >> 2) & 63;
        q.t2 = min(t >> 8, NT - 1);
        q.k = k0 + Mfma<T>::row(q.l2, q.v);
        q.slot = s0 + NT * (q.l2 & 15) + q.t2;
        q.ok = t < 256 * NT && q.k < n && q.slot < a.nact;
        q.u = static_cast<const cplx<T>*>(
            a.U)[((long long)n * (a.line[side] - 1) + (q.ok ? q.k : 0)) * a.nact + (q.ok ? q.slot : 0)];
    }
    // FP32: three real products per complex one (p1 = (ar + ai) br,
    // p2 = ar (bi - br), p3 = ai (br + bi); re = p1 - p3, im = p1 + p2), the
    // matrix-core work of the step down by a quarter; FP64: the four products
    KTile3 kacc[NT];
    CTile<T> acc[NT];
#pragma unroll
    for (int t2 = 0; t2 < NT; ++t2) {
        acc[t2].zero();
        kacc[t2].zero();
    }
    struct Batch {
        cplx<T> av[4], bv[4][NT];
        bool ok[4];
    };
    auto load = [&](Batch& B, int c0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + 4 * u + lk;
            const int cc = min(c, ce - 1);
            B.av[u] = Tt[(long long)cc * 16];
#pragma unroll
            for (int t2 = 0; t2 < NT; ++t2) B.bv[u][t2] = Wi[(long long)cc * ws + s0 + NT * li + t2];
            B.ok[u] = c < ce;
        }
    };
    auto multiply = [&](const Batch& B) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const cplx<T> av = csel(B.ok[u], B.av[u], mk<T>(T(0), T(0)));
#pragma unroll
            for (int t2 = 0; t2 < NT; ++t2) {
                if constexpr (sizeof(T) == 4)
                    kmac3(kacc[t2], av, B.bv[u][t2]);
                else
                    cmac(acc[t2], av, B.bv[u][t2]);
            }
        }
    };
    // SPL: the two batches (32 columns) as the k range of one split product;
    // slot j < 4 of a lane holds batch 0's column 4 j + lk, slot j >= 4 batch 1's
    auto multiply_split = [&](const Batch& B0, const Batch& B1) {
        if constexpr (SPL) {
#pragma unroll
            for (int t2 = 0; t2 < NT; ++t2) {
                float ar[8], ai[8], br[8], bi[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const Batch& B = j < 4 ? B0 : B1;
                    const int u = j & 3;
                    const cplx<T> av = csel(B.ok[u], B.av[u], mk<T>(T(0), T(0)));
                    ar[j] = av.x;
                    ai[j] = av.y;
                    br[j] = B.bv[u][t2].x;
                    bi[j] = B.bv[u][t2].y;
                }
                cmac_split(acc[t2], ar, ai, br, bi);
            }
        }
    };
    Batch b0, b1;
    load(b0, cb);
    load(b1, cb + 16);
    // nothing outstanding on entry: the waits in the loop count its own loads
    __builtin_amdgcn_s_waitcnt(0);
    for (int c0 = cb; c0 < cb + per; c0 += 32) {
        if constexpr (SPL) {
            multiply_split(b0, b1);
            __builtin_amdgcn_sched_barrier(0);
            load(b0, c0 + 32);
            load(b1, c0 + 48);
            __builtin_amdgcn_sched_barrier(0);
        } else {
            multiply(b0);
            __builtin_amdgcn_sched_barrier(0);
            load(b0, c0 + 32);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (NT == 1)
                if (c0 + 16 >= cb + per) break;
            multiply(b1);
            __builtin_amdgcn_sched_barrier(0);
            load(b1, c0 + 48);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (sizeof(T) == 4 && !SPL) {
#pragma unroll
        for (int t2 = 0; t2 < NT; ++t2)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                acc[t2].re[v] = kacc[t2].p1[v] - kacc[t2].p3[v];
                acc[t2].im[v] = kacc[t2].p1[v] + kacc[t2].p2[v];
            }
    }
#pragma unroll
    for (int t2 = 0; t2 < NT; ++t2)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wv][t2][l][v] = mk<T>(acc[t2].re[v], acc[t2].im[v]);
    __syncthreads();
#pragma unroll
    for (int o = 0; o < OPT; ++o) {
        const Out& q = out[o];
        if (!q.ok) continue;
        cplx<T> sum = red[0][q.t2][q.l2][q.v];
#pragma unroll
        for (int w = 1; w < NWV; ++w) sum = sum + red[w][q.t2][q.l2][q.v];
        const zd val = ccast<double>(sum) + ccast<double>(q.u);
        a.W[a.w_out[side] + (long long)q.k * a.nact + q.slot] = val;
        reinterpret_cast<cplx<T>*>(a.Wt_out[side])[(long long)q.k * ws + q.slot] = ccast<T>(val);
    }
}

// W rows of the first sweep step: u~_{1,1} on the last line of X_1 (right-going)
// and u~_{m,m} on the first line of X_m (left-going), plus their copies in the
// factor precision (padding slots zero); one thread per (i1, slot)
template <typename T>
__global__ void sweep_seed_kernel(const cplx<T>* __restrict__ U, zd* __restrict__ W,
                                  long long outR, long long outL, int lineR, int lineL,
                                  cplx<T>* __restrict__ WtR, cplx<T>* __restrict__ WtL, int nact, int ws,
                                  int n) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long long)n * ws) return;
    const int k = (int)(i / ws), slot = (int)(i - (long long)k * ws);
    if (slot >= nact) {
        WtR[i] = mk<T>(0, 0);
        WtL[i] = mk<T>(0, 0);
        return;
    }
    const cplx<T> vR = U[((long long)n * (lineR - 1) + k) * nact + slot];
    const cplx<T> vL = U[((long long)n * (lineL - 1) + k) * nact + slot];
    W[outR + (long long)k * nact + slot] = ccast<double>(vR);
    W[outL + (long long)k * nact + slot] = ccast<double>(vL);
    WtR[i] = vR;
    WtL[i] = vL;
}

// Sequential sweep step: the boundary line R_{t+1} hands to R_{t+2} (its
// output a plus u~ on the last line of its layer) and the one L_{m-t} hands to
// L_{m-t-1} (c plus u~ on the first line of its layer) into their W rows
template <typename T>
__global__ void sweep_hand_kernel(const cplx<T>* __restrict__ A, const cplx<T>* __restrict__ C,
                                  const cplx<T>* __restrict__ U, zd* __restrict__ W, long long rowR,
                                  int lineR, long long rowL, int lineL, int nact, int n) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long len = (long long)n * nact;
    if (i >= len) return;
    const long long gR = len * (lineR - 1) + i, gL = len * (lineL - 1) + i;
    W[rowR + i] = ccast<double>(A[gR]) + ccast<double>(U[gR]);
    W[rowL + i] = ccast<double>(C[gL]) + ccast<double>(U[gL]);
}

// the caller's boundary values (n per right-hand side) into a W row
__global__ void boundary_row_kernel(const zd* __restrict__ w, zd* __restrict__ W, int nact, int n) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long long)n * nact) return;
    const int k = (int)(i / nact), slot = (int)(i - (long long)k * nact);
    W[i] = w[(long long)slot * n + k];
}

// ----------------------------------------------------------------------------
// Between the caller's vectors (right-hand side after right-hand side, i1
// fastest) and the slot-fastest ones of an apply: both sides of the move are
// contiguous runs, the transposition goes through LDS.  A block moves 1024
// entries: nc <= 16 slots of 1024 / nc grid points of one line (nc rounded up
// to a power of two), so that one right-hand side fills its threads too.
// Blocks (points, lines, slots / 16).
// ----------------------------------------------------------------------------
constexpr int MOVE = 1024;
struct MoveArgs {
    const zd* r;           // pack: the caller's vectors
    zd* z;                 // unpack: the caller's vectors
    long long stride;      // entries between the caller's vectors
    int line_off;          // sweep line of the caller's first line, less one
    const int* act;        // the caller's vector of each slot (NULL: id0 + slot)
    int id0, nact, n;
    int pshift;            // 2^pshift grid points per block
    const void *U, *A, *C; // unpack: their sum (A, C on some lines only)
    void* out;             // pack: slot-fastest copy
    int a_from, c_to;      // A on lines >= a_from, C on lines <= c_to
    int line0;             // first sweep line of the launch
};

// the block's tile: points k0 .. k0 + np of nc slots from s0; LDS row stride
// 2^pshift + 4 spreads the slots of a point over the banks
struct MoveTile {
    int k0, line, s0, nc, np, pmask, str;
    __device__ explicit MoveTile(const MoveArgs& a) {
        const int pts = 1 << a.pshift;
        k0 = blockIdx.x << a.pshift;
        line = a.line0 + blockIdx.y;
        s0 = blockIdx.z * 16;
        nc = min(16, a.nact - s0);
        np = min(pts, a.n - k0);
        pmask = pts - 1;
        str = pts + 4;
    }
};
constexpr int MOVE_LDS = MOVE + 4 * 16;

template <typename T>
__global__ __launch_bounds__(256) void pack_kernel(MoveArgs a) {
    __shared__ cplx<T> tile[MOVE_LDS];
    const MoveTile t(a);
    for (int e = threadIdx.x; e < t.nc << a.pshift; e += 256) {
        const int q = e >> a.pshift, k = e & t.pmask;
        if (k >= t.np) continue;
        const int id = a.act ? a.act[t.s0 + q] : a.id0 + t.s0 + q;
        tile[q * t.str + k] =
            ccast<T>(a.r[id * a.stride + (long long)(t.line - 1 - a.line_off) * a.n + t.k0 + k]);
    }
    __syncthreads();
    cplx<T>* out = static_cast<cplx<T>*>(a.out) + ((long long)(t.line - 1) * a.n + t.k0) * a.nact + t.s0;
    for (int e = threadIdx.x; e < t.nc * t.np; e += 256) {
        const int k = e / t.nc, q = e - k * t.nc;
        out[(long long)k * a.nact + q] = tile[q * t.str + k];
    }
}

// z = U + C on the lines before a_from, A + C + U between, A + U after c_to
template <typename T>
__global__ __launch_bounds__(256) void unpack_kernel(MoveArgs a) {
    __shared__ zd tile[MOVE_LDS];
    const MoveTile t(a);
    const bool ha = a.A && t.line >= a.a_from, hc = a.C && t.line <= a.c_to;
    const long long base = ((long long)(t.line - 1) * a.n + t.k0) * a.nact + t.s0;
    for (int e = threadIdx.x; e < t.nc * t.np; e += 256) {
        const int k = e / t.nc, q = e - k * t.nc;
        const long long g = base + (long long)k * a.nact + q;
        const zd u = ccast<double>(static_cast<const cplx<T>*>(a.U)[g]);
        zd v = u;
        if (ha && hc)
            v = (ccast<double>(static_cast<const cplx<T>*>(a.A)[g]) +
                 ccast<double>(static_cast<const cplx<T>*>(a.C)[g])) + u;
        else if (ha || hc)
            v = ccast<double>(static_cast<const cplx<T>*>(ha ? a.A : a.C)[g]) + u;
        tile[q * t.str + k] = v;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < t.nc << a.pshift; e += 256) {
        const int q = e >> a.pshift, k = e & t.pmask;
        if (k >= t.np) continue;
        const int id = a.act ? a.act[t.s0 + q] : a.id0 + t.s0 + q;
        a.z[id * a.stride + (long long)(t.line - 1 - a.line_off) * a.n + t.k0 + k] = tile[q * t.str + k];
    }
}

}  // namespace

hipError_t launch_sweep_hand(const asp_plan* P, const Apply2& v, int rowR, int lineR, int rowL, int lineL,
                             hipStream_t st) {
    const long long len = (long long)P->n * v.nact;
    const dim3 grid((unsigned)((len + 255) / 256));
    if (P->prec != ASP_PREC_FP64)
        hipLaunchKernelGGL(sweep_hand_kernel<float>, grid, dim3(256), 0, st, (const zf*)v.A, (const zf*)v.C,
                           (const zf*)v.U, v.W, rowR * len, lineR, rowL * len, lineL, v.nact, P->n);
    else
        hipLaunchKernelGGL(sweep_hand_kernel<double>, grid, dim3(256), 0, st, (const zd*)v.A, (const zd*)v.C,
                           (const zd*)v.U, v.W, rowR * len, lineR, rowL * len, lineL, v.nact, P->n);
    return hipGetLastError();
}

hipError_t launch_boundary2d(const asp_plan* P, const Apply2& v, const zd* w, int row, hipStream_t st) {
    const long long len = (long long)P->n * v.nact;
    hipLaunchKernelGGL(boundary_row_kernel, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, st, w,
                       v.W + row * len, v.nact, P->n);
    return hipGetLastError();
}

// log2 of the grid points a move block takes: 1024 entries over up to 16 slots
static int move_shift(int nact) {
    int s = 6;
    for (int c = std::min(nact, 16); c <= 8 && s < 10; c *= 2) ++s;
    return s;
}

hipError_t launch_pack2d(const asp_plan* P, const Apply2& v, const zd* r, long long stride, int line0, int line1,
                         int line_off, const int* act, int id0, hipStream_t st) {
    MoveArgs a{};
    a.r = r;
    a.stride = stride;
    a.line_off = line_off;
    a.act = act;
    a.id0 = id0;
    a.nact = v.nact;
    a.n = P->n;
    a.pshift = move_shift(v.nact);
    a.out = v.R;
    a.line0 = line0;
    const dim3 grid((P->n + (1 << a.pshift) - 1) >> a.pshift, line1 - line0 + 1, (v.nact + 15) / 16);
    if (P->prec != ASP_PREC_FP64) hipLaunchKernelGGL(pack_kernel<float>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(pack_kernel<double>, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_unpack2d(const asp_plan* P, const Apply2& v, const void* U, const void* A, const void* C,
                           int a_from, int c_to, zd* z, long long stride, int line0, int line1, int line_off,
                           const int* act, int id0, hipStream_t st) {
    MoveArgs a{};
    a.z = z;
    a.stride = stride;
    a.line_off = line_off;
    a.act = act;
    a.id0 = id0;
    a.nact = v.nact;
    a.n = P->n;
    a.pshift = move_shift(v.nact);
    a.U = U;
    a.A = A;
    a.C = C;
    a.a_from = a_from;
    a.c_to = c_to;
    a.line0 = line0;
    const dim3 grid((P->n + (1 << a.pshift) - 1) >> a.pshift, line1 - line0 + 1, (v.nact + 15) / 16);
    if (P->prec != ASP_PREC_FP64) hipLaunchKernelGGL(unpack_kernel<float>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(unpack_kernel<double>, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_factor2d(const asp_plan* P, hipStream_t st) {
    AxisTables ax{P->d_axis, P->d_axis + (P->n + 1), P->d_axis + (2 * P->n + 1)};
    const int LX = std::max(P->LR_M, P->LR_RL);
    auto cls = [&](int first, int count, int LR) {
        FactorClass c{first, count, LR, 0, 0};
        for (int s = first; s < first + count; ++s) c.npair = std::max(c.npair, (P->subs[s].L + 1) / 2);
        c.blocks = (count + LX / LR - 1) / (LX / LR);
        return c;
    };
    const FactorClass cm = cls(0, P->m, P->LR_M);
    const FactorClass cr = cls(P->m, (int)P->subs.size() - P->m, P->LR_RL);
    auto go = [&](auto* k, auto* fac) {
        hipLaunchKernelGGL(k, dim3(cm.blocks + cr.blocks), dim3(8 * LX), 0, st, P->d_desc, cm, cr, ax,
                           P->d_subtab, P->d_ksq, P->n, fac, P->d_flag);
    };
    if (P->prec != ASP_PREC_FP64) {
        zf* f = reinterpret_cast<zf*>(P->d_fac);
        if (LX == 16) go(factor2d_kernel<float, 16>, f);
        else if (LX == 32) go(factor2d_kernel<float, 32>, f);
        else go(factor2d_kernel<float, 64>, f);
    } else {
        zd* f = reinterpret_cast<zd*>(P->d_fac);
        if (LX == 16) go(factor2d_kernel<double, 16>, f);
        else if (LX == 32) go(factor2d_kernel<double, 32>, f);
        else go(factor2d_kernel<double, 64>, f);
    }
    return hipGetLastError();
}

template <typename TS>
static hipError_t launch_rgf_t(const asp_plan* P, const int* jobs0, const int* jobs1, int nlists,
                               int njobs, hipStream_t st) {
    AxisTables ax{P->d_axis, P->d_axis + (P->n + 1), P->d_axis + (2 * P->n + 1)};
    const cplx<TS>* fac = reinterpret_cast<const cplx<TS>*>(P->d_fac);
    cplx<TS>* tb = reinterpret_cast<cplx<TS>*>(P->d_T);
    const dim3 grid(njobs, nlists, 2);
    if (P->LR_RL == 16)
        hipLaunchKernelGGL((rgf2d_kernel<TS, 16>), grid, dim3(FB), 0, st, P->d_desc, jobs0, jobs1, ax,
                           P->d_subtab, P->n, fac, tb);
    else if (P->LR_RL == 32)
        hipLaunchKernelGGL((rgf2d_kernel<TS, 32>), grid, dim3(FB), 0, st, P->d_desc, jobs0, jobs1, ax,
                           P->d_subtab, P->n, fac, tb);
    else
        hipLaunchKernelGGL((rgf2d_kernel<TS, 64>), grid, dim3(FB), 0, st, P->d_desc, jobs0, jobs1, ax,
                           P->d_subtab, P->n, fac, tb);
    return hipGetLastError();
}

hipError_t launch_rgf2d(const asp_plan* P, int job0, int job1, int njobs, hipStream_t st) {
    if (njobs <= 0) return hipSuccess;
    const int* j0 = P->d_jobs + job0;
    const int* j1 = job1 >= 0 ? P->d_jobs + job1 : j0;
    const int nl = job1 >= 0 ? 2 : 1;
    if (P->prec != ASP_PREC_FP64) return launch_rgf_t<float>(P, j0, j1, nl, njobs, st);
    return launch_rgf_t<double>(P, j0, j1, nl, njobs, st);
}

static int map_chunks(int n) { return (mid_block(n) + RC - 1) / RC; }   // of a half's columns

// one kernel per (precision, row count, input mode): the M-solves, the R/L
// solves and the map chains are separate kernels
template <typename T, int LR, int INM, bool SPL, int KW>
static hipError_t launch_solve_t(const SolveArgs& a, int nchunk, hipStream_t st) {
    if (INM == IN_TWIST) {
        const unsigned blocks = a.twist_kind == 0 ? 4u * a.njobs * map_chunks(a.n) : 2u * a.njobs * nchunk;
        hipLaunchKernelGGL((solve2d_bwd_kernel<T, LR, INM, SPL, KW>), dim3(blocks), dim3(4 * LR * KW), 0, st, a);
        return hipGetLastError();
    }
    constexpr int FWD = INM == IN_TWIST ? IN_GRID : INM;   // map chains have no forward pass
    const unsigned blocks = (2u * a.njobs * nchunk + 7) / 8 * 8;
    hipLaunchKernelGGL((solve2d_fwd_kernel<T, LR, FWD, SPL, KW>), dim3(blocks), dim3(4 * LR * KW), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((solve2d_bwd_kernel<T, LR, INM, SPL, KW>), dim3(blocks), dim3(4 * LR * KW), 0, st, a);
    return hipGetLastError();
}

// Wavefronts per 16-row tile of a launch: several shorten the chain of products of
// a block step (FP64: 64 cycles each) but repeat the loads of its data.  A rule on
// the plan alone, so that a result does not depend on the batch.  (ms per apply with
// one / two / four wavefronts; layers of 4 lines and gamma = 12 unless stated.)
//
// M, R and L, FP32, 16 and 32 rows: four while the tiles of the launch's problems,
// two halves each and one chunk of right-hand sides, leave half of the SIMDs idle;
// past that one, the step being bound by its memory instructions.  64 (8)
// right-hand sides:
//   M, 32 rows      n = 511 (492 tiles)   0.99 / 1.19 / 1.13  (0.48 / 0.40 / 0.34)
//                   n = 640 (620)         1.57 / 1.81 / 1.78  (0.78 / 0.72 / 0.69)
//                   n = 1023 (1004)       3.89 / 4.51 / 4.51  (1.26 / 1.28 / 1.25)
//   R and L, 16     n = 511 (488)         0.67 / 0.67 / 0.72  (0.27 / 0.27 / 0.24)
//                   n = 640 (616)         1.05 / 1.05 / 1.12  (0.35 / 0.36 / 0.36)
//                   n = 1023 (1000)       2.58 / 2.74 / 2.82  (0.87 / 0.83 / 0.86)
//   sequential sweep (two problems per launch at any size), n = 300, layers of one
//   line, 40 right-hand sides: 42.5 / 34.3 / 30.3
// FP32, 64 rows: one, the four tiles already sharing a step (M, 16 and 64 right-hand
// sides: n = 180, gamma = 20 0.32 / 0.40 and 0.56 / 0.82; n = 400, gamma = 24, b = 1
// 2.19 / 2.93 and 7.65 / 11.0).
// FP64: four (64 rows: two; four would be sixteen wavefronts and 128 KB of shares).
// More are faster with few right-hand sides and slower with many at every size past
// 512 tiles (M, one / four: n = 255 0.35 / 0.26 with 16 right-hand sides; n = 700
// 1.51 / 1.30 with 4, 1.79 / 1.87 with 24; n = 1023 2.25 / 2.01 with one, 3.64 / 3.74
// with 24, 6.27 / 7.53 with 64; R and L within 4%; 64 rows, n = 600, gamma = 20, b = 8,
// one / two: 1.62 / 1.53 with 16, 4.89 / 4.58 with 64).
//
// Map chains, which come four per problem and 16 columns of a half: two while their
// products of 16 x 16 tiles per step are few, else one; one for 64 rows.  ms per
// factorization with one / two:
//   FP32  n = 255 (3648) 0.48 / 0.44, 300 (5440) 0.67 / 0.67, 511 with b = 8 and
//         gamma = 9 (7680) 1.10 / 1.06, 383 (8544) 0.98 / 0.98, 511 (15488) 1.67 / 1.74,
//         1023 11.2 / 11.7; 32 rows: n = 250, gamma = 20, b = 8 (6400) 1.51 / 1.48,
//         n = 300, gamma = 17, b = 3 (28160) 2.32 / 2.55
//   FP64  n = 120 (736) 0.25 / 0.23, 255 (3648) 0.62 / 0.61, 300 (5440) 0.90 / 0.94,
//         1023 19.3 / 20.5; 32 rows: n = 200, gamma = 20, b = 8 (4256) 1.36 / 1.34,
//         n = 300, gamma = 5, b = 14 (6080) 1.51 / 1.64
//   64 rows, n = 300, gamma = 13, b = 24: FP32 8.8 / 9.1, FP64 9.1 / 9.2
//
// The bf16-split products run over 32 columns at once: one wavefront.
constexpr int SOLVE_SPLIT_WAVES = 512;
constexpr int MAP_SPLIT_PRODUCTS = 8192;   // FP64: half, its products taking twice as long

int solve_wavefronts(const asp_plan* P, int in_mode) {
    if (P->prec == ASP_PREC_BF16X3) return 1;
    const bool f64 = P->prec == ASP_PREC_FP64;
    const int LR = in_mode == IN_GRID ? P->LR_M : P->LR_RL, tiles = LR / 16;
    if (in_mode == IN_TWIST) {
        const long long products = 4LL * (2 * P->m - 4) * map_chunks(P->n) * tiles * tiles;
        return LR < 64 && products <= (f64 ? MAP_SPLIT_PRODUCTS / 2 : MAP_SPLIT_PRODUCTS) ? 2 : 1;
    }
    if (f64) return LR == 64 ? 2 : 4;
    const long long problems = in_mode == IN_GRID ? P->m : P->sweep_seq ? 2 : 2 * P->m - 2;
    return LR < 64 && 2 * problems * tiles <= SOLVE_SPLIT_WAVES ? 4 : 1;
}

template <int LR, int INM>
static hipError_t launch_solve_lr(const asp_plan* P, const SolveArgs& a, int nchunk, hipStream_t st) {
    if (P->prec == ASP_PREC_BF16X3) return launch_solve_t<float, LR, INM, true, 1>(a, nchunk, st);
    const bool f64 = P->prec == ASP_PREC_FP64, one = solve_wavefronts(P, INM) == 1;
    if constexpr (INM == IN_TWIST) {
        if constexpr (LR < 64)
            if (!one)
                return f64 ? launch_solve_t<double, LR, INM, false, 2>(a, nchunk, st)
                           : launch_solve_t<float, LR, INM, false, 2>(a, nchunk, st);
        return f64 ? launch_solve_t<double, LR, INM, false, 1>(a, nchunk, st)
                   : launch_solve_t<float, LR, INM, false, 1>(a, nchunk, st);
    } else {
        if (f64) return launch_solve_t<double, LR, INM, false, LR == 64 ? 2 : 4>(a, nchunk, st);
        if constexpr (LR < 64)
            if (!one) return launch_solve_t<float, LR, INM, false, 4>(a, nchunk, st);
        return launch_solve_t<float, LR, INM, false, 1>(a, nchunk, st);
    }
}

template <int LR>
static hipError_t launch_solve_mode(const asp_plan* P, const SolveArgs& a, int in_mode, int nchunk,
                                    hipStream_t st) {
    if (in_mode == IN_GRID) return launch_solve_lr<LR, IN_GRID>(P, a, nchunk, st);
    if (in_mode == IN_BOUNDARY) return launch_solve_lr<LR, IN_BOUNDARY>(P, a, nchunk, st);
    if (in_mode == IN_TWIST) return launch_solve_lr<LR, IN_TWIST>(P, a, nchunk, st);
    return hipErrorInvalidValue;
}

template <typename T>
static hipError_t launch_cross_t(int LR, const SolveArgs& a, hipStream_t st) {
    const dim3 grid(((a.n + 15) / 16 + 3) / 4, a.njobs);
    if (LR == 16) hipLaunchKernelGGL((map_cross_kernel<T, 16>), grid, dim3(256), 0, st, a);
    else if (LR == 32) hipLaunchKernelGGL((map_cross_kernel<T, 32>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((map_cross_kernel<T, 64>), grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

// forward results: n blocks of LR rows x 16 right-hand sides per problem and chunk
long long solve_scratch_elems(const asp_plan* P, int nrhs) {
    const long long m = P->m, mr = std::max(m * P->LR_M, (2 * m - 2) * P->LR_RL);
    return mr * ((nrhs + RC - 1) / RC * RC) * P->n;
}

static SolveArgs solve_args(const asp_plan* P, const SolveLaunch& L) {
    SolveArgs a;
    a.desc = P->d_desc;
    a.jobs = P->d_jobs + L.job0;
    a.njobs = L.njobs;
    a.njobs0 = L.njobs0 ? L.njobs0 : L.njobs;
    a.jobs1 = L.job1 - L.job0;
    a.nact = L.nact;
    a.fac = P->d_fac;
    a.ax = AxisTables{P->d_axis, P->d_axis + (P->n + 1), P->d_axis + (2 * P->n + 1)};
    a.subtab = P->d_subtab;
    a.r = L.r;
    a.W = L.W;
    a.out = L.out;
    a.out_L = L.out_L ? L.out_L : L.out;
    a.Tout = P->d_T;
    a.y = P->d_y;
    const size_t esz = P->prec != ASP_PREC_FP64 ? sizeof(zf) : sizeof(zd);
    a.buf_ok = (long long)((P->n + 15) / 16 * 16) * P->n * (long long)esz < (1LL << 31) ? 1 : 0;
    a.twist_kind = L.twist_kind;
    a.n = P->n;
    return a;
}

// the most right-hand sides of one apply pass: a problem's lines of X (and a
// boundary row, in double) within the 31-bit range of a buffer resource
int apply_max_rhs(const asp_plan* P) {
    long long lines = 1;
    for (const auto& x : P->X) lines = std::max(lines, (long long)x[1] - x[0] + 1);
    const long long s = ((1LL << 31) - 1) / (lines * P->n * (long long)sizeof(zd));
    return (int)std::min<long long>(std::max<long long>(s, 1), 4096);
}

// problems per launch for which the forward-result scratch has room (all of
// them, but for a workspace of a fixed size that is nearly too small)
static long long solve_room(const asp_plan* P, const SolveLaunch& L) {
    const long long nchunk = (L.nact + RC - 1) / RC;
    return P->y_elems / (nchunk * P->n * (L.rl ? P->LR_RL : P->LR_M) * RC);
}

int solve_launches(const asp_plan* P, const SolveLaunch& L) {
    const long long room = std::max(solve_room(P, L), 1LL);
    return 2 * (int)((L.njobs + room - 1) / room);
}

hipError_t launch_solve2d(const asp_plan* P, const SolveLaunch& L, hipStream_t st) {
    if (L.njobs <= 0 || L.nact <= 0) return hipSuccess;
    const int LR = L.rl ? P->LR_RL : P->LR_M;   // every job of one launch shares its row count
    const int nchunk = (L.nact + RC - 1) / RC;
    SolveLaunch part = L;
    if (L.in_mode != IN_TWIST) {
        const long long room = solve_room(P, L);
        if (room < 1 || L.nact > apply_max_rhs(P)) return hipErrorInvalidValue;
        part.njobs = (int)std::min<long long>(L.njobs, room);
    }
    for (int j = 0; j < L.njobs; j += part.njobs) {
        part.job0 = L.job0 + j;
        part.njobs = std::min(part.njobs, L.njobs - j);
        const SolveArgs a = solve_args(P, part);
        const hipError_t e = LR == 16 ? launch_solve_mode<16>(P, a, L.in_mode, nchunk, st)
                             : LR == 32 ? launch_solve_mode<32>(P, a, L.in_mode, nchunk, st)
                                        : launch_solve_mode<64>(P, a, L.in_mode, nchunk, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_map_cross(const asp_plan* P, const SolveLaunch& L, hipStream_t st) {
    if (L.njobs <= 0) return hipSuccess;
    const SolveArgs a = solve_args(P, L);
    if (P->prec != ASP_PREC_FP64) return launch_cross_t<float>(P->LR_RL, a, st);
    return launch_cross_t<double>(P->LR_RL, a, st);
}

static int sweep_slots(int nact) { return (nact + SW_RT - 1) / SW_RT * SW_RT; }

long long sweep_wt_line(const asp_plan* P, int nact) { return (long long)P->n * sweep_slots(nact); }

int sweep_wt_len(const asp_plan* P, int nrhs) { return 4 * P->n * sweep_slots(nrhs); }

// transposed sweep buffers: [side][ping-pong][n][ws]
static void* wt_buf(const asp_plan* P, int side, int pp, int ws) {
    const size_t esz = P->prec != ASP_PREC_FP64 ? sizeof(zf) : sizeof(zd);
    return static_cast<char*>(P->d_wt) + ((size_t)(side * 2 + pp) * P->n * ws) * esz;
}

hipError_t launch_sweep_seed(const asp_plan* P, const Apply2& v, int rowR, int rowL, hipStream_t st) {
    if (v.nact <= 0) return hipSuccess;
    const int lineR = P->X[0][1];
    const int lineL = P->X[P->m - 1][0];
    const int ws = sweep_slots(v.nact);
    if ((long long)4 * P->n * ws > P->wt_elems) return hipErrorInvalidValue;
    const long long len = (long long)P->n * v.nact;
    const dim3 grid((unsigned)(((long long)P->n * ws + 255) / 256));
    if (P->prec != ASP_PREC_FP64)
        hipLaunchKernelGGL(sweep_seed_kernel<float>, grid, dim3(256), 0, st, (const zf*)v.U, v.W, rowR * len,
                           rowL * len, lineR, lineL, (zf*)wt_buf(P, 0, 0, ws), (zf*)wt_buf(P, 1, 0, ws),
                           v.nact, ws, P->n);
    else
        hipLaunchKernelGGL(sweep_seed_kernel<double>, grid, dim3(256), 0, st, (const zd*)v.U, v.W, rowR * len,
                           rowL * len, lineR, lineL, (zd*)wt_buf(P, 0, 0, ws), (zd*)wt_buf(P, 1, 0, ws),
                           v.nact, ws, P->n);
    return hipGetLastError();
}

template <typename T, bool SPL, int NWV>
static void launch_sweep_w(const SweepArgs& a, hipStream_t st) {
    const int tiles = (a.n + SW_ROWS - 1) / SW_ROWS, ct = (a.nact + 15) / 16;
    if (2 * tiles * ct <= SW_ONE_TILE)
        hipLaunchKernelGGL((sweep_step_kernel<T, SPL, 1, NWV>), dim3(tiles, ct, 2), dim3(64 * NWV), 0, st, a);
    else
        hipLaunchKernelGGL((sweep_step_kernel<T, SPL, 2, NWV>), dim3(tiles, (ct + 1) / 2, 2), dim3(64 * NWV), 0, st, a);
}

template <typename T, bool SPL>
static void launch_sweep_t(const SweepArgs& a, hipStream_t st) {
    if (a.n <= SW_FEW_COLUMNS) launch_sweep_w<T, SPL, 4>(a, st);
    else launch_sweep_w<T, SPL, 8>(a, st);
}

hipError_t launch_sweep_step(const asp_plan* P, const Apply2& v, int t, hipStream_t st) {
    // step t moves the right-going sweep from layer p = t+1 to p+1 and the
    // left-going sweep from layer p' = m-t to p'-1; the transposed inputs of
    // step t are ping-pong buffer (t-1) & 1
    const int m = P->m;
    const int pR = t + 1, pL = m - t;
    const int ws = sweep_slots(v.nact);
    if ((long long)4 * P->n * ws > P->wt_elems) return hipErrorInvalidValue;
    SweepArgs a;
    a.T = P->d_T;
    a.t_off[0] = P->subs[P->idx_R(pR)].tr_off;
    a.t_off[1] = P->subs[P->idx_L(pL)].tr_off;
    for (int side = 0; side < 2; ++side) {
        a.Wt_in[side] = wt_buf(P, side, (t - 1) & 1, ws);
        a.Wt_out[side] = wt_buf(P, side, t & 1, ws);
    }
    a.W = v.W;
    a.w_out[0] = (long long)P->wrow(P->idx_R(pR + 1)) * v.nact * P->n;
    a.w_out[1] = (long long)P->wrow(P->idx_L(pL - 1)) * v.nact * P->n;
    a.line[0] = P->X[pR - 1][1];
    a.line[1] = P->X[pL - 1][0];
    a.U = v.U;
    a.nact = v.nact;
    a.ws = ws;
    a.n = P->n;
    if (P->prec == ASP_PREC_BF16X3) launch_sweep_t<float, true>(a, st);
    else if (P->prec != ASP_PREC_FP64) launch_sweep_t<float, false>(a, st);
    else launch_sweep_t<double, false>(a, st);
    return hipGetLastError();
}
