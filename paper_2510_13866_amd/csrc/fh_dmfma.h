// FP64 circulant on the FP64 matrix cores, shared by the FP64 forward filter, the FP64 adjoint
// and the FP64 re-filter of blocks that leave FP32's range (fh_kernels.hip, fh_mfma.hip).
//
// v_mfma_f64_16x16x4_f64 reads A[i][k] from lane i + 16 k, B[k][j] from lane j + 16 k, and
// leaves D[i][j] in lane j + 16 (i mod 4), register i / 4 (checked on the device). A 32 x 32
// matrix in that accumulator layout is four 16 x 16 tiles (I, J), tile index 2 I + J; element
// (16 I + 4 r + lane / 16, 16 J + lane % 16) sits in register r of tile (I, J). Register r of
// tile (K, I) is then directly the A operand of X^T with K-index 16 K + 4 r + lane / 16, so
//   (X^T C)(I, J) = sum over K, r of mfma(X(K, I)[r], Cb[(4 K + r) * 2 + J])
// with Cb the matching B operands of the circulant C[k][j] = g((k - j) mod L) (zero outside
// L x L): 32 products per multiplication, no operand splitting, every product and sum in FP64.
// Two multiplications give (F^T C)^T C = C F C, C being symmetric.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

namespace fh {

typedef __attribute__((ext_vector_type(4))) double f64x4;

struct Tile64 {
    f64x4 t[4];
};

__device__ inline Tile64 circ64(const Tile64& X, const double (&Cb)[16]) {
    Tile64 Y;
#pragma unroll
    for (int I = 0; I < 2; ++I)
#pragma unroll
        for (int J = 0; J < 2; ++J) {
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int K = 0; K < 2; ++K)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X.t[2 * K + I][r],
                                                               Cb[(4 * K + r) * 2 + J], acc, 0, 0, 0);
            Y.t[2 * I + J] = acc;
        }
    return Y;
}

// A 64-bit lane exchange by DPP (every lane has its source lane under these controls).
template <int CTRL>
__device__ inline double dpp_swap_f64(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, (uint64_t)(uint32_t)lo | ((uint64_t)(uint32_t)hi << 32));
}
__device__ inline double lane_f64(double v, int lane) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
// Sum over the wavefront, the same bits in every lane: each 16-lane row by DPP exchanges (an
// addition and its mirror give the same bits), then the four row sums in one fixed order. No
// LDS round trip (the FP64 recursions wait on this sum every step).
__device__ inline double wave_sum_f64(double v) {
    v += dpp_swap_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v += dpp_swap_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v += dpp_swap_f64<0x141>(v);  // row_half_mirror
    v += dpp_swap_f64<0x140>(v);  // row_mirror
    return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}

// Sum of a lane's sixteen values, in one order for every form of the recursion and four additions
// deep (the normaliser waits on it every step; one after another they take sixteen: a sweep of 3 FP64
// chains of 32 x 32 x 332 with every worldline its own recursion took 4500 us, 4450 this way).
__device__ inline double tile_sum(const Tile64& F) {
#pragma clang fp contract(off)
    double s[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] = (F.t[q][0] + F.t[q][1]) + (F.t[q][2] + F.t[q][3]);
    return (s[0] + s[1]) + (s[2] + s[3]);
}

// Tile coordinates of element (tile q, register r) of a lane: x = 16 (q & 1) + lane % 16,
// y = 16 (q >> 1) + 4 r + lane / 16.
__device__ inline int t64_x(int q, int lane) { return 16 * (q & 1) + (lane & 15); }
__device__ inline int t64_y(int q, int r, int lane) { return 16 * (q >> 1) + 4 * r + (lane >> 4); }

// C F C of a lattice with L <= 16, which fills tile (0, 0) only: every product with another tile
// is an exact zero, so the two multiplications take ceil(L / 4) instructions each instead of 32
// and leave the bits of circ64(circ64(F)). Cb[r]: the B operands Cb[2 r] of the 32 x 32 layout.
__device__ inline f64x4 circ16(const f64x4& F, const double (&Cb)[4], int L) {
    f64x4 X = {0.0, 0.0, 0.0, 0.0}, H = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (4 * r < L) X = __builtin_amdgcn_mfma_f64_16x16x4f64(F[r], Cb[r], X, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (4 * r < L) H = __builtin_amdgcn_mfma_f64_16x16x4f64(X[r], Cb[r], H, 0, 0, 0);
    return H;
}

// dmfma_block_forward_end for L <= 16 (wtab(l, w) fills w[r] at the lane's element (0, r)), with
// the next slice's W~ loaded a step ahead: at 2 ceil(L / 4) products a step the load latency
// would show. A step of a lone 4 x 4 recursion takes 0.6 us (3.0 us on the full tiling, whose
// 64 products bound it).
template <typename WTab, typename Put, typename PutEnd>
__device__ inline double dmfma16_block_forward_end(const double (&Cb)[4], int L, int L_tau,
                                                   int start, int len, int a, int e, double la,
                                                   const double* __restrict__ shift, WTab wtab,
                                                   Put put, PutEnd put_end, double* la_end,
                                                   bool* ok) {
#pragma clang fp contract(off)  // the same bits from every form of the recursion
    const int lane = threadIdx.x & 63;
    auto inside = [&](int r) { return t64_x(0, lane) < L && t64_y(0, r, lane) < L; };
    const int ax = a % L, ay = a / L;
    f64x4 F;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        F[r] = (t64_x(0, lane) == ax && t64_y(0, r, lane) == ay) ? 1.0 : 0.0;
    bool good = true;
    double wa[4], wb[4];
    int l = (start + 1) % L_tau;
    wtab(l, wa);
    auto step = [&](int j, const double (&w)[4], double (&wf)[4]) {
        const double sh = shift[l];
        l = l + 1 == L_tau ? 0 : l + 1;
        wtab(l, wf);  // the last step fetches a slice it does not use
        const f64x4 H = circ16(F, Cb, L);
        double sum = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            F[r] = H[r] * w[r];
            sum += F[r];
        }
        const double tot = wave_sum_f64(sum);
        good = good && tot > 0.0 && isfinite(tot);
        const double inv = 1.0 / tot;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            F[r] *= inv;
            if (inside(r)) put(j, 0, r, F[r]);
        }
        la += log(tot) + sh;
    };
    int j = 1;
    for (; j + 1 < len; j += 2) {
        step(j, wa, wb);
        step(j + 1, wb, wa);
    }
    if (j < len) step(j, wa, wb);
    const f64x4 H = circ16(F, Cb, L);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (inside(r)) put_end(0, r, H[r]);
    *la_end = la;
    const int ex = e % L, ey = e / L, re = ey >> 2;
    double hv = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (r == re) hv = H[r];
    hv = __shfl(hv, ex + 16 * (ey & 3), 64);
    good = good && hv > 0.0;
    *ok = good;
    return la + log(hv);
}

// The forward recursion of one block on the FP64 circulant, one wavefront (Sec. 3.5.2, site
// basis, with the per-step sum normaliser and the log-shifted potentials W~ = W exp(-m_l)):
//   f~_0 = delta_a; h_j = W~_{start+j} . (C f~_{j-1} C); c_j = sum h_j; f~_j = h_j / c_j
//   log Z = la + sum_j (log c_j + m_{start+j}) + log (C f~_{len-1} C)(e),
// where la is log W_start(a), supplied by the caller. wtab(l, w) fills w[4 q + r] with W~ of
// slice l at the lane's element (q, r) (any finite value at padded positions, where C f C is an
// exact zero); put(j, q, r, v) receives element (q, r) of row f~_j, j = 1 .. len - 1, at the
// lane's positions inside the L x L lattice only; put_end(q, r, v) the same elements of the end
// tile C f~_{len-1} C (L <= 16: w holds the four elements of tile 0 only, and only those are
// put), and *la_end log Z without the end weight (for worldlines that share these
// rows but end elsewhere). Returns log Z; *ok becomes false when a normaliser or the end weight
// is not a positive finite number.
template <typename WTab, typename Put, typename PutEnd>
__device__ inline double dmfma_block_forward_end(const double (&Cb)[16], int L, int L_tau,
                                                 int start, int len, int a, int e, double la,
                                                 const double* __restrict__ shift, WTab wtab,
                                                 Put put, PutEnd put_end, double* la_end,
                                                 bool* ok) {
#pragma clang fp contract(off)  // the same bits from every form of the recursion
    const int lane = threadIdx.x & 63;
    if (L <= 16) {
        const double C4[4] = {Cb[0], Cb[2], Cb[4], Cb[6]};
        return dmfma16_block_forward_end(C4, L, L_tau, start, len, a, e, la, shift, wtab, put,
                                         put_end, la_end, ok);
    }
    auto inside = [&](int q, int r) { return t64_x(q, lane) < L && t64_y(q, r, lane) < L; };
    const int ax = a % L, ay = a / L;
    Tile64 F;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            F.t[q][r] = (t64_x(q, lane) == ax && t64_y(q, r, lane) == ay) ? 1.0 : 0.0;
    bool good = true;
    for (int j = 1; j < len; ++j) {
        const int l = (start + j) % L_tau;
        double w[16];
        wtab(l, w);
        const Tile64 H = circ64(circ64(F, Cb), Cb);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) F.t[q][r] = H.t[q][r] * w[4 * q + r];
        const double tot = wave_sum_f64(tile_sum(F));
        good = good && tot > 0.0 && isfinite(tot);
        const double inv = 1.0 / tot;
        la += log(tot) + shift[l];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                F.t[q][r] *= inv;
                if (inside(q, r)) put(j, q, r, F.t[q][r]);
            }
    }
    // end weight (C f~ C)(e)
    const Tile64 H = circ64(circ64(F, Cb), Cb);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (inside(q, r)) put_end(q, r, H.t[q][r]);
    *la_end = la;
    const int ex = e % L, ey = e / L;
    const int qe = 2 * (ey >> 4) + (ex >> 4), re = (ey & 15) >> 2;
    double hv = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (q == qe && r == re) hv = H.t[q][r];
    hv = __shfl(hv, (ex & 15) + 16 * (ey & 3), 64);
    good = good && hv > 0.0;
    *ok = good;
    return la + log(hv);
}

// dmfma_block_forward_end without the end tile.
template <typename WTab, typename Put>
__device__ inline double dmfma_block_forward(const double (&Cb)[16], int L, int L_tau, int start,
                                             int len, int a, int e, double la,
                                             const double* __restrict__ shift, WTab wtab, Put put,
                                             bool* ok) {
    double la_end;
    return dmfma_block_forward_end(Cb, L, L_tau, start, len, a, e, la, shift, wtab, put,
                                   [](int, int, double) {}, &la_end, ok);
}

// The recursion of dmfma_block_forward_end by one workgroup of four wavefronts, for passes with
// too few recursions to fill the chip with one wavefront each. Wavefront wq owns the 16 x 16 tile
// wq = 2 I + J of the padded 32 x 32 filter: every wavefront holds the whole filter F, forms the
// two tiles X(0, I), X(1, I) of X = F^T C that its tile of H = X^T C needs, then that tile: 24
// products per step where one wavefront takes 64. The four W-weighted tiles meet in LDS (xch,
// double-buffered; *buf is kept between calls), and every wavefront sums all of them in the order
// of dmfma_block_forward_end, so the normaliser, the rows, the end tile and log Z are bit for bit
// those of the one-wavefront recursion. cm: the chain's B operands [16][64]; Wl0: W~ of slice 0;
// row f~_j goes to rows + (j - 1) N, the end tile C f~_{len-1} C to end (nullable). *la enters
// as log W_start(a) and leaves as log Z without the end weight. Returns true on the wavefront
// that holds the end weight, *hv (every lane).
__device__ inline bool dmfma4_block_forward(const double* __restrict__ cm, int L, int L_tau,
                                            int start, int len, int a, int e,
                                            const double* __restrict__ Wl0,
                                            const double* __restrict__ shift,
                                            double* __restrict__ rows, double* __restrict__ end,
                                            f64x4 (*xch)[4][64], int wq, int lane, int* buf,
                                            double* la, double* hv, bool* ok) {
#pragma clang fp contract(off)  // the same bits from every form of the recursion
    const int N = L * L, I = wq >> 1, J = wq & 1;
    // the B operands this wavefront's products take: column block I of C for X(K, I), column
    // block J for its tile of H (loaded by index, not picked from registers at a run-time index,
    // which would put them in scratch)
    double CbI[8], CbJ[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        CbI[k] = cm[(k * 2 + I) * 64 + lane];
        CbJ[k] = cm[(k * 2 + J) * 64 + lane];
    }
    // this wavefront's elements: site of register r of tile wq (-1 where padded; W is read at
    // site 0 there and multiplies an exact zero)
    int site[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int x = t64_x(wq, lane), y = t64_y(wq, r, lane);
        site[r] = (x < L && y < L) ? y * L + x : -1;
    }
    auto load_w = [&](int l, double (&w)[4]) {
        const double* Wl = Wl0 + (int64_t)l * N;
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = Wl[max(site[r], 0)];
    };
    // this wavefront's tile of H = (F^T C)^T C = C F C
    auto own_tile = [&](const Tile64& F) {
        f64x4 X[2];
#pragma unroll
        for (int K = 0; K < 2; ++K) {
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int K2 = 0; K2 < 2; ++K2)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(F.t[2 * K2 + K][r], CbI[4 * K2 + r],
                                                               acc, 0, 0, 0);
            X[K] = acc;
        }
        f64x4 H = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int K = 0; K < 2; ++K)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                H = __builtin_amdgcn_mfma_f64_16x16x4f64(X[K][r], CbJ[4 * K + r], H, 0, 0, 0);
        return H;
    };
    Tile64 F;
    const int ax = a % L, ay = a / L;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            F.t[q][r] = (t64_x(q, lane) == ax && t64_y(q, r, lane) == ay) ? 1.0 : 0.0;
    bool good = true;
    double lz = *la;
    int bf = *buf;
    // W of the next slice loaded one step ahead, in two buffers that swap roles
    double wa[4], wb[4];
    load_w((start + 1) % L_tau, wa);
    auto step = [&](int j, const double (&w)[4], double (&wf)[4]) {
        const int l = (start + j) % L_tau;
        const f64x4 H = own_tile(F);
        load_w((l + 1) % L_tau, wf);  // the last step fetches a slice it does not use
        f64x4 P;
#pragma unroll
        for (int r = 0; r < 4; ++r) P[r] = H[r] * w[r];
        xch[bf][wq][lane] = P;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) F.t[q] = xch[bf][q][lane];
        bf ^= 1;
        const double tot = wave_sum_f64(tile_sum(F));
        good = good && tot > 0.0 && isfinite(tot);
        const double inv = 1.0 / tot;
        lz += log(tot) + shift[l];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) F.t[q][r] *= inv;
        // this wavefront's tile of the row: its own products scaled as F.t[wq] (read from the
        // products it holds, as F.t[wq] at a run-time index would live in scratch)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (site[r] >= 0) rows[(int64_t)(j - 1) * N + site[r]] = P[r] * inv;
    };
    int j = 1;
    for (; j + 1 < len; j += 2) {
        step(j, wa, wb);
        step(j + 1, wb, wa);
    }
    if (j < len) step(j, wa, wb);
    // end weight (C f~ C)(e): the end tile, and the element at e from its tile's wavefront
    const f64x4 H = own_tile(F);
    if (end) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (site[r] >= 0) end[site[r]] = H[r];
    }
    *buf = bf;
    *la = lz;
    *ok = good;
    const int ex = e % L, ey = e / L, re = (ey & 15) >> 2;
    double h = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (r == re) h = H[r];
    *hv = __shfl(h, (ex & 15) + 16 * (ey & 3), 64);
    return wq == 2 * (ey >> 4) + (ex >> 4);
}

// One recursion by one workgroup: four wavefronts for L > 16, the first one alone for L <= 16
// (one tile). Arguments as dmfma4_block_forward; *lz receives log Z (valid, with *ok, on the
// wavefront that gets true).
__device__ inline bool dmfma_wg_forward(const double* __restrict__ cm, int L, int L_tau, int start,
                                        int len, int a, int e, const double* __restrict__ Wl0,
                                        const double* __restrict__ shift,
                                        double* __restrict__ rows, double* __restrict__ end,
                                        f64x4 (*xch)[4][64], int wq, int lane, int* buf,
                                        double* la, double* lz, bool* ok) {
    if (L <= 16) {
        if (wq != 0) return false;
        const int N = L * L;
        double Cb[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) Cb[r] = cm[2 * r * 64 + lane];
        auto site = [&](int r) { return t64_y(0, r, lane) * L + t64_x(0, lane); };
        auto wtab = [&](int l, double (&w)[4]) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool in = t64_x(0, lane) < L && t64_y(0, r, lane) < L;
                w[r] = Wl0[(int64_t)l * N + (in ? site(r) : 0)];
            }
        };
        auto put = [&](int j, int, int r, double v) { rows[(int64_t)(j - 1) * N + site(r)] = v; };
        auto put_end = [&](int, int r, double v) {
            if (end) end[site(r)] = v;
        };
        *lz = dmfma16_block_forward_end(Cb, L, L_tau, start, len, a, e, *la, shift, wtab, put,
                                        put_end, la, ok);
        return true;
    }
    double hv;
    const bool mine = dmfma4_block_forward(cm, L, L_tau, start, len, a, e, Wl0, shift, rows, end,
                                           xch, wq, lane, buf, la, &hv, ok);
    *ok = *ok && hv > 0.0;
    *lz = *la + log(hv);
    return mine;
}

// Lattices of side L = 16 NT with NT = 3 or 4 (L = 48, 64) on the same instruction. The filter
// is NT x NT tiles of 16 x 16, tile q = NT I + J holding rows 16 I .. and columns 16 J .., its
// element (16 I + 4 r + lane / 16, 16 J + lane % 16) in register r, as above. C[k][j] =
// g((k - j) mod L) is then block-circulant: its 16 x 16 block (K, J) depends only on
// D = (K - J) mod NT, and the B operands are Cb[4 D + r], lane j + 16 k holding
// g((16 D + 4 r + k - j) mod L):
//   (X^T C)(I, J) = sum over K, r of mfma(X(K, I)[r], Cb[4 ((K - J) mod NT) + r]),
// 4 NT^3 products per multiplication, every product and sum in FP64, as for L <= 32.
template <int NT>
struct TileBig {
    f64x4 t[NT * NT];
};

template <int NT>
__device__ inline void circ_big(const TileBig<NT>& X, const double (&Cb)[16], TileBig<NT>& Y) {
#pragma unroll
    for (int I = 0; I < NT; ++I)
#pragma unroll
        for (int J = 0; J < NT; ++J) {
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int K = 0; K < NT; ++K)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(
                        X.t[NT * K + I][r], Cb[4 * ((K - J + NT) % NT) + r], acc, 0, 0, 0);
            Y.t[NT * I + J] = acc;
        }
}

// Site coordinates of element (tile q, register r) of a lane in the NT x NT tiling.
template <int NT>
__device__ inline int tb_x(int q, int lane) { return 16 * (q % NT) + (lane & 15); }
template <int NT>
__device__ inline int tb_y(int q, int r, int lane) { return 16 * (q / NT) + 4 * r + (lane >> 4); }

// dmfma_block_forward_end for L = 16 NT: the same recursion, normaliser, log Z and outputs.
// wtab(l, w) fills w[4 q + r] with W~ of slice l at the lane's element (q, r); every element is
// a lattice site, so put and put_end see all of them.
template <int NT, typename WTab, typename Put, typename PutEnd>
__device__ inline double dmfma_big_block_forward_end(const double (&Cb)[16], int L_tau,
                                                     int start, int len, int a, int e, double la,
                                                     const double* __restrict__ shift, WTab wtab,
                                                     Put put, PutEnd put_end, double* la_end,
                                                     bool* ok) {
#pragma clang fp contract(off)  // the same bits from every form of the recursion
    constexpr int L = 16 * NT, NQ = NT * NT;
    const int lane = threadIdx.x & 63;
    const int ax = a % L, ay = a / L;
    TileBig<NT> F, X;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            F.t[q][r] = (tb_x<NT>(q, lane) == ax && tb_y<NT>(q, r, lane) == ay) ? 1.0 : 0.0;
    bool good = true;
    for (int j = 1; j < len; ++j) {
        const int l = (start + j) % L_tau;
        circ_big<NT>(F, Cb, X);
        circ_big<NT>(X, Cb, F);
        // W after the products: loaded before them, the slice would need 2 NT^2 more registers
        double w[4 * NQ];
        wtab(l, w);
        double sum = 0.0;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                F.t[q][r] *= w[4 * q + r];
                sum += F.t[q][r];
            }
        const double tot = wave_sum_f64(sum);
        good = good && tot > 0.0 && isfinite(tot);
        const double inv = 1.0 / tot;
        la += log(tot) + shift[l];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                F.t[q][r] *= inv;
                put(j, q, r, F.t[q][r]);
            }
    }
    // end weight (C f~ C)(e)
    circ_big<NT>(F, Cb, X);
    circ_big<NT>(X, Cb, F);
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) put_end(q, r, F.t[q][r]);
    *la_end = la;
    const int ex = e % L, ey = e / L;
    const int qe = NT * (ey >> 4) + (ex >> 4), re = (ey & 15) >> 2;
    double hv = 0.0;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (q == qe && r == re) hv = F.t[q][r];
    hv = __shfl(hv, (ex & 15) + 16 * (ey & 3), 64);
    good = good && hv > 0.0;
    *ok = good;
    return la + log(hv);
}

// dmfma_big_block_forward_end by one workgroup, for passes with few recursions: wavefront w < NT
// owns row block w of the NT x NT tiles. It forms column block w of X = F^T C and, from exactly
// those tiles, row block w of H = X^T C: 8 NT^2 products, the whole step's 8 NT^3 split without
// repeats. The W-weighted tiles meet in LDS (xch, [2][NT^2][64], double-buffered; *buf is kept
// between calls), and every wavefront sums all of them in the one-wavefront order, so every bit is
// the same. Wl0: W~ of slice 0; rows f~_j go to rows + (j - 1) N, the end tile to end (nullable).
// *la enters as log W_start(a) and leaves as log Z without the end weight; *lz receives log Z on
// the wavefront that gets true. Wavefronts past NT only meet the barriers.
// Bound: FP64 products, 2 NT^2 (NT = 4: 128) of 64 cycles a wavefront and step; a 64 x 64 step took
// 18.6 us on one wavefront, 4.6 us here.
template <int NT>
__device__ inline bool dmfma_big_wg_forward(const double (&Cb)[16], int L_tau, int start, int len,
                                            int a, int e, const double* __restrict__ Wl0,
                                            const double* __restrict__ shift,
                                            double* __restrict__ rows, double* __restrict__ end,
                                            f64x4 (*xch)[NT * NT][64], int w, int lane, int* buf,
                                            double* la, double* lz, bool* ok) {
#pragma clang fp contract(off)
    constexpr int L = 16 * NT, N = L * L, NQ = NT * NT;
    const bool works = w < NT;
    const int row = works ? w : 0;  // this wavefront's row block
    // its elements: tile (row, J), register r; every position is a lattice site
    const int y0 = 16 * row + (lane >> 4), x0 = lane & 15;
    auto site = [&](int J, int r) { return (y0 + 4 * r) * L + 16 * J + x0; };
    TileBig<NT> F;
    const int ax = a % L, ay = a / L;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            F.t[q][r] = (tb_x<NT>(q, lane) == ax && tb_y<NT>(q, r, lane) == ay) ? 1.0 : 0.0;
    // column block `row` of C is Cb rotated by it: the operands of the X tiles, picked once (a
    // run-time index into registers would put them in scratch)
    double Cr[16];
#pragma unroll
    for (int D = 0; D < NT; ++D)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double v = 0.0;
#pragma unroll
            for (int s = 0; s < NT; ++s)
                if (s == row) v = Cb[4 * ((D - s + NT) % NT) + r];
            Cr[4 * D + r] = v;  // block (D, row)
        }
    auto own_tiles = [&](f64x4 (&H)[NT]) {
        f64x4 X[NT];  // X(K, row)
#pragma unroll
        for (int K = 0; K < NT; ++K) {
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int K2 = 0; K2 < NT; ++K2)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(F.t[NT * K2 + K][r], Cr[4 * K2 + r],
                                                               acc, 0, 0, 0);
            X[K] = acc;
        }
#pragma unroll
        for (int J = 0; J < NT; ++J) {
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int K = 0; K < NT; ++K)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(
                        X[K][r], Cb[4 * ((K - J + NT) % NT) + r], acc, 0, 0, 0);
            H[J] = acc;
        }
    };
    bool good = true;
    double lzv = *la;
    int bf = *buf;
    for (int j = 1; j < len; ++j) {
        const int l = (start + j) % L_tau;
        f64x4 P[NT];
        if (works) {
            double wv[NT][4];
#pragma unroll
            for (int J = 0; J < NT; ++J)
#pragma unroll
                for (int r = 0; r < 4; ++r) wv[J][r] = Wl0[(int64_t)l * N + site(J, r)];
            __builtin_amdgcn_sched_barrier(0);  // W in flight during the matrix work
            own_tiles(P);
#pragma unroll
            for (int J = 0; J < NT; ++J) {
#pragma unroll
                for (int r = 0; r < 4; ++r) P[J][r] *= wv[J][r];
                xch[bf][NT * row + J][lane] = P[J];
            }
        }
        __syncthreads();
        if (works) {
            double sum = 0.0;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                F.t[q] = xch[bf][q][lane];
#pragma unroll
                for (int r = 0; r < 4; ++r) sum += F.t[q][r];
            }
            const double tot = wave_sum_f64(sum);
            good = good && tot > 0.0 && isfinite(tot);
            const double inv = 1.0 / tot;
            lzv += log(tot) + shift[l];
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) F.t[q][r] *= inv;
#pragma unroll
            for (int J = 0; J < NT; ++J)
#pragma unroll
                for (int r = 0; r < 4; ++r) rows[(int64_t)(j - 1) * N + site(J, r)] = P[J][r] * inv;
        }
        bf ^= 1;
    }
    *buf = bf;
    if (!works) return false;
    f64x4 H[NT];  // end weight (C f~ C)(e)
    own_tiles(H);
    const int ex = e % L, ey = e / L, re = (ey & 15) >> 2;
    double hv = 0.0;
#pragma unroll
    for (int J = 0; J < NT; ++J)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (end) end[site(J, r)] = H[J][r];
            if (J == (ex >> 4) && r == re) hv = H[J][r];
        }
    hv = __shfl(hv, (ex & 15) + 16 * (ey & 3), 64);
    *la = lzv;
    *ok = good && hv > 0.0;
    *lz = lzv + log(hv);
    return row == (ey >> 4);
}

}  // namespace fh
