// k_variational.hip -- one-level variational refinement of the interpolated
// field (Sec. 4 of the paper): an energy of a data term (colour and
// gradient constancy with a normalisation, the paper citing its form) and a
// smoothness term on the flow gradient norm weighted by alpha(x) =
// exp(-kappa ||grad I1||), minimised from the interpolated field u0 without
// coarse-to-fine by `fixed_point` steps (the non-linear weights of the
// Euler-Lagrange equations re-evaluated) of `sor` successive
// over-relaxation sweeps.
//
// The discrete problem (the reading this library takes of the cited data
// term, and its discretisation):
//   I2w = I2(x + u0(x)) bilinear, coordinates clamped; central differences
//   with the border pixel repeated; Ixx, Iyy, Ixy of I2w; Iz = I2w - I1;
//   Ixz, Iyz the gradient differences of I2w and I1;
//   colour   sum_c theta_c (Iz + Ix du + Iy dv)^2,      theta_c  = 1/(Ix^2+Iy^2+zeta^2)
//   gradient sum_c thetax_c (Ixz + Ixx du + Ixy dv)^2 + thetay_c (Iyz + Ixy du + Iyy dv)^2,
//            thetax = 1/(Ixx^2+Ixy^2+zeta^2), thetay = 1/(Ixy^2+Iyy^2+zeta^2)
//   E = sum_x delta psi(colour) + gamma psi(gradient)
//     + sum over 4-neighbour edges lam (alpha_i+alpha_j)/2 psi(|U_j-U_i|^2 + |V_j-V_i|^2)
//   psi(s^2) = sqrt(s^2 + eps^2), U = u0 + du, V = v0 + dv.
// Each fixed-point step evaluates psi' at the current (du, dv) and solves
//   (A11 + sum_j g_ij) du_i + A12 dv_i = b1 + sum_j g_ij (U_j - u0_i), likewise dv,
// by red-black SOR sweeps (red: x + y even), du before dv at each pixel; an
// equation with a zero diagonal leaves its unknown unchanged.  The sums are
// taken as sum_j g_ij (u0_j - u0_i) + sum_j g_ij du_j: the first part is
// fixed for a fixed-point step and folded into the right-hand side, and the
// small increments du carry the sweeps (no cancellation against u0).
//
// Kernels (FP32):
//   k_var_coef     I2w and I1 of a 32 x 8 tile and the pixels around it into
//                  LDS, then per pixel the colour and gradient systems J (6
//                  entries each) and alpha, in 3 records of 16 bytes and a
//                  plane.  Bound by its reads' latency: 11.7 us at 1024 x 436
//                  (a kernel for I2w and one that read both images from memory
//                  took 7.0 + 14.1)
//   k_var_weights  per fixed-point step and pixel the numbers its update
//                  needs: omega / D1 and omega / D2 for the diagonals
//                  D1 = A11 + sum g, D2 = A22 + sum g (one division per
//                  step, not per sweep), A12, right-hand sides B1, B2, and
//                  its edge weights (each edge evaluated in one canonical
//                  order, so both endpoints see the same value), in two
//                  records of 16 bytes
//   k_var_sor      up to 16 half-sweeps per launch with the sweeps blocked
//                  in time: a workgroup loads its tile and a halo of 16
//                  pixels, relaxes the whole region (each half-sweep
//                  corrupts at most one more ring from the region's edge
//                  inwards, so the tile's values equal those of global
//                  half-sweeps) and writes the tile to the other buffer of
//                  a ping-pong pair, the last launch u0 + du instead.  A
//                  launch per half-sweep would spend most of its time in
//                  launching and in re-reading the system from memory.
//   k_var_copy     u0, for a call without sweeps
#include <type_traits>

#include "epic_dev.h"

namespace epic {

namespace {

__device__ __forceinline__ float psi_d(float s2, float eps) {
    return 0.5f / sqrtf(fmaxf(s2, 0.0f) + eps * eps);
}

__device__ __forceinline__ float quad(const float* J, float du, float dv) {
    return J[0] * du * du + 2.0f * J[1] * du * dv + J[2] * dv * dv + 2.0f * J[3] * du + 2.0f * J[4] * dv + J[5];
}

}  // namespace

// The input field's two numbers at pixel i in one load (the field need only be
// aligned to a float).
struct __attribute__((packed, aligned(4))) Flow2 { float u, v; };
__device__ __forceinline__ float2 field(const float* f, long long i) {
    const Flow2 t = reinterpret_cast<const Flow2*>(f)[i];
    return make_float2(t.u, t.v);
}

constexpr int kCoefX = 32, kCoefY = 8;                      // pixels per workgroup
constexpr int kCoefW = kCoefX + 2, kCoefN = kCoefW * (kCoefY + 2);

template <int C, bool SLICED>
__global__ __launch_bounds__(256) void k_var_coef(VarArgs A, unsigned tile0) {
    __shared__ float Lw[C][kCoefN], L1[C][kCoefN];
    const int W = A.W, H = A.H, tid = threadIdx.x;
    const int tiles_x = (W + kCoefX - 1) / kCoefX;
    const unsigned tile = SLICED ? tile0 + blockIdx.x : blockIdx.x;
    const int X0 = (int)(tile % tiles_x) * kCoefX, Y0 = (int)(tile / tiles_x) * kCoefY;
    // I2w and I1 of the tile and one pixel around it, the border repeated
    for (int e = tid; e < kCoefN; e += 256) {
        const int x = min(max(X0 + e % kCoefW - 1, 0), W - 1), y = min(max(Y0 + e / kCoefW - 1, 0), H - 1);
        const long long i = (long long)y * W + x;
        const float2 u = field(A.u0, i);
        const float fxp = fminf(fmaxf((float)x + u.x, 0.0f), (float)(W - 1));
        const float fyp = fminf(fmaxf((float)y + u.y, 0.0f), (float)(H - 1));
        const int x0 = min((int)floorf(fxp), W > 1 ? W - 2 : 0), y0 = min((int)floorf(fyp), H > 1 ? H - 2 : 0);
        const int x1 = min(x0 + 1, W - 1), y1 = min(y0 + 1, H - 1);
        const float fx = fxp - (float)x0, fy = fyp - (float)y0;
        const float *ra = A.I2 + ((long long)y0 * W + x0) * C, *rb = A.I2 + ((long long)y0 * W + x1) * C;
        const float *rd = A.I2 + ((long long)y1 * W + x0) * C, *re = A.I2 + ((long long)y1 * W + x1) * C;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            L1[c][e] = A.I1[i * C + c];
            Lw[c][e] = (1.0f - fy) * ((1.0f - fx) * ra[c] + fx * rb[c]) + fy * ((1.0f - fx) * rd[c] + fx * re[c]);
        }
    }
    __syncthreads();
    const int x = X0 + tid % kCoefX, y = Y0 + tid / kCoefX;
    if (x >= W || y >= H) return;
    const long long i = (long long)y * W + x;
    const int e = (tid / kCoefX + 1) * kCoefW + tid % kCoefX + 1;
    float J[12];
    for (int k = 0; k < 12; ++k) J[k] = 0.0f;
    float gn = 0.0f;
    const float z2 = A.zeta * A.zeta;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const float *q = Lw[c] + e, *q1 = L1[c] + e;
        const float w = q[0];
        const float Ix = 0.5f * (q[1] - q[-1]);
        const float Iy = 0.5f * (q[kCoefW] - q[-kCoefW]);
        const float gx1 = 0.5f * (q1[1] - q1[-1]);
        const float gy1 = 0.5f * (q1[kCoefW] - q1[-kCoefW]);
        const float Iz = w - q1[0];
        const float Ixx = q[1] - 2.0f * w + q[-1];
        const float Iyy = q[kCoefW] - 2.0f * w + q[-kCoefW];
        const float Ixy = 0.25f * (q[kCoefW + 1] - q[kCoefW - 1] - q[-kCoefW + 1] + q[-kCoefW - 1]);
        const float Ixz = Ix - gx1, Iyz = Iy - gy1;
        const float th = 1.0f / (Ix * Ix + Iy * Iy + z2);
        const float thx = 1.0f / (Ixx * Ixx + Ixy * Ixy + z2);
        const float thy = 1.0f / (Ixy * Ixy + Iyy * Iyy + z2);
        // colour system: th [Ix Iy Iz]^T [Ix Iy Iz]
        J[0] += th * Ix * Ix; J[1] += th * Ix * Iy; J[2] += th * Iy * Iy;
        J[3] += th * Ix * Iz; J[4] += th * Iy * Iz; J[5] += th * Iz * Iz;
        // gradient system: thx [Ixx Ixy Ixz]^T [..] + thy [Ixy Iyy Iyz]^T [..]
        J[6] += thx * Ixx * Ixx + thy * Ixy * Ixy;
        J[7] += thx * Ixx * Ixy + thy * Ixy * Iyy;
        J[8] += thx * Ixy * Ixy + thy * Iyy * Iyy;
        J[9] += thx * Ixx * Ixz + thy * Ixy * Iyz;
        J[10] += thx * Ixy * Ixz + thy * Iyy * Iyz;
        J[11] += thx * Ixz * Ixz + thy * Iyz * Iyz;
        gn += gx1 * gx1 + gy1 * gy1;
    }
    float4* S = reinterpret_cast<float4*>(A.coef);
    S[i] = make_float4(J[0], J[1], J[2], J[3]);
    S[A.HW + i] = make_float4(J[4], J[5], J[6], J[7]);
    S[2 * A.HW + i] = make_float4(J[8], J[9], J[10], J[11]);
    A.coef[12LL * A.HW + i] = expf(-A.kappa * sqrtf(gn));
    A.d[0][i] = make_float2(0.0f, 0.0f);
}

// A pixel as the smoothness weights see it: alpha, (u0, v0) and (du, dv).
struct VarPixel {
    float alpha;
    float2 u, d;
};

__device__ __forceinline__ VarPixel var_pixel(const VarArgs& A, const float2* d, long long i) {
    return {A.coef[12LL * A.HW + i], field(A.u0, i), d[i]};
}

// Edge (p, q) with p the left or upper pixel: lam (alpha_p + alpha_q) / 2
// psi'(|U_q - U_p|^2 + |V_q - V_p|^2), in this one order for both ends.
__device__ __forceinline__ float edge_weight(const VarArgs& A, const VarPixel& p, const VarPixel& q) {
    const float dU = (q.u.x + q.d.x) - (p.u.x + p.d.x);
    const float dV = (q.u.y + q.d.y) - (p.u.y + p.d.y);
    return A.lam * 0.5f * (p.alpha + q.alpha) * psi_d(dU * dU + dV * dV, A.eps);
}

// A pixel's update, two records of A.sys:
//   [i]       omega / D1, omega / D2 (0 for an empty equation, which keeps
//             its unknown), A12, B1
//   [HW + i]  B2 and the weights of its right, lower and left edge (the
//             upper edge is the lower one of the pixel above)
__global__ __launch_bounds__(256) void k_var_weights(VarArgs A, const float2* __restrict__ d) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= A.HW) return;
    const int W = A.W, H = A.H;
    const int x = (int)(i % W), y = (int)(i / W);
    const float4* S = reinterpret_cast<const float4*>(A.coef);
    const float4 s0 = S[i], s1 = S[A.HW + i], s2 = S[2 * A.HW + i];
    const float JC[6] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y};
    const float JG[6] = {s1.z, s1.w, s2.x, s2.y, s2.z, s2.w};
    // a neighbour outside the image: the pixel itself (its weight is not used)
    const VarPixel P = var_pixel(A, d, i);
    const VarPixel Pl = var_pixel(A, d, x > 0 ? i - 1 : i), Pr = var_pixel(A, d, x + 1 < W ? i + 1 : i);
    const VarPixel Pu = var_pixel(A, d, y > 0 ? i - W : i), Pd = var_pixel(A, d, y + 1 < H ? i + W : i);
    const float dui = P.d.x, dvi = P.d.y;
    const float wc = A.delta * psi_d(quad(JC, dui, dvi), A.eps);
    const float wg = A.gamma * psi_d(quad(JG, dui, dvi), A.eps);
    const float a11 = wc * JC[0] + wg * JG[0];
    const float a12 = wc * JC[1] + wg * JG[1];
    const float a22 = wc * JC[2] + wg * JG[2];
    float b1 = -(wc * JC[3] + wg * JG[3]);
    float b2 = -(wc * JC[4] + wg * JG[4]);
    // the 4 edges (0 where there is no neighbour) and the fixed part of the
    // neighbour sums, sum_j g (u0_j - u0_i)
    const float gl = x > 0 ? edge_weight(A, Pl, P) : 0.0f;
    const float gr = x + 1 < W ? edge_weight(A, P, Pr) : 0.0f;
    const float gu = y > 0 ? edge_weight(A, Pu, P) : 0.0f;
    const float gd = y + 1 < H ? edge_weight(A, P, Pd) : 0.0f;
    auto fold = [&](float g, const VarPixel& q) {
        b1 += g * (q.u.x - P.u.x);
        b2 += g * (q.u.y - P.u.y);
    };
    if (x > 0) fold(gl, Pl);
    if (x + 1 < W) fold(gr, Pr);
    if (y > 0) fold(gu, Pu);
    if (y + 1 < H) fold(gd, Pd);
    const float sw = ((gl + gr) + gu) + gd;
    const float d1 = a11 + sw, d2 = a22 + sw;
    float4* R = reinterpret_cast<float4*>(A.sys);
    R[i] = make_float4(d1 > 0.0f ? A.omega / d1 : 0.0f, d2 > 0.0f ? A.omega / d2 : 0.0f, a12, b1);
    R[A.HW + i] = make_float4(b2, gr, gd, gl);
}

// The sweeps' tile: TX x TY pixels and a halo of S (the most half-sweeps a
// launch runs; even, so every launch starts with red) make the region RX x RY
// of NR strips of KP rows.  Thread (strip, s) holds pixels 2s and 2s + 1 of
// its strip's rows -- one of each colour per row -- with their update records
// in registers.  All tile and strip edges are even, so which of the two is
// red is known at compile time, and of a pixel's four neighbours the other
// one of its pair and, inside the strip, the ones above and below are the
// thread's own registers: 1 + 2 / KP instead of 4 LDS reads per update.  An
// edge between two pixels of a thread is held once.  A wave whose rows can no
// longer reach the tile in the sweeps that are left skips them.
//
// What bounds it: 16 half-sweeps take 6.3 of a launch's 15 us at 1024 x 436
// (FP32 FMAs and a barrier each), the records 1.4 (2 x 16 bytes a pixel), and
// most of the rest is the launch itself, so a launch runs 16 (S = 20 saves a
// quarter of the launches and gives it back in halo: 364 against 359 us a call
// with 64 x 28 tiles).  With records in nine planes, all four neighbours from
// LDS, S = 12 and 64 x 32 tiles a call took 626 us; then 359 (348 with the warp
// and the coefficients in one kernel).
template <int TX_, int S_, int KP_, int NR_>
struct VarTile {
    static constexpr int TX = TX_, S = S_, KP = KP_, NR = NR_;
    static_assert(TX % 2 == 0 && S % 2 == 0 && KP % 2 == 0, "even tile width, halo and strip");
    static constexpr int RX = TX + 2 * S, RY = NR * KP, TY = RY - 2 * S, RXh = RX / 2;
    static constexpr int NT = (NR * RXh + 63) / 64 * 64;
    static_assert(TY > 0 && NT <= 1024, "tile");
    static long long tiles(int H, int W) { return (long long)((W + TX - 1) / TX) * ((H + TY - 1) / TY); }
};
// 32 x 16 pixels, 768 threads of 2 rows: less work per CU where there are CUs to
// spare.  32 x 32 pixels, 1024 threads of 2 rows: two workgroups fit a CU.  64 x
// 28 pixels, 720 threads of 4 rows: one per CU, and a third less halo.
using VarFine = VarTile<32, 16, 2, 24>;
using VarSmall = VarTile<32, 16, 2, 32>;
using VarWide = VarTile<64, 16, 4, 15>;
constexpr int kVarCus = 256;

template <class T, bool SLICED>
__global__ __launch_bounds__(T::NT) void k_var_sor(VarArgs A, const float2* __restrict__ in, float2* __restrict__ out,
                                                   int nh, int last, unsigned tile0) {
    constexpr int TX = T::TX, S = T::S, KP = T::KP, NR = T::NR, RY = T::RY, TY = T::TY, RXh = T::RXh, NT = T::NT;
    constexpr int LW = RXh + 2, LN = (RY + 2) * LW;
    __shared__ float2 L[2][LN];
    const int tid = threadIdx.x;
    const int W = A.W, H = A.H;
    const int tiles_x = (W + TX - 1) / TX;
    const unsigned tile = SLICED ? tile0 + blockIdx.x : blockIdx.x;
    const int X0 = (int)(tile % tiles_x) * TX - S, Y0 = (int)(tile / tiles_x) * TY - S;
    // the pads around the region: read by its outermost ring only
    for (int k = tid; k < 2 * (2 * LW + 2 * RY); k += NT) {
        const int a = k & 1, q = k >> 1;
        const int e = q < LW ? q : q < 2 * LW ? (RY + 1) * LW + q - LW
                                              : (1 + (q - 2 * LW) / 2) * LW + ((q & 1) ? LW - 1 : 0);
        L[a][e] = make_float2(0.0f, 0.0f);
    }
    const int strip = tid / RXh, s = tid % RXh, y0 = strip * KP;
    const bool act = strip < NR;
    const int cell = (y0 + 1) * LW + s + 1;
    const float4* R = reinterpret_cast<const float4*>(A.sys);
    // this thread's pixels [row][x & 1]
    float2 v[KP][2];
    float w1[KP][2], w2[KP][2], a12[KP][2], b1[KP][2], b2[KP][2], gr[KP][2], gd[KP][2], gl[KP], gu[2] = {0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < KP; ++k) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int y = y0 + k, gx = X0 + 2 * s + p, gy = Y0 + y;
            float4 r0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), r1 = r0;
            v[k][p] = make_float2(0.0f, 0.0f);
            // rows past the reach of this launch's sweeps are not needed
            if (act && y >= S - nh && y < RY - S + nh && gx >= 0 && gx < W && gy >= 0 && gy < H) {
                const long long i = (long long)gy * W + gx;
                r0 = R[i];
                r1 = R[A.HW + i];
                v[k][p] = in[i];
                if (k == 0 && gy > 0) gu[p] = R[A.HW + i - W].z;
            }
            w1[k][p] = r0.x; w2[k][p] = r0.y; a12[k][p] = r0.z; b1[k][p] = r0.w;
            b2[k][p] = r1.x; gr[k][p] = r1.y; gd[k][p] = r1.z;
            if (p == 0) gl[k] = r1.w;
            if (act) L[p][cell + k * LW] = v[k][p];
        }
    }
    __syncthreads();
    const float om1 = 1.0f - A.omega;
    // the rows of this wave
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wy0 = wave * 64 / RXh * KP, wy1 = min((wave * 64 + 63) / RXh, NR - 1) * KP + KP;
    auto half = [&](auto colour, int left) {
        constexpr int c = decltype(colour)::value;
        // rows within `left` half-sweeps' reach of the tile
        if (wy1 > S - left && wy0 < RY - S + left && act) {
            float2 far[KP], up, dn;
#pragma unroll
            for (int k = 0; k < KP; ++k) far[k] = (c + k) & 1 ? L[0][cell + k * LW + 1] : L[1][cell + k * LW - 1];
            up = L[c][cell - LW];
            dn = L[(c + KP - 1) & 1][cell + KP * LW];
#pragma unroll
            for (int k = 0; k < KP; ++k) {
                const int p = (c + k) & 1;
                const float2 l = p ? v[k][0] : far[k], r = p ? far[k] : v[k][1];
                const float2 u = k ? v[k - (k > 0)][p] : up, d = k < KP - 1 ? v[k + (k < KP - 1)][p] : dn;
                const float g0 = p ? gr[k][0] : gl[k], g2 = k ? gd[k - (k > 0)][p] : gu[p];
                // every rounding spelled out, so the result does not depend on
                // how the compiler schedules (and fuses) the unrolled slots:
                // any tiling gives the same bits
                const float su = __fmaf_rn(gd[k][p], d.x, __fmaf_rn(g2, u.x, __fmaf_rn(gr[k][p], r.x,
                                                                                       __fmul_rn(g0, l.x))));
                const float sv = __fmaf_rn(gd[k][p], d.y, __fmaf_rn(g2, u.y, __fmaf_rn(gr[k][p], r.y,
                                                                                       __fmul_rn(g0, l.y))));
                float2 t = v[k][p];
                if (w1[k][p] > 0.0f)
                    t.x = __fmaf_rn(__fadd_rn(__fmaf_rn(-a12[k][p], t.y, b1[k][p]), su), w1[k][p], __fmul_rn(om1, t.x));
                if (w2[k][p] > 0.0f)
                    t.y = __fmaf_rn(__fadd_rn(__fmaf_rn(-a12[k][p], t.x, b2[k][p]), sv), w2[k][p], __fmul_rn(om1, t.y));
                v[k][p] = t;
                L[p][cell + k * LW] = t;
            }
        }
        __syncthreads();
    };
    for (int h = nh; h > 0; h -= 2) {     // nh is even: red, then black
        half(std::integral_constant<int, 0>{}, h - 1);
        half(std::integral_constant<int, 1>{}, h - 2);
    }
    // the tile (distance >= S from the region's edge) is exact
#pragma unroll
    for (int k = 0; k < KP; ++k) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int x = 2 * s + p, y = y0 + k, gx = X0 + x, gy = Y0 + y;
            if (act && x >= S && x < S + TX && y >= S && y < S + TY && gx < W && gy < H) {
                const long long i = (long long)gy * W + gx;
                if (last) {
                    const float2 u = field(A.u0, i);
                    reinterpret_cast<Flow2*>(A.flow)[i] = {u.x + v[k][p].x, u.y + v[k][p].y};
                } else {
                    out[i] = v[k][p];
                }
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_var_copy(VarArgs A) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= A.HW) return;
    A.flow[2 * i] = A.u0[2 * i] + 0.0f;
    A.flow[2 * i + 1] = A.u0[2 * i + 1] + 0.0f;
}

// One launch, or (SLICED kernels, told the first tile) several of at most 2^21
// tiles: a launch has fewer than 2^32 threads, which very narrow images would
// pass (a tile is 32 pixels wide at least: 1 pixel by 2^27 is 2^22 tiles of
// 1024 threads).  Kernels of their own: reading the first tile costs a sweep
// launch 0.08 us.
template <class F>
static void in_slices(long long tiles, F launch) {
    constexpr long long SLICE = 1 << 21;
    if (tiles <= SLICE) {
        launch(std::false_type{}, dim3((unsigned)tiles), 0u);
        return;
    }
    for (long long t = 0; t < tiles; t += SLICE)
        launch(std::true_type{}, dim3((unsigned)(tiles - t < SLICE ? tiles - t : SLICE)), (unsigned)t);
}

template <class T>
static void sweeps(const VarArgs& A, hipStream_t s) {
    const dim3 g((unsigned)((A.HW + 255) / 256)), b(256);
    int cur = 0;
    for (int f = 0; f < A.fixed_point; ++f) {
        hipLaunchKernelGGL(k_var_weights, g, b, 0, s, A, A.d[cur]);
        for (int h = 0; h < 2 * A.sor; h += T::S) {
            const int nh = 2 * A.sor - h < T::S ? 2 * A.sor - h : T::S;
            const int last = f + 1 == A.fixed_point && h + T::S >= 2 * A.sor;
            in_slices(T::tiles(A.H, A.W), [&](auto sliced, dim3 tiles, unsigned tile0) {
                hipLaunchKernelGGL((k_var_sor<T, decltype(sliced)::value>), tiles, dim3(T::NT), 0, s, A, A.d[cur],
                                   A.d[cur ^ 1], nh, last, tile0);
            });
            cur ^= 1;
        }
    }
}

hipError_t launch_variational(const VarArgs& A, hipStream_t s) {
    const dim3 g((unsigned)((A.HW + 255) / 256)), b(256);
    if (A.fixed_point == 0 || A.sor == 0) {
        hipLaunchKernelGGL(k_var_copy, g, b, 0, s, A);
        return hipGetLastError();
    }
    const long long coef_tiles = (long long)((A.W + kCoefX - 1) / kCoefX) * ((A.H + kCoefY - 1) / kCoefY);
    in_slices(coef_tiles, [&](auto sliced, dim3 tiles, unsigned tile0) {
        constexpr bool S = decltype(sliced)::value;
        switch (A.C) {
            case 1: hipLaunchKernelGGL((k_var_coef<1, S>), tiles, b, 0, s, A, tile0); break;
            case 2: hipLaunchKernelGGL((k_var_coef<2, S>), tiles, b, 0, s, A, tile0); break;
            case 3: hipLaunchKernelGGL((k_var_coef<3, S>), tiles, b, 0, s, A, tile0); break;
            default: hipLaunchKernelGGL((k_var_coef<4, S>), tiles, b, 0, s, A, tile0); break;
        }
    });
    // A launch takes as long as its busiest CU, so the smallest tile that leaves
    // every CU at most one workgroup: the fine one (128 x 96: 188 us against 217
    // with the small one, 400 x 300: 235 against 254), the small one (640 x 300:
    // 278 against 334 with the wide one), the wide one (1024 x 436: 359 against
    // 392 with the small one).  For larger images the small tile, of which two
    // workgroups share a CU (1280 x 720: 707 against 974 with the wide one).
    if (VarFine::tiles(A.H, A.W) <= kVarCus) sweeps<VarFine>(A, s);
    else if (VarWide::tiles(A.H, A.W) <= kVarCus && VarSmall::tiles(A.H, A.W) > kVarCus) sweeps<VarWide>(A, s);
    else sweeps<VarSmall>(A, s);
    return hipGetLastError();
}

}  // namespace epic
