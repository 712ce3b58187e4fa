// k_image_cost.hip -- the cost map from the image gradient: C(p) =
// ||grad I(p)||_2 + eps (Table 2 of the paper, the norm-of-gradient contour
// row; Sec. 4 uses the same gradient norm for its smoothness weight).  The
// gradient is taken by central differences, (I(x+1) - I(x-1)) / 2 and
// (I(y+1) - I(y-1)) / 2, with the border pixel repeated outside the image,
// and the norm runs over both directions and all channels (interleaved,
// 1 to 4 per pixel).
//
// A streaming stencil bound by HBM: 4*ch bytes read and 4 written per
// pixel.  A workgroup takes a tile of 256 x 8 pixels: its rows and the
// pixels around them come in 16-byte loads of consecutive lanes, all issued
// before the first is used, and go to LDS; then a thread walks 4 rows of one
// column, with the rows above and below in registers.  64 RGB images (20.9
// Mpx, 1242 x 375 to 256 x 192): 74 us, 4.5 TB/s, 92 % of a large copy's
// rate.  One pixel per thread with four loads of its own took 91 us (3.7
// TB/s): a wavefront lived for its latencies, the search for its image among
// up to 64 and one round of loads, on 64 pixels.  Four pixels by 1, 2 or 4
// rows per thread, loaded 16 bytes at a time 48 bytes apart: 121, 112 and 77
// us.  Tiles of 128 x 16, 128 x 8 and 256 x 8 with 256 threads: 84, 75 and 77
// us.  FP32, one rounding per operation (the square root's too: sqrtf, where
// __fsqrt_rn is the hardware's root, which is one unit off for one in seven).
#include "epic_dev.h"

namespace epic {

namespace {

constexpr int kTileW = 256, kTileH = 8;    // pixels per workgroup
constexpr int kBlock = 512;
constexpr int kRows = kTileW * kTileH / kBlock;      // rows per thread

// 4 floats at an address that is a multiple of 4 bytes.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

}  // namespace

template <int CH>
__global__ __launch_bounds__(kBlock) void k_image_cost(ImageCostArgs args) {
    // one rounding per operation (no fused multiply-adds)
#pragma clang fp contract(off)
    constexpr int SEG = (kTileW + 2) * CH;             // floats of a tile's row with its neighbours
    constexpr int CPR = (SEG + 3) / 4, PITCH = CPR * 4;
    constexpr int NROW = kTileH + 2, NC = NROW * CPR, LI = (NC + kBlock - 1) / kBlock;
    __shared__ alignas(16) float S[NROW * PITCH];
    // the image whose pixels this block takes: a binary search over the
    // ascending block bases
    const int im = find_pair(args.n, (int)blockIdx.x, [&](int i) { return args.img[i].block_base; });
    const ImageDesc& D = args.img[im];
    const int H = D.H, W = D.W;
    const int tx = (W + kTileW - 1) / kTileW;
    const int b = (int)blockIdx.x - D.block_base;
    const int x0 = (b % tx) * kTileW, y0 = (b / tx) * kTileH;
    const EPIC_GLOBAL float* const img = gmem(D.image);
    const int tid = threadIdx.x;
    // the tile's columns and one on each side, as far as the image reaches;
    // rows outside it repeat the border row
    const int xs = max(x0 - 1, 0), n = (min(x0 + kTileW + 1, W) - xs) * CH;
    f32x4u v[LI];
#pragma unroll
    for (int it = 0; it < LI; ++it) {
        const int i = tid + it * kBlock, ry = i / CPR, f = (i - ry * CPR) * 4;
        v[it] = f32x4u{0.0f, 0.0f, 0.0f, 0.0f};
        if (i < NC && f < n) {
            const int yy = min(max(y0 + ry - 1, 0), H - 1);
            const EPIC_GLOBAL float* const g = img + (long long)yy * W * CH + (xs * CH + f);
            if (f + 4 <= n) {
                v[it] = *reinterpret_cast<const EPIC_GLOBAL f32x4u*>(g);
            } else {
                v[it].x = g[0];
                if (f + 1 < n) v[it].y = g[1];
                if (f + 2 < n) v[it].z = g[2];
            }
        }
    }
#pragma unroll
    for (int it = 0; it < LI; ++it) {
        const int i = tid + it * kBlock;
        if (i < NC) *reinterpret_cast<float4*>(&S[i * 4]) = make_float4(v[it].x, v[it].y, v[it].z, v[it].w);
    }
    __syncthreads();
    const int x = x0 + tid % kTileW, r0 = tid / kTileW * kRows;
    if (x >= W) return;
    // the column's place in a row, and its neighbours' (the border pixel repeated)
    const int c = (x - xs) * CH, l = (max(x - 1, 0) - xs) * CH, r = (min(x + 1, W - 1) - xs) * CH;
    float up[CH], mid[CH], down[CH];
#pragma unroll
    for (int k = 0; k < CH; ++k) {
        up[k] = S[r0 * PITCH + c + k];
        mid[k] = S[(r0 + 1) * PITCH + c + k];
    }
    EPIC_GLOBAL float* const cost = gmem(D.cost);
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        const float* const row = &S[(r0 + j + 1) * PITCH];
        float s = 0.0f;
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            down[k] = row[PITCH + c + k];
            const float gx = 0.5f * (row[r + k] - row[l + k]);
            const float gy = 0.5f * (down[k] - up[k]);
            s = s + (gx * gx + gy * gy);
        }
        const int y = y0 + r0 + j;
        if (y < H) cost[(long long)y * W + x] = sqrtf(s) + args.eps;
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            up[k] = mid[k];
            mid[k] = down[k];
        }
    }
}

int image_cost_blocks(int H, int W) {
    return ((W + kTileW - 1) / kTileW) * ((H + kTileH - 1) / kTileH);
}

hipError_t launch_image_cost(const ImageCostArgs& args, int channels, int total_blocks, hipStream_t s) {
    switch (channels) {
        case 1: hipLaunchKernelGGL(k_image_cost<1>, dim3(total_blocks), dim3(kBlock), 0, s, args); break;
        case 2: hipLaunchKernelGGL(k_image_cost<2>, dim3(total_blocks), dim3(kBlock), 0, s, args); break;
        case 3: hipLaunchKernelGGL(k_image_cost<3>, dim3(total_blocks), dim3(kBlock), 0, s, args); break;
        case 4: hipLaunchKernelGGL(k_image_cost<4>, dim3(total_blocks), dim3(kBlock), 0, s, args); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace epic
