// D-SSIM part of the photometric loss (Sec. III-C: L_3DGS = (1 - lambda) L1 + lambda D-SSIM)
// and its adjoint with respect to the rendered colour, for all views in one launch.
//
// Per pixel p and channel: with G the 11 x 11 Gaussian window (sigma 1.5, weights summing to
// 1, zero padding), mu_x = G * x, E_xx = G * x^2, E_xy = G * (x y) (y = target),
//   A1 = 2 mu_x mu_y + C1,  A2 = 2 (E_xy - mu_x mu_y) + C2,
//   B1 = mu_x^2 + mu_y^2 + C1,  B2 = (E_xx - mu_x^2) + (E_yy - mu_y^2) + C2,  s = A1 A2 / (B1 B2).
// The loss adds sum_p m_p (1 - s_p) per channel, m_p = lambda w_l1 / (3 n_b) on the pixels of
// the L1 mask (all pixels without one).  Its adjoint: with the partial derivatives of s at
// fixed window moments
//   D_mu = 2 mu_y (A2 - A1) / (B1 B2) + 2 mu_x s (1 / B2 - 1 / B1),
//   D_xx = -s / B2,   D_xy = 2 A1 / (B1 B2),
// dL/dx_q = -[G * (m D_mu)](q) - 2 x_q [G * (m D_xx)](q) - y_q [G * (m D_xy)](q)
// (the window is symmetric, so the transposed blur is the blur).
//
// One workgroup of four waves per 44 x 30 output tile and colour channel.  The inputs with a 10-pixel
// halo are 64 columns wide, one per lane, so the column pass of the window moments runs from registers
// (a lane: 20 rows in, 10 rows out) and only its results go to LDS; the row pass forms the moments and
// D over the tile plus a 5-pixel halo, and D is blurred back onto the tile by rows, then columns, and
// combined with x and y.  A thread runs a blur over a short segment of one row or column with the
// segment's inputs in registers, so every LDS value read feeds several outputs.  E_xx and E_yy enter
// through their sum alone (B2), so x^2 + y^2 is blurred as one map: four maps, not five.
//
// What bounds it is vector issue, and the waits of the phases between barriers: 360 instructions a pixel
// and channel, halo included.  An f32 fma takes 2 cycles a wave with vector operands and 4 with a scalar
// one, so the window's six distinct weights are kept in vector registers.  The phases share 26 KB of LDS
// (two of the four maps at a time, then D, then its row blur), so that five workgroups of four waves
// run on a CU; with 50 KB and six waves it was two.  Three 1119 x 701 views: 136 us as 32 x 32 tiles of
// 512 threads with the inputs staged in LDS, 101 with the column pass from registers, 95 with the
// shared LDS, 78 with four waves; one 960 x 600 view 36 -> 26.
#include "common.h"

namespace ags {

constexpr int kSsimR = 5;                     // window radius
constexpr int kSsimTW = 44, kSsimTH = 30;     // output tile
constexpr int kSsimIW = kSsimTW + 4 * kSsimR; // 64: input columns with the double halo
constexpr int kSsimMW = kSsimTW + 2 * kSsimR; // 54 x 40: moments / D with the single halo
constexpr int kSsimMH = kSsimTH + 2 * kSsimR;
constexpr int kSsimThreads = 256;
constexpr int kSsimA = 10;  // column pass: rows a lane
constexpr int kSsimB = 9;   // moments: columns a lane
constexpr int kSsimC = 11;  // row pass of D: columns a lane
constexpr int kSsimD = 6;   // last column pass: rows a lane
constexpr float kSsimC1 = 0.01f * 0.01f;
constexpr float kSsimC2 = 0.03f * 0.03f;
static_assert(kSsimIW == 64 && kSsimMH == kSsimA * (kSsimThreads / 64), "a wave a row segment, a lane a column");
static_assert(kSsimMW % kSsimB == 0 && kSsimMW / kSsimB * kSsimMH <= kSsimThreads, "one item a thread");
static_assert(kSsimTW % kSsimC == 0 && kSsimTH % kSsimD == 0 && kSsimTH / kSsimD * kSsimTW <= kSsimThreads, "");

int ssim_tiles(const ViewTable& vt, int b) {
    return ((vt.width[b] + kSsimTW - 1) / kSsimTW) * ((vt.height[b] + kSsimTH - 1) / kSsimTH);
}

long long ssim_blocks(const ViewTable& vt) {
    long long t = 0;
    for (int b = 0; b < vt.n_views; ++b) t += ssim_tiles(vt, b);
    return 3 * t;
}

// Odd row strides, so that lanes of consecutive rows touch different banks.  26 KB.
union SsimShared {
    float v[2][kSsimMH][kSsimIW + 1];  // two of the column-blurred x, y, x^2 + y^2, x y
    float d[3][kSsimMH][kSsimMW + 1];
    float h[3][kSsimMH][kSsimTW + 1];  // row-blurred D
};

// Output o of an 11-tap blur whose inputs start at in[o]; wt[k] = weight of the taps at distance 5 - k.
template <int N>
__device__ __forceinline__ float ssim_tap(const float (&in)[N], int o, const float (&wt)[kSsimR + 1]) {
    float acc = wt[0] * in[o];
#pragma unroll
    for (int k = 1; k < 2 * kSsimR + 1; ++k) acc += wt[k <= kSsimR ? k : 2 * kSsimR - k] * in[o + k];
    return acc;
}

__global__ __launch_bounds__(kSsimThreads) void ssim_kernel(SsimArgs a) {
    __shared__ SsimShared sh;
    __shared__ unsigned long long son[kSsimMH];  // per middle row: input columns that take part in the loss
    __shared__ float sred[kSsimThreads / 64];
    const ViewTable& vt = a.vt;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = blockIdx.y;  // colour channel
    // view and tile of this workgroup
    int b = 0, t = blockIdx.x;
    while (b + 1 < vt.n_views && t >= a.tile_base[b + 1]) ++b;
    t -= a.tile_base[b];
    const int W = vt.width[b], H = vt.height[b];
    const int ntx = (W + kSsimTW - 1) / kSsimTW;
    const int ox = (t % ntx) * kSsimTW, oy = (t / ntx) * kSsimTH;
    const long long plane = (long long)W * H;
    const float* X = a.rgb + 3 * vt.pix_base[b] + c * plane;
    const float* Y = a.gt_rgb + 3 * vt.pix_base[b] + c * plane;
    float w[kSsimR + 1];
#pragma unroll
    for (int k = 0; k <= kSsimR; ++k) {
        w[k] = a.w[k];
        asm volatile("" : "+v"(w[k]));
    }

    float vs[2][kSsimA];
    // 1. column pass of x, y, x^2 + y^2, x y: input columns [ox - 2R, ox + TW + 2R), rows
    //    [oy - R, oy + TH + R); the inputs are zero outside the image
    {
        constexpr int kN = kSsimA + 2 * kSsimR;
        const int x = ox - 2 * kSsimR + lane, r0 = wave * kSsimA, y0 = oy - 2 * kSsimR + r0;
        const bool inx = x >= 0 && x < W;
        // rows are wave-uniform: a scalar row address and the lane's clamped column; what lies outside
        // the image becomes zero afterwards, in the workgroups that have any
        const uint32_t xc = (uint32_t)(x < 0 ? 0 : x < W ? x : W - 1);
        float u[kN], v[kN];
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            const int y = y0 + k < 0 ? 0 : y0 + k < H ? y0 + k : H - 1;
            u[k] = (X + (long long)y * W)[xc];
            v[k] = (Y + (long long)y * W)[xc];
        }
        if (ox < 2 * kSsimR || ox + kSsimTW + 2 * kSsimR > W || y0 < 0 || y0 + kN > H) {
#pragma unroll
            for (int k = 0; k < kN; ++k) {
                const bool in = inx && y0 + k >= 0 && y0 + k < H;
                u[k] = in ? u[k] : 0.f;
                v[k] = in ? v[k] : 0.f;
            }
        }
        // the mask is read here, where lanes hold consecutive columns
        bool on[kSsimA];
#pragma unroll
        for (int o = 0; o < kSsimA; ++o) {
            const int y = y0 + kSsimR + o;
            on[o] = inx && y >= 0 && y < H;
            if (a.mask && on[o]) on[o] = a.mask[vt.pix_base[b] + (long long)y * W + x] != 0;
        }
#pragma unroll
        for (int o = 0; o < kSsimA; ++o) {
            const unsigned long long bits = __builtin_amdgcn_ballot_w64(on[o]);
            if (lane == 0) son[r0 + o] = bits;
        }
#pragma unroll
        for (int o = 0; o < kSsimA; ++o) {
            sh.v[0][r0 + o][lane] = ssim_tap(u, o, w);
            sh.v[1][r0 + o][lane] = ssim_tap(v, o, w);
        }
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            const float xx = u[k] * u[k], xy = u[k] * v[k];
            u[k] = xx + v[k] * v[k];
            v[k] = xy;
        }
#pragma unroll
        for (int o = 0; o < kSsimA; ++o) {
            vs[0][o] = ssim_tap(u, o, w);
            vs[1][o] = ssim_tap(v, o, w);
        }
    }
    __syncthreads();

    // 2. row pass -> moments over the middle region; s, D and the loss there
    const float mscale = a.scale[b];
    float part = 0.f;
    float D[3][kSsimB];
    float mom[4][kSsimB];
    const int r2 = tid % kSsimMH, q2 = tid / kSsimMH * kSsimB;
    const bool item2 = q2 < kSsimMW;
    auto rows = [&](int to) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            float row[kSsimB + 2 * kSsimR];
#pragma unroll
            for (int k = 0; k < kSsimB + 2 * kSsimR; ++k) row[k] = sh.v[m][r2][q2 + k];
#pragma unroll
            for (int o = 0; o < kSsimB; ++o) mom[to + m][o] = ssim_tap(row, o, w);
        }
    };
    if (item2) rows(0);
    __syncthreads();
#pragma unroll
    for (int o = 0; o < kSsimA; ++o) {
        sh.v[0][wave * kSsimA + o][lane] = vs[0][o];
        sh.v[1][wave * kSsimA + o][lane] = vs[1][o];
    }
    __syncthreads();
    if (item2) {
        rows(2);
        const uint32_t on = (uint32_t)(son[r2] >> (q2 + kSsimR));
#pragma unroll
        for (int o = 0; o < kSsimB; ++o) {
            const int q = q2 + o;
            const float mx = mom[0][o], my = mom[1][o];
            const float A1 = 2.f * mx * my + kSsimC1;
            const float A2 = 2.f * (mom[3][o] - mx * my) + kSsimC2;
            const float B1 = mx * mx + my * my + kSsimC1;
            const float B2 = (mom[2][o] - mx * mx) - my * my + kSsimC2;
            const float rB1 = __builtin_amdgcn_rcpf(B1), rB2 = __builtin_amdgcn_rcpf(B2);
            const float iB = rB1 * rB2;
            const float s = A1 * A2 * iB;
            const float m = (on >> o) & 1u ? mscale : 0.f;
            D[0][o] = m * (2.f * my * (A2 - A1) * iB + 2.f * mx * s * (rB2 - rB1));
            D[1][o] = m * (-s * rB2);
            D[2][o] = m * (2.f * A1 * iB);
            if (r2 >= kSsimR && r2 < kSsimR + kSsimTH && q >= kSsimR && q < kSsimR + kSsimTW) part += m * (1.f - s);
        }
    }
    __syncthreads();  // D takes the place of the column-blurred maps
    if (item2) {
#pragma unroll
        for (int m = 0; m < 3; ++m)
#pragma unroll
            for (int o = 0; o < kSsimB; ++o) sh.d[m][r2][q2 + o] = D[m][o];
    }
    __syncthreads();

    // the last pass's x and y are asked for before the row pass, to arrive behind it
    const int q4 = tid % kSsimTW, r4 = tid / kSsimTW * kSsimD, x4 = ox + q4;
    const bool item4 = r4 < kSsimTH;
    float xv[kSsimD], yv[kSsimD];
#pragma unroll
    for (int o = 0; o < kSsimD; ++o) {
        const int y = oy + r4 + o;
        const bool in = item4 && x4 < W && y < H;
        const long long p = (long long)y * W + x4;
        xv[o] = in ? X[p] : 0.f;
        yv[o] = in ? Y[p] : 0.f;
    }

    // 3. row pass of m D onto the tile's columns
    constexpr int kN3 = 3 * kSsimMH * (kSsimTW / kSsimC), kRounds = (kN3 + kSsimThreads - 1) / kSsimThreads;
    float h[kRounds][kSsimC];
#pragma unroll
    for (int j = 0; j < kRounds; ++j) {
        const int it = tid + j * kSsimThreads;
        if (it < kN3) {
            const int r = it % kSsimMH, m = it / kSsimMH % 3, c0 = it / (3 * kSsimMH) * kSsimC;
            float row[kSsimC + 2 * kSsimR];
#pragma unroll
            for (int k = 0; k < kSsimC + 2 * kSsimR; ++k) row[k] = sh.d[m][r][c0 + k];
#pragma unroll
            for (int o = 0; o < kSsimC; ++o) h[j][o] = ssim_tap(row, o, w);
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kRounds; ++j) {
        const int it = tid + j * kSsimThreads;
        if (it < kN3) {
            const int r = it % kSsimMH, m = it / kSsimMH % 3, c0 = it / (3 * kSsimMH) * kSsimC;
#pragma unroll
            for (int o = 0; o < kSsimC; ++o) sh.h[m][r][c0 + o] = h[j][o];
        }
    }
    __syncthreads();

    // 4. column pass onto the tile; combine with x and y
    if (item4) {
        float g[3][kSsimD];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            float col[kSsimD + 2 * kSsimR];
#pragma unroll
            for (int k = 0; k < kSsimD + 2 * kSsimR; ++k) col[k] = sh.h[m][r4 + k][q4];
#pragma unroll
            for (int o = 0; o < kSsimD; ++o) g[m][o] = ssim_tap(col, o, w);
        }
#pragma unroll
        for (int o = 0; o < kSsimD; ++o) {
            const int y = oy + r4 + o;
            if (x4 < W && y < H)
                a.d_rgb[3 * vt.pix_base[b] + c * plane + (long long)y * W + x4] =
                    -(g[0][o] + 2.f * xv[o] * g[1][o] + yv[o] * g[2][o]);
        }
    }

    // workgroup sum of the loss part, one partial per workgroup
    part = wave_sum(part);
    if (lane == 0) sred[wave] = part;
    __syncthreads();
    if (tid == 0) {
        float s = 0.f;
        for (int i = 0; i < kSsimThreads / 64; ++i) s += sred[i];
        a.partials[(long long)blockIdx.y * gridDim.x + blockIdx.x] = s;
    }
}

void launch_ssim(SsimArgs a, hipStream_t s) {
    int tb = 0;
    for (int b = 0; b < a.vt.n_views; ++b) {
        a.tile_base[b] = tb;
        tb += ssim_tiles(a.vt, b);
    }
    a.tile_base[a.vt.n_views] = tb;
    if (tb == 0) return;
    // the zero-mean-free Gaussian window, normalised in double
    double wd[2 * kSsimR + 1], sum = 0.0;
    for (int k = 0; k <= 2 * kSsimR; ++k) {
        const double d = k - kSsimR;
        wd[k] = std::exp(-d * d / (2.0 * 1.5 * 1.5));
        sum += wd[k];
    }
    for (int k = 0; k <= 2 * kSsimR; ++k) a.w[k] = (float)(wd[k] / sum);
    hipLaunchKernelGGL(ssim_kernel, dim3(tb, 3), dim3(kSsimThreads), 0, s, a);
}

}  // namespace ags
