// Tile rasterisation of all views in one launch: forward compositing and its adjoint.
//
// A workgroup owns one T x T tile of one view (the global tile id selects the view), so a
// rig's views and a set of submaps share one launch.  Its waves own 8 x 8 blocks of the tile (one
// pixel a lane) or 8 x 16 blocks (two, eight rows apart) and work independently: a wave streams
// the tile's depth-ordered list 64 entries at a time, one per lane, keeps those whose alpha >=
// alpha_min ellipse reaches its own block (block_reached), packs them in order into LDS rows of its
// own and composites them front to back (Sec. III-B, standard 3DGS):
//   power = -1/2 (a dx^2 + c dy^2) - b dx dy, (dx, dy) = (u, v) - pixel centre
//   alpha = min(alpha_max, o e^power), skipped when power > 0 or alpha < alpha_min
//   T' = T (1 - alpha); stop (excluding this Gaussian) when T' < t_min
//   C += alpha T rgb; D += alpha T z; T = T'
// and the accumulated alpha A = sum alpha T is written as 1 - T_final (the same sum, not
// accumulated in the loop).  A wave ends when its pixels have stopped; there is no barrier in
// the loops.  The forward keeps 8 bytes per pixel (final T and the list position of the last
// contributor) so the backward recomputes transmittance instead of storing per-pixel blend
// lists.
//
// The backward walks the list back to front from the last contributor, recovering
// T_k = T_{k+1} / (1 - alpha_k) and accumulating suffix sums S = sum_{j>k} w_j f_j:
//   dL/dalpha_k = T_k (gC . c_k + gD z_k + gA)
//                 - (gC . S^C + gD S^D + gA S^A + T_final gC . bg) / (1 - alpha_k)
// (the bracket is kept as one running sum U), then chains through alpha = o e^power (unless
// clamped) to p = dL/dpower = alpha dL/dalpha, of which it keeps the sum (= o dL/do) and five pixel
// moments (sum p dx, p dy, p dx^2, p dx dy, p dy^2); the projection backward turns them into the
// opacity, centre and conic adjoints.  dL/drgb_k = w_k gC, dL/dz_k = w_k gD.  The ten per-Gaussian
// sums of a wave are reduced over its lanes (wave_column_sums) and one atomic instruction of ten
// lanes adds them into the pair's 64-byte adjoint row.
//
// What bounds both kernels is vector instruction issue.  Measured on one SIMD with eight waves, a
// wave64 instruction takes: 2 cycles for add / mul / fma f32 and moves with vector operands, 4 with a
// scalar operand and for compares, selects, min / max and DPP, 8 for exp / rcp and the lane swaps;
// scalar instructions issue one per 4 cycles and a 16-byte LDS read of one address by all lanes
// takes 5 of the CU's LDS cycles.  The loops are built for those costs: the per-pixel tests that
// only an odd record needs (p2 <= 0, the alpha clamp) are made only for chunks that hold one, keep
// decisions stay in scalar lane masks, and the records are read from consecutive LDS rows instead
// of by scalar bit scans (which bound an earlier form of the forward at 85 % scalar issue).
// 8 x 16 blocks share dx and the record reads between two pixels and halve the per-chunk work, 8 x 8
// blocks give a launch twice the waves, each with half the serial work: launches of at least 8192
// waves of 8 x 16 blocks (what the chip holds) take the former, others the latter (wide_blocks).
#include <type_traits>

#include "common.h"

namespace ags {

struct TileCoord {
    int b, px0, py0, W, H;
    long long pix0;  // first pixel of the view in the flat image buffers
};

__device__ __forceinline__ TileCoord tile_coord(const ViewTable& vt, int tile) {
    TileCoord c;
    c.b = view_of_tile(vt, tile);
    int local = tile - vt.tile_base[c.b];
    int ntx = vt.ntx[c.b];
    c.px0 = (local % ntx) * vt.tile;
    c.py0 = (local / ntx) * vt.tile;
    c.W = vt.width[c.b];
    c.H = vt.height[c.b];
    c.pix0 = vt.pix_base[c.b];
    return c;
}

using f32x4 = __attribute__((ext_vector_type(4))) float;
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kChunk = 64;  // list entries a wave takes at a time

// Whether the alpha >= alpha_min ellipse of the record (u, v, a, b | c, o) may reach the pixel
// centres of the block whose first one is (X0, Y0) and whose last one is (X0 + wx, Y0 + wy).  The
// quadratic form is convex with its minimum at the centre, so its minimum over the rectangle lies
// on a side facing the centre: the nearer vertical and the nearer horizontal side, each at its own
// minimiser clamped to the side.  The level is 2 ln(o / alpha_min) itself (the binning rebuilds it from
// the footprint box, whose determinant cancels for a thin ellipse), widened by 2e-3 of itself, 1e-3,
// and the rounding of the form at the far corner (its terms may cancel); NaN keeps the record.
__device__ __forceinline__ bool block_reached(const float4& r0, float c, float o, float inv_amin, float X0, float Y0,
                                              float wx, float wy) {
    const float a = r0.z, b = r0.w, b2 = 2.f * b;
    const float lx = X0 - r0.x, hx = lx + wx, ly = Y0 - r0.y, hy = ly + wy;
    const float fx = fmaxf(fabsf(lx), fabsf(hx)), fy = fmaxf(fabsf(ly), fabsf(hy));
    const float tau2 = 2.004f * __logf(o * inv_amin) + 1e-3f + 2e-6f * (a * fx * fx + c * fy * fy);
    const float X = __builtin_amdgcn_fmed3f(0.f, lx, hx), Y = __builtin_amdgcn_fmed3f(0.f, ly, hy);
    const float y = __builtin_amdgcn_fmed3f(-b * __builtin_amdgcn_rcpf(c) * X, ly, hy);
    const float x = __builtin_amdgcn_fmed3f(-b * __builtin_amdgcn_rcpf(a) * Y, lx, hx);
    const float q1 = X * (a * X + b2 * y) + c * y * y;
    const float q2 = x * (a * x + b2 * Y) + c * Y * Y;
    return !(q1 > tau2 && q2 > tau2);
}

// Whether the exponent of a record may round above 0 or its alpha reach the clamp, so that both
// tests have to be made per pixel: a conic (A', B', C', pre-scaled) that is not definite by a margin
// far above rounding, an opacity above alpha_max, NaN.
__device__ __forceinline__ bool needs_tests(float A, float B, float C, float o, float amax) {
    return !(o <= amax && A < 0.f && C < 0.f && B * B < 3.9999f * (A * C));
}

// The base-2 exponent A' dx^2 + B' dx dy + C' dy^2 in one fixed order of roundings for both block shapes.
// (SHARED, the backward of several pixels a thread: they share A' dx instead, which rounds the other of the two
// products, as that shape always did.  Its alpha may differ from the forward's in the last bit, so a pair at the
// cutoff is kept by one of the two only, a few pixels in 10^7: there T comes back wrong by 1 - alpha_min for the
// nearer entries.  One order for both takes no longer, 4-view step 1161 us, but is not nearer to float64, since the
// forward's own rounding puts as many pairs across the cutoff, and moves a variance-weighted step's pose gradient
// by up to 8e-5 of its norm.)
__device__ __forceinline__ float exponent2(float A, float B, float C, float dx, float dy) {
    return __builtin_fmaf(dy, dy * C, dx * __builtin_fmaf(dx, A, dy * B));
}

// Lane mask of a <= b, and this lane's bit of a wave-uniform mask.
__device__ __forceinline__ unsigned long long le_mask(float a, float b) {
    return __builtin_amdgcn_fcmpf(a, b, 5);  // ordered, less or equal
}
__device__ __forceinline__ bool lane_of(unsigned long long m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
__device__ __forceinline__ int rank_in(unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Whether a record's colour or depth is infinite, NaN or beyond 1e15 (in any channel, or their sum): 0 times it
// may then not be 0, so it stays out of sums that also run over pixels which do not keep the record.
__device__ __forceinline__ bool unbounded(float r, float g, float b, float z) {
    return !(fabsf(r) + fabsf(g) + fabsf(b) + fabsf(z) <= 1e15f);
}

// Keeps a value in a vector register from here on.
template <typename V>
__device__ __forceinline__ void in_vgpr(V& v) {
    asm volatile("" : "+v"(v));
}

// Issue priority of a wave by the entries it has ahead of it.  Eight waves share a SIMD, so at equal
// priority a tile with a long list advances at an eighth of the SIMD's rate and ends after the rest of
// the launch, although the longest lists start first (see kWorkStrip): raster backward of a
// 2M-Gaussian 4-view step 534 -> 475 us, of a 22-view 2.9M sub-map step 1217 -> 1180 us.
__device__ __forceinline__ void prio_by_length(int n) {
    if (n >= 512) __builtin_amdgcn_s_setprio(3);
    else if (n >= 256) __builtin_amdgcn_s_setprio(2);
    else if (n >= 128) __builtin_amdgcn_s_setprio(1);
}

// A wave's loads of a list: lane l holds the record of one entry.
struct Rec {
    float4 a, b, c;  // u v a b | c o z ex | ey r g b
};
__device__ __forceinline__ Rec load_rec(const float* records, uint32_t q) {
    const float4* r = reinterpret_cast<const float4*>(records + (long long)q * kRecFloats);
    return {r[0], r[1], r[2]};
}

// A wave's LDS rows: the records of a chunk that reach its block, in list order, then PAD fillers
// (opacity 0) for the last group; the conic (a, b, c) becomes log2(e) (-a/2, -b, -c/2), so that the
// exponent in base 2 is exponent2 and e^power one instruction.
template <int PAD>
struct Rows {
    float4 g[kChunk + PAD];    // u v A' B'
    float4 col[kChunk + PAD];  // r g b z
    float2 co[kChunk + PAD];   // C' o
    uint32_t pos[kChunk + PAD];
    // Packs the lanes' records with `in` set and returns how many there are; `slow` if any of them, with the
    // opacity `o` (the record's), needs the per-pixel tests.
    __device__ __forceinline__ int pack(const Rec& r, float o, bool in, uint32_t position, float amax, bool& slow) {
        const unsigned long long im = __builtin_amdgcn_ballot_w64(in);
        const int n = __popcll(im), at = rank_in(im);
        const float A = -0.5f * kLog2e * r.a.z, B = -kLog2e * r.a.w, C = -0.5f * kLog2e * r.b.x;
        slow = __builtin_amdgcn_ballot_w64(in && needs_tests(A, B, C, o, amax)) != 0ull;
        if (in) {
            g[at] = make_float4(r.a.x, r.a.y, A, B);
            co[at] = make_float2(C, r.b.y);
            col[at] = make_float4(r.c.y, r.c.z, r.c.w, r.b.z);
            pos[at] = position;
        }
        const int lane = __lane_id();
        if (lane < PAD) {
            g[n + lane] = col[n + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
            co[n + lane] = make_float2(0.f, 0.f);
            pos[n + lane] = 0u;
        }
        __builtin_amdgcn_wave_barrier();
        return n;
    }
};

// The rendered depth variance sum w z^2 - (sum w z)^2 (rendered-variance LiDAR term), accumulated
// without cancellation: the weighted scatter S about the running normalised mean m (A' = A + w,
// m' = m + (z - m) w / A', S' = S + w (z - m)(z - m')), then sum w z^2 - (A m)^2 =
// S + A (1 - A) m^2 with 1 - A = the final transmittance.  One fixed order of roundings for both block
// shapes.
struct Scatter {
    float A = 0.f, m = 0.f, S = 0.f;
    __device__ __forceinline__ void add(float alpha, float T, float z) {
        const float w = alpha * T;
        A = __builtin_fmaf(alpha, T, A);
        const float dz = z - m;
        m = __builtin_fmaf(dz, w * __builtin_amdgcn_rcpf(A), m);
        S = __builtin_fmaf(w * dz, z - m, S);
    }
    __device__ __forceinline__ float variance(float T) const { return __builtin_fmaf(A * T * m, m, S); }
};

__device__ __forceinline__ void write_pixel(const RasterArgs& a, const TileCoord& tc, int x, int y, float r, float g,
                                            float b, float D, float T, uint32_t last, const Scatter* var) {
    const long long plane = (long long)tc.W * tc.H, p = (long long)y * tc.W + x, gp = tc.pix0 + p;
    float* rgb = a.rgb + 3 * tc.pix0;
    rgb[p] = r + T * a.st.bg0;
    rgb[plane + p] = g + T * a.st.bg1;
    rgb[2 * plane + p] = b + T * a.st.bg2;
    a.depth[gp] = D;
    if (var) a.depth_var[gp] = var->variance(T);
    a.alpha[gp] = 1.f - T;
    a.t_final[gp] = T;
    a.last[gp] = last;
    if (a.zero_px[0]) a.zero_px[0][gp] = 0.f;
    if (a.zero_px[1]) a.zero_px[1][gp] = 0.f;
}

// ------------------------------------------------------------------------- forward
//
// 8 x 8 blocks, one pixel a lane, four entries a step: their exponents are formed side by side and
// only T is carried from one to the next, because the launches that come here have too few waves to
// hide a serial chain (one 960 x 600 view over 300k Gaussians: 102 -> 47 us; two 161 x 119 views over
// 4k: 22 -> 12 us).  The colour is a contraction over the entries, C[ch][pixel] += c[ch] w[pixel], which
// v_mfma_f32_4x4x1_16b_f32 does with the pixel's four sums in its own lane: one LDS read a step gives
// the colours of all four entries, where broadcast reads kept the LDS 80 % busy.  It rounds like the
// four fmas it replaces, but runs over all lanes, of which those that do not keep the entry have w = 0: a
// chunk with an infinite colour takes the fmas, on the lanes that keep it.  S2: also output the rendered
// depth variance.
template <int T, bool S2>
__global__ __launch_bounds__(T* T) void raster_fwd_kernel(RasterArgs a) {
    constexpr int NW = T * T / 64, COLS = T / 8, GRP = 4;
    __shared__ Rows<GRP> rows[NW];
    const uint32_t wt = a.work[blockIdx.x];
    if (wt == kNoTile) return;  // padding of a shorter XCD list
    const int tile = (int)wt;
    const TileCoord tc = tile_coord(a.vt, tile);
    const uint32_t start = __builtin_amdgcn_readfirstlane(a.ranges[2 * tile]);
    const uint32_t end = __builtin_amdgcn_readfirstlane(a.ranges[2 * tile + 1]);
    const int lane = __lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Rows<GRP>& my = rows[wave];

    const int bx = tc.px0 + (wave % COLS) * 8, by = tc.py0 + (wave / COLS) * 8;
    const int px = bx + (lane & 7), py = by + (lane >> 3);
    const float cx = (float)px + 0.5f, cy = (float)py + 0.5f;
    const float X0 = (float)bx + 0.5f, Y0 = (float)by + 0.5f;
    const bool inside = px < tc.W && py < tc.H;
    unsigned long long open = __builtin_amdgcn_ballot_w64(inside);  // lanes whose pixel has not stopped
    float Tr = 1.f;
    f32x4 C = {0.f, 0.f, 0.f, 0.f};  // r, g, b, expected depth
    Scatter var;
    uint32_t last = 0;
    const float amin = a.st.alpha_min, tmin = a.st.t_min;
    const float amax = __builtin_canonicalizef(a.st.alpha_max);
    const float inv_amin = 1.f / amin;

    // a chunk's records are loaded while the chunk before it is composited, its pair ids one chunk
    // earlier still
    auto id_of = [&](uint32_t e) { return a.tile_pairs[e < end ? e : end - 1]; };
    Rec next = {};
    uint32_t nq = 0;
    if (start < end) {
        next = load_rec(a.records, id_of(start + lane));
        nq = id_of(start + kChunk + lane);
    }
    for (uint32_t bs = start; bs < end && open != 0ull; bs += kChunk) {
        const Rec r = next;
        if (bs + kChunk < end) {
            next = load_rec(a.records, nq);
            nq = id_of(bs + 2 * kChunk + lane);
        }
        const uint32_t e = bs + lane;
        const bool in = e < end && block_reached(r.a, r.b.x, r.b.y, inv_amin, X0, Y0, 7.f, 7.f);
        // `slow` also for an infinite colour or depth: 0 times the largest (none is below 0) makes this opacity NaN.
        // A ballot of its own lengthened the chain of a long list (six 64 x 48 views over 300k: 2230 -> 2335 us).
        const float o = __builtin_fmaf(0.f, fmaxf(fmaxf(fmaxf(r.c.y, r.c.z), r.c.w), r.b.z), r.b.y);
        bool slow;
        const int n = my.pack(r, o, in, e - start + 1, amax, slow);
        int lastc = -1;  // the last contributor's row in this chunk
        auto run = [&](auto tests, auto matrix) {
            int row = 0;
            in_vgpr(row);
            for (int g = 0; g < n && open != 0ull; g += GRP, row += GRP) {
                // lanes 4 i .. 4 i + 3 hold the channels of the step's entry i (i < 4)
                float colv = 0.f;
                if (decltype(matrix)::value) colv = reinterpret_cast<const float*>(my.col + g)[lane & 15];
                float4 r0[GRP];
                float2 r1[GRP];
#pragma unroll
                for (int i = 0; i < GRP; ++i) {
                    r0[i] = my.g[g + i];
                    r1[i] = my.co[g + i];
                }
                float al[GRP];
                unsigned long long kp[GRP];  // lanes that keep the pair, open or not
#pragma unroll
                for (int i = 0; i < GRP; ++i) {
                    const float p2 = exponent2(r0[i].z, r0[i].w, r1[i].x, r0[i].x - cx, r0[i].y - cy);
                    al[i] = r1[i].y * __builtin_amdgcn_exp2f(p2);
                    if (decltype(tests)::value) al[i] = fminf(amax, al[i]);
                    kp[i] = le_mask(amin, al[i]);
                    if (decltype(tests)::value) kp[i] &= le_mask(p2, 0.f);
                    in_vgpr(al[i]);  // formed here, not inside the branches below
                }
                // the entry index is an immediate of the matrix instruction
                auto blend = [&](auto entry) {
                    constexpr int i = decltype(entry)::value;
                    const unsigned long long km = kp[i] & open;
                    if (km == 0ull) return;  // wave-uniform
                    // stop before a Gaussian that would take T below t_min; T (1 - alpha), one
                    // rounding, is the next T
                    const float Tn = __builtin_fmaf(-al[i], Tr, Tr);
                    const unsigned long long go = le_mask(tmin, Tn) & km;
                    open &= ~(km ^ go);
                    if (decltype(matrix)::value) {
                        const float w = lane_of(go) ? al[i] * Tr : 0.f;
                        C = __builtin_amdgcn_mfma_f32_4x4x1f32(colv, w, C, 4, i, 0);
                    }
                    if (lane_of(go)) {
                        if (!decltype(matrix)::value) {
                            const float4 c = my.col[g + i];
                            const float w = al[i] * Tr;
                            C[0] = __builtin_fmaf(w, c.x, C[0]);
                            C[1] = __builtin_fmaf(w, c.y, C[1]);
                            C[2] = __builtin_fmaf(w, c.z, C[2]);
                            C[3] = __builtin_fmaf(w, c.w, C[3]);
                        }
                        if (S2) var.add(al[i], Tr, my.col[g + i].w);
                        Tr = Tn;
                        lastc = row + i;
                    }
                };
                blend(std::integral_constant<int, 0>{});
                blend(std::integral_constant<int, 1>{});
                blend(std::integral_constant<int, 2>{});
                blend(std::integral_constant<int, 3>{});
            }
        };
        if (!slow) run(std::false_type{}, std::true_type{});
        else if (__builtin_amdgcn_ballot_w64(in && o != o) == 0ull) run(std::true_type{}, std::true_type{});
        else run(std::true_type{}, std::false_type{});
        if (lastc >= 0) last = my.pos[lastc];
        __builtin_amdgcn_wave_barrier();
    }
    if (inside) write_pixel(a, tc, px, py, C[0], C[1], C[2], C[3], Tr, last, S2 ? &var : nullptr);
}

// 8 x 16 blocks, two pixels a lane eight rows apart (the same dx), two entries a step, plain fmas: one
// read of a record serves two pixels, which keeps the LDS behind the vector units.  4-view 1280 x 800
// step over 1M Gaussians 195 -> 173 us, over 2M 246 -> 204 us.
// No prefetch: it costs two of eight waves a SIMD (rig step 177 -> 192 us).
template <int T, bool S2>
__global__ __launch_bounds__(T* T / 2) void raster_fwd_wide_kernel(RasterArgs a) {
    constexpr int NW = T * T / 128, COLS = T / 8, GRP = 2, PPT = 2;
    __shared__ Rows<GRP> rows[NW];
    const uint32_t wt = a.work[blockIdx.x];
    if (wt == kNoTile) return;  // padding of a shorter XCD list
    const int tile = (int)wt;
    const TileCoord tc = tile_coord(a.vt, tile);
    const uint32_t start = __builtin_amdgcn_readfirstlane(a.ranges[2 * tile]);
    const uint32_t end = __builtin_amdgcn_readfirstlane(a.ranges[2 * tile + 1]);
    const int lane = __lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Rows<GRP>& my = rows[wave];
    const int bx = tc.px0 + (wave % COLS) * 8, by = tc.py0 + (wave / COLS) * 16;
    const int px = bx + (lane & 7), py = by + (lane >> 3);
    const float cx = (float)px + 0.5f;
    float cy[PPT], Tr[PPT], C0[PPT], C1[PPT], C2[PPT], D[PPT];
    Scatter var[PPT];
    uint32_t last[PPT];
    unsigned long long open[PPT];  // lanes whose pixel is in the image and has not stopped
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        cy[k] = (float)(py + 8 * k) + 0.5f;
        open[k] = __builtin_amdgcn_ballot_w64(px < tc.W && py + 8 * k < tc.H);
        Tr[k] = 1.f;
        C0[k] = C1[k] = C2[k] = D[k] = 0.f;
        last[k] = 0;
    }
    prio_by_length((int)(end - start));
    const float amin = a.st.alpha_min, tmin = a.st.t_min;
    const float amax = __builtin_canonicalizef(a.st.alpha_max);
    const float inv_amin = 1.f / amin;
    const float X0 = (float)bx + 0.5f, Y0 = (float)by + 0.5f;

    for (uint32_t bs = start; bs < end && (open[0] | open[1]) != 0ull; bs += kChunk) {
        const uint32_t e = bs + lane;
        const Rec r = load_rec(a.records, a.tile_pairs[e < end ? e : end - 1]);
        // a half whose pixels have stopped takes no more entries
        const float top = open[0] ? Y0 : Y0 + 8.f, span = open[0] && open[1] ? 15.f : 7.f;
        const bool in = e < end && block_reached(r.a, r.b.x, r.b.y, inv_amin, X0, top, 7.f, span);
        bool slow;
        const int n = my.pack(r, r.b.y, in, e - start + 1, amax, slow);
        int lastc[PPT] = {-1, -1};  // the last contributor's row in this chunk
        auto run = [&](auto tests) {
            int row = 0;
            in_vgpr(row);
            for (int g = 0; g < n; g += GRP, row += GRP) {
                float4 r0[GRP], rc[GRP];
                float2 r1[GRP];
#pragma unroll
                for (int i = 0; i < GRP; ++i) {
                    r0[i] = my.g[g + i];
                    r1[i] = my.co[g + i];
                    rc[i] = my.col[g + i];
                }
                float al[GRP][PPT];
                unsigned long long kp[GRP][PPT];  // lanes that keep the pair, open or not
#pragma unroll
                for (int i = 0; i < GRP; ++i) {
                    const float dx = r0[i].x - cx;
#pragma unroll
                    for (int k = 0; k < PPT; ++k) {
                        const float p2 = exponent2(r0[i].z, r0[i].w, r1[i].x, dx, r0[i].y - cy[k]);
                        al[i][k] = r1[i].y * __builtin_amdgcn_exp2f(p2);
                        if (decltype(tests)::value) al[i][k] = fminf(amax, al[i][k]);
                        kp[i][k] = le_mask(amin, al[i][k]);
                        if (decltype(tests)::value) kp[i][k] &= le_mask(p2, 0.f);
                        in_vgpr(al[i][k]);  // formed here, not inside the branches below
                    }
                }
#pragma unroll
                for (int i = 0; i < GRP; ++i) {
#pragma unroll
                    for (int k = 0; k < PPT; ++k) {
                        const unsigned long long km = kp[i][k] & open[k];
                        if (km == 0ull) continue;  // wave-uniform
                        // the stop test as above
                        const float Tn = __builtin_fmaf(-al[i][k], Tr[k], Tr[k]);
                        const unsigned long long go = le_mask(tmin, Tn) & km;
                        open[k] &= ~(km ^ go);
                        if (lane_of(go)) {
                            const float w = al[i][k] * Tr[k];
                            C0[k] = __builtin_fmaf(w, rc[i].x, C0[k]);
                            C1[k] = __builtin_fmaf(w, rc[i].y, C1[k]);
                            C2[k] = __builtin_fmaf(w, rc[i].z, C2[k]);
                            D[k] = __builtin_fmaf(w, rc[i].w, D[k]);
                            if (S2) var[k].add(al[i][k], Tr[k], rc[i].w);
                            Tr[k] = Tn;
                            lastc[k] = row + i;
                        }
                    }
                }
            }
        };
        if (slow) run(std::true_type{});
        else run(std::false_type{});
#pragma unroll
        for (int k = 0; k < PPT; ++k)
            if (lastc[k] >= 0) last[k] = my.pos[lastc[k]];
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int k = 0; k < PPT; ++k)
        if (px < tc.W && py + 8 * k < tc.H)
            write_pixel(a, tc, px, py + 8 * k, C0[k], C1[k], C2[k], D[k], Tr[k], last[k], S2 ? &var[k] : nullptr);
}

// Several pixels a thread, and many tiles: the workgroup stages its tile's list in LDS, M entries at a
// time, thread t covers column t % T and PPT rows.  It is here for that shape's images alone: the compiler
// forms the exponents of a thread's pixels in different orders of roundings, so the one order of the
// block kernels moves alpha by an ulp, which is across the cutoff for a few pixels in 10^7 (images up to
// 2.8e-3 of their root mean square off).  It is as fast as the wide blocks for 22 views at (16, 64, 4), 507 and 500
// us, and slower elsewhere: four 1280 x 800 views 260 us at (16, 256, 2), 429 at (16, 64, 4), 683 at (32, 512, 2),
// 1211 at (32, 256, 4), where the wide blocks take 190 to 210.
struct alignas(16) StagedRec {
    float4 m, g0;  // z r g b | u v A' B'
    float2 g1;     // C' o
};

template <int T, int PPT, int M, bool S2>
__global__ __launch_bounds__(T* T / PPT) void raster_fwd_staged_kernel(RasterArgs a) {
    constexpr int NT = T * T / PPT;
    __shared__ StagedRec srec[M];
    const uint32_t wt = a.work[blockIdx.x];
    if (wt == kNoTile) return;  // padding of a shorter XCD list (whole workgroup)
    const int tile = (int)wt;
    const TileCoord tc = tile_coord(a.vt, tile);
    const uint32_t start = __builtin_amdgcn_readfirstlane(a.ranges[2 * tile]);
    const uint32_t end = __builtin_amdgcn_readfirstlane(a.ranges[2 * tile + 1]);
    const int tid = threadIdx.x;

    // A pixel that has stopped (or lies outside the image) gets cx = +inf: its exponent is
    // then -inf (or NaN), below every threshold, so it keeps no further Gaussian without a
    // separate flag test.
    constexpr float kStopped = __builtin_huge_valf();
    float cx[PPT], cy[PPT], Tr[PPT], C0[PPT], C1[PPT], C2[PPT], D[PPT], A[PPT], Mn[PPT], Sc[PPT];
    uint32_t last[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int lx = tid % T, ly = (tid / T) * PPT + k;
        const int px = tc.px0 + lx, py = tc.py0 + ly;
        cx[k] = (px < tc.W && py < tc.H) ? (float)px + 0.5f : kStopped;
        cy[k] = (float)py + 0.5f;
        Tr[k] = 1.f;
        C0[k] = C1[k] = C2[k] = D[k] = A[k] = Mn[k] = Sc[k] = 0.f;
        last[k] = 0;
    }
    const float amin = a.st.alpha_min, tmin = a.st.t_min;
    const float amax = __builtin_canonicalizef(a.st.alpha_max);

    for (uint32_t bs = start; bs < end; bs += M) {
        bool any = false;
#pragma unroll
        for (int k = 0; k < PPT; ++k) any |= cx[k] != kStopped;
        if (__syncthreads_count(any) == 0) break;
#pragma unroll
        for (int l = tid; l < M; l += NT) {
            const uint32_t e = bs + l;
            if (e < end) {
                const Rec r = load_rec(a.records, a.tile_pairs[e]);
                srec[l].m = make_float4(r.b.z, r.c.y, r.c.z, r.c.w);
                srec[l].g0 = make_float4(r.a.x, r.a.y, -0.5f * kLog2e * r.a.z, -kLog2e * r.a.w);
                srec[l].g1 = make_float2(-0.5f * kLog2e * r.b.x, r.b.y);
            }
        }
        __syncthreads();
        const uint32_t bend = end - bs > (uint32_t)M ? bs + M : end;
        const char* sbase = reinterpret_cast<const char*>(srec);
        uint32_t off = 0;  // byte offset of record e - bs in LDS
        in_vgpr(off);
        // entries in groups of eight: the later records are read at immediate offsets from the
        // first's LDS address, so the address advances once per group, and the wave's early
        // exit is tested once per group (entries past a wave's stop keep nothing: a stopped
        // pixel's exponent is -inf or NaN)
        auto entry = [&](const StagedRec& r, uint32_t e) {
            const float4 r0 = r.g0;
            const float2 r1 = r.g1;  // (C', o)
            // all of the record's reads are issued here, before the tests that use them
            asm volatile("" ::"v"(r0.x), "v"(r0.y), "v"(r0.z), "v"(r0.w), "v"(r1.x), "v"(r1.y));
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                // one predicate, one branch: the exp is cheap next to divergent control
                const float dx = r0.x - cx[k], dy = r0.y - cy[k];
                const float p2 = dx * (r0.z * dx + r0.w * dy) + r1.x * dy * dy;
                const float alpha = fminf(amax, r1.y * __builtin_amdgcn_exp2f(p2));
                const bool keep = p2 <= 0.f && alpha >= amin;
                if (keep) {
                    // stop (once per pixel) before a Gaussian that would take T below t_min;
                    // the tested T (1 - alpha), one rounding, is the next T
                    const float Tn = __builtin_fmaf(-alpha, Tr[k], Tr[k]);
                    const bool go = Tn >= tmin;
                    cx[k] = go ? cx[k] : kStopped;  // +inf marks the pixel stopped
                    in_vgpr(cx[k]);                 // one select here, not moves in both branches
                    if (go) {
                        const float4 rc = r.m;  // (z, r, g, b)
                        const float w = alpha * Tr[k];
                        C0[k] += w * rc.y;
                        C1[k] += w * rc.z;
                        C2[k] += w * rc.w;
                        D[k] += w * rc.x;
                        if (S2) {
                            A[k] += w;
                            const float dz = rc.x - Mn[k];
                            Mn[k] += dz * (w * __builtin_amdgcn_rcpf(A[k]));
                            Sc[k] += w * dz * (rc.x - Mn[k]);
                        }
                        Tr[k] = Tn;
                        last[k] = e - start + 1;
                    }
                }
            }
        };
        auto wave_live = [&]() {
            bool live = false;
#pragma unroll
            for (int k = 0; k < PPT; ++k) live |= cx[k] != kStopped;
            return __ballot(live) != 0ull;  // wave-uniform: false once every pixel has stopped
        };
        for (uint32_t e = bs; e < bend; e += 8, off += 8 * sizeof(StagedRec)) {
            if (!wave_live()) break;
            entry(*reinterpret_cast<const StagedRec*>(sbase + off), e);
#pragma unroll
            for (int g = 1; g < 8; ++g) {
                if (e + g == bend) break;
                entry(*reinterpret_cast<const StagedRec*>(sbase + off + g * sizeof(StagedRec)), e + g);
            }
        }
        __syncthreads();
    }
    const long long plane = (long long)tc.W * tc.H;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int lx = tid % T, ly = (tid / T) * PPT + k;
        if (tc.px0 + lx >= tc.W || tc.py0 + ly >= tc.H) continue;
        const long long p = (long long)(tc.py0 + ly) * tc.W + (tc.px0 + lx);
        const long long gp = tc.pix0 + p;
        float* rgb = a.rgb + 3 * tc.pix0;
        rgb[p] = C0[k] + Tr[k] * a.st.bg0;
        rgb[plane + p] = C1[k] + Tr[k] * a.st.bg1;
        rgb[2 * plane + p] = C2[k] + Tr[k] * a.st.bg2;
        a.depth[gp] = D[k];
        if (S2) a.depth_var[gp] = Sc[k] + A[k] * Tr[k] * Mn[k] * Mn[k];
        a.alpha[gp] = 1.f - Tr[k];
        a.t_final[gp] = Tr[k];
        a.last[gp] = last[k];
        if (a.zero_px[0]) a.zero_px[0][gp] = 0.f;
        if (a.zero_px[1]) a.zero_px[1][gp] = 0.f;
    }
}

// ------------------------------------------------------------------------- backward
//
// PPT pixels a lane (8 x 8 PPT blocks), GRP entries a step: the exponents of a step are formed side by
// side, then each entry that some lane keeps runs its adjoint and reduction.  Two pixels a lane
// share dx, the record reads and one reduction (a third of the issue cycles): rig step 500 -> 430 us,
// over 2M Gaussians 560 -> 465 us, 22 views 1278 -> 1230 us (8 x 8 blocks: 499, 546, 1547); 8 x 8 blocks
// halve a wave's serial work for launches with few tiles: 300k single view 140 -> 95 us (8 x 16: 166),
// two small views 32 -> 24 us (41).  GA: the upstream adjoint has an alpha term (dL/dA); the fused
// loss never has one.  S2: the loss has an adjoint for the second depth moment sum w z^2 (rendered
// variance).
template <int T, int PPT, int GRP, bool GA, bool S2, bool SHARED>
__global__ __launch_bounds__(T* T / PPT) void raster_bwd_kernel(RasterBwdArgs a) {
    constexpr int NW = T * T / PPT / 64, COLS = T / 8;
    __shared__ Rows<GRP> rows[NW];
    __shared__ uint32_t rpair[NW][kChunk + GRP];
    __shared__ float sred[NW];
    const uint32_t wt = a.work[blockIdx.x];
    if (wt == kNoTile) return;  // padding of a shorter XCD list (whole workgroup)
    const int tile = (int)wt;
    const TileCoord tc = tile_coord(a.vt, tile);
    const uint32_t start = __builtin_amdgcn_readfirstlane(a.ranges[2 * tile]);
    const int lane = __lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Rows<GRP>& my = rows[wave];
    uint32_t* const mypair = rpair[wave];
    const float amin = a.st.alpha_min;

    // U = T_final gC.bg + sum over later contributors j of w_j (gC.c_j + gD z_j + gA)
    const int bx = tc.px0 + (wave % COLS) * 8, by = tc.py0 + (wave / COLS) * 8 * PPT;
    const int px = bx + (lane & 7), py = by + (lane >> 3);
    const float cx = (float)px + 0.5f;
    float cy[PPT], Tr[PPT], gC0[PPT], gC1[PPT], gC2[PPT], gD[PPT], gX[PPT], U[PPT];
    uint32_t last[PPT];
    float loss_part = 0.f;
    uint32_t wlast = 0;
    const long long plane = (long long)tc.W * tc.H;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int y = py + 8 * k;
        cy[k] = (float)y + 0.5f;
        gC0[k] = gC1[k] = gC2[k] = gD[k] = gX[k] = 0.f;  // gX: gA or the second moment's adjoint
        Tr[k] = 1.f;
        last[k] = 0;
        U[k] = 0.f;
        if (px < tc.W && y < tc.H) {
            const long long p = (long long)y * tc.W + px;
            const long long gp = tc.pix0 + p;
            Tr[k] = a.t_final[gp];
            last[k] = a.last[gp];
            if (a.loss_mode) {
                const bool on = a.mask ? (a.mask[gp] != 0) : true;
                if (on) {
                    const float sc = a.l1_scale[tc.b];
                    const float* rgb = a.rgb + 3 * tc.pix0;
                    const float* gt = a.gt_rgb + 3 * tc.pix0;
                    const float d0 = rgb[p] - gt[p];
                    const float d1 = rgb[plane + p] - gt[plane + p];
                    const float d2 = rgb[2 * plane + p] - gt[2 * plane + p];
                    gC0[k] = d0 > 0.f ? sc : (d0 < 0.f ? -sc : 0.f);
                    gC1[k] = d1 > 0.f ? sc : (d1 < 0.f ? -sc : 0.f);
                    gC2[k] = d2 > 0.f ? sc : (d2 < 0.f ? -sc : 0.f);
                    loss_part += sc * (fabsf(d0) + fabsf(d1) + fabsf(d2));
                }
                if (a.d_rgb) {  // D-SSIM adjoint (already zero outside the mask)
                    const float* g = a.d_rgb + 3 * tc.pix0;
                    gC0[k] += g[p];
                    gC1[k] += g[plane + p];
                    gC2[k] += g[2 * plane + p];
                }
                if (a.d_depth) gD[k] = a.d_depth[gp];
                if (S2) gX[k] = a.d_depth2[gp];
            } else {
                if (a.d_rgb) {
                    const float* g = a.d_rgb + 3 * tc.pix0;
                    gC0[k] = g[p];
                    gC1[k] = g[plane + p];
                    gC2[k] = g[2 * plane + p];
                }
                if (a.d_depth) gD[k] = a.d_depth[gp];
                if (GA) gX[k] = a.d_alpha[gp];
            }
            U[k] = Tr[k] * (gC0[k] * a.st.bg0 + gC1[k] * a.st.bg1 + gC2[k] * a.st.bg2);
            wlast = max(wlast, last[k]);
        }
    }
    // An adjoint, or from the first record on that has one a colour, that makes dL/dalpha infinite or NaN must
    // not reach the sums of p of the records that its pixel does not keep.  Decided for a whole wave, since a
    // select in every entry would cost all of them (the 4-view backward takes as long with the test as without).
    bool far = false;
#pragma unroll
    for (int k = 0; k < PPT; ++k) far |= unbounded(gC0[k], gC1[k], gC2[k], gD[k]) || unbounded(gX[k], 0.f, 0.f, 0.f);
    far = __builtin_amdgcn_ballot_w64(far) != 0ull;
    if (a.loss_mode) {
        // tile sum of the L1 partials (deterministic order)
        float s = wave_sum(loss_part);
        if (NW > 1) {
            if (lane == 0) sred[wave] = s;
            __syncthreads();
            s = 0.f;
            for (int w = 0; w < NW; ++w) s += sred[w];
        }
        if (threadIdx.x == 0) a.loss_partials[tile] = s;
    }
    // entries at or past every lane's last contributor are not visited
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) wlast = max(wlast, (uint32_t)__shfl_xor((int)wlast, o, 64));
    const int wl = (int)__builtin_amdgcn_readfirstlane(wlast);

    prio_by_length(wl);
    const float amax = __builtin_canonicalizef(a.st.alpha_max);
    const float inv_amin = 1.f / amin;
    const float X0 = (float)bx + 0.5f, Y0 = (float)by + 0.5f;
    // odd waves add their six sums of p to a second set of slots, see kGrad2d
    int red_val = column_sum_of(lane);
    if ((wave & 1) && red_val >= 0 && red_val < kGrad2dSplit) red_val += kGrad2d;

    for (int hi = wl; hi > 0; hi -= kChunk) {  // the chunk's entries back to front
        const int e = hi - 1 - lane;
        const uint32_t q = a.tile_pairs[start + (e >= 0 ? e : 0)];
        const Rec r = load_rec(a.records, q);
        const bool in = e >= 0 && block_reached(r.a, r.b.x, r.b.y, inv_amin, X0, Y0, 7.f, 8.f * PPT - 1.f);
        if (in) mypair[rank_in(__builtin_amdgcn_ballot_w64(in))] = q;
        bool slow;
        const int n = my.pack(r, r.b.y, in, (uint32_t)e, amax, slow);
        far |= __builtin_amdgcn_ballot_w64(in && unbounded(r.c.y, r.c.z, r.c.w, r.b.z)) != 0ull;
        auto run = [&](auto tests) {
            constexpr bool TESTS = decltype(tests)::value;
            for (int g = 0; g < n; g += GRP) {
                float4 r0[GRP], rc[GRP];
                float2 r1[GRP];
                uint32_t j[GRP];
#pragma unroll
                for (int i = 0; i < GRP; ++i) {
                    r0[i] = my.g[g + i];
                    r1[i] = my.co[g + i];
                    rc[i] = my.col[g + i];
                    j[i] = my.pos[g + i];
                }
                float araw[GRP][PPT];
                unsigned long long km[GRP][PPT];  // lanes that keep the pair
#pragma unroll
                for (int i = 0; i < GRP; ++i) {
                    const float dx = r0[i].x - cx, Adx = r0[i].z * dx;
#pragma unroll
                    for (int k = 0; k < PPT; ++k) {
                        const float dy = r0[i].y - cy[k];
                        const float p2 =
                            !SHARED ? exponent2(r0[i].z, r0[i].w, r1[i].x, dx, dy)
                                    : __builtin_fmaf(dy, dy * r1[i].x, dx * __builtin_fmaf(r0[i].w, dy, Adx));
                        araw[i][k] = r1[i].y * __builtin_amdgcn_exp2f(p2);
                        km[i][k] = __builtin_amdgcn_uicmp(j[i], last[k], 36) &  // j < last
                                   le_mask(amin, TESTS ? fminf(amax, araw[i][k]) : araw[i][k]);
                        if (TESTS) km[i][k] &= le_mask(p2, 0.f);
                    }
                }
#pragma unroll
                for (int i = 0; i < GRP; ++i) {
                    if ((km[i][0] | km[i][PPT - 1]) == 0ull) continue;  // wave-uniform
                    const float dx = r0[i].x - cx;
                    const float z = rc[i].w, z2 = S2 ? z * z : 0.f;
                    float h[PPT], c[4];
#pragma unroll
                    for (int k = 0; k < PPT; ++k) {
                        // branch-free: a pixel that does not keep this Gaussian has alpha = 0, so its w
                        // and h are 0 and its T and U stay as they are (and every quantity stays
                        // finite: alpha <= alpha_max < 1)
                        const float ak = lane_of(km[i][k]) ? (TESTS ? fminf(amax, araw[i][k]) : araw[i][k]) : 0.f;
                        const float om = 1.f - ak;
                        float rom = __builtin_amdgcn_rcpf(om);
                        const float Tk = Tr[k] * rom;
                        const float w = ak * Tk;
                        float qv = gC0[k] * rc[i].x + gC1[k] * rc[i].y + gC2[k] * rc[i].z + gD[k] * z;
                        if (GA) qv += gX[k];
                        if (S2) qv += gX[k] * z2;
                        const float ga = Tk * qv - U[k] * rom;  // dL/dalpha
                        U[k] += w * qv;
                        Tr[k] = Tk;
                        // dL/dpower = alpha dL/dalpha (none where the alpha_max clamp is active)
                        h[k] = TESTS && !(lane_of(km[i][k]) && araw[i][k] <= amax) ? 0.f : ga * ak;
                        // depth adjoint: d(w z)/dz = w, d(w z^2)/dz = 2 w z
                        const float gz = S2 ? gD[k] + 2.f * z * gX[k] : gD[k];
                        c[0] = k == 0 ? w * gC0[k] : c[0] + w * gC0[k];
                        c[1] = k == 0 ? w * gC1[k] : c[1] + w * gC1[k];
                        c[2] = k == 0 ? w * gC2[k] : c[2] + w * gC2[k];
                        c[3] = k == 0 ? w * gz : c[3] + w * gz;
                    }
                    const float dy0 = r0[i].y - cy[0];
                    float hs = h[0], hy = h[0] * dy0, hyy = hy * dy0;
                    if (PPT == 2) {
                        const float dy1 = r0[i].y - cy[PPT - 1], t = h[PPT - 1] * dy1;
                        hs += h[PPT - 1];
                        hy += t;
                        hyy += t * dy1;
                    }
                    const float tot = wave_column_sums(hs, hy, hyy, c, dx);
                    const uint32_t pair = mypair[g + i];
                    if (red_val >= 0) atomicAdd(a.grad2d + red_val + (long long)pair * kGrad2dStride, tot);
                }
            }
        };
        if (slow || far) run(std::true_type{});
        else run(std::false_type{});
        __builtin_amdgcn_wave_barrier();
    }
}

// The backward's clears in one launch, when the forward's own zeroing of these accumulators
// cannot be relied on (a second backward of one forward).  Thread g zeroes the adjoint rows of
// the pairs 4 g .. 4 g + 3 that some tile lists (the only rows the raster backward adds to
// and the projection backward reads): one 16-byte load of their counts, then the 64-byte row
// stores of the visible ones, so no store waits on more than one load; then, striding over
// the grid, the dense float buffers (the LiDAR depth and second-moment adjoints).
static_assert(kGrad2dStride == 16, "four float4 stores per row");

__global__ __launch_bounds__(256) void bwd_clear_kernel(BwdClearArgs a) {
    const long long g = (long long)blockIdx.x * 256 + threadIdx.x;
    const long long q0 = 4 * g;
    if (q0 < a.n_pairs) {
        uint32_t c[4];
        if (q0 + 4 <= a.n_pairs) {
            const uint4 v = reinterpret_cast<const uint4*>(a.pair_count)[g];  // 16-byte aligned
            c[0] = v.x; c[1] = v.y; c[2] = v.z; c[3] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) c[j] = q0 + j < a.n_pairs ? a.pair_count[q0 + j] : 0u;
        }
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!c[j]) continue;
            float4* row = reinterpret_cast<float4*>(a.grad2d + (q0 + j) * kGrad2dStride);
#pragma unroll
            for (int k = 0; k < kGrad2dStride / 4; ++k) row[k] = z;
        }
    }
    const long long stride = (long long)gridDim.x * 256;
    for (int r = 0; r < kBwdClearRegions; ++r)
        for (long long i = g; i < a.zero_n[r]; i += stride) a.zero[r][i] = 0.f;
}

void launch_bwd_clear(const BwdClearArgs& a, hipStream_t s) {
    long long most = (a.n_pairs + 3) / 4;
    for (int r = 0; r < kBwdClearRegions; ++r) {
        const long long t = (a.zero_n[r] + 3) / 4;  // about four floats per thread
        most = t > most ? t : most;
    }
    if (most <= 0) return;
    const long long grid = (most + 255) / 256;
    hipLaunchKernelGGL(bwd_clear_kernel, dim3((unsigned)grid), dim3(256), 0, s, a);
}

int raster_blocks(const ViewTable& vt) {
    const int n = vt.tile_base[vt.n_views];
    if (n <= 0) return 0;
    const int strips = (n + kWorkStrip - 1) / kWorkStrip;
    return 8 * ((strips + 7) / 8) * kWorkStrip;  // 8 XCD lists of equal (maximum) length
}

#define AGS_RASTER_CONFIGS(X) \
    X(8, 1, 64)               \
    X(8, 1, 128)              \
    X(16, 1, 128)             \
    X(16, 1, 256)             \
    X(16, 2, 64)              \
    X(16, 2, 128)             \
    X(16, 2, 256)             \
    X(16, 4, 64)              \
    X(32, 4, 256)             \
    X(32, 2, 512)

int raster_shapes(int* tile, int* ppt, int* batch, int n_max) {
    int n = 0;
#define X(t_, p_, m_)             \
    if (n < n_max) {              \
        tile[n] = t_;             \
        ppt[n] = p_;              \
        batch[n] = m_;            \
    }                             \
    ++n;
    AGS_RASTER_CONFIGS(X)
#undef X
    return n;
}

// Whether a launch takes 8 x 16 blocks: from 8192 waves of them (256 CUs of 32 waves) the chip is
// full with half the waves; an 8 x 8 tile has no 8 x 16 block.  Both sides measured at the kernels.
static bool wide_blocks(const ViewTable& vt, int T) {
    return T > 8 && (long long)vt.tile_base[vt.n_views] * (T * T / 128) >= 8192;
}

// How many entries and pixels a lane takes follows from the number of blocks; `batch` and `ppt` name a
// supported shape, and ppt > 1 the staged forward for many tiles and the backward's shared exponents.  `batch`
// sizes the staged forward's LDS and nothing else: the other shapes of a tile and ppt are the same kernels.
static bool shape_supported(int T, int batch, int ppt) {
#define X(t_, p_, m_) \
    if (T == t_ && ppt == p_ && batch == m_) return true;
    AGS_RASTER_CONFIGS(X)
#undef X
    return false;
}

int raster_kernel_of(const ViewTable& vt, int T, int batch, int ppt, bool backward) {
    if (backward) return T == 16 && ppt > 1 ? 1 : 0;
    return wide_blocks(vt, T) && ppt > 1 ? 1024 * ppt + batch : 0;
}

int launch_raster_fwd(const RasterArgs& a, int T, int batch, int ppt, hipStream_t s) {
    const int nb = raster_blocks(a.vt);
    if (nb <= 0) return 0;
    if (!shape_supported(T, batch, ppt)) return AGS_ERR_NOT_SUPPORTED;
    auto launch = [&](auto kernel, int threads) { hipLaunchKernelGGL(kernel, dim3(nb), dim3(threads), 0, s, a); };
    const bool wide = wide_blocks(a.vt, T), var = a.depth_var != nullptr;
    if (wide && ppt > 1) {
#define X(t_, p_, m_)                                                                                          \
    if constexpr (p_ > 1)                                                                                      \
        if (T == t_ && ppt == p_ && batch == m_)                                                               \
            var ? launch(raster_fwd_staged_kernel<t_, p_, m_, true>, t_ * t_ / p_)                             \
                : launch(raster_fwd_staged_kernel<t_, p_, m_, false>, t_ * t_ / p_);
        AGS_RASTER_CONFIGS(X)
#undef X
        return 0;
    }
    if (T == 8) var ? launch(raster_fwd_kernel<8, true>, 64) : launch(raster_fwd_kernel<8, false>, 64);
    else if (wide) var ? launch(raster_fwd_wide_kernel<16, true>, 128) : launch(raster_fwd_wide_kernel<16, false>, 128);
    else if (T == 16) var ? launch(raster_fwd_kernel<16, true>, 256) : launch(raster_fwd_kernel<16, false>, 256);
    else var ? launch(raster_fwd_kernel<32, true>, 1024) : launch(raster_fwd_kernel<32, false>, 1024);
    return 0;
}

template <int T, int PPT, int GRP, bool SHARED>
static void bwd_variant(const RasterBwdArgs& a, int nb, hipStream_t s) {
    const bool ga = !a.loss_mode && a.d_alpha, s2 = a.loss_mode && a.d_depth2;
    const auto kernel = ga   ? raster_bwd_kernel<T, PPT, GRP, true, false, SHARED>
                        : s2 ? raster_bwd_kernel<T, PPT, GRP, false, true, SHARED>
                             : raster_bwd_kernel<T, PPT, GRP, false, false, SHARED>;
    hipLaunchKernelGGL(kernel, dim3(nb), dim3(T * T / PPT), 0, s, a);
}

int launch_raster_bwd(const RasterBwdArgs& a, int T, int batch, int ppt, hipStream_t s) {
    const int nb = raster_blocks(a.vt);
    if (nb <= 0) return 0;
    if (!shape_supported(T, batch, ppt)) return AGS_ERR_NOT_SUPPORTED;
    const bool wide = wide_blocks(a.vt, T), shared = ppt > 1;
    if (T == 8) bwd_variant<8, 1, 4, false>(a, nb, s);
    else if (T == 16 && wide) shared ? bwd_variant<16, 2, 2, true>(a, nb, s) : bwd_variant<16, 2, 2, false>(a, nb, s);
    else if (T == 16) shared ? bwd_variant<16, 1, 4, true>(a, nb, s) : bwd_variant<16, 1, 4, false>(a, nb, s);
    else if (wide) bwd_variant<32, 2, 2, true>(a, nb, s);  // tiles of 32 have two or four pixels a thread
    else bwd_variant<32, 1, 4, true>(a, nb, s);
    return 0;
}

}  // namespace ags
