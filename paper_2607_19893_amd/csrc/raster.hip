// Rendering phase part 2 (forward alpha blending), the L1 image loss, and the
// backward phase (pixel replay + per-primitive chain rule).
//
// Forward: one 256-thread workgroup per 16x16 tile, one pixel per thread, each
// wave an 8x8 quadrant.  The tile's sorted pairs are staged through LDS in batches
// of 256 (sigma's polynomial about the tile centre, opacity, colour, and the blocks
// of the tile the footprint can reach); a wave walks the list of the pairs that
// reach its quadrant, and a workgroup-wide count of finished pixels ends the batch
// loop early.
//
// Backward: same tile/pixel mapping, walking each tile's pairs back to front in
// batches of 64; each 16-lane row of a wave has its own list, of the pairs that
// reach its 8x2 strip of pixels.  Each pixel recovers the transmittance in front of
// a pair by dividing by (1 - alpha) and keeps the projection of the suffix colour
// sum on its upstream gradient; per pair, eight moment and colour sums are taken
// over each 16-lane row with DPP, stored in the strip's LDS record of the pair,
// combined over the strips in a fixed order, and written to the pair's slot at its
// emission position (a primitive's pairs side by side).  Per visible primitive,
// k_slot_sum adds its slots in a fixed order -- deterministic, no floating-point atomics
// in global memory -- and k_project_bwd applies the projection and colour chain
// rule (geometry in fp64) and writes one compact gradient row.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace gsmi {

namespace {

constexpr float kAlphaMin = 1.0f / 255.0f;
constexpr float kAlphaMax = 0.99f;
constexpr float kTMin = 1e-4f;
constexpr float kCutMargin = 1e-3f;   // extra sigma beyond the 1/255 cut-off when bounding a footprint

// One pair's primitive as staged in LDS for the 8x8 walk: 64 bytes, read by a
// whole wave at one address (a broadcast).
//   q[0..5]: sigma as a polynomial in the pixel's offset (X, Y) from the tile
//   centre, in fp64:
//     sigma = q0 + q1 X + q2 Y + q3 X^2 + q4 XY + q5 Y^2
//   then the opacity and the colour.
// fp64 because the terms of sigma cancel for elongated footprints far from their
// centre (fp32 loses up to ~1e-3 of sigma there); the coefficients are formed
// once per staged pair from the exact fp32 mean and conic, so a pixel's sigma costs
// five fused multiply-adds and one conversion.
struct __align__(16) Splat {
    double q[6];
    float o, r, g, b;
};

// A pair is skipped where sigma < 0, which its exact sigma is only if its conic is not
// positive definite.  The polynomial's rounding error is at most 16 * 2^-53 of
//   size = A/2 x^2 + |B| x y + C/2 y^2,  (x, y) = (|u| + 7.5, |v| + 7.5),
// (u, v) the centre from the tile's: nine roundings on the way to the coefficients
// and five of the evaluation, each of a sum of terms that lie within size.  Up to
// kNearSize that is below 5e-9: a definite pair's sigma neither overflows nor turns
// visibly negative, and needs no test.  Batches that hold another pair
// (kChecked) test sigma.  An indefinite pair, whose record carries -o, is skipped below
// kSigmaNeg (a zero of sigma can come out as a tiny negative number).  A definite pair
// further out has its negative sigmas, which are rounding, taken as 0, and those beyond
// kSigmaFar, possibly past the fp32 range, as kSigmaFar, at which alpha is 0.  A colour
// that is not finite is kChecked too: those batches take it only where the pair is
// included, since 0 times it is a NaN.
constexpr float kSigmaNeg = -1e-9f, kSigmaFar = 1e4f, kNearSize = 2.5e6f;
constexpr uint32_t kChecked = 1u << 16;

// Fills rec from a pair's mean, conic and colour, relative to the tile centre
// (xc, yc), and returns the tile's blocks of 8 x BH pixels that hold a pixel centre
// with sigma <= cut = ln(255 o) + kCutMargin: a block that is left out has no pixel
// at or above alpha = 1/255.  Bit b is the block of wave b / (8 / BH) (quadrant
// (w & 1, w >> 1)), counted downwards inside the quadrant; kChecked comes on top.
//
// sigma's minimum over a rectangle lies at its centre if that is inside, else on
// the vertical or horizontal edge line nearest to the centre: along each of the
// two lines it is at the line's vertex clamped to the rectangle.  In fp32, with
// the rounding of sigma's terms (bounded by their largest values over the tile)
// added to the cut.  A conic that is not positive definite reaches every block, an
// infinite centre or conic none.
template <int BH>
__device__ __forceinline__ uint32_t stage_pair(Splat* rec, float2 m, float4 co, const float* __restrict__ rgb3,
                                               double xc, double yc) {
    constexpr int kPer = 8 / BH;                     // blocks of a quadrant
    constexpr uint32_t kAll = (1u << (4 * kPer)) - 1u;
    const double du = (double)m.x - xc, dv = (double)m.y - yc;
    const double qa = 0.5 * (double)co.x, qb = (double)co.y, qc = 0.5 * (double)co.z;
    const double ax = fma(qa, du, qb * dv), cy = qc * dv;
    rec->q[0] = fma(du, ax, cy * dv);
    rec->q[1] = -fma(qa, du, ax);
    rec->q[2] = -fma(qb, du, 2.0 * cy);
    rec->q[3] = qa;
    rec->q[4] = qb;
    rec->q[5] = qc;
    rec->o = co.w;
    rec->r = rgb3[0];
    rec->g = rgb3[1];
    rec->b = rgb3[2];
    constexpr float kLn2 = 0.693147180559945309417f;
    const float cut = fmaf(__builtin_amdgcn_logf(255.0f * co.w), kLn2, kCutMargin);
    if (!(cut > 0.0f)) return 0u;              // opacity below 1/255: no pixel can take it
    const float A = co.x, B = co.y, C = co.z, u = (float)du, v = (float)dv;
    const float hA = 0.5f * A, hC = 0.5f * C;
    const float mx = fabsf(u) + 7.5f, my = fabsf(v) + 7.5f;
    const float size = hA * mx * mx + fabsf(B) * mx * my + hC * my * my;
    const float lim = fmaf(1e-6f, size, cut);
    const bool definite = A > 0.0f && (double)A * C - (double)B * B > 0.0;
    const float no_colour = (rec->r - rec->r) + (rec->g - rec->g) + (rec->b - rec->b);     // 0, or a NaN
    uint32_t mask = no_colour == 0.0f ? 0u : kChecked;
    if (!definite || !(size <= kNearSize)) {
        if (isinf(u) || isinf(v) || isinf(A) || isinf(B) || isinf(C)) return 0u;
        mask = kChecked;
        if (!definite) {
            const bool nan = u != u || v != v || (A > 0.0f && (B != B || C != C));
            rec->o = -co.w;
            return nan ? 0u : kAll | mask;
        }
        if (isinf(lim)) return kAll | mask;
    }
    const float sx = -B * __builtin_amdgcn_rcpf(A), sy = -B * __builtin_amdgcn_rcpf(C);
#pragma unroll
    for (int r = 0; r < 2 * kPer; ++r) {
        // offsets (splat - pixel) over the block's rows and columns
        const float ylo = v + (7.5f - (float)(r * BH + BH - 1)), yhi = ylo + (float)(BH - 1);
        const float dyn = __builtin_amdgcn_fmed3f(0.0f, ylo, yhi);
        const float bdy = B * dyn, cdy = hC * dyn * dyn, vx = sx * dyn;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float xlo = c ? u - 7.5f : u + 0.5f, xhi = xlo + 7.0f;
            const float dxn = __builtin_amdgcn_fmed3f(0.0f, xlo, xhi);
            const float dyv = __builtin_amdgcn_fmed3f(sy * dxn, ylo, yhi);
            const float dxv = __builtin_amdgcn_fmed3f(vx, xlo, xhi);
            const float s1 = fmaf(fmaf(hC, dyv, B * dxn), dyv, hA * dxn * dxn);
            const float s2 = fmaf(fmaf(hA, dxv, bdy), dxv, cdy);
            if (fminf(s1, s2) <= lim) mask |= 1u << ((2 * (r / kPer) + c) * kPer + r % kPer);
        }
    }
    return mask;
}

// A pixel's offset from its tile's centre and its products, for the pairs' sigma.
struct PixelPoly {
    double X, Y, XX, XY, YY;
    __device__ __forceinline__ PixelPoly(int x, int y) {
        X = x - 7.5;
        Y = y - 7.5;
        XX = X * X;
        XY = X * Y;
        YY = Y * Y;
    }
    __device__ __forceinline__ float eval(const Splat& S) const {
        return (float)fma(S.q[5], YY, fma(S.q[4], XY, fma(S.q[3], XX, fma(S.q[2], Y, fma(S.q[1], X, S.q[0])))));
    }
};

// sigma of a staged pair, for a batch whose pairs need a test (see kChecked): false
// if the pair is skipped; o is set to its opacity.  A NaN stays one.
__device__ __forceinline__ bool check_sigma(const Splat& S, float& sigma, float& o) {
    const bool skip = S.o < 0.0f && sigma < kSigmaNeg;
    o = fabsf(S.o);
    sigma = sigma > kSigmaFar ? kSigmaFar : (sigma < 0.0f ? 0.0f : sigma);
    return !skip;
}

// Pairs a walk takes per iteration; the lists are padded to a multiple of it.
constexpr int kPad = 4;

// The list of the nb staged pairs that reach quadrant w, in order, as byte
// offsets of their records; padded with the offset of record GS_BLOCK.  One wave
// builds and reads its own list.
__device__ __forceinline__ uint32_t quad_list(const uint8_t* quad, uint32_t* list, uint32_t nb, int w) {
    const int lane = lane_id();
    const uint64_t lt = lanemask_lt();
    uint32_t n = 0;
    for (uint32_t c = 0; c < nb; c += GS_WAVE) {
        const bool on = (quad[c + lane] >> w) & 1u;
        const uint64_t m = __ballot(on);
        if (on) list[n + popc64(m & lt)] = (uint32_t)((c + lane) * sizeof(Splat));
        n += popc64(m);
    }
    if (lane < kPad) list[n + lane] = (uint32_t)(GS_BLOCK * sizeof(Splat));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    return __builtin_amdgcn_readfirstlane(n);
}

// exp(-sigma) = 2^-t with t = sigma log2(e) carried as hi + lo (log2(e)
// split into an fp32 head and tail; hi = sigma * head rounded, lo its exact
// rounding error plus sigma * tail, |lo| < 2e-5 for the sigmas that matter).
// 2^-t = 2^-hi * 2^-lo with 2^-lo = 1 - lo ln2 up to (lo ln2)^2 / 2 < 1e-10;
// the hardware base-2 exponential (1 ulp) takes -hi directly.  About two ulps
// in all, far inside the alpha decision band; forward and backward call the
// same code, so they take identical decisions.  Sigmas from 104 on give 0; past 2.3e38
// hi overflows and the result is a NaN, which the caller's kSigmaFar keeps out.
__device__ __forceinline__ float exp_neg(float sigma) {
    constexpr float kLog2eHi = 1.44269502162933349609375f;    // log2(e) rounded to fp32
    constexpr float kLog2eLo = 1.925963033500011e-08f;        // log2(e) - kLog2eHi
    constexpr float kLn2 = 0.693147180559945309417f;
    const float hi = sigma * kLog2eHi;
    float lo = fmaf(sigma, kLog2eHi, -hi);
    lo = fmaf(sigma, kLog2eLo, lo);
    return __builtin_amdgcn_exp2f(-hi) * fmaf(-lo, kLn2, 1.0f);
}

// |a - t| and the sign of a - t scaled by inv (0 for a tie): one L1 term and its derivative.
__device__ __forceinline__ float l1_elem(float a, float t, float inv, float& dl) {
    const float d = a - t;
    dl = d > 0.0f ? inv : (d < 0.0f ? -inv : 0.0f);
    return fabsf(d);
}

// The tile a workgroup renders: the grid covers the tiles once, in the
// caller's dispatch order (longest first from gs_bin_sort), else row-major.
// Pixels, losses and pair records are per tile, so the order changes no
// result, only how the longest tiles overlap the rest.
__device__ __forceinline__ uint32_t dispatch_tile(const uint32_t* __restrict__ tile_order) {
    return tile_order ? tile_order[blockIdx.x] : blockIdx.x;
}

// Position of this thread's pixel in its tile: wave w renders the 8x8 quadrant
// (w & 1, w >> 1), lane l its pixel (l & 7, l >> 3).
__device__ __forceinline__ int quad_x(int tid) { return ((tid >> 6) & 1) * 8 + (tid & 7); }
__device__ __forceinline__ int quad_y(int tid) { return (tid >> 7) * 8 + ((tid >> 3) & 7); }

// What bounds it is VALU issue: 27 instructions per (wave, pair) step (sigma 6, the
// exponential 6, blending 14).  An 8x8 block takes more
// steps than lists per 16x1 row of the tile did (their rows found 54% of the lanes
// included, a block 34%), but a wave-uniform list needs no per-row lockstep, no list
// building per row and no per-pair address arithmetic, and sigma as a polynomial no
// per-pair offsets, so a step got shorter by more: 7.8e7 -> 6.4e7 VALU a view on a
// 1M-primitive 1080p room.  Four pairs an iteration keep four records' loads and
// footprints in flight beside the serial T chain; their registers allow six waves per
// SIMD, which measured better than two pairs at eight waves, most of all where few tiles
// leave a wave or two per SIMD (256 tiles: 34 us against 39).  Measured, 16x1 rows
// before and this: room 139 -> 105 us, 3840x2160 render of 500k primitives 305 -> 217,
// 475 tiles of 400x304 66 -> 38, 256 tiles of 256x256 50 -> 35.
//
// LOSS: the L1 loss of the view is taken in the same pass (the image loss of
// the view, Section 2.1): each pixel compares its three fp32 channels with
// the target exactly as k_loss_l1 does, writes dL/dimg, and each tile leaves
// its sum of |img - target| in loss_partial[tile] for k_loss_final.
template <bool STATS, bool LOSS>
__global__ void __launch_bounds__(GS_BLOCK, STATS ? 5 : 6) k_raster_fwd(
    const uint32_t* __restrict__ tile_order, const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ vals,
    const float2* __restrict__ mean2d, const float4* __restrict__ conic_op, const float* __restrict__ rgb, int32_t W,
    int32_t H, int32_t TX, float bg0, float bg1, float bg2, float* __restrict__ img, float* __restrict__ final_T,
    uint32_t* __restrict__ n_contrib,
    uint8_t* __restrict__ active, unsigned long long* __restrict__ pair_stats, const float* __restrict__ target,
    float inv_total, float* __restrict__ dL, float* __restrict__ loss_partial) {
    __shared__ Splat L[GS_BLOCK + 1];                    // the last record blends nothing: it pads the lists
    __shared__ uint8_t s_quad[GS_BLOCK];                 // quadrants each staged pair can reach
    __shared__ uint8_t s_hit[GS_BLOCK + 1];              // pairs some pixel included (active flags)
    __shared__ __align__(16) uint32_t s_list[4][GS_BLOCK + kPad];  // per wave: its pairs' records, as offsets into L
    __shared__ uint32_t s_stat[4][4];
    const uint32_t tile = dispatch_tile(tile_order);
    if (tile >= gridDim.x) return;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid / GS_WAVE);
    const int lane = lane_id();
    const int tx = (int)tile % TX, ty = (int)tile / TX;
    const int px = tx * GS_TILE + quad_x(tid);
    const int py = ty * GS_TILE + quad_y(tid);
    const bool inside = px < W && py < H;
    const double xc = tx * GS_TILE + 8, yc = ty * GS_TILE + 8;
    const PixelPoly P(quad_x(tid), quad_y(tid));
    const uint32_t start = ranges[2 * tile], end = ranges[2 * tile + 1];
    // T, negated once the pixel is finished: every later T (1 - alpha) is then below kTMin
    float T = inside ? 1.0f : -1.0f;
    float c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
    uint32_t last = 0, n_inc = 0, term_at = 0, w_iter = 0, w_hit = 0;
    if (tid < 16) reinterpret_cast<float*>(&L[GS_BLOCK])[tid] = 0.0f;
    // the ids of the next batch load while this one is walked
    uint32_t g = start + tid < end ? vals[start + tid] : 0u;
    for (uint32_t bs = start; bs < end; bs += GS_BLOCK) {
        if (__syncthreads_count(T < 0.0f) == GS_BLOCK) break;
        const uint32_t j = bs + tid;
        const uint32_t gj = g;
        uint32_t quad = 0u;
        if (j < end) quad = stage_pair<8>(&L[tid], mean2d[gj], conic_op[gj], rgb + 3 * (size_t)gj, xc, yc);
        if (j + GS_BLOCK < end) g = vals[j + GS_BLOCK];
        s_quad[tid] = (uint8_t)quad;
        s_hit[tid] = 0;
        const bool check = __syncthreads_or((int)(quad & kChecked));
        if (__ballot(T > 0.0f) != 0ull) {
            const uint32_t n_list = quad_list(s_quad, s_list[w], min((uint32_t)GS_BLOCK, end - bs), w);
            uint32_t lk = 0xFFFFFFFFu;      // record offset of the pixel's last included pair of this batch
            auto walk = [&](auto checked) {
                constexpr bool CHECK = decltype(checked)::value;
                // kPad pairs at a time: their records load together and their footprints are
                // evaluated side by side; the blending then takes them in order
                for (uint32_t i0 = 0; i0 < n_list; i0 += kPad) {
                    uint32_t ats[kPad];
                    __builtin_memcpy(ats, __builtin_assume_aligned(&s_list[w][i0], 4 * kPad), sizeof(ats));
                    uint32_t hit = 0u;      // of the kPad pairs, those some pixel included
#pragma unroll
                    for (int i = 0; i < kPad; ++i) {
                        const uint32_t at = ats[i];
                        const Splat& S = *reinterpret_cast<const Splat*>(reinterpret_cast<const char*>(L) + at);
                        float sigma = P.eval(S), o = S.o;
                        const bool on = !CHECK || check_sigma(S, sigma, o);
                        float al = fminf(kAlphaMax, o * exp_neg(sigma));
                        uint64_t ok_mask = __builtin_amdgcn_ballot_w64(!(al < kAlphaMin));
                        bool ok = !(al < kAlphaMin);
                        if (CHECK) {
                            ok_mask &= __builtin_amdgcn_ballot_w64(on);
                            ok = ok & on;
                        }
                        al = ok ? al : 0.0f;
                        const float Tn = T * (1.0f - al);
                        const bool go = !(Tn < kTMin);       // stop in front of a pair that would leave less
                        if (STATS && !go && T > 0.0f) term_at = bs - start + at / (uint32_t)sizeof(Splat) + 1u;
                        const float wgt = go ? al * T : 0.0f;
                        ok = ok && go;
                        c0 = fmaf(wgt, !CHECK || ok ? S.r : 0.0f, c0);
                        c1 = fmaf(wgt, !CHECK || ok ? S.g : 0.0f, c1);
                        c2 = fmaf(wgt, !CHECK || ok ? S.b : 0.0f, c2);
                        T = go ? Tn : -fabsf(T);
                        lk = ok ? at : lk;
                        hit |= (ok_mask & __builtin_amdgcn_ballot_w64(go)) != 0ull ? 1u << i : 0u;
                        if (STATS && i0 + i < n_list) {
                            n_inc += ok ? 1u : 0u;
                            const uint64_t om = __ballot(ok);
#pragma unroll
                            for (int q = 0; q < 4; ++q) w_hit += ((om >> (16 * q)) & 0xFFFFull) ? 1u : 0u;
                            w_iter += 4u;
                        }
                    }
                    // every wave that stores here stores the same value
                    if (active != nullptr && lane < kPad && ((hit >> lane) & 1u)) s_hit[s_list[w][i0 + lane] / (uint32_t)sizeof(Splat)] = 1;
                    if (__ballot(T > 0.0f) == 0ull) break;
                }
            };
            if (check)
                walk(std::true_type{});
            else
                walk(std::false_type{});
            last = lk != 0xFFFFFFFFu ? bs - start + lk / (uint32_t)sizeof(Splat) + 1u : last;
        }
        __syncthreads();
        if (active && j < end && s_hit[tid]) active[gj] = 1;
    }
    if (STATS) {
        // entries the per-pixel definition examines: up to and including the
        // terminating one, else the whole list
        const uint32_t n_eval = !inside ? 0u : (T < 0.0f ? term_at : end - start);
        const uint32_t e = wave_sum_u32(n_eval), i = wave_sum_u32(n_inc);
        if (lane_id() == 0) {
            s_stat[0][w] = e;
            s_stat[1][w] = i;
            s_stat[2][w] = w_iter;      // wave-uniform counts
            s_stat[3][w] = w_hit;
        }
        __syncthreads();
        if (tid < 4)
            atomicAdd(&pair_stats[tid], (unsigned long long)s_stat[tid][0] + s_stat[tid][1] + s_stat[tid][2] +
                                            s_stat[tid][3]);
    }
    T = fabsf(T);
    float lsum = 0.0f;
    if (inside) {
        const size_t HW = (size_t)W * H, p = (size_t)py * W + px;
        const float o0 = fmaf(T, bg0, c0), o1 = fmaf(T, bg1, c1), o2 = fmaf(T, bg2, c2);
        img[p] = o0;
        img[HW + p] = o1;
        img[2 * HW + p] = o2;
        final_T[p] = T;
        n_contrib[p] = last;
        if (LOSS) {
            float g0, g1, g2;
            lsum += l1_elem(o0, target[p], inv_total, g0);
            lsum += l1_elem(o1, target[HW + p], inv_total, g1);
            lsum += l1_elem(o2, target[2 * HW + p], inv_total, g2);
            dL[p] = g0;
            dL[HW + p] = g1;
            dL[2 * HW + p] = g2;
        }
    }
    if (LOSS) {
        __shared__ float s_loss[4];
        lsum = wave_sum(lsum);
        if (lane_id() == 0) s_loss[w] = lsum;
        __syncthreads();
        if (tid == 0) loss_partial[tile] = (s_loss[0] + s_loss[1]) + (s_loss[2] + s_loss[3]);
    }
}

// ---------------------------------------------------------------------------
// L1 loss
// ---------------------------------------------------------------------------


// Block b covers elements [b*2048, b*2048+2048): with VEC, as 512 float4
// (all three arrays 16-byte aligned; elements past the last whole float4
// are done one by one by the last block), else element by element.
template <bool VEC>
__global__ void __launch_bounds__(GS_BLOCK) k_loss_l1(const float* __restrict__ img, const float* __restrict__ tgt,
                                                      uint32_t total, float inv, float* __restrict__ dL,
                                                      float* __restrict__ partial) {
    __shared__ float s_red[4];
    float acc = 0.0f;
    if (VEC) {
        const uint32_t n4 = total / 4;
        const float4* a4 = reinterpret_cast<const float4*>(img);
        const float4* t4 = reinterpret_cast<const float4*>(tgt);
        float4* d4 = reinterpret_cast<float4*>(dL);
        const uint32_t base = blockIdx.x * (GS_TILE_ITEMS / 4) + threadIdx.x;
#pragma unroll
        for (int k = 0; k < GS_ITEMS / 4; ++k) {
            const uint32_t i = base + k * GS_BLOCK;
            if (i < n4) {
                const float4 a = a4[i], t = t4[i];
                float4 g;
                acc += l1_elem(a.x, t.x, inv, g.x);
                acc += l1_elem(a.y, t.y, inv, g.y);
                acc += l1_elem(a.z, t.z, inv, g.z);
                acc += l1_elem(a.w, t.w, inv, g.w);
                d4[i] = g;
            }
        }
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x < total - 4 * n4) {
            const uint32_t i = 4 * n4 + threadIdx.x;
            float g;
            acc += l1_elem(img[i], tgt[i], inv, g);
            dL[i] = g;
        }
    } else {
        const uint32_t base = blockIdx.x * GS_TILE_ITEMS + threadIdx.x;
#pragma unroll
        for (int k = 0; k < GS_ITEMS; ++k) {
            const uint32_t i = base + k * GS_BLOCK;
            if (i < total) {
                float g;
                acc += l1_elem(img[i], tgt[i], inv, g);
                dL[i] = g;
            }
        }
    }
    acc = wave_sum(acc);
    if (lane_id() == 0) s_red[threadIdx.x / GS_WAVE] = acc;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
}

__global__ void __launch_bounds__(GS_BLOCK) k_loss_final(const float* __restrict__ partial, uint32_t nb,
                                                         double inv_total, float* __restrict__ loss) {
    __shared__ double s[GS_BLOCK / GS_WAVE];
    constexpr int U = 8;
    double acc = 0.0;
    // all of a thread's loads are issued before its sums (float4 when aligned)
    uint32_t done = 0;
    if ((reinterpret_cast<uintptr_t>(partial) & 15u) == 0u) {
        const uint32_t n4 = nb / 4u;
        const float4* p4 = reinterpret_cast<const float4*>(partial);
        for (uint32_t i0 = threadIdx.x; i0 < n4; i0 += U * GS_BLOCK) {
            float4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t i = i0 + (uint32_t)u * GS_BLOCK;
                v[u] = i < n4 ? p4[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                acc += ((double)v[u].x + (double)v[u].y) + ((double)v[u].z + (double)v[u].w);
        }
        done = 4u * n4;
    }
    for (uint32_t i = done + threadIdx.x; i < nb; i += GS_BLOCK) acc += (double)partial[i];
#pragma unroll
    for (int d = GS_WAVE / 2; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, GS_WAVE);
    if (lane_id() == 0) s[threadIdx.x / GS_WAVE] = acc;
    __syncthreads();
    if (threadIdx.x == 0) *loss = (float)(((s[0] + s[1]) + (s[2] + s[3])) * inv_total);
}

// ---------------------------------------------------------------------------
// backward, part 1: per pixel, back to front
// ---------------------------------------------------------------------------

constexpr int kG = 9;   // du dv dA dB dC dopacity dr dg db
constexpr int kSlot = 12;          // floats per pair slot (9 used, padded for 16-byte stores)
constexpr int kBwdBatch = GS_WAVE;    // pairs walked between two combinations of the strips' sums
constexpr int kBwdPad = 2;            // pairs per iteration of the walk
constexpr int kStrips = 4;            // 8x2 strips of a wave's 8x8 quadrant, one per 16-lane row
constexpr int kSums = 8;              // floats a strip keeps per pair

// Per pixel, walking back to front: T is recovered in front of each included
// pair as T / (1 - alpha), and instead of the three suffix colour sums S_c
// (the colour still to come behind the pair, background included) the pixel
// keeps their projection gS = sum_c dL/dC_c S_c on its upstream gradient,
// which is all that d alpha needs:
//   dL/dalpha = T_k (g . rgb) - gS / (1 - alpha),  gS += alpha T_k (g . rgb).
//
// The 2D gradient of a pair is linear in moments of ds = dL/dsigma over its
// pixels: with sigma = (A dx^2 + 2B dx dy + C dy^2) / 2 and (dx, dy) the offset
// of the splat centre from the pixel centre,
//   dL/du = A m_x + B m_y,  dL/dv = B m_x + C m_y,
//   dL/dA = m_xx / 2,  dL/dB = m_xy,  dL/dC = m_yy / 2,  dL/dopacity = -m / o,
// with m = sum ds, m_x = sum ds dx, m_xy = sum ds dx dy and so on (the opacity
// line because ds = -dL/dalpha * o e^-sigma below the 0.99 cap, and both are 0
// at it).  Each 16-lane row of a wave renders an 8x2 strip of pixels and walks its
// own list of the batch.  The pixels of one of the strip's two pixel rows share dy, so
// eight sums hold all moments: of ds and ds dx over each pixel row, and of ds dx^2 and
// the three colour terms over the strip.  dx and dy are differences of the fp32 centre and
// the pixel centre's exact coordinate, rounded once.  A strip takes a pair at most once per batch, so
// its sums go to the (strip, pair) record with plain LDS writes; after the walk
// four threads per pair add the 16 strips' records in a fixed order.  A pair slot holds
// (m_x, m_y, m_xx, m_xy, m_yy, m, colour); k_project_bwd expands it with the
// conic once per primitive.
//
// What bounds it is VALU issue: 53 instructions per (wave, pair) step, 18 of them for
// the eight sums (24 while they held ds h and ds dx h, h the pixel row's offset from the
// strip's middle, which also cost the y moments their last bits).  Two pairs are
// evaluated side by side in front of the serial T and gS chain.  The strip is 8x2 because it weighs the steps against the sums:
// 16x1 rows need six sums but 1.26 times the steps, 4x4 blocks nine for 0.93 times, 8x8
// blocks nine over 64 lanes for 1.33 times.  The sums are DPP additions because nothing
// else here is cheaper: the 32-bit matrix product does not run beside other waves' VALU
// on this chip (one 16x16x4 product costs 34 cycles of it, and the four products that
// sum 64 pixels took the walk from 209 to 293 us), and an LDS float add costs 3 cycles a
// lane.  The records (33 KB) allow four workgroups per CU.  Measured, 16x1 rows with a
// butterfly each before and this: 1M-primitive 1080p room (with the overlapped commit)
// 264 -> 208 us, 3M walk-through 151 -> 91, 200k ring at 720p 169 -> 122, 60k ring at
// 651x433 143 -> 80, 10k box at 256x256 82 -> 45.

// Eight sums over each 16-lane row, in 12 DPP additions: of m and x over each half of the
// row, of e..h over all of it.  The halves of two of e..h are added into the two halves of
// one register; then the quarters of two registers (m and x as they are) into the
// quarters of one, and two steps inside each quarter finish.  Returns quarter by quarter
// m, x of the low half and m, x of the high half in the even lanes, and e, g, f, h in the
// odd ones.  A DPP source must have been written at least two instructions earlier
// (s_nop where the order does not see to it).
__device__ __forceinline__ float row_sum8(float m, float x, float e, float f, float g, float h, bool odd) {
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %1, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %2, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %0, %0, %0 row_shl:4 row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %0, %3, %3 row_shr:4 row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %1, %1, %1 row_shl:4 row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %1, %2, %2 row_shr:4 row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_add_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_add_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
        : "+&v"(m), "+&v"(e), "+&v"(g)
        : "v"(x), "v"(f), "v"(h));
    return odd ? e : m;
}

__device__ __forceinline__ float quad_add(float v) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true));
}

__global__ void __launch_bounds__(GS_BLOCK, 4) k_raster_bwd(
    const uint32_t* __restrict__ tile_order, const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ vals,
    const float2* __restrict__ mean2d, const float4* __restrict__ conic_op, const float* __restrict__ rgb, int32_t W,
    int32_t H, int32_t TX, float bg0,
    float bg1, float bg2, const float* __restrict__ final_T, const uint32_t* __restrict__ n_contrib,
    const float* __restrict__ dL_dimg, const uint32_t* __restrict__ pair_emit, float* __restrict__ slots) {
    // record and sums kBwdBatch belong to a pair that blends nothing: it pads the lists
    __shared__ Splat L[kBwdBatch + 1];
    __shared__ __align__(16) float s_sum[4 * kStrips][kBwdBatch + 1][kSums];
    __shared__ float s_u[kBwdBatch + 1], s_v[kBwdBatch];      // splat centres
    __shared__ __align__(4) uint16_t s_list[4 * kStrips][kBwdBatch + kBwdPad];   // per strip: byte offsets of its pairs' sums
    __shared__ uint32_t s_emit[kBwdBatch];
    __shared__ uint32_t s_max[4];
    __shared__ uint32_t s_checked;
    __shared__ uint16_t s_mask[kBwdBatch];
    constexpr uint32_t kStep = kSums * sizeof(float);          // a list entry is pair k's k * kStep
    static_assert(sizeof(Splat) == 2 * kStep, "a record lies at twice its sums' offset");
    const uint32_t tile = dispatch_tile(tile_order);
    if (tile >= gridDim.x) return;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid / GS_WAVE);
    const int lane = lane_id();
    const int strip = lane >> 4;
    const int tx = (int)tile % TX, ty = (int)tile / TX;
    const int px = tx * GS_TILE + quad_x(tid);
    const int py = ty * GS_TILE + quad_y(tid);
    const bool inside = px < W && py < H;
    const double xc = tx * GS_TILE + 8, yc = ty * GS_TILE + 8;
    const PixelPoly P(quad_x(tid), quad_y(tid));
    const uint32_t start = ranges[2 * tile], n = ranges[2 * tile + 1] - start;
    const size_t HW = (size_t)W * H, pix = (size_t)py * W + px;
    float T = inside ? final_T[pix] : 1.0f;
    const uint32_t last = inside ? n_contrib[pix] : 0u;
    const float gC0 = inside ? dL_dimg[pix] : 0.0f;
    const float gC1 = inside ? dL_dimg[HW + pix] : 0.0f;
    const float gC2 = inside ? dL_dimg[2 * HW + pix] : 0.0f;
    float gS = T * (gC0 * bg0 + gC1 * bg1 + gC2 * bg2);
    // largest n_contrib of each strip of the wave, and of the tile
    uint32_t rl = last;
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) rl = max(rl, (uint32_t)__shfl_xor((int)rl, d, GS_WAVE));
    uint32_t strip_last[kStrips], wl = 0u;
#pragma unroll
    for (int q = 0; q < kStrips; ++q) {
        strip_last[q] = (uint32_t)__builtin_amdgcn_readlane((int)rl, 16 * q);
        wl = max(wl, strip_last[q]);
    }
    if (lane == 0) s_max[w] = wl;
    if (tid < 16) reinterpret_cast<float*>(&L[kBwdBatch])[tid] = 0.0f;
    if (tid == 16) s_u[kBwdBatch] = 0.0f;
    if (tid < 4 * kStrips * kBwdPad) s_list[tid / kBwdPad][kBwdBatch + tid % kBwdPad] = (uint16_t)(kBwdBatch * kStep);
    __syncthreads();
    const uint32_t maxlast = max(max(s_max[0], s_max[1]), max(s_max[2], s_max[3]));
    const float xj = (float)px + 0.5f;      // (exact: an image side has at most 16 bits)
    // where this lane stores its sum: row_sum8 leaves sum (bank, odd) in every lane of a bank's parity
    const bool odd = (lane & 1) != 0;
    const int bank = (lane >> 2) & 3;
    char* const my_sums = reinterpret_cast<char*>(&s_sum[w * kStrips + strip][0][bank + (odd ? 4 : 0)]);
    if (n == 0) return;
    for (int32_t gs = (int32_t)((n - 1) / GS_BLOCK * GS_BLOCK); gs >= 0; gs -= GS_BLOCK) {
        // the next 256 pairs' primitives, one per thread; wave b then stages batch b
        const uint32_t pos = (uint32_t)gs + tid;
        float2 m = make_float2(0.0f, 0.0f);
        float4 co = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        float cr[3] = {0.0f, 0.0f, 0.0f};
        const uint32_t emit = pos < n ? pair_emit[start + pos] : 0u;
        if (pos < n && pos < maxlast) {
            const uint32_t g = vals[start + pos];
            m = mean2d[g];
            co = conic_op[g];
            cr[0] = rgb[3 * (size_t)g];
            cr[1] = rgb[3 * (size_t)g + 1];
            cr[2] = rgb[3 * (size_t)g + 2];
        }
        for (int b = (int)min(3u, (n - 1u - (uint32_t)gs) / kBwdBatch); b >= 0; --b) {
            const uint32_t bs = (uint32_t)gs + b * kBwdBatch;
            const uint32_t cnt = min((uint32_t)kBwdBatch, n - bs);
            if (bs >= maxlast) {
                // no pixel included any of these
                if (w == b && (uint32_t)lane < cnt) {
                    float4* dst = reinterpret_cast<float4*>(slots + (size_t)emit * kSlot);
                    dst[0] = dst[1] = dst[2] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                }
                continue;
            }
            if (w == b) {
                uint32_t mask = 0u;
                if ((uint32_t)lane < cnt && pos < maxlast) mask = stage_pair<2>(&L[lane], m, co, cr, xc, yc);
                s_u[lane] = m.x;
                s_v[lane] = mask ? m.y : 0.0f;      // (of a pair no pixel takes it may be infinite)
                s_mask[lane] = (uint16_t)mask;
                s_emit[lane] = emit;
                const uint64_t check = __ballot((mask & kChecked) != 0u);
                if (lane == 0) s_checked = check != 0ull ? 1u : 0u;
            }
            __syncthreads();
            // the strips' lists, back to front and filled up with the pad; pairs a strip does not take leave zero sums
            const uint32_t mask = (uint32_t)s_mask[lane] >> (kStrips * w);
            uint32_t n_list = 0u;
#pragma unroll
            for (int q = 0; q < kStrips; ++q) {
                const bool on = bs + (uint32_t)lane < strip_last[q] && ((mask >> q) & 1u);
                const uint64_t taken = __ballot(on);
                const uint32_t nq = popc64(taken), before = popc64(taken & lanemask_lt());
                s_list[w * kStrips + q][on ? nq - 1u - before : nq + lane - before] =
                    (uint16_t)((on ? lane : kBwdBatch) * kStep);
                if (!on) {
                    float4* z = reinterpret_cast<float4*>(&s_sum[w * kStrips + q][lane][0]);
                    z[0] = z[1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                }
                n_list = max(n_list, nq);
            }
            n_list = __builtin_amdgcn_readfirstlane(n_list);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // the pixel's pairs of this batch: offsets below last_b
            const uint32_t last_b = (last > bs ? min(last - bs, (uint32_t)kBwdBatch) : 0u) * kStep;
            const uint16_t* list = s_list[w * kStrips + strip];
            auto walk = [&](auto checked) {
                constexpr bool CHECK = decltype(checked)::value;
                for (uint32_t i0 = 0; i0 < n_list; i0 += kBwdPad) {
                    const uint32_t at2 = *reinterpret_cast<const uint32_t*>(list + i0);
                    // the pairs' records and footprints side by side, then the chain through T and gS
                    float capped[kBwdPad], u[kBwdPad], c0[kBwdPad], c1[kBwdPad], c2[kBwdPad];
                    bool on[kBwdPad];
#pragma unroll
                    for (int i = 0; i < kBwdPad; ++i) {
                        const uint32_t at = i ? at2 >> 16 : at2 & 0xFFFFu;
                        const Splat& S = *reinterpret_cast<const Splat*>(reinterpret_cast<const char*>(L) + 2 * at);
                        u[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(s_u) + at / kSums);
                        c0[i] = S.r;
                        c1[i] = S.g;
                        c2[i] = S.b;
                        float sigma = P.eval(S), o = S.o;
                        on[i] = !CHECK || check_sigma(S, sigma, o);
                        capped[i] = fminf(kAlphaMax, o * exp_neg(sigma));
                    }
#pragma unroll
                    for (int i = 0; i < kBwdPad; ++i) {
                        const uint32_t at = i ? at2 >> 16 : at2 & 0xFFFFu;
                        // a lane without the pair takes alpha = 0: its T stays, its weight and ds are 0
                        bool ok = (at < last_b) & !(capped[i] < kAlphaMin);
                        if (CHECK) ok = ok & on[i];
                        const float al = ok ? capped[i] : 0.0f;
                        const float inv_om = __builtin_amdgcn_rcpf(1.0f - al);
                        T = T * inv_om;
                        float gcol = gC0 * c0[i] + gC1 * c1[i] + gC2 * c2[i];
                        if (CHECK) gcol = ok ? gcol : 0.0f;
                        const float dalpha = gS * inv_om - T * gcol;        // -dL/dalpha
                        const float wgt = al * T;
                        gS = fmaf(wgt, gcol, gS);
                        // the 0.99 cap stops d/d(opacity, sigma); a pixel whose gS is not finite passes
                        // that on to the pairs it includes only
                        const float ds = ok & (capped[i] < kAlphaMax) ? dalpha * al : 0.0f;
                        const float dx = u[i] - xj;
                        const float dsx = ds * dx;
                        *reinterpret_cast<float*>(my_sums + at) =
                            row_sum8(ds, dsx, dsx * dx, wgt * gC1, wgt * gC0, wgt * gC2, odd);
                    }
                }
            };
            if (s_checked)
                walk(std::true_type{});
            else
                walk(std::false_type{});
            __syncthreads();
            // four threads per pair, two strips' rows of the tile each (both quadrants
            // beside each other share the rows); the slot is the pair's emission
            // position: a primitive's pairs end up side by side for k_slot_sum
            const uint32_t k = (uint32_t)tid >> 2;
            uint32_t part = (uint32_t)tid & 3u;
            loaded(part);       // (formed here and not kept through the walk, whose two pairs need the registers)
            if (k < cnt) {
                float acc[kG] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
                const float v = s_v[k];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const uint32_t row = 2u * part + i;                          // strip of the tile, downwards
                    const uint32_t sl = (row >> 2) * 2u * kStrips + (row & 3u);  // in the left quadrant; the right one follows
                    const float4 a0 = *reinterpret_cast<const float4*>(&s_sum[sl][k][0]);
                    const float4 a1 = *reinterpret_cast<const float4*>(&s_sum[sl][k][4]);
                    const float4 b0 = *reinterpret_cast<const float4*>(&s_sum[sl + kStrips][k][0]);
                    const float4 b1 = *reinterpret_cast<const float4*>(&s_sum[sl + kStrips][k][4]);
                    // as stored: m, m_x of the upper and of the lower pixel row; m_xx and the colours
                    const float m0 = a0.x + b0.x, x0 = a0.y + b0.y, m1 = a0.z + b0.z, x1 = a0.w + b0.w;
                    const float y = (float)(ty * GS_TILE + 2 * (int)row) + 0.5f;
                    const float dy0 = v - y, dy1 = v - (y + 1.0f);
                    const float y0 = dy0 * m0, y1 = dy1 * m1;
                    acc[0] += x0 + x1;
                    acc[1] += y0 + y1;
                    acc[2] += a1.x + b1.x;
                    acc[3] += fmaf(dy0, x0, dy1 * x1);
                    acc[4] += fmaf(dy0, y0, dy1 * y1);
                    acc[5] += m0 + m1;
                    acc[6] += a1.y + b1.y;
                    acc[7] += a1.z + b1.z;
                    acc[8] += a1.w + b1.w;
                }
#pragma unroll
                for (int q = 0; q < kG; ++q) acc[q] = quad_add(acc[q]);
                const float4 out = part == 0u   ? make_float4(acc[0], acc[1], acc[2], acc[3])
                                   : part == 1u ? make_float4(acc[4], acc[5], acc[6], acc[7])
                                                : make_float4(acc[8], 0.0f, 0.0f, 0.0f);
                if (part < 3u) reinterpret_cast<float4*>(slots + (size_t)s_emit[k] * kSlot)[part] = out;
            }
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------
// backward, part 2: per visible primitive
// ---------------------------------------------------------------------------

constexpr float kY1 = 0.48860251190291992f;
constexpr float kY2a = 1.0925484305920792f;
constexpr float kY2b = 0.31539156525252005f;
constexpr float kY2c = 0.54627421529603959f;
constexpr float kY3a = 0.59004358992664352f;
constexpr float kY3b = 2.8906114426405538f;
constexpr float kY3c = 0.45704579946446572f;
constexpr float kY3d = 0.37317633259011546f;
constexpr float kY3e = 1.4453057213202769f;

// SH basis values and gradients of their polynomial form at d.
template <int DEG>
__device__ __forceinline__ void sh_basis_grad(float x, float y, float z, float* Y, float (*G)[3]) {
    Y[0] = 0.28209479177387814f;
    G[0][0] = G[0][1] = G[0][2] = 0.0f;
    if (DEG < 1) return;
    Y[1] = -kY1 * y; G[1][0] = 0.0f; G[1][1] = -kY1; G[1][2] = 0.0f;
    Y[2] = kY1 * z;  G[2][0] = 0.0f; G[2][1] = 0.0f; G[2][2] = kY1;
    Y[3] = -kY1 * x; G[3][0] = -kY1; G[3][1] = 0.0f; G[3][2] = 0.0f;
    if (DEG < 2) return;
    const float xx = x * x, yy = y * y, zz = z * z;
    Y[4] = kY2a * x * y;  G[4][0] = kY2a * y; G[4][1] = kY2a * x; G[4][2] = 0.0f;
    Y[5] = -kY2a * y * z; G[5][0] = 0.0f; G[5][1] = -kY2a * z; G[5][2] = -kY2a * y;
    Y[6] = kY2b * (2.0f * zz - xx - yy);
    G[6][0] = -2.0f * kY2b * x; G[6][1] = -2.0f * kY2b * y; G[6][2] = 4.0f * kY2b * z;
    Y[7] = -kY2a * x * z; G[7][0] = -kY2a * z; G[7][1] = 0.0f; G[7][2] = -kY2a * x;
    Y[8] = kY2c * (xx - yy); G[8][0] = 2.0f * kY2c * x; G[8][1] = -2.0f * kY2c * y; G[8][2] = 0.0f;
    if (DEG < 3) return;
    Y[9] = -kY3a * y * (3.0f * xx - yy);
    G[9][0] = -6.0f * kY3a * x * y; G[9][1] = -3.0f * kY3a * (xx - yy); G[9][2] = 0.0f;
    Y[10] = kY3b * x * y * z;
    G[10][0] = kY3b * y * z; G[10][1] = kY3b * x * z; G[10][2] = kY3b * x * y;
    Y[11] = -kY3c * y * (4.0f * zz - xx - yy);
    G[11][0] = 2.0f * kY3c * x * y; G[11][1] = -kY3c * (4.0f * zz - xx - 3.0f * yy); G[11][2] = -8.0f * kY3c * y * z;
    Y[12] = kY3d * z * (2.0f * zz - 3.0f * xx - 3.0f * yy);
    G[12][0] = -6.0f * kY3d * x * z; G[12][1] = -6.0f * kY3d * y * z; G[12][2] = kY3d * (6.0f * zz - 3.0f * xx - 3.0f * yy);
    Y[13] = -kY3c * x * (4.0f * zz - xx - yy);
    G[13][0] = -kY3c * (4.0f * zz - 3.0f * xx - yy); G[13][1] = 2.0f * kY3c * x * y; G[13][2] = -8.0f * kY3c * x * z;
    Y[14] = kY3e * z * (xx - yy);
    G[14][0] = 2.0f * kY3e * x * z; G[14][1] = -2.0f * kY3e * y * z; G[14][2] = kY3e * (xx - yy);
    Y[15] = -kY3a * x * (xx - 3.0f * yy);
    G[15][0] = -3.0f * kY3a * (xx - yy); G[15][1] = 6.0f * kY3a * x * y; G[15][2] = 0.0f;
}

__device__ __forceinline__ float dot3(const float* a, const float* b) { return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]; }

// Per-primitive work: k_slot_sum adds each visible primitive's pair slots, and
// k_project_bwd, one thread per visible row, applies the chain rule to the sums.

template <int DEG>
struct RowLayout {
    static constexpr int K = (DEG + 1) * (DEG + 1);
    static constexpr int SH = 3 * K;
    static constexpr int ROW = 11 + SH;                        // mean 3, log_scale 3, quat 4, opacity 1, sh
    static constexpr int ROW4 = (ROW + 3) / 4 * 4;
};

// Chain rule from one primitive's 2D gradient (du, dv, dA, dB, dC in g2) back
// to mean, log-scale and quaternion, evaluated in scalar type Rl.  gpw
// receives the projection path's camera-space mean gradient (the world-space
// one is R^T gpw, formed by the caller together with the colour path's part);
// out receives log_scale (3..5) and quat (6..9) gradients.
template <typename Rl>
__device__ __forceinline__ void geometry_bwd(const float* mu_f, const float* ls_f, const float* qr_f,
                                             const float* g2, const CamArgs& c, Rl* gpw, float* out) {
    Rl R[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) R[k] = (Rl)c.R[k];
    const Rl mu[3] = {(Rl)mu_f[0], (Rl)mu_f[1], (Rl)mu_f[2]};
    const Rl fx = (Rl)c.fx, fy = (Rl)c.fy;
    Rl p[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) p[k] = R[3 * k] * mu[0] + R[3 * k + 1] * mu[1] + R[3 * k + 2] * mu[2] + (Rl)c.t[k];
    const Rl s[3] = {exp((Rl)ls_f[0]), exp((Rl)ls_f[1]), exp((Rl)ls_f[2])};
    const Rl q0 = (Rl)qr_f[0], q1 = (Rl)qr_f[1], q2 = (Rl)qr_f[2], q3 = (Rl)qr_f[3];
    const Rl iq = (Rl)1 / sqrt(q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3);
    const Rl w = q0 * iq, x = q1 * iq, y = q2 * iq, z = q3 * iq;
    const Rl Rq[3][3] = {{1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)},
                         {2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)},
                         {2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)}};
    Rl M[3][3], Sg[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) M[a][b] = Rq[a][b] * s[b];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) Sg[a][b] = M[a][0] * M[b][0] + M[a][1] * M[b][1] + M[a][2] * M[b][2];
    const Rl tz = p[2], itz = (Rl)1 / tz;
    const Rl lx = (Rl)(1.3f * c.tan_fovx), ly = (Rl)(1.3f * c.tan_fovy);
    const Rl rx = p[0] * itz, ry = p[1] * itz;
    const bool clx = rx < -lx || rx > lx, cly = ry < -ly || ry > ly;
    const Rl xr = rx < -lx ? -lx : (rx > lx ? lx : rx);
    const Rl yr = ry < -ly ? -ly : (ry > ly ? ly : ry);
    const Rl j00 = fx * itz, j11 = fy * itz;
    const Rl j02 = -fx * xr * itz, j12 = -fy * yr * itz;
    Rl T0[3], T1[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        T0[k] = j00 * R[k] + j02 * R[6 + k];
        T1[k] = j11 * R[3 + k] + j12 * R[6 + k];
    }
    Rl ST0[3], ST1[3];   // Sigma T0, Sigma T1
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        ST0[a] = Sg[a][0] * T0[0] + Sg[a][1] * T0[1] + Sg[a][2] * T0[2];
        ST1[a] = Sg[a][0] * T1[0] + Sg[a][1] * T1[1] + Sg[a][2] * T1[2];
    }
    const Rl ca = T0[0] * ST0[0] + T0[1] * ST0[1] + T0[2] * ST0[2] + (Rl)0.3f;
    const Rl cb = T0[0] * ST1[0] + T0[1] * ST1[1] + T0[2] * ST1[2];
    const Rl cc = T1[0] * ST1[0] + T1[1] * ST1[1] + T1[2] * ST1[2] + (Rl)0.3f;
    const Rl det = ca * cc - cb * cb;
    const Rl id2 = (Rl)1 / (det * det);
    // conic (A,B,C) = (c, -b, a)/det  ->  gradient w.r.t. (a, b, c)
    const Rl gA = g2[2], gB = g2[3], gC = g2[4];
    const Rl ga = (-gA * cc * cc + gB * cb * cc - gC * cb * cb) * id2;
    const Rl gb = (2 * gA * cb * cc - gB * (ca * cc + cb * cb) + 2 * gC * ca * cb) * id2;
    const Rl gcv = (-gA * cb * cb + gB * ca * cb - gC * ca * ca) * id2;
    // a = T0.S.T0, b = T0.S.T1, c = T1.S.T1
    Rl gT0[3], gT1[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        gT0[a] = 2 * ga * ST0[a] + gb * ST1[a];
        gT1[a] = gb * ST0[a] + 2 * gcv * ST1[a];
    }
    const Rl gj00 = gT0[0] * R[0] + gT0[1] * R[1] + gT0[2] * R[2];
    const Rl gj02 = gT0[0] * R[6] + gT0[1] * R[7] + gT0[2] * R[8];
    const Rl gj11 = gT1[0] * R[3] + gT1[1] * R[4] + gT1[2] * R[5];
    const Rl gj12 = gT1[0] * R[6] + gT1[1] * R[7] + gT1[2] * R[8];
    const Rl itz2 = itz * itz;
    Rl gp[3] = {0, 0, 0};
    gp[2] -= (gj00 * fx + gj11 * fy) * itz2;
    if (clx) {
        gp[2] += gj02 * fx * xr * itz2;
    } else {
        gp[0] -= gj02 * fx * itz2;
        gp[2] += 2 * gj02 * fx * p[0] * itz2 * itz;
    }
    if (cly) {
        gp[2] += gj12 * fy * yr * itz2;
    } else {
        gp[1] -= gj12 * fy * itz2;
        gp[2] += 2 * gj12 * fy * p[1] * itz2 * itz;
    }
    const Rl gu = g2[0], gv = g2[1];
    gp[0] += gu * fx * itz;
    gp[1] += gv * fy * itz;
    gp[2] -= (gu * fx * p[0] + gv * fy * p[1]) * itz2;
    gpw[0] = gp[0];
    gpw[1] = gp[1];
    gpw[2] = gp[2];
    // Sigma = M M^T with symmetric gradient Gs = ga T0T0^T + gb (T0T1^T + T1T0^T)/2 + gc T1T1^T
    Rl Gs[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
            Gs[a][b] = ga * T0[a] * T0[b] + (Rl)0.5 * gb * (T0[a] * T1[b] + T1[a] * T0[b]) + gcv * T1[a] * T1[b];
    Rl gR[3][3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        Rl gsb = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const Rl gM = 2 * (Gs[a][0] * M[0][b] + Gs[a][1] * M[1][b] + Gs[a][2] * M[2][b]);
            gR[a][b] = gM * s[b];
            gsb += gM * Rq[a][b];
        }
        out[3 + b] = (float)(gsb * s[b]);
    }
    const Rl gw = 2 * (x * (gR[2][1] - gR[1][2]) + y * (gR[0][2] - gR[2][0]) + z * (gR[1][0] - gR[0][1]));
    const Rl gx = 2 * (w * (gR[2][1] - gR[1][2]) - 2 * x * (gR[1][1] + gR[2][2]) + y * (gR[0][1] + gR[1][0]) +
                       z * (gR[0][2] + gR[2][0]));
    const Rl gy = 2 * (w * (gR[0][2] - gR[2][0]) + x * (gR[0][1] + gR[1][0]) - 2 * y * (gR[0][0] + gR[2][2]) +
                       z * (gR[1][2] + gR[2][1]));
    const Rl gz = 2 * (w * (gR[1][0] - gR[0][1]) + x * (gR[0][2] + gR[2][0]) + y * (gR[1][2] + gR[2][1]) -
                       2 * z * (gR[0][0] + gR[1][1]));
    const Rl along = w * gw + x * gx + y * gy + z * gz;
    out[6] = (float)((gw - w * along) * iq);
    out[7] = (float)((gx - x * along) * iq);
    out[8] = (float)((gy - y * along) * iq);
    out[9] = (float)((gz - z * along) * iq);
}

template <int N>
__device__ __forceinline__ void load_row(const float* __restrict__ src, float* dst) {
    if constexpr (N % 4 == 0) {
        const float4* s4 = reinterpret_cast<const float4*>(src);
#pragma unroll
        for (int k = 0; k < N / 4; ++k) {
            const float4 v = s4[k];
            dst[4 * k] = v.x; dst[4 * k + 1] = v.y; dst[4 * k + 2] = v.z; dst[4 * k + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < N; ++k) dst[k] = src[k];
    }
}

// Position of id in the ascending list u[0..m), or m if absent.
__device__ __forceinline__ uint32_t find_row(const uint32_t* __restrict__ u, uint32_t m, uint32_t id) {
    uint32_t lo = 0, hi = m;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (u[mid] < id) lo = mid + 1; else hi = mid;
    }
    return (lo < m && u[lo] == id) ? lo : m;
}

// A primitive's slots are added by 8 lanes: one slot per lane first, then four more
// per lane; a primitive with more goes to a whole wave.
constexpr uint32_t kOctSlots = 8, kOctSlots2 = 5 * kOctSlots;
// Visible rows up to which 8 lanes take 4 primitives instead of 8, so that twice the
// workgroups share them and one round of loads does; with more rows the chip is full
// either way and the workgroups' own start costs.  Measured, 4 against 8, at 2 and at 6
// slots a primitive on average: 32k rows 4.6 against 5.9 us and 6.3 against 8.7, 98k 7.0
// against 8.4 and 12.4 against 13.5, 131k (the line) 9.0 against 8.7 and 15.0 against
// 14.9, 197k 12.8 against 11.0 and 19.7 against 18.8, 524k 24.0 against 21.2 and 43.2
// against 42.7.
constexpr uint32_t kFewRows = 1u << 17;

// The value of lane I of each 8 lanes, in all of them.
template <int I>
__device__ __forceinline__ uint32_t oct_bcast(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (I << 5) | 0x18);
}

// The sum over each 8 lanes, in all of them.
__device__ __forceinline__ float oct_sum(float v) {
    v = quad_add(v);
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, true));
}

template <int C>
__device__ __forceinline__ double dpp_add64(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), C, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), C, 0xF, 0xF, true);
    return v + __hiloint2double(hi, lo);
}
// a's halves (rows of 16 with ROWS) added in the low one (the even ones), b's in the other:
// the swap leaves the low half of a beside that of b, and so the high halves.
template <bool ROWS>
__device__ __forceinline__ double swap_add64(double a, double b) {
    const uint32_t al = __double2loint(a), ah = __double2hiint(a), bl = __double2loint(b), bh = __double2hiint(b);
    const auto lo = ROWS ? __builtin_amdgcn_permlane16_swap(al, bl, false, false)
                         : __builtin_amdgcn_permlane32_swap(al, bl, false, false);
    const auto hi = ROWS ? __builtin_amdgcn_permlane16_swap(ah, bh, false, false)
                         : __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// The sum over each 8 lanes, in all of them.
__device__ __forceinline__ double oct_sum64(double v) {
    return dpp_add64<0x141>(dpp_add64<0x4E>(dpp_add64<0xB1>(v)));
}
// The sums of a[0..9) over the wave: returned in lane l is that of a[slot_of(l)], a8 is the
// ninth's in all lanes.  Two values share a register from each of the first three steps on,
// so that one step inside 8 lanes serves all eight of them.
__device__ __forceinline__ uint32_t slot_of(uint32_t lane) {
    return ((lane >> 5) & 1u) | ((lane >> 4) & 1u) << 1 | ((lane >> 3) & 1u) << 2;
}
__device__ __forceinline__ double wave_sum9(const double (&a)[kG], uint32_t lane, double& a8) {
    const double t0 = swap_add64<true>(swap_add64<false>(a[0], a[1]), swap_add64<false>(a[2], a[3]));
    const double t1 = swap_add64<true>(swap_add64<false>(a[4], a[5]), swap_add64<false>(a[6], a[7]));
    const double s8 = swap_add64<false>(a[8], a[8]);
    const double r8 = swap_add64<true>(s8, s8);
    const bool high = (lane & 8u) != 0u;
    const double keep = high ? t1 : t0, send = high ? t0 : t1;
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(send), 0x128, 0xF, 0xF, true);     // row_ror:8
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(send), 0x128, 0xF, 0xF, true);
    a8 = oct_sum64(dpp_add64<0x128>(r8));
    return oct_sum64(keep + __hiloint2double(hi, lo));
}

__device__ __forceinline__ void add_slot(float (&a)[kG], const float4& x, const float4& y, float z) {
    a[0] += x.x; a[1] += x.y; a[2] += x.z; a[3] += x.w;
    a[4] += y.x; a[5] += y.y; a[6] += y.z; a[7] += y.w;
    a[8] += z;
}

// Per visible row r: the sum of the primitive's pair slots (emission
// positions pair_offset[id] .. + tiles[id], side by side; none if the pair
// list overflowed its capacity), as one kSlot-float row at sums + kSlot r.
// A kernel of its own: the chain rule's registers would leave the slot
// stream too few waves to keep its loads in flight.
//
// Latency bounds it, so the lists are spread over lanes: each 8 lanes take 8 (or 4)
// consecutive primitives, whose slots share cache lines, four at a time, with one
// lane per slot and every load of the four in flight; longer lists get one round of
// four slots per lane more, and the rare ones beyond that are left in LDS for the
// workgroup's waves, 256 slots a round: a lane's four in fp32, the lanes and rounds in fp64.
// These are the wide footprints near the camera, whose geometry gradients cancel by up to
// 1e3, so that the order of an fp32 sum decided the error of a whole view's gradients.  Its
// geometric mean against 64 bits over 12 seeds each, all in fp32, all in fp64 and this: 400k
// aerial 4.2, 3.7, 3.7e-6, 150k aerial 6.8, 5.3, 5.2e-6, 300k walk-through 7.1, 6.5, 6.5e-7.
// The kernel on 100k primitives of an aerial capture at 1910x1400, where most lists are long:
// 42.7, 47.4 (nine 64-bit butterflies and 36 conversions a lane), 42.2 us.
// Every order is fixed, so the sums do not
// depend on scheduling.  A thread per primitive with lists of more than 8 slots taken
// whole by the wave one after the other, before, and this: 200k ring at 720p (6 slots
// a primitive on average) 51 -> 18 us, 1M room 58 -> 37, 3M walk-through (2 slots)
// 27 -> 23, 10k box 6.5 -> 4.8.
__global__ void __launch_bounds__(GS_BLOCK) k_slot_sum(const uint32_t* __restrict__ vis_idx,
                                                       const uint32_t* __restrict__ vis_count,
                                                       const uint32_t* __restrict__ tiles,
                                                       const uint32_t* __restrict__ pair_offset,
                                                       const float* __restrict__ slots, uint32_t capacity,
                                                       float* __restrict__ sums) {
    __shared__ uint3 s_long[GS_BLOCK];      // row, first slot and count of each list left for the waves
    __shared__ uint32_t s_n;
    const uint32_t V = *vis_count;
    // Workgroup b takes chunks b, b + NB, b + 2 NB, ... of consecutive rows (NB the
    // workgroups needed): in a spatially ordered pool the long slot lists of
    // neighbours near the camera come in runs, which one workgroup would
    // otherwise add one after the other while the rest of the chip idles.
    const uint32_t per = V <= kFewRows ? 4u : 8u;
    const uint32_t per_block = GS_BLOCK / kOctSlots * per;
    const uint32_t nb = (V + per_block - 1u) / per_block;
    if (blockIdx.x >= nb) return;
    if (threadIdx.x == 0) s_n = 0u;
    __syncthreads();
    const uint32_t lane = lane_id(), at = lane & 7u;
    const uint32_t r0 = ((threadIdx.x >> 3) * nb + blockIdx.x) * per;
    // lane i of 8: the chunk's primitive i
    const bool valid = at < per && r0 + at < V;
    const uint32_t id = valid ? vis_idx[r0 + at] : 0u;
    uint32_t first = valid ? pair_offset[id] : 0u;
    uint32_t nt = valid ? tiles[id] : 0u;
    if (!((uint64_t)first + nt <= capacity)) first = nt = 0u;
    const bool is_long = nt > kOctSlots2;
    if (is_long) {
        s_long[atomicAdd(&s_n, 1u)] = make_uint3(r0 + at, first, nt);
        first = nt = 0u;
    }
    const uint64_t longs = __ballot(is_long);
    auto four = [&](auto i4) {
        constexpr int I = decltype(i4)::value * 4;
        const uint32_t f[4] = {oct_bcast<I>(first), oct_bcast<I + 1>(first), oct_bcast<I + 2>(first),
                               oct_bcast<I + 3>(first)};
        const uint32_t c[4] = {oct_bcast<I>(nt), oct_bcast<I + 1>(nt), oct_bcast<I + 2>(nt), oct_bcast<I + 3>(nt)};
        float4 v[4][2];
        float v8[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float4* sl = reinterpret_cast<const float4*>(
                slots + (size_t)(f[u] + min(at, c[u] > 0u ? c[u] - 1u : 0u)) * kSlot);   // past the list: its last slot, unused
            v[u][0] = sl[0];
            v[u][1] = sl[1];
            v8[u] = sl[2].x;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float a[kG] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
            if (at < c[u]) add_slot(a, v[u][0], v[u][1], v8[u]);
            if (__ballot(c[u] > kOctSlots) != 0ull) {
                float4 x[4][2];
                float x8[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float4* sl = reinterpret_cast<const float4*>(
                        slots + (size_t)(f[u] + min(at + kOctSlots * (k + 1), c[u] > 0u ? c[u] - 1u : 0u)) * kSlot);
                    x[k][0] = sl[0];
                    x[k][1] = sl[1];
                    x8[k] = sl[2].x;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (at + kOctSlots * (k + 1) < c[u]) add_slot(a, x[k][0], x[k][1], x8[k]);
            }
#pragma unroll
            for (int q = 0; q < kG; ++q) a[q] = oct_sum(a[q]);
            const uint32_t r = r0 + I + u;
            const bool left = ((longs >> ((lane & 56u) + I + u)) & 1ull) != 0ull;
            if (at < 3u && r < V && !left)
                reinterpret_cast<float4*>(sums + (size_t)r * kSlot)[at] =
                    at == 0u   ? make_float4(a[0], a[1], a[2], a[3])
                    : at == 1u ? make_float4(a[4], a[5], a[6], a[7])
                               : make_float4(a[8], 0.0f, 0.0f, 0.0f);
        }
    };
    four(std::integral_constant<int, 0>{});
    if (per == 8u) four(std::integral_constant<int, 1>{});
    __syncthreads();
    for (uint32_t l = threadIdx.x / GS_WAVE; l < s_n; l += GS_BLOCK / GS_WAVE) {
        const uint3 e = s_long[l];
        double a[kG] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        for (uint32_t k0 = 0; k0 < e.z; k0 += 4 * GS_WAVE) {
            float4 x[4][2];
            float x8[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4* sl = reinterpret_cast<const float4*>(
                    slots + (size_t)(e.y + min(k0 + j * GS_WAVE + lane, e.z - 1u)) * kSlot);
                x[j][0] = sl[0];
                x[j][1] = sl[1];
                x8[j] = sl[2].x;
            }
            float f[kG] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (k0 + j * GS_WAVE + lane < e.z) add_slot(f, x[j][0], x[j][1], x8[j]);
#pragma unroll
            for (int q = 0; q < kG; ++q) a[q] += f[q];
        }
        double a8;
        const float v = (float)wave_sum9(a, lane, a8);
        float* dst = sums + (size_t)e.x * kSlot;
        if (at == 0u) dst[slot_of(lane)] = v;
        if (lane == 1u) *reinterpret_cast<float4*>(dst + 8) = make_float4((float)a8, 0.0f, 0.0f, 0.0f);
    }
}

// Per visible row r: the primitive's 2D gradient (from its slot sums, row r
// of k_slot_sum), then the chain rule to the parameters; writes the row's
// gradient record at grad_rows + r * ld.  ACCUM (a task unit
// of several views): the record is added to row u instead, u the position of
// id in the unit's ascending union list, and |dL/d(u,v)| is added to
// grad_norm[id].
template <int DEG, bool ACCUM>
__global__ void __launch_bounds__(GS_BLOCK) k_project_bwd(
    const uint32_t* __restrict__ vis_idx, const uint32_t* __restrict__ vis_count, const float* __restrict__ sums,
    const float4* __restrict__ conic_op, const uint8_t* __restrict__ clampm, const float* __restrict__ mean, const float* __restrict__ log_scale,
    const float* __restrict__ quat, const float* __restrict__ opacity, const float* __restrict__ sh, SceneLd pld,
    CamArgs c, float* __restrict__ grad_rows, int32_t ld, float* __restrict__ grad2d, float* __restrict__ grad_norm,
    const uint32_t* __restrict__ union_idx, const uint32_t* __restrict__ union_count) {
    using L = RowLayout<DEG>;
    constexpr int K = L::K;
    const uint32_t V = *vis_count;
    const uint32_t r = blockIdx.x * GS_BLOCK + threadIdx.x;
    if (r >= V) return;
    const uint32_t id = vis_idx[r];
    float g2[kG];
    {
        const float4* src = reinterpret_cast<const float4*>(sums + (size_t)r * kSlot);
        const float4 a0 = src[0], a1 = src[1], a2 = src[2];
        g2[0] = a0.x; g2[1] = a0.y; g2[2] = a0.z; g2[3] = a0.w;
        g2[4] = a1.x; g2[5] = a1.y; g2[6] = a1.z; g2[7] = a1.w; g2[8] = a2.x;
    }
    {
        // moments -> 2D gradient, with the conic the pixels used; fp64 because
        // A m_x and B m_y can nearly cancel for elongated footprints
        const float4 co = conic_op[id];
        const double mx = g2[0], my = g2[1];
        g2[0] = (float)((double)co.x * mx + (double)co.y * my);
        g2[1] = (float)((double)co.y * mx + (double)co.z * my);
        g2[2] = 0.5f * g2[2];
        g2[4] = 0.5f * g2[4];
        g2[5] = co.w > 0.0f ? -g2[5] / co.w : 0.0f;
    }
    uint32_t row = r;
    if (ACCUM) {
        const uint32_t m = *union_count;
        row = find_row(union_idx, m, id);
        if (row == m) return;                 // not in the unit's union: nothing to add to
    }
    if (grad2d) {
#pragma unroll
        for (int q = 0; q < kG; ++q) grad2d[(size_t)id * kG + q] = g2[q];
    }
    if (grad_norm) {
        const float gn = sqrtf(g2[0] * g2[0] + g2[1] * g2[1]);
        grad_norm[id] = ACCUM ? grad_norm[id] + gn : gn;
    }
    float mu[3], ls[3], qr[4];
    load_row<3>(mean + (size_t)id * pld.mean, mu);
    load_row<4>(quat + (size_t)id * pld.quat, qr);
    float logit;
    if (pld.head) {
        float h[4];
        load_row<4>(quat + (size_t)id * pld.quat + 4, h);
        ls[0] = h[0]; ls[1] = h[1]; ls[2] = h[2]; logit = h[3];
    } else {
        load_row<3>(log_scale + (size_t)id * pld.log_scale, ls);
        logit = opacity[(size_t)id * pld.opacity];
    }
    const uint8_t cm = clampm[id];
    float out[L::ROW4];

    // 1. geometry, in fp64: for wide footprints the conic gradient is large
    //    while the scale / rotation gradients it produces are tiny, and the
    //    chain cancels too much for fp32
    double gp[3];
    geometry_bwd<double>(mu, ls, qr, g2, c, gp, out);

    // 2. opacity
    const float o = 1.0f / (1.0f + expf(-logit));
    out[10] = g2[5] * o * (1.0f - o);

    // 3. colour: dL/dsh and the view-direction path to the mean
    float gmu[3];
    {
        float v[3] = {mu[0] - c.campos[0], mu[1] - c.campos[1], mu[2] - c.campos[2]};
        const float len = sqrtf(dot3(v, v));
        const float il = 1.0f / len;
        const float d[3] = {v[0] * il, v[1] * il, v[2] * il};
        float Y[16], G[16][3];
        sh_basis_grad<DEG>(d[0], d[1], d[2], Y, G);
        const float gc[3] = {(cm & 1) ? 0.0f : g2[6], (cm & 2) ? 0.0f : g2[7], (cm & 4) ? 0.0f : g2[8]};
        float co[3 * K];
        load_row<3 * K>(sh + (size_t)id * pld.sh, co);
        float gd[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float a = gc[0] * co[3 * k] + gc[1] * co[3 * k + 1] + gc[2] * co[3 * k + 2];
            gd[0] += a * G[k][0];
            gd[1] += a * G[k][1];
            gd[2] += a * G[k][2];
            out[11 + 3 * k + 0] = gc[0] * Y[k];
            out[11 + 3 * k + 1] = gc[1] * Y[k];
            out[11 + 3 * k + 2] = gc[2] * Y[k];
        }
        const float rad = dot3(gd, d);
        gmu[0] = (gd[0] - d[0] * rad) * il;
        gmu[1] = (gd[1] - d[1] * rad) * il;
        gmu[2] = (gd[2] - d[2] * rad) * il;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
        out[k] = (float)((double)gmu[k] + (double)c.R[k] * gp[0] + (double)c.R[3 + k] * gp[1] +
                         (double)c.R[6 + k] * gp[2]);
#pragma unroll
    for (int k = L::ROW; k < L::ROW4; ++k) out[k] = 0.0f;

    float4* dst = reinterpret_cast<float4*>(grad_rows + (size_t)row * ld);
    if (ACCUM) {
#pragma unroll
        for (int k = 0; k < L::ROW4 / 4; ++k) {
            const float4 a = dst[k];
            dst[k] = make_float4(a.x + out[4 * k], a.y + out[4 * k + 1], a.z + out[4 * k + 2], a.w + out[4 * k + 3]);
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < L::ROW4 / 4; ++k) dst[k] = make_float4(out[4 * k], out[4 * k + 1], out[4 * k + 2], out[4 * k + 3]);
    for (int k = L::ROW4 / 4; k < ld / 4; ++k) dst[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

// First view of a task unit: the union's gradient rows (all ld columns) and
// the grad_norm entries of its ids start at zero.
__global__ void __launch_bounds__(GS_BLOCK) k_clear_union_rows(const uint32_t* __restrict__ union_idx,
                                                               const uint32_t* __restrict__ union_count,
                                                               float* __restrict__ grad_rows, int32_t ld,
                                                               float* __restrict__ grad_norm) {
    const uint32_t m = *union_count;
    const uint32_t q4 = (uint32_t)ld / 4;
    const uint64_t total = (uint64_t)m * q4;
    float4* rows = reinterpret_cast<float4*>(grad_rows);
    for (uint64_t i = (uint64_t)blockIdx.x * GS_BLOCK + threadIdx.x; i < total; i += (uint64_t)gridDim.x * GS_BLOCK) {
        rows[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (grad_norm && i % q4 == 0) grad_norm[union_idx[i / q4]] = 0.0f;
    }
}

}  // namespace

hipError_t launch_raster_fwd(const gs_proj& proj, const uint32_t* vals, const uint32_t* ranges,
                             const uint32_t* tile_order, int32_t width, int32_t height, const float bg[3],
                             float* img, float* final_T, uint32_t* n_contrib, uint8_t* active, uint64_t* pair_stats,
                             hipStream_t st) {
    const int32_t TX = (width + GS_TILE - 1) / GS_TILE, TY = (height + GS_TILE - 1) / GS_TILE;
    if (TX * TY == 0) return hipSuccess;
    if (pair_stats)
        hipLaunchKernelGGL((k_raster_fwd<true, false>), dim3(TX * TY), dim3(GS_BLOCK), 0, st, tile_order, ranges, vals,
                           reinterpret_cast<const float2*>(proj.mean2d),
                           reinterpret_cast<const float4*>(proj.conic_opacity), proj.rgb, width, height, TX, bg[0],
                           bg[1], bg[2], img, final_T, n_contrib, active,
                           reinterpret_cast<unsigned long long*>(pair_stats), nullptr, 0.0f, nullptr, nullptr);
    else
        hipLaunchKernelGGL((k_raster_fwd<false, false>), dim3(TX * TY), dim3(GS_BLOCK), 0, st, tile_order, ranges, vals,
                           reinterpret_cast<const float2*>(proj.mean2d),
                           reinterpret_cast<const float4*>(proj.conic_opacity), proj.rgb, width, height, TX, bg[0],
                           bg[1], bg[2], img, final_T, n_contrib, active, nullptr, nullptr, 0.0f, nullptr, nullptr);
    return hipGetLastError();
}

size_t raster_fwd_l1_ws_bytes(int32_t width, int32_t height) {
    const uint64_t T = (uint64_t)div_up((uint64_t)(width > 0 ? width : 0), GS_TILE) *
                       div_up((uint64_t)(height > 0 ? height : 0), GS_TILE);
    return align256(sizeof(float) * (T + 1));
}

hipError_t launch_raster_fwd_l1(const gs_proj& proj, const uint32_t* vals, const uint32_t* ranges,
                                const uint32_t* tile_order, int32_t width, int32_t height, const float bg[3],
                                const float* target, float* img, float* final_T, uint32_t* n_contrib, uint8_t* active,
                                float* loss, float* dL, void* ws, hipStream_t st) {
    const int32_t TX = (width + GS_TILE - 1) / GS_TILE, TY = (height + GS_TILE - 1) / GS_TILE;
    const uint64_t total = 3ull * (uint64_t)width * (uint64_t)height;
    float* partial = static_cast<float*>(ws);
    if (TX * TY > 0)
        hipLaunchKernelGGL((k_raster_fwd<false, true>), dim3(TX * TY), dim3(GS_BLOCK), 0, st, tile_order, ranges, vals,
                           reinterpret_cast<const float2*>(proj.mean2d),
                           reinterpret_cast<const float4*>(proj.conic_opacity), proj.rgb, width, height, TX, bg[0],
                           bg[1], bg[2], img, final_T, n_contrib, active, nullptr, target,
                           (float)(1.0 / (double)(total ? total : 1)), dL, partial);
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(GS_BLOCK), 0, st, partial, (uint32_t)(TX * TY),
                       total ? 1.0 / (double)total : 0.0, loss);
    return hipGetLastError();
}

size_t loss_ws_bytes(int32_t width, int32_t height) {
    return align256(sizeof(float) * (div_up(3ull * (uint64_t)width * (uint64_t)height, GS_TILE_ITEMS) + 1));
}

hipError_t launch_loss_l1(const float* img, const float* target, int32_t width, int32_t height, float* loss,
                          float* dL, void* ws, hipStream_t st) {
    const uint64_t total = 3ull * (uint64_t)width * (uint64_t)height;
    const uint32_t nb = div_up(total, GS_TILE_ITEMS);
    float* partial = static_cast<float*>(ws);
    const float inv = (float)(1.0 / (double)total);
    if (nb > 0)
    {
        const bool vec = ((reinterpret_cast<uintptr_t>(img) | reinterpret_cast<uintptr_t>(target) |
                           reinterpret_cast<uintptr_t>(dL)) & 15u) == 0;
        if (vec)
            hipLaunchKernelGGL(k_loss_l1<true>, dim3(nb), dim3(GS_BLOCK), 0, st, img, target, (uint32_t)total, inv,
                               dL, partial);
        else
            hipLaunchKernelGGL(k_loss_l1<false>, dim3(nb), dim3(GS_BLOCK), 0, st, img, target, (uint32_t)total, inv,
                               dL, partial);
    }
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(GS_BLOCK), 0, st, partial, nb,
                       total ? 1.0 / (double)total : 0.0, loss);
    return hipGetLastError();
}

// Workspace: the pair slots (capacity x kSlot floats), then the slot sums of
// the visible rows (n x kSlot floats; the pixel half alone needs only the
// slots, n = 0).
size_t raster_bwd_ws_bytes(int32_t n, uint32_t capacity) {
    return align256(sizeof(float) * kSlot * (size_t)(capacity > 0 ? capacity : 1)) +
           (n > 0 ? align256(sizeof(float) * kSlot * (size_t)n) : 0);
}

hipError_t launch_raster_bwd(const gs_scene& scene, const CamArgs& cam, const gs_proj& proj, const uint32_t* vals,
                             const uint32_t* ranges, const uint32_t* tile_order, const uint32_t* pair_offset,
                             const uint32_t* pair_emit, const uint32_t* vis_idx, const uint32_t* vis_count,
                             uint32_t capacity, const float* final_T, const uint32_t* n_contrib, const float* dL_dimg,
                             const float bg[3], float* grad_rows, int32_t grad_ld, float* grad2d, float* grad_norm,
                             void* ws, int stages, hipStream_t st, const uint32_t* union_idx, const uint32_t* union_count, int first) {
    float* slots = static_cast<float*>(ws);
    const int32_t T = cam.tiles_x * cam.tiles_y;
    if ((stages & 1) && T > 0)
        hipLaunchKernelGGL(k_raster_bwd, dim3(T), dim3(GS_BLOCK), 0, st, tile_order, ranges, vals,
                           reinterpret_cast<const float2*>(proj.mean2d),
                           reinterpret_cast<const float4*>(proj.conic_opacity), proj.rgb, cam.width, cam.height,
                           cam.tiles_x, bg[0], bg[1], bg[2], final_T, n_contrib, dL_dimg, pair_emit, slots);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || scene.n == 0 || !(stages & 2)) return e;
    const dim3 grid(div_up(scene.n, GS_BLOCK));
    float* sums = slots + align256(sizeof(float) * kSlot * (size_t)(capacity > 0 ? capacity : 1)) / sizeof(float);
    // the kernel decides on the visible rows, known on the device only: workgroups for either split
    const dim3 sum_grid(std::max(grid.x, div_up(std::min((uint32_t)scene.n, kFewRows), GS_BLOCK / 2)));
    hipLaunchKernelGGL(k_slot_sum, sum_grid, dim3(GS_BLOCK), 0, st, vis_idx, vis_count, proj.tiles, pair_offset, slots,
                       capacity, sums);
    if (union_idx) {
        if (first) {
            uint32_t cb = div_up((uint64_t)scene.n * (uint64_t)(grad_ld / 4), GS_BLOCK);
            if (cb > 8192) cb = 8192;
            hipLaunchKernelGGL(k_clear_union_rows, dim3(cb), dim3(GS_BLOCK), 0, st, union_idx, union_count, grad_rows,
                               grad_ld, grad_norm);
        }
    }
#define GS_LAUNCH_PBWD(D, A)                                                                                     \
    hipLaunchKernelGGL((k_project_bwd<D, A>), grid, dim3(GS_BLOCK), 0, st, vis_idx, vis_count, sums,             \
                       reinterpret_cast<const float4*>(proj.conic_opacity),                                       \
                       proj.clamp, scene.mean, scene.log_scale, scene.quat, scene.opacity, scene.sh,              \
                       scene_ld(scene), cam,                                                                      \
                       grad_rows, grad_ld, grad2d, grad_norm, union_idx, union_count)
    if (union_idx) {
        switch (scene.sh_degree) {
            case 0: GS_LAUNCH_PBWD(0, true); break;
            case 1: GS_LAUNCH_PBWD(1, true); break;
            case 2: GS_LAUNCH_PBWD(2, true); break;
            default: GS_LAUNCH_PBWD(3, true); break;
        }
    } else {
        switch (scene.sh_degree) {
            case 0: GS_LAUNCH_PBWD(0, false); break;
            case 1: GS_LAUNCH_PBWD(1, false); break;
            case 2: GS_LAUNCH_PBWD(2, false); break;
            default: GS_LAUNCH_PBWD(3, false); break;
        }
    }
#undef GS_LAUNCH_PBWD
    return hipGetLastError();
}

}  // namespace gsmi
