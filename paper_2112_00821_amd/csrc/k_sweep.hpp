// Fused plane-sweep matching on gfx950 (Alg. 1 of the paper): for a tile of
// reference pixels and each plane label, every matching view is warped onto
// the tile (plus the window halo) into LDS; the matching cost of each pixel
// is taken in LDS -- the census of the warped view and its Hamming distance
// to the reference census (v_bcnt), or the negated, truncated and scaled
// NCC against the reference window -- the per-side sums combined by the
// occlusion-robust minimum, and the cost written to the label-innermost
// uint8 volume S[y][x][label].
//
// Tile 64 x 4*NW pixels, NW wavefronts (4 or 8, the caller's choice per
// level); a wavefront owns four rows, a lane one column of them, so an LDS row
// read serves up to four census windows.  The label range of a block is the
// union of its pixels' windows (dynamic cost volume); pixels whose window
// misses a label skip the store.
//
// What bounds it: VALU issue at the clock the chip holds under it (about 2.1
// GHz).  A census unit -- one pixel, label and view -- is 62 subtractions and
// 62 v_alignbit; the subtraction issues beside another wavefront's v_alignbit
// (two VALU instructions a quad-cycle, where one is a plain add, subtract,
// multiply, xor or move), so about 62 + 45 (1.5 samples of about 30
// instructions) issue slots are needed and the chip spends about 165.  Hence:
//  - a (label, view) pair's texel loads are requested before the previous
//    pair's costs are computed and interpolated after them, so no load is
//    waited for: wavefronts stall for 28 % of their cycles with four a SIMD;
//  - a bilinear sample is one aligned 32-bit load (packed 2x2 texels,
//    launch_pack_quads) instead of four byte loads, the border baked in;
//  - homographies arrive by scalar loads one pair ahead, and the part of them
//    that a region row shares is computed once per row and pair;
//  - costs leave 16 labels of a pixel at a time.
// 1920x1080, 4 views, 128 labels, 9x7, level 0: 6.1 ms with byte loads, loads
// waited for in place and 4-byte stores, 4.9 ms so; 2704x1520, 384 labels:
// 33.5 and 27.8 ms; 1280x720, 64 labels, 5x5: 1.3 and 0.80 ms.
//
// Warped values are double-buffered so one barrier per (label, view) pair
// suffices.  Blocks are remapped so that neighbouring tiles share an XCD's L2.
#pragma once
#include "dev_common.hpp"
#include "kernels.hpp"

#include <climits>
#include <type_traits>

namespace fmvs {

// Where the samples come from: packed 2x2 texels, pre-warped views, or the
// views' own bytes, four loads a sample.  The bytes are for the stage calls'
// views that there is no room to pack, or whose packed texels lie beyond
// 32-bit byte offsets (2^30 texels).  A stage call packed, packing included,
// and in bytes: 160x120, 2 views, 32 labels, 5x5 51 and 47 us; 640x480, 2, 64,
// 9x7 238 and 251; 1920x1080, 4, 128, 9x7 4.09 and 4.74 ms.
enum SweepSource : int { kPacked, kWarped, kBytes };

namespace {
constexpr int TW = 64;       // tile width: a wavefront's row
constexpr int RPT = 4;       // rows per thread
constexpr int kSweepWaves = 4;   // wavefronts per SIMD the registers are held to
// Uniform data (kernel arguments, homographies) is read through the constant
// address space, so it arrives by scalar loads and stays in scalar registers
// although the kernel also stores to global memory.
#define FMVS_CONST_AS __attribute__((address_space(4)))
typedef const FMVS_CONST_AS SweepArgs ArgsC;

// Values computed by this point of the program: the compiler otherwise moves
// the arithmetic past the next block and keeps its many inputs in registers.
template <typename V>
__device__ __forceinline__ void pin(V &v) {
    asm volatile("" : "+v"(v));
}

__device__ __forceinline__ uint32_t insert_sign(uint32_t acc, float v, float c) {
    // (acc << 1) | [v < c]: the sign of v - c (exact for distinct floats,
    // +0 when equal) shifted in through alignbit
    return __builtin_amdgcn_alignbit(acc, __float_as_uint(v - c), 31);
}

// Combined cost of the left and right subset sums: min over non-empty X of
// floor(s^X m / |X|) (census; m = max subset size) or floor(s^X / |X|) (NCC,
// m = 1).  The quotient is (s c) >> 17 with c = m ceil(2^17 / |X|): with
// s <= 8 * 255 and |X| <= 8, s m (|X| - 1) < 2^17, so the floor is exact, and
// the product stays below 2^32.
struct Combine {
    uint32_t cL, cR, oL, oR;   // factors; all ones for an empty subset
    bool equal;
    __device__ __forceinline__ Combine(int nL, int nR, int m)
        : cL(nL > 0 ? (uint32_t)m * ((131071u + nL) / nL) : 0u), cR(nR > 0 ? (uint32_t)m * ((131071u + nR) / nR) : 0u),
          oL(nL > 0 ? 0u : ~0u), oR(nR > 0 ? 0u : ~0u), equal(nL == m && nR == m) {}
    __device__ __forceinline__ uint32_t operator()(uint32_t sLR) const {
        const uint32_t sL = sLR & 0xFFFFu, sR = sLR >> 16;
        if (equal) return min(sL, sR);
        return min((__umul24(sL, cL) >> 17) | oL, (__umul24(sR, cR) >> 17) | oR);
    }
};

// Shape of a workgroup's tile and of the region its windows read.  The
// region's samples are dealt to the wavefronts in steps of one sample a lane:
// step st < RH is the first 64 columns of region row st, the NH steps after
// them are HR rows each of the last E columns.  Wavefront w takes the steps
// w, w + NW, ...; NST bounds its share (the last steps are repeated where the
// count does not divide, so that no step is conditional).
template <int CW, int CH, int NW>
struct SweepTile {
    static constexpr int NT = 64 * NW, TH = RPT * NW;
    static constexpr int RX = CW / 2, RY = CH / 2;
    static constexpr int RW = TW + 2 * RX, RH = TH + 2 * RY, NS = RW * RH;
    static constexpr int E = 2 * RX, HR = 64 / E;
    static constexpr int NH = (RH + HR - 1) / HR;
    static constexpr int NST = (RH + NH + NW - 1) / NW;
    static constexpr int NFULL = RH / NW;   // steps that are a row's first 64 columns for every wavefront
};

// What a wavefront holds of the samples it has requested: the packed 2x2
// texels (four bytes each in a register of its own; the value itself, from
// pre-warped views) and the fractions.
template <int NST, int SRC>
struct Pending {
    uint32_t tex[NST][SRC == kBytes ? 4 : 1];
    float ax[NST], ay[NST];
};
}  // namespace

// NCC cost of one view at one pixel from its window sums (the oracle's
// definition, the same operations in the same order): sA and vA = n sAA -
// sA^2 are exact integers of the reference window.
__device__ __forceinline__ int ncc_cost_exact(double cov, double p) {
    double rho = cov / sqrt(p);
    rho = fmin(1.0, fmax(-1.0, rho));
    const double c = fmin(1.0, 1.0 - rho);
    return (int)floor(255.0 * c + 0.5);
}
// The correctly rounded square root and division (about 60 instructions, half
// of a 5x5 window's sums) decide the cost only where
// 255 (1 - rho) + 0.5 lies next to a whole number: rho in float is off by at
// most 4.5 x 2^-24 of it (the covariance's conversion 1, the product's under
// the root 1/2, the reciprocal square root within an ulp 2, the product 1),
// 6.9e-5 of 255, and that number's own rounding adds 0.8e-5, so 1e-4 further
// from a whole number its floor is the same, and only the remaining pixels take them.
// 1920x1080, 3 views, 128 labels, 5x5, three levels: 8.6 ms with them for
// every pixel and a rolled row loop, 5.1 ms so.
__device__ __forceinline__ int ncc_finish(int sA_i, int vA_i, double sB, double sBB, double sAB, double n) {
    const double sA = (double)sA_i;
    const double vA = (double)vA_i;
    const double vB = n * sBB - sB * sB;
    const double cov = n * sAB - sA * sB;
    const double p = vA * vB;
    const float t = __builtin_fmaf((float)cov * __builtin_amdgcn_rsqf((float)p), -255.0f, 255.5f);
    const float tc = fminf(255.5f, fmaxf(0.5f, t));
    int cost = (int)tc;
    const bool flat = !(vA > 0.0 && vB > 0.0);
    const float fr = __builtin_amdgcn_fractf(tc);
    if (!flat && !(fr > 1e-4f && fr < 1.0f - 1e-4f)) cost = ncc_cost_exact(cov, p);
    return flat ? 255 : cost;
}

// XCD-aware remap: hardware dispatches workgroup b to XCD b % 8; give each
// XCD a contiguous range of logical work items.
__device__ __forceinline__ int xcd_logical(int b, int nb) {
    const int q = nb >> 3, r8 = nb & 7, xcd = b & 7, slot = b >> 3;
    return xcd * q + min(xcd, r8) + slot;
}

// One workgroup's share of the sweep of one frame: logical = tile *
// n_chunks + chunk.
template <int CW, int CH, int NW, int SRC, int COST>
__device__ __forceinline__ void sweep_block(ArgsC &a, const int logical) {
    constexpr bool WARPED = SRC == kWarped;
    typedef SweepTile<CW, CH, NW> T;
    constexpr int NT = T::NT, RX = T::RX, RY = T::RY, RW = T::RW, RH = T::RH, NS = T::NS;
    constexpr int NST = T::NST, NFULL = T::NFULL, E = T::E, HR = T::HR;
    constexpr int NB = CW * CH - 1;
    constexpr int NHI = NB > 32 ? NB - 32 : 0;
    constexpr int FW = 64;   // planes whose flags are held at a time
    __shared__ float wbuf[2][NS];
    __shared__ float aref[COST == 1 ? NS : 1];   // reference intensities of the region (NCC)
    __shared__ double s_row[2][3][RH];            // homography row terms of the region's rows, per pair
    constexpr int RUN = 5;   // words per pixel of its run (an odd stride between pixels)
    __shared__ uint32_t s_run[T::NT * RPT * RUN];
    __shared__ int s_lo[kMaxFam], s_hi[kMaxFam];
    __shared__ int s_flag[FW];   // bit k: the region maps inside view k for this plane

    const int aw = a.w, ah = a.h, n_fam = a.n_fam, n_views = a.n_views;
    const int chunk = logical % a.n_chunks;
    const int tile = logical / a.n_chunks;
    const int x0 = (tile % a.tiles_x) * TW;
    const int y0 = (tile / a.tiles_x) * T::TH;

    const int tid = threadIdx.x;
    const int tx = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int x = x0 + tx;
    const size_t N = (size_t)aw * ah;

    if (tid < kMaxFam) {
        s_lo[tid] = INT_MAX;
        s_hi[tid] = INT_MIN;
    }
    if (COST == 1) {
        for (int s2 = tid; s2 < NS; s2 += NT) {
            const int rx = s2 % RW, ry = s2 / RW;
            const int qx = min(max(x0 - RX + rx, 0), aw - 1), qy = min(max(y0 - RY + ry, 0), ah - 1);
            aref[s2] = (float)a.ref[(size_t)qy * aw + qx];
        }
    }
    __syncthreads();

    uint32_t ref_hi[RPT], ref_lo[RPT];   // census cost: the reference census words
    int refA[RPT], refV[RPT];            // NCC cost: sum and n * sum of squares - sum^2 of the window
    const int yt = y0 + wv * RPT;
    const uint32_t pix0 = (uint32_t)(yt * aw + x);   // pixel of the thread's first row
    const int rows = x < aw ? min(max(ah - yt, 0), RPT) : 0;   // rows of this thread inside the image
    const int32_t *__restrict__ offs = a.offs;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        if (COST == 0) {
            const uint64_t ct = j < rows ? a.ct_ref[pix0 + (uint32_t)(j * aw)] : 0;
            ref_hi[j] = (uint32_t)(ct >> 32);
            ref_lo[j] = (uint32_t)ct;
        } else {
            int sA = 0, sAA = 0;
#pragma unroll 1
            for (int dy = 0; dy < CH; ++dy)
                for (int dx = 0; dx < CW; ++dx) {
                    const int v = (int)aref[(wv * RPT + j + dy) * RW + tx + dx];
                    sA += v;
                    sAA += v * v;
                }
            refA[j] = sA;
            refV[j] = CW * CH * sAA - sA * sA;
        }
    }
    // union of the pixels' label windows per family
    for (int f = 0; f < n_fam; ++f) {
        int lo = INT_MAX, hi = INT_MIN;
        if (offs) {
#pragma unroll
            for (int j = 0; j < RPT; ++j)
                if (j < rows) {
                    const int o = offs[(size_t)f * N + pix0 + (uint32_t)(j * aw)];
                    lo = min(lo, o);
                    hi = max(hi, o);
                }
            lo = wave_min_i32(lo);
            hi = ~wave_min_i32(~hi);
        } else {
            lo = hi = 0;
        }
        if (tx == 0 && hi != INT_MIN) {
            atomicMin(&s_lo[f], lo);
            atomicMax(&s_hi[f], hi + a.W[f]);
        }
    }
    __syncthreads();

    // this block's share of the concatenated union of label ranges
    int total = 0;
    for (int f = 0; f < n_fam; ++f) total += s_hi[f] > s_lo[f] ? s_hi[f] - s_lo[f] : 0;
    total = __builtin_amdgcn_readfirstlane(total);
    // (in whole words of four labels, as even as these allow)
    const int words = (total + 3) >> 2;
    const int pos0 = 4 * (chunk * words / a.n_chunks);
    const int pos1 = min(total, 4 * ((chunk + 1) * words / a.n_chunks));
    if (pos0 >= pos1) return;
    if (a.work && tid == 0) {
        int nv = min(TW, aw - x0) * min(T::TH, ah - y0);
        atomicAdd(a.work, (unsigned long long)(pos1 - pos0) * (unsigned long long)nv);
    }
    auto flo = [&](int f_) { return __builtin_amdgcn_readfirstlane(s_lo[f_]); };
    auto fhi = [&](int f_) { return __builtin_amdgcn_readfirstlane(s_hi[f_]); };

    int f = 0, fbase = 0;
    while (f < n_fam && pos0 >= fbase + (fhi(f) - flo(f))) {
        fbase += fhi(f) - flo(f);
        ++f;
    }
    int g = flo(f) + (pos0 - fbase);
    int g_end = fhi(f);   // end of the family's range in this tile
    int g_last = flo(f) + min(pos1 - fbase, g_end - flo(f)) - 1;
    int off[RPT];   // window offsets of the current family (out of reach for rows outside the image)
    auto load_off = [&](int f_) {
#pragma unroll
        for (int j = 0; j < RPT; ++j)
            off[j] = j < rows ? (offs ? offs[(size_t)f_ * N + pix0 + (uint32_t)(j * aw)] : 0) : 0x40000000;
    };
    load_off(f);
    // Costs are written 16 labels at a time: acc holds the last four of a
    // pixel, the newest in the top byte; full words wait in LDS (each thread
    // reads back its own only).  All pixels write at the same labels (a
    // pixel's window may start anywhere, so the runs are not aligned); where
    // the labels do not all lie in the pixel's window the ones that do are
    // written in words and singly.
    const int D = a.D;
    uint32_t acc[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) acc[j] = 0;
    uint32_t *const run = s_run + tid * RUN;   // pixel j at j * NT * RUN
    // this wavefront's first row of the tile in S
    uint8_t *__restrict__ S_rows = a.S + ((size_t)(y0 + wv * RPT) * aw + x0) * D;

    const Combine combine(a.nL, a.nR, COST == 0 ? a.m : 1);
    const FMVS_CONST_AS double *H0 = (const FMVS_CONST_AS double *)a.H;

    // Which views the region maps inside of, for the FW planes from position
    // p on: thread t tests view t / FW's corners for plane t % FW.  The flag
    // only selects between two forms of the same values.
    auto mark_inside = [&](int p) __attribute__((always_inline)) {
        if (WARPED) return;
        for (int i = tid; i < FW; i += NT) s_flag[i] = 0;
        __syncthreads();
        // (opaque: nothing of this is worth registers across the plane loop)
        int xl = max(x0 - RX, 0), xh = min(x0 - RX + RW - 1, aw - 1);
        int yl = max(y0 - RY, 0), yh = min(y0 - RY + RH - 1, ah - 1);
        pin(xl);
        pin(xh);
        pin(yl);
        pin(yh);
        const double qx_lo = (double)xl + 0.5, qx_hi = (double)xh + 0.5;
        const double qy_lo = (double)yl + 0.5, qy_hi = (double)yh + 0.5;
        for (int i = tid; i < FW * n_views; i += NT) {
            int q = p + (i & (FW - 1));
            const int k = i / FW;
            if (q >= pos1) continue;
            int f_ = 0, len = s_hi[0] > s_lo[0] ? s_hi[0] - s_lo[0] : 0;
            while (q >= len) {
                q -= len;
                ++f_;
                len = s_hi[f_] > s_lo[f_] ? s_hi[f_] - s_lo[f_] : 0;
            }
            const double *Hm = a.H + ((size_t)k * a.sumG + a.goff[f_] + s_lo[f_] + q) * 9;
            double hm[9];
            for (int e = 0; e < 9; ++e) hm[e] = Hm[e];
            if (warp_region_inside(hm, qx_lo, qx_hi, qy_lo, qy_hi, aw, ah)) atomicOr(&s_flag[i & (FW - 1)], 1 << k);
        }
        __syncthreads();
    };

    // Lane constants of the sample steps.  Steps from NFULL on differ between
    // wavefronts: their column coordinate, region row, and word in the
    // region's buffer (-1: not written).
    constexpr int NMIX = NST - NFULL;
    const double qxm = (double)min(max(x0 - RX + tx, 0), aw - 1) + 0.5;
    double qx_mix[NMIX];
    int row_mix[NMIX], word_mix[NMIX];
#pragma unroll
    for (int i = 0; i < NMIX; ++i) {
        const int st = min((NFULL + i) * NW + wv, RH + T::NH - 1);
        const bool halo = st >= RH;
        const int col = halo ? TW + tx % E : tx, row = halo ? (st - RH) * HR + tx / E : st;
        qx_mix[i] = (double)min(max(x0 - RX + col, 0), aw - 1) + 0.5;
        row_mix[i] = min(row, RH - 1);
        word_mix[i] = (NFULL + i) * NW + wv < RH + T::NH && row < RH && (!halo || tx < HR * E) ? row * RW + col : -1;
    }

    // The next (plane, view) pair to request: its homography and packed view
    // are fetched by scalar loads one pair ahead of the request that uses
    // them, the row terms h1 qy + h2 (and likewise) are put into s_row by the
    // last wavefront in between.
    struct Pair {
        int pos, k, f, g, end;
    } nx;
    double h0 = 0.0, h3 = 0.0, h6 = 0.0;
    const uint32_t *quads = nullptr;
    const uint8_t *bytes = nullptr;
    const float *warped = nullptr;
    bool inside = false;
    int vflag = 0;   // lane i: the views' flags of the i-th plane of this window
    int pb = pos0;
    auto fetch = [&](int slot) __attribute__((always_inline)) {
        const int lab = nx.k * a.sumG + a.goff[nx.f] + nx.g;
        if (WARPED) {
            warped = a.warped + (size_t)lab * N;
        } else {
            const FMVS_CONST_AS double *Hm = H0 + (uint32_t)__builtin_amdgcn_readfirstlane(lab * 9);
            if (SRC == kBytes)
                bytes = a.views[nx.k];
            else
                quads = a.quads[nx.k];
            inside = ((__builtin_amdgcn_readlane(vflag, nx.pos - pb) >> nx.k) & 1) != 0;
            h0 = Hm[0];
            h3 = Hm[3];
            h6 = Hm[6];
            if (wv == NW - 1 && tx < RH) {
                const double qy = (double)min(max(y0 - RY + tx, 0), ah - 1) + 0.5;
                s_row[slot][0][tx] = __builtin_fma(Hm[1], qy, Hm[2]);
                s_row[slot][1][tx] = __builtin_fma(Hm[4], qy, Hm[5]);
                s_row[slot][2][tx] = __builtin_fma(Hm[7], qy, Hm[8]);
            }
        }
        // the pair after it, in this block's order
        if (++nx.k == n_views) {
            nx.k = 0;
            ++nx.pos;
            if (++nx.g >= nx.end && nx.pos < pos1) {
                do ++nx.f;
                while (fhi(nx.f) <= flo(nx.f));
                nx.g = flo(nx.f);
                nx.end = fhi(nx.f);
            }
        }
    };

    Pending<NST, SRC> pend;
    // Request the fetched pair's samples: coordinates, fractions and one
    // packed-texel load each.
    auto request = [&](int slot) __attribute__((always_inline)) {
        if (WARPED) {
#pragma unroll
            for (int i = 0; i < NST; ++i) {
                const int r = i < NFULL ? wv + i * NW : row_mix[i < NFULL ? 0 : i - NFULL];
                const double qx = i < NFULL ? qxm : qx_mix[i < NFULL ? 0 : i - NFULL];
                pend.tex[i][0] = __float_as_uint(warped[(size_t)min(max(y0 - RY + r, 0), ah - 1) * aw + (int)qx]);
            }
            return;
        }
        const __amdgpu_buffer_rsrc_t rs =
            SRC == kBytes
                ? __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(bytes), 0, (int)(uint32_t)N, 0x00020000)
                : __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(quads), 0, (int)(uint32_t)(N * 4), 0x00020000);
        auto steps = [&](auto in) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < NST; ++i) {
                const int r = i < NFULL ? wv + i * NW : row_mix[i < NFULL ? 0 : i - NFULL];
                const double qx = i < NFULL ? qxm : qx_mix[i < NFULL ? 0 : i - NFULL];
                const Sample q = warp_point<decltype(in)::value>(
                    aw, ah, __builtin_fma(h0, qx, s_row[slot][0][r]), __builtin_fma(h3, qx, s_row[slot][1][r]),
                    __builtin_fma(h6, qx, s_row[slot][2][r]));
                pend.ax[i] = q.ax;
                pend.ay[i] = q.ay;
                pin(pend.ax[i]);
                pin(pend.ay[i]);
                if (SRC == kBytes) {
                    const uint32_t xb = min(q.x + 1u, (uint32_t)(aw - 1)), yb = min(q.y + 1u, (uint32_t)(ah - 1));
                    const uint32_t ra = __umul24(q.y, (uint32_t)aw), rb = __umul24(yb, (uint32_t)aw);
                    const uint32_t at[4] = {ra + q.x, ra + xb, rb + q.x, rb + xb};
#pragma unroll
                    for (int e = 0; e < (SRC == kBytes ? 4 : 1); ++e)
                        pend.tex[i][e] = __builtin_amdgcn_raw_buffer_load_b8(rs, at[e], 0, 0);
                } else {
                    pend.tex[i][0] = __builtin_amdgcn_raw_buffer_load_b32(rs, quad_offset(q, aw), 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (inside) {
            steps(std::true_type());
        } else {
            steps(std::false_type());
        }
    };
    // Interpolate the requested samples into buf.
    auto deliver = [&](float *buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NST; ++i) {
            uint32_t t = pend.tex[i][0];
            if constexpr (SRC == kBytes) t |= pend.tex[i][1] << 8 | pend.tex[i][2] << 16 | pend.tex[i][3] << 24;
            const float v = WARPED ? __uint_as_float(t) : quad_value(t, pend.ax[i], pend.ay[i]);
            if (i < NFULL)
                buf[(wv + i * NW) * RW + tx] = v;
            else if (word_mix[i < NFULL ? 0 : i - NFULL] >= 0)
                buf[word_mix[i < NFULL ? 0 : i - NFULL]] = v;
        }
    };
    uint32_t right = 0;   // bit k: view k counts to the right subset
    for (int k = 0; k < n_views; ++k) right |= a.side[k] < 0 ? 0u : 1u << k;

    nx = {pos0, 0, f, g, g_end};
    int held = 0;   // costs in acc not yet written
    for (; pb < pos1; pb += FW) {
        const int pe = min(pb + FW, pos1);
        mark_inside(pb);
        if (!WARPED) vflag = s_flag[tx];
        fetch(0);
        __syncthreads();
        request(0);
        bool more = nx.pos < pe;
        if (more) fetch(1);
        deliver(wbuf[0]);
        __syncthreads();
        // left-view sums in the low 16 bits, right-view sums in the high 16
        // (at most 8 views of at most 255 each): one shift-add per view and
        // pixel, the subset decided by a uniform shift
        uint32_t sLR[RPT];
#pragma unroll
        for (int j = 0; j < RPT; ++j) sLR[j] = 0;
        int k = 0, it = 0;
        for (;;) {
            // the next pair's samples are requested before this pair's costs
            // and delivered after them, and the pair after it is fetched
            const bool now = more;
            if (now) {
                request((it + 1) & 1);
                more = nx.pos < pe;
                if (more) fetch(it & 1);
            }
            const float *buf = wbuf[it & 1];
            const uint32_t sh = ((right >> k) & 1u) << 4;
            const float *base = buf + (wv * RPT) * RW + tx;
            if (COST == 0) {
                // census of the warped view for this thread's pixels
                float c[RPT];
#pragma unroll
                for (int j = 0; j < RPT; ++j) c[j] = base[(j + RY) * RW + RX];
                uint32_t hi[RPT], lo[RPT];
#pragma unroll
                for (int j = 0; j < RPT; ++j) hi[j] = lo[j] = 0;
                // one window row is read ahead of the one being compared; the
                // barriers keep the compiler from reading them all first,
                // which costs the registers of two more waves a SIMD
                float v[CW], vn[CW];
#pragma unroll
                for (int cx = 0; cx < CW; ++cx) vn[cx] = base[cx];
#pragma unroll
                for (int rr = 0; rr < RPT + 2 * RY; ++rr) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int cx = 0; cx < CW; ++cx) {
                        v[cx] = vn[cx];
                        if (rr + 1 < RPT + 2 * RY) vn[cx] = base[(rr + 1) * RW + cx];
                    }
#pragma unroll
                    for (int j = 0; j < RPT; ++j) {
                        const int wy = rr - j;
                        if (wy < 0 || wy >= CH) continue;
#pragma unroll
                        for (int cx = 0; cx < CW; ++cx) {
                            if (wy == RY && cx == RX) continue;
                            const int bpos = wy * CW + cx - ((wy > RY || (wy == RY && cx > RX)) ? 1 : 0);
                            if (bpos < NHI)
                                hi[j] = insert_sign(hi[j], v[cx], c[j]);
                            else
                                lo[j] = insert_sign(lo[j], v[cx], c[j]);
                        }
                    }
                }
#pragma unroll
                for (int j = 0; j < RPT; ++j) {
                    const uint32_t cst = __popc(hi[j] ^ ref_hi[j]) + __popc(lo[j] ^ ref_lo[j]);
                    sLR[j] += cst << sh;
                    pin(sLR[j]);
                }
            } else {
                // NCC: row sums of the window rows, left to right, then the
                // window sums over the rows top to bottom, in double (a
                // window's sums start at its first row's).  One row at a
                // time, as above.
                const float *abase = aref + (wv * RPT) * RW + tx;
                double wB[RPT], wBB[RPT], wAB[RPT];
#pragma unroll
                for (int rr = 0; rr < RPT + 2 * RY; ++rr) {
                    __builtin_amdgcn_sched_barrier(0);
                    double rB = 0.0, rBB = 0.0, rAB = 0.0;
#pragma unroll
                    for (int cx = 0; cx < CW; ++cx) {
                        const double vb = (double)base[rr * RW + cx];
                        const double va = (double)abase[rr * RW + cx];
                        rB = cx ? rB + vb : vb;
                        rBB = cx ? __builtin_fma(vb, vb, rBB) : vb * vb;
                        rAB = cx ? __builtin_fma(va, vb, rAB) : va * vb;
                    }
#pragma unroll
                    for (int j = 0; j < RPT; ++j) {
                        if (rr < j || rr - j >= CH) continue;
                        wB[j] = rr > j ? wB[j] + rB : rB;
                        wBB[j] = rr > j ? wBB[j] + rBB : rBB;
                        wAB[j] = rr > j ? wAB[j] + rAB : rAB;
                        pin(wB[j]);
                        pin(wBB[j]);
                        pin(wAB[j]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < RPT; ++j) {
                    const uint32_t cst = (uint32_t)ncc_finish(refA[j], refV[j], wB[j], wBB[j], wAB[j], (double)(CW * CH));
                    sLR[j] += cst << sh;
                    pin(sLR[j]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (now) deliver(wbuf[(it + 1) & 1]);
            __syncthreads();
            ++it;
            if (++k < n_views) continue;
            k = 0;
#pragma unroll
            for (int j = 0; j < RPT; ++j) {
                acc[j] = __builtin_amdgcn_perm(combine(sLR[j]), acc[j], 0x04030201u);
                sLR[j] = 0;
            }
            ++held;
            if ((held & 3) == 0 || g == g_last) {
                if ((held & 3) != 0) {
#pragma unroll
                    for (int j = 0; j < RPT; ++j) acc[j] >>= 8 * (4 - (held & 3));
                }
#pragma unroll
                for (int j = 0; j < RPT; ++j) run[j * (NT * RUN) + ((held - 1) >> 2)] = acc[j];
            }
            if (held == 16 || g == g_last) {
                const int Wf = a.W[f], fo = a.foff[f];
                const int first = g - held + 1;   // the run's labels are first .. g
#pragma unroll
                for (int j = 0; j < RPT; ++j) {
                    const int rel = first - off[j];   // the first one in the pixel's window
                    // (row base 16 bytes back: a run may start before the window)
                    uint8_t *dst = (S_rows - 16 + (size_t)j * aw * D) + (uint32_t)(tx * D + fo + rel + 16);
                    const uint32_t *w = run + j * (NT * RUN);
                    if (held == 16 && rel >= 0 && rel + 16 <= Wf) {
                        const uint32_t v[4] = {w[0], w[1], w[2], w[3]};
                        __builtin_memcpy(dst, v, 16);
                    } else if (rel > -held && rel < Wf) {
#pragma unroll 1
                        for (int b = 0; b < held; b += 4) {
                            const uint32_t v = w[b >> 2];
                            const int n = min(held - b, 4);
                            if (n == 4 && rel + b >= 0 && rel + b + 4 <= Wf) {
                                __builtin_memcpy(dst + b, &v, 4);
                            } else {
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    if (e < n && rel + b + e >= 0 && rel + b + e < Wf)
                                        dst[b + e] = (uint8_t)(v >> (8 * e));
                            }
                        }
                    }
                }
                held = 0;
            }
            // the plane after it (none after the block's last)
            if (++g >= g_end && (now || pb + FW < pos1)) {
                do {
                    fbase += fhi(f) > flo(f) ? fhi(f) - flo(f) : 0;
                    ++f;
                } while (fhi(f) <= flo(f));
                g = flo(f);
                g_end = fhi(f);
                g_last = g + min(pos1 - fbase, g_end - g) - 1;
                load_off(f);
            }
            if (!now) break;
        }
    }
}

template <int CW, int CH, int NW, int SRC, int COST>
__global__ __launch_bounds__(64 * NW, SRC == kBytes ? 2 : kSweepWaves) void k_sweep(const SweepArgs) {
    // the arguments, in place
    ArgsC &a = *(ArgsC *)__builtin_amdgcn_kernarg_segment_ptr();
    sweep_block<CW, CH, NW, SRC, COST>(a, xcd_logical(blockIdx.x, gridDim.x));
}

// Several frames in one launch: the workgroups of frame f are the logical
// items prefix[f] .. prefix[f + 1] - 1 (each frame's tiles x chunks), the
// whole grid remapped to XCDs as one.
template <int CW, int CH, int NW, int COST>
__global__ __launch_bounds__(64 * NW, kSweepWaves) void k_sweep_batch(const SweepArgs *__restrict__ list,
                                                             const int *__restrict__ prefix, int n) {
    const int logical = xcd_logical(blockIdx.x, gridDim.x);
    int f = 0;
    while (f + 1 < n && logical >= prefix[f + 1]) ++f;
    f = __builtin_amdgcn_readfirstlane(f);
    sweep_block<CW, CH, NW, kPacked, COST>(*(ArgsC *)(list + f), logical - prefix[f]);
}

// Launch one window size and cost: tiles of 64 x 4*rpt pixels (rpt 4 or 8:
// 4 or 8 wavefronts), from packed view texels or from pre-warped views.  Each
// (window, cost) pair is instantiated in a translation unit of its own so the
// sweep variants compile in parallel.
template <int CW, int CH, int COST>
hipError_t sweep_launch_cfg(const SweepArgs &a, dim3 grid, int rpt, hipStream_t s) {
    if (rpt == 4) {
        if (a.warped)
            hipLaunchKernelGGL((k_sweep<CW, CH, 4, kWarped, COST>), grid, dim3(256), 0, s, a);
        else if (a.views[0])
            hipLaunchKernelGGL((k_sweep<CW, CH, 4, kBytes, COST>), grid, dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL((k_sweep<CW, CH, 4, kPacked, COST>), grid, dim3(256), 0, s, a);
    } else {
        if (a.warped)
            hipLaunchKernelGGL((k_sweep<CW, CH, 8, kWarped, COST>), grid, dim3(512), 0, s, a);
        else
            hipLaunchKernelGGL((k_sweep<CW, CH, 8, kPacked, COST>), grid, dim3(512), 0, s, a);
    }
    return hipGetLastError();
}

template <int CW, int CH, int COST>
hipError_t sweep_launch_batch_cfg(const SweepArgs *list, const int *prefix, int n, int blocks, int rpt,
                                  hipStream_t s) {
    if (rpt == 4)
        hipLaunchKernelGGL((k_sweep_batch<CW, CH, 4, COST>), dim3(blocks), dim3(256), 0, s, list, prefix, n);
    else
        hipLaunchKernelGGL((k_sweep_batch<CW, CH, 8, COST>), dim3(blocks), dim3(512), 0, s, list, prefix, n);
    return hipGetLastError();
}

}  // namespace fmvs
