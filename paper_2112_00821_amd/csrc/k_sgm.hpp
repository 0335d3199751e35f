// Semi-global aggregation on gfx950 (Eq. sgm-path / sgm-smooth-fp /
// sgm-smooth-sn / sgm-aggr / sgm-wta of the paper, adaptive P2 of
// Eq. p2-grad).
//
// One wavefront walks one path; label i of the pixel sits in lane i % 64 of
// register i / 64.  The predecessor's path costs live in a per-wave LDS
// buffer with three guard entries on each side of every family segment, so
// the zero-cost transition shifted by the window offsets and the
// surface-normal offset (a per-pixel, per-family shift) is a plain indexed
// LDS read.  The predecessor minimum comes from a DPP reduction.
//
// All directions run in one launch, each writing its own buffer of path costs,
// 16 bits each or (sgm_narrow) 9 (no read-modify-write of a shared aggregate,
// so every path of every direction proceeds concurrently); a streaming kernel
// then adds the buffers and takes the winner-takes-all argmin, so the aggregate
// volume is never written.
#pragma once
#include "dev_common.hpp"
#include "kernels.hpp"

#include <algorithm>
#include <cstdlib>

namespace fmvs {

namespace {
constexpr uint32_t INF = 0x3FFFFFFFu;
constexpr int WAVES = 4;
// cache-policy bit of the buffer intrinsics for non-temporal (streaming)
// accesses on gfx950
constexpr int kNonTemporal = 2;
constexpr int GUARD = 3;
constexpr int LBUF = kMaxLabels + 2 * GUARD * kMaxFam;

struct PathGeom {
    int sx, sy, dx, dy, len;
};

__device__ __forceinline__ PathGeom path_geom(int dir, int pi, int w, int h) {
    PathGeom g;
    g.dx = dir_dx(dir);
    g.dy = dir_dy(dir);
    if (g.dy == 0) {
        g.sx = g.dx > 0 ? 0 : w - 1;
        g.sy = pi;
        g.len = w;
    } else if (g.dx == 0) {
        g.sx = pi;
        g.sy = g.dy > 0 ? 0 : h - 1;
        g.len = h;
    } else {
        if (pi < w) {
            // longest paths first within each direction (the dispatcher
            // starts workgroups in index order, so short paths fill the tail)
            g.sx = g.dx > 0 ? pi : w - 1 - pi;
            g.sy = g.dy > 0 ? 0 : h - 1;
        } else {
            int j = pi - w;
            g.sx = g.dx > 0 ? 0 : w - 1;
            g.sy = g.dy > 0 ? j + 1 : h - 2 - j;
        }
        int lx = g.dx > 0 ? w - g.sx : g.sx + 1;
        int ly = g.dy > 0 ? h - g.sy : g.sy + 1;
        g.len = lx < ly ? lx : ly;
    }
    return g;
}
}  // namespace


// Path costs of one direction, written to that direction's buffer.  Loads
// run ahead of the recursion: a ring of PF steps holds each lane's cost
// bytes, and the per-step uniform values (the P2 penalty of the step's
// intensity change, window offsets, surface-normal offsets) of 64 steps are
// fetched by one vector load per quantity (lane j holds step t0 + j) and
// read back with readlane.
// NF bounds the plane families (1, or up to the maximum), which sizes the
// per-family registers.
template <int K, int NF, bool WIN, bool SN, bool PG>
__global__ __launch_bounds__(64 * WAVES) void k_sgm(const SgmArgs a) {
    constexpr int PF = 8;
    __shared__ uint32_t lbuf[WAVES][2][LBUF];
    __shared__ double pdelta[PG ? kMaxPgPlanes : 1];
    if (PG) {
        for (int i = threadIdx.x; i < a.sumG; i += 64 * WAVES) pdelta[i] = a.delta[i];
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int path = blockIdx.x * WAVES + wid;
    if (path >= a.path_begin[a.n_dirs]) return;
    int slot = 0;
    while (path >= a.path_begin[slot + 1]) ++slot;
    const int dir = a.dirs[slot];
    const PathGeom pg = path_geom(dir, path - a.path_begin[slot], a.w, a.h);
    const size_t N = (size_t)a.w * a.h;
    const int D = a.D;
    const int F = NF == 1 ? 1 : a.n_fam;
    const long pstride = (long)pg.dy * a.w + pg.dx;
    const long p0 = (long)pg.sy * a.w + pg.sx;
    const int len = pg.len;

    int fam[K], li[K], wf[K], seg[K];
    bool lv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int i = k * 64 + lane;
        lv[k] = i < D;
        int f = 0;
        while (f + 1 < F && i >= a.foff[f + 1]) ++f;
        fam[k] = f;
        li[k] = i - a.foff[f];
        wf[k] = a.W[f];
        int sb = GUARD;
        for (int ff = 0; ff < f; ++ff) sb += a.W[ff] + 2 * GUARD;
        seg[k] = sb;
    }
    uint32_t *buf0 = lbuf[wid][0];
    uint32_t *buf1 = lbuf[wid][1];
    for (int i = lane; i < LBUF; i += 64) {
        buf0[i] = INF;
        buf1[i] = INF;
    }
    __builtin_amdgcn_wave_barrier();

    const uint8_t *__restrict__ S = a.S;
    uint16_t *__restrict__ out = a.out[slot];

    // per-step uniform values, 64 steps per chunk
    auto load_chunk = [&](int t0, int &ref_v, int (&off_v)[NF], int (&di_v)[NF]) {
        // ref_v: the penalty P2 of step t = t0 + lane, from the intensity
        // step between its pixel and the previous one on the path
        const int t = t0 + lane < len ? t0 + lane : len - 1;
        const long p = p0 + (long)t * pstride;
        const long pp = p0 + (long)(t > 0 ? t - 1 : 0) * pstride;
        const int di = (int)a.ref[p] - (int)a.ref[pp];
        ref_v = a.lut[di < 0 ? -di : di];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            off_v[f] = (WIN && f < F) ? a.offs[(size_t)f * N + p] : 0;
            di_v[f] = (SN && f < F) ? (int)a.dI[((size_t)dir * N + p) * F + f] : 0;
        }
    };
    int c_ref, n_ref;
    int c_off[NF], n_off[NF], c_di[NF], n_di[NF];
    load_chunk(0, c_ref, c_off, c_di);
    if (len > 64) load_chunk(64, n_ref, n_off, n_di);

    // ring of cost bytes, PF steps ahead
    uint32_t ring[PF][K];
#pragma unroll
    for (int u = 0; u < PF; ++u) {
        long p = p0 + (long)(u < len ? u : len - 1) * pstride;
#pragma unroll
        for (int k = 0; k < K; ++k) ring[u][k] = lv[k] ? S[(size_t)p * D + k * 64 + lane] : 0u;
    }

    uint32_t L[K];
    uint32_t Mq = 0;
    int oq[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) oq[f] = 0;
    // path-gradient state: depths of the last two minimum-cost points
    double dq1 = 0.0, dq2 = 0.0;

    for (int t0 = 0; t0 < len; t0 += PF) {
        if (t0 > 0 && (t0 & 63) == 0) {
            c_ref = n_ref;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                c_off[f] = n_off[f];
                c_di[f] = n_di[f];
            }
            if (t0 + 64 < len) load_chunk(t0 + 64, n_ref, n_off, n_di);
        }
        const int lb = t0 & 63;   // PF divides 64
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int t = t0 + u;
            if (t >= len) break;
            const long p = p0 + (long)t * pstride;
            uint32_t sv[K];
#pragma unroll
            for (int k = 0; k < K; ++k) sv[k] = ring[u][k];
            if (t + PF < len) {
                const long pn = p + (long)PF * pstride;
#pragma unroll
                for (int k = 0; k < K; ++k) ring[u][k] = lv[k] ? S[(size_t)pn * D + k * 64 + lane] : 0u;
            }
            const uint32_t P2 = (uint32_t)__builtin_amdgcn_readlane(c_ref, lb + u);
            int op[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) op[f] = WIN ? __builtin_amdgcn_readlane(c_off[f], lb + u) : 0;
            uint32_t *cur = (t & 1) ? buf1 : buf0;
            const uint32_t *prev = (t & 1) ? buf0 : buf1;
            if (t == 0) {
#pragma unroll
                for (int k = 0; k < K; ++k) L[k] = sv[k];
            } else {
                const uint32_t P1 = (uint32_t)a.p1;
                int sh[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    int v = WIN ? op[f] - oq[f] : 0;
                    if (SN) v += __builtin_amdgcn_readlane(c_di[f], lb + u);
                    sh[f] = v;
                }
                if (PG && t >= 2 && dq1 > 0.0 && dq2 > 0.0) {
                    // extrapolated inverse depth of the path's minimum-cost
                    // points, as a plane-index jump per family
                    const int px = pg.sx + t * pg.dx, py = pg.sy + t * pg.dy;
                    double rp[3], rq[3];
                    ray_of(a.Kinv, px + 0.5, py + 0.5, rp);
                    ray_of(a.Kinv, (px - pg.dx) + 0.5, (py - pg.dy) + 0.5, rq);
                    const double inv = 2.0 / dq1 - 1.0 / dq2;
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        if (f >= F) break;
                        const double *n = a.fam_n[f];
                        const double cp = -(n[0] * rp[0] + n[1] * rp[1] + n[2] * rp[2]);
                        const double cq = -(n[0] * rq[0] + n[1] * rq[1] + n[2] * rq[2]);
                        if (!(cp > 0.0) || !(cq > 0.0)) continue;
                        const double ip = inv / cp;
                        const double iq = 1.0 / (dq1 * cq);
                        double v = (ip - iq) / a.step[f];
                        v = fmin(fmax(v, -7.0), 7.0);
                        sh[f] += (int)round(v);
                    }
                }
                const uint32_t floor2 = Mq + P2;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    int sft = sh[0];
#pragma unroll
                    for (int f = 1; f < NF; ++f)
                        if (fam[k] == f) sft = sh[f];
                    int j = li[k] + sft;
                    j = j < -2 ? -2 : (j > wf[k] + 1 ? wf[k] + 1 : j);
                    const uint32_t *q = prev + seg[k] + j;
                    uint32_t c0 = q[0];
                    uint32_t cm = q[-1];
                    uint32_t cp = q[1];
                    uint32_t c1 = (cm < cp ? cm : cp) + P1;
                    uint32_t best = c0 < c1 ? c0 : c1;
                    best = best < floor2 ? best : floor2;
                    L[k] = sv[k] + best - Mq;
                }
            }
            uint32_t m = INF;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (lv[k]) {
                    cur[seg[k] + li[k]] = L[k];
                    out[(size_t)p * D + k * 64 + lane] = (uint16_t)L[k];
                }
                uint32_t v = lv[k] ? L[k] : INF;
                m = v < m ? v : m;
            }
            __builtin_amdgcn_wave_barrier();
            if (PG) {
                // minimum and its label in one reduction (smallest label on ties)
                uint32_t key = 0xFFFFFFFFu;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const uint32_t kk = lv[k] ? ((L[k] << 16) | (uint32_t)(k * 64 + lane)) : 0xFFFFFFFFu;
                    key = kk < key ? kk : key;
                }
                key = wave_min_u32(key);
                Mq = key >> 16;
                const int bi = (int)(key & 0xFFFFu);
                int f = 0;
                while (f + 1 < F && bi >= a.foff[f + 1]) ++f;
                const int g = (WIN ? op[f] : 0) + (bi - a.foff[f]);
                const int px = pg.sx + t * pg.dx, py = pg.sy + t * pg.dy;
                double rr[3];
                ray_of(a.Kinv, px + 0.5, py + 0.5, rr);
                const double den = a.fam_n[f][0] * rr[0] + a.fam_n[f][1] * rr[1] + a.fam_n[f][2] * rr[2];
                dq2 = dq1;
                dq1 = den < 0.0 ? -pdelta[a.goff[f] + g] / den : 0.0;
            } else {
                Mq = wave_min_u32(m);
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) oq[f] = op[f];
        }
    }
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u16x2 as_u16x2(uint32_t v) { return __builtin_bit_cast(u16x2, v); }
__device__ __forceinline__ uint32_t as_u32(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }

// Path costs of one direction with two labels per lane as packed 16-bit
// values (labels 2i, 2i+1 of pair i = 64k + lane in register k).  Same
// recursion and results as k_sgm; every family window must hold an even
// number of labels so no pair straddles two families.  The predecessor
// buffer holds 16-bit costs with six +inf guards around each family
// segment; a pair's three taps (j-1, j), (j, j+1), (j+1, j+2) come from
// three aligned 32-bit LDS reads and byte permutes whose selectors follow
// the parity of the shifted index j.  P1 is added with unsigned saturation
// so the guards stay +inf; every finite sum stays below 2^16 by the
// configuration bound.  Global traffic goes through buffer resources built
// per step on the scalar unit from row pointers that advance by one add
// (row base = pixel of the step): the lane offset is the only vector
// operand, and lanes past the label count read 0 and drop their stores by
// the resource's range check.  With PG the same kernel runs the
// path-gradient variant (Eq. sgm-smooth-pg): its plane jump is five 64-bit
// quotients a step, the same in every lane, so a step was bound by their
// issue (960x540 x 128 labels, 3 levels: 1.83 ms against about 0.4 ms of the
// recursion alone).  The reciprocals of a pixel's divisors are taken once
// per block, a lane a step, those of the plane list once per workgroup, and
// the quotients follow in two fused multiply-adds, with the division's bits
// (recip_from has the one exception): 1.10 ms.
// With NARROW the path costs leave as 9-bit heights above S (sgm_narrow): a
// byte a label at once, the 9th bits gathered by two ballots a step in lane
// 4u .. 4u + 3 of step u of the block (even and odd labels of pairs 0-31, then
// of pairs 32-63) and stored once per block.  On large frames the 16-bit form
// is bound by its bytes (1920x1080 x 128 labels, level 0: 7.26 GB in 1.58 ms,
// 4.6 of the 4.9 TB/s a copy reaches); the narrow form moves 5.60 GB in 1.30 ms (4.3
// TB/s), the packing's instructions beside its bytes (VALU busy 0.75).
// Without windows and surface-normal shifts the taps are the same in every
// step and cost no address arithmetic (640x480 x 16 to 96 labels: reading a
// shift of 0 each step took the stage 1.09 times as long).

// Wave-uniform copies of values read from an argument block (its arrays
// indexed by a uniform index stay uniform, wherever the block lives).
__device__ __forceinline__ int rfl(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T>
__device__ __forceinline__ T *rflp(T *p) {
    const uint64_t u = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return (T *)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void *p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}

constexpr int PK_G2 = 6;
constexpr int PK_LW = (kMaxLabels + 2 * PK_G2 * kMaxFam) / 2 + 1;   // 32-bit words per buffer, last one a sink

// Path gradient: a plane's delta and its reciprocal.
struct PgPlane {
    double delta, recip;
};

__device__ __forceinline__ double lane_f64(double v, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// x / b, correctly rounded, from r = 1 / b correctly rounded: the remainder
// of the first quotient is exact in a fused multiply-add, and the corrected
// quotient rounds as the division does (P. Markstein, IBM J. Res. Dev. 34
// (1990); the product x r is up to 1.5 units in the last place off where the
// theorem asks for one: no operands are known where that shows, none of all
// with mantissas of 5 to 8 bits nor of 2 x 10^8 with 53).  Zeros, infinities
// and NaN as the division gives them; divisors and quotients are normal
// numbers.
__device__ __forceinline__ double div_by(double x, double b, double r) {
    const double q = x * r;
    return __builtin_amdgcn_div_fixup(__builtin_fma(__builtin_fma(-q, b, x), r, q), b, x);
}

// 1 / b from an estimate a few units in the last place off: two steps of
// Newton's iteration, the second on a faithful value.  Correctly rounded but
// for the divisors with every mantissa bit set, one in 2^52: their reciprocal
// may come out as the power of two one unit below it.  (Putting the unit back
// takes five instructions of the serial step, the 960x540 frame 3.82 -> 3.99
// ms; a label could only turn on it where a jump also lies within 10^-15 of
// half a plane.)
__device__ __forceinline__ double recip_from(double b, double r) {
    r = __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
    r = __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
    return __builtin_amdgcn_div_fixup(r, b, 1.0);
}

// A shift's three aligned words of taps: their byte step from the words of
// no shift, and the byte selector of the first tap pair (the others follow).
// The four 16-bit entries q .. q + 3 start at q = j - 1, j even for a shift
// of 0.
struct Taps {
    int step;
    uint32_t sel;
};
__device__ __forceinline__ Taps taps_of(int shift) {
    return Taps{4 * ((shift - 1) >> 1), 0x03020100u + (uint32_t)(~shift & 1) * 0x02020202u};
}
typedef __attribute__((address_space(3))) uint32_t LdsWord;

// (the compiler's own operation; it has no builtin)
__device__ uint32_t write_lane(uint32_t value, uint32_t lane, uint32_t old) __asm("llvm.amdgcn.writelane.i32");

// Where the 9th bits start in a direction's narrow path costs of N pixels.
__host__ __device__ inline size_t narrow_bits_at(size_t N, int D) { return (N * D + 15) & ~(size_t)15; }

// One wavefront's LDS: two predecessor buffers (the last step's path costs,
// this step's) and a block's shifts by family (path gradient: their plain
// values in .step).
struct PkLds {
    uint32_t cost[2][PK_LW];
    Taps shift[16][kMaxFam];
};

// Smaller 16-bit half of a word.  A lane-crossing read of the result needs
// two wait states; they are in the block unless another instruction comes
// first (OTHER).
template <bool OTHER>
__device__ __forceinline__ uint32_t min_of_halves(uint32_t v) {
    uint32_t r;
    if (OTHER)
        asm("v_min_u32_sdwa %0, %1, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1"
            : "=v"(r) : "v"(v));
    else
        asm("v_min_u32_sdwa %0, %1, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1\n\ts_nop 1"
            : "=v"(r) : "v"(v));
    return r;
}

__device__ __forceinline__ int med3_i32(int v, int lo, int hi) {
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "v"(lo), "v"(hi));
    return r;
}

// One path of the two-label kernel: path index `path` of the frame a (all
// its directions' paths numbered by a.path_begin), run by one wavefront with
// the P2 table s_lut and (path gradient) the plane lists in LDS, and its own
// LDS buffers.
template <int KP, int NF, bool WIN, bool SN, bool PG, bool NARROW>
__device__ __forceinline__ void sgm_pk_path(const SgmArgs a, const int path, const int *s_lut,
                                            const PgPlane *planes, PkLds &lds) {
    constexpr int PF = KP >= 2 ? 8 : 16;   // steps per block (ring depth): fewer registers for many labels
    constexpr int G2 = PK_G2;
    constexpr int LW = PK_LW;
    constexpr bool SHIFTS = WIN || SN;   // else every shift is 0 (the path gradient's jump aside)
    const int lane = threadIdx.x & 63;
    // the argument block's scalars as wave-uniform locals (the block may sit
    // in registers, private memory or global memory depending on the caller)
    const int aw = rfl(a.w), ah = rfl(a.h);
    const uint8_t *__restrict__ aref = rflp(a.ref);
    const int32_t *__restrict__ aoffs = rflp(a.offs);
    const int8_t *__restrict__ adI = rflp(a.dI);
    int slot = 0;
    while (path >= rfl(a.path_begin[slot + 1])) ++slot;
    const int dir = rfl(a.dirs[slot]);
    const PathGeom pg = path_geom(dir, path - rfl(a.path_begin[slot]), aw, ah);
    const size_t N = (size_t)aw * ah;
    const int D = rfl(a.D);
    const int F = NF == 1 ? 1 : rfl(a.n_fam);
    const long pstride = (long)pg.dy * aw + pg.dx;
    const long p0 = (long)pg.sy * aw + pg.sx;
    const int len = pg.len;

    int fam[KP], widx[KP];
    // LDS byte addresses in the first predecessor buffer: of the pair's own
    // word, and the range of its taps' first word (beyond it they are guards
    // only)
    const int cost0 = (int)(uint32_t)(uintptr_t)(LdsWord *)lds.cost[0];
    int at0[KP], at_lo[KP], at_hi[KP];
    uint32_t lo8[KP];   // byte offset of the pair inside a pixel's cost row
    bool lv[KP];
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        const int i = 2 * (k * 64 + lane);   // first label of the pair
        lo8[k] = (uint32_t)i;
        lv[k] = i < D;
        int f = 0;
        while (f + 1 < F && i >= a.foff[f + 1]) ++f;
        fam[k] = f;
        const int li = i - a.foff[f];
        int sb = G2;
        for (int ff = 0; ff < f; ++ff) sb += a.W[ff] + 2 * G2;
        at0[k] = cost0 + 2 * (sb + li);
        at_lo[k] = cost0 + 2 * (sb - G2);
        at_hi[k] = cost0 + 2 * (sb + a.W[f]);
        widx[k] = lv[k] ? (sb + li) >> 1 : LW - 1;
    }
    for (int i = lane; i < LW; i += 64) {
        lds.cost[0][i] = 0xFFFFFFFFu;
        lds.cost[1][i] = 0xFFFFFFFFu;
    }
    __builtin_amdgcn_wave_barrier();

    const uint8_t *__restrict__ S = rflp(a.S);
    // path costs: 2 bytes a label, or (NARROW) a byte each and the pairs' 9th
    // bits behind them
    constexpr int kOut = NARROW ? 1 : 2;
    uint8_t *__restrict__ out = (uint8_t *)rflp(a.out[slot]);
    uint32_t *__restrict__ bits = (uint32_t *)(out + narrow_bits_at(N, D));
    uint32_t high[KP];   // a block's 9th bits: four words a step, a word a lane
#pragma unroll
    for (int k = 0; k < KP; ++k) high[k] = 0;

    // Uniform per-step values of one block of PF steps, one vector load per
    // quantity (lane j holds step t0 + j, j < PF): the penalty P2 of the
    // intensity change from the previous pixel and the families' shifts (the
    // step of the window offset and the surface-normal offset).  The loads of
    // a block are issued one block ahead and finished (the P2 lookup in LDS)
    // when the block starts, so no load is waited for before its use.  One
    // family: P2 and the shift leave their lane in one word; several: each
    // lane reads its family's shift of the step from LDS.  The first step of
    // the path gets P2 = 0: with the predecessor minimum at 0 the recursion
    // then reduces to L = S there, so the first step needs no code of its
    // own.
    struct BlockRaw {
        int i0, i1;   // intensities at the step and at its predecessor
        bool first;
        int off[NF], offp[NF], di[NF];
    };
    auto issue_block = [&](int t0, BlockRaw &r) {
        const int tl = t0 + (lane & (PF - 1));
        const int t = tl < len ? tl : len - 1;
        const long p = p0 + (long)t * pstride;
        const long pp = p0 + (long)(t > 0 ? t - 1 : 0) * pstride;
        r.i0 = aref[p];
        r.i1 = aref[pp];
        r.first = t == 0;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            r.off[f] = (WIN && f < F) ? aoffs[(size_t)f * N + p] : 0;
            r.offp[f] = (WIN && f < F) ? aoffs[(size_t)f * N + pp] : 0;
            r.di[f] = (SN && f < F) ? (int)adI[((size_t)dir * N + p) * F + f] : 0;
        }
    };
    int c_ref;       // P2 in the low half, one family's shift in the high half
    int c_off[NF];   // path gradient: the window offsets
    // path gradient: -n^T K^-1 p of the block's pixels and its reciprocal
    double b_c[NF], b_r[NF];
    auto finish_block = [&](int t0, const BlockRaw &r) {
        const int d = r.i0 - r.i1;
        const int p2 = r.first ? 0 : s_lut[d < 0 ? -d : d];
        c_ref = p2;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            c_off[f] = r.off[f];
            if (!SHIFTS) continue;
            // (no window is as wide as the bound)
            const int sh = min(max(r.off[f] - r.offp[f] + r.di[f], -2 * kMaxLabels), 2 * kMaxLabels);
            if (NF == 1)
                c_ref = (int)__builtin_amdgcn_perm((uint32_t)sh, (uint32_t)p2, 0x05040100u);
            else
                lds.shift[lane & (PF - 1)][f] = PG ? Taps{sh, 0u} : taps_of(sh);
        }
        if (PG) {
            const int t = t0 + (lane & (PF - 1));
            double rp[3];
            ray_of(a.Kinv, (pg.sx + t * pg.dx) + 0.5, (pg.sy + t * pg.dy) + 0.5, rp);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const double *n = a.fam_n[f < F ? f : 0];
                b_c[f] = -(n[0] * rp[0] + n[1] * rp[1] + n[2] * rp[2]);
                b_r[f] = 1.0 / b_c[f];
            }
        }
    };
    BlockRaw raw;
    issue_block(0, raw);
    finish_block(0, raw);

    // ring of cost byte pairs, PF steps ahead (steps past the path's end
    // re-read its last pixel)
    uint16_t ring[PF][KP];
#pragma unroll
    for (int u = 0; u < PF; ++u) {
        const long p = p0 + (long)(u < len ? u : len - 1) * pstride;
        const __amdgpu_buffer_rsrc_t rs = row_rsrc(S + (size_t)p * D, D);
#pragma unroll
        for (int k = 0; k < KP; ++k) ring[u][k] = __builtin_amdgcn_raw_buffer_load_b16(rs, lo8[k], 0, 0);
    }

    u16x2 L[KP];
    uint32_t Mq = 0;
    // path-gradient state: depths of the last two minimum-cost points, 2/d
    // of each, and -n^T K^-1 p of the previous pixel per family with its
    // reciprocal.  Values carried from one step to the next are the same
    // doubles the formulas would recompute (the ray and its dot products of a
    // pixel, and 1/d = (2/d) / 2, exact in binary floating point).
    double dq1 = 0.0, dq2 = 0.0, a1 = 0.0, a2 = 0.0;
    double c_prev[NF], r_prev[NF], r_step[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        c_prev[f] = r_prev[f] = 0.0;
        r_step[f] = PG ? 1.0 / a.step[f < F ? f : 0] : 0.0;
    }

    // Row pointers advance by one path step at a time (two scalar adds)
    // instead of being recomputed from the step index: s_ahead is the cost
    // row the ring loads next (PF steps ahead, held at the path's last
    // pixel), o_cur the output row of the current step.
    const long sstride = pstride * D;
    const uint8_t *s_ahead = S + (size_t)(p0 + (long)(PF < len ? PF : len - 1) * pstride) * D;
    uint8_t *o_cur = out + (size_t)p0 * D * kOut;

    // one step of the recursion at path position t (ring slot and block
    // lane u); clamp: the ring row may reach the path's last pixel in this
    // step (else it advances unconditionally)
    auto step = [&](const int t, const int u, const bool clamp) __attribute__((always_inline)) {
        u16x2 sv[KP], dl[KP];   // costs, and the path costs above them (at most P2)
#pragma unroll
        for (int k = 0; k < KP; ++k) sv[k] = as_u16x2(__builtin_amdgcn_perm(0u, ring[u][k], 0x0c010c00u));
        {
            // the reload of ring[u] may not move above its use (an empty
            // asm that takes sv and yields the offset), so the slot keeps
            // one register across the loop
            uint32_t off[KP];
#pragma unroll
            for (int k = 0; k < KP; ++k) {
                off[k] = lo8[k];
                asm volatile("" : "+v"(off[k]) : "v"(sv[k]));
            }
            const __amdgpu_buffer_rsrc_t rs = row_rsrc(s_ahead, D);
#pragma unroll
            for (int k = 0; k < KP; ++k) ring[u][k] = __builtin_amdgcn_raw_buffer_load_b16(rs, off[k], 0, 0);
            if (!clamp || t + PF + 1 < len) s_ahead += sstride;
            // one live row pointer (the compiler would otherwise keep a
            // precomputed address per unrolled step in scalar registers)
            asm volatile("" : "+s"(s_ahead));
        }
        const int word = __builtin_amdgcn_readlane(c_ref, u);
        const uint32_t P2 = (uint32_t)word & 0xFFFFu;
        uint32_t *cur = lds.cost[u & 1];
        double c_cur[NF], r_cur[NF];   // path gradient: -n^T K^-1 p of this step's pixel and its reciprocal
        {
            // splats of uniform 16-bit values (the packed instructions take
            // them as one scalar operand)
            const uint32_t P1 = (uint32_t)rfl(a.p1);
            const u16x2 p1v = (u16x2)(uint16_t)P1;
            const u16x2 mqv = (u16x2)(uint16_t)Mq;
            const uint16_t fl = (uint16_t)(Mq + P2);
            const u16x2 flv = (u16x2)fl;
            int jump[NF];   // path gradient: the planes' jump
#pragma unroll
            for (int f = 0; f < NF; ++f) jump[f] = 0;
            if (PG) {
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    c_cur[f] = lane_f64(b_c[f], u);
                    r_cur[f] = lane_f64(b_r[f], u);
                }
            }
            if (PG && t >= 2 && dq1 > 0.0 && dq2 > 0.0) {
                // extrapolated inverse depth of the path's minimum-cost
                // points, as a plane-index jump per family:
                // 1/d* = 2/dq1 - 1/dq2
                const double inv = a1 - 0.5 * a2;
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    if (f >= F) break;
                    const double cp = c_cur[f], cq = c_prev[f];
                    if (!(cp > 0.0) || !(cq > 0.0)) continue;
                    const double ip = div_by(inv, cp, r_cur[f]);
                    const double iq = recip_from(dq1 * cq, 0.5 * a1 * r_prev[f]);
                    double v = div_by(ip - iq, a.step[f], r_step[f]);
                    v = fmin(fmax(v, -7.0), 7.0);
                    // round half away from zero
                    jump[f] = (int)(v + __builtin_copysign(0x1.fffffffffffffp-2, v));
                }
            }
#pragma unroll
            for (int k = 0; k < KP; ++k) {
                Taps tp{0, 0u};
                if (NF > 1 && SHIFTS) tp = lds.shift[u][fam[k]];
                if (NF == 1 || PG || !SHIFTS) {
                    int jf = PG ? jump[0] : 0;
#pragma unroll
                    for (int f = 1; f < NF; ++f)
                        if (PG && fam[k] == f) jf = jump[f];
                    tp = taps_of((!SHIFTS ? 0 : NF == 1 ? word >> 16 : tp.step) + jf);
                }
                // The taps (j-1, j), (j, j+1), (j+1, j+2) of the pair come from
                // three aligned words; byte permutes pick them whatever the
                // parity of the shift.  (One read of 8 bytes at a 2-byte step
                // takes the LDS longer: 1.88 -> 2.62 ms at 1920x1080 x 128.)
                const int at = med3_i32(at0[k] + tp.step, at_lo[k], at_hi[k]);
                const LdsWord *q = (const LdsWord *)(uintptr_t)(uint32_t)(at + (u & 1 ? 0 : (int)sizeof lds.cost[0]));
                const uint32_t A = q[0], B = q[1], C = q[2];
                const uint32_t wm = __builtin_amdgcn_perm(B, A, tp.sel);
                const uint32_t w0 = __builtin_amdgcn_perm(B, A, tp.sel + 0x02020202u);
                const uint32_t wp = __builtin_amdgcn_perm(C, B, tp.sel);
                const u16x2 cm = as_u16x2(wm), c0 = as_u16x2(w0), cp = as_u16x2(wp);
                const u16x2 c1 = __builtin_elementwise_add_sat(__builtin_elementwise_min(cm, cp), p1v);
                u16x2 best = __builtin_elementwise_min(c0, c1);
                best = __builtin_elementwise_min(best, flv);
                dl[k] = best - mqv;
                L[k] = sv[k] + dl[k];
            }
        }
        u16x2 m2 = as_u16x2(0xFFFFFFFFu);
        const __amdgpu_buffer_rsrc_t ro = row_rsrc(o_cur, kOut * D);
        o_cur += kOut * sstride;
        asm volatile("" : "+s"(o_cur));
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            cur[widx[k]] = as_u32(L[k]);
            // non-temporal: the path costs are read once, by the
            // winner-takes-all pass, long after the caches have turned over
            if (NARROW) {
                const uint32_t d = as_u32(dl[k]);
                __builtin_amdgcn_raw_buffer_store_b16((uint16_t)__builtin_amdgcn_perm(0u, d, 0x0c0c0200u), ro, lo8[k], 0,
                                                      kNonTemporal);
                const uint64_t even = __builtin_amdgcn_ballot_w64((uint16_t)d > 255);
                const uint64_t odd = __builtin_amdgcn_ballot_w64((uint16_t)(d >> 16) > 255);
                high[k] = write_lane((uint32_t)even, 4u * u, high[k]);
                high[k] = write_lane((uint32_t)odd, 4 * u + 1, high[k]);
                high[k] = write_lane((uint32_t)(even >> 32), 4 * u + 2, high[k]);
                high[k] = write_lane((uint32_t)(odd >> 32), 4 * u + 3, high[k]);
            } else {
                __builtin_amdgcn_raw_buffer_store_b32(as_u32(L[k]), ro, 2 * lo8[k], 0, kNonTemporal);
            }
            m2 = __builtin_elementwise_min(m2, (lv[k]) ? L[k] : as_u16x2(0xFFFFFFFFu));
        }
        __builtin_amdgcn_wave_barrier();
        if (PG) {
            // minimum and its label in one reduction (smallest label on ties)
            uint32_t key = 0xFFFFFFFFu;
#pragma unroll
            for (int k = 0; k < KP; ++k) {
                const uint32_t lw = as_u32(L[k]);
                const uint32_t i0 = lo8[k];
                const uint32_t k0 = (lw << 16) | i0, k1 = (lw & 0xFFFF0000u) | (i0 + 1);
                const bool ok = lv[k];
                key = ok && k0 < key ? k0 : key;
                key = ok && k1 < key ? k1 : key;
            }
            key = wave_min_u32(key);
            Mq = key >> 16;
            const int bi = (int)(key & 0xFFFFu);
            int f = 0;
            while (f + 1 < F && bi >= a.foff[f + 1]) ++f;
            int of = 0;
#pragma unroll
            for (int ff = 0; ff < NF; ++ff)
                if (WIN && ff == f) of = __builtin_amdgcn_readlane(c_off[ff], u);
            const int g = of + (bi - a.foff[f]);
            double cf = c_cur[0], rf = r_cur[0];
#pragma unroll
            for (int ff = 1; ff < NF; ++ff) {
                if (ff == f) {
                    cf = c_cur[ff];
                    rf = r_cur[ff];
                }
            }
            const PgPlane pl = planes[a.goff[f] + g];
            dq2 = dq1;
            a2 = a1;
            dq1 = cf > 0.0 ? div_by(pl.delta, cf, rf) : 0.0;
            a1 = dq1 > 0.0 ? 2.0 * recip_from(dq1, cf * pl.recip) : 0.0;
#pragma unroll
            for (int ff = 0; ff < NF; ++ff) {
                c_prev[ff] = c_cur[ff];
                r_prev[ff] = r_cur[ff];
            }
        } else {
            // (one pair a lane: the select stands between the halves' minimum
            // and the reduction)
            const uint32_t m = min_of_halves<KP == 1>(as_u32(KP == 1 ? L[0] : m2));
            Mq = wave_min_u32(KP > 1 || lv[0] ? m : 0xFFFFu);
        }
    };

    // the 9th bits of the block at t0
    auto store_high = [&](int t0) {
        const int t = t0 + (lane >> 2);
        if (lane >= 4 * PF || t >= len) return;
        const long p = p0 + (long)t * pstride;
#pragma unroll
        for (int k = 0; k < KP; ++k)
            __builtin_nontemporal_store(high[k], bits + ((size_t)p * KP + k) * 4 + (lane & 3));
    };

    // Whole blocks of PF steps, then the tail.  The loop body is one
    // straight run of PF steps, so every ring slot and block value keeps its
    // register from one block to the next and no load is waited for before
    // its use PF steps later.
    int t0 = 0;
    for (; t0 + 2 * PF + 1 <= len; t0 += PF) {
        issue_block(t0 + PF, raw);
#pragma unroll
        for (int u = 0; u < PF; ++u) step(t0 + u, u, false);
        if (NARROW) store_high(t0);
        finish_block(t0 + PF, raw);
    }
    for (; t0 + PF <= len; t0 += PF) {
        issue_block(t0 + PF, raw);
#pragma unroll
        for (int u = 0; u < PF; ++u) step(t0 + u, u, true);
        if (NARROW) store_high(t0);
        finish_block(t0 + PF, raw);
    }
#pragma unroll
    for (int u = 0; u < PF; ++u) {
        if (t0 + u >= len) break;
        step(t0 + u, u, true);
    }
    if (NARROW) store_high(t0);
}

template <int KP, int NF, bool WIN, bool SN, bool PG, bool NARROW>
__global__ __launch_bounds__(64 * WAVES) void k_sgm_pk(const SgmArgs a) {
    __shared__ PkLds lbuf[WAVES];
    __shared__ int s_lut[256];   // P2 by intensity change
    extern __shared__ PgPlane planes[];   // path gradient: the level's plane lists (a.sumG entries)
    for (int i = threadIdx.x; i < 256; i += 64 * WAVES) s_lut[i] = a.lut[i];
    if (PG)
        for (int i = threadIdx.x; i < a.sumG; i += 64 * WAVES) planes[i] = PgPlane{a.delta[i], 1.0 / a.delta[i]};
    __syncthreads();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int path = blockIdx.x * WAVES + wid;
    if (path >= a.path_begin[a.n_dirs]) return;
    sgm_pk_path<KP, NF, WIN, SN, PG, NARROW>(a, path, s_lut, planes, lbuf[wid]);
}

// The fields the aggregation reads of a frame's arguments in device memory,
// as wave-uniform values (the frame index is uniform, so are its fields).
__device__ __forceinline__ SgmArgs uniform_sgm_args(const SgmArgs *__restrict__ p) {
    SgmArgs a;
    a.w = rfl(p->w);
    a.h = rfl(p->h);
    a.D = rfl(p->D);
    a.n_fam = rfl(p->n_fam);
    for (int f = 0; f < kMaxFam; ++f) {
        a.W[f] = rfl(p->W[f]);
        a.foff[f] = rfl(p->foff[f]);
    }
    a.S = rflp(p->S);
    a.offs = rflp(p->offs);
    a.dI = rflp(p->dI);
    a.ref = rflp(p->ref);
    a.p1 = rfl(p->p1);
    a.n_dirs = rfl(p->n_dirs);
    for (int d = 0; d < 8; ++d) {
        a.dirs[d] = rfl(p->dirs[d]);
        a.out[d] = rflp(p->out[d]);
    }
    for (int d = 0; d < 9; ++d) a.path_begin[d] = rfl(p->path_begin[d]);
    a.pg = 0;
    return a;
}

// Persistent form over the paths of several frames: every wavefront takes
// the next job (a path of some frame: jobs prefix[f] .. prefix[f + 1] - 1
// are frame f's) from the counter until none is left, and loads the frame's
// P2 table into its own LDS slice when the frame changes.  The counter
// starts at 0 (the host clears it before the launch).
template <int KP, int NF, bool WIN, bool SN>
__global__ __launch_bounds__(64 * WAVES) void k_sgm_pk_jobs(const SgmArgs *__restrict__ list,
                                                            const int *__restrict__ prefix, int n,
                                                            unsigned *__restrict__ counter) {
    __shared__ PkLds lbuf[WAVES];
    __shared__ int s_lut[WAVES][256];
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int total = rfl(prefix[n]);
    int cur = -1;
    for (;;) {
        unsigned j = 0;
        if (lane == 0) j = atomicAdd(counter, 1u);
        const int job = __builtin_amdgcn_readfirstlane((int)j);
        if (job >= total) break;
        int f = 0;
        while (f + 1 < n && job >= rfl(prefix[f + 1])) ++f;
        if (f != cur) {
            for (int i = lane; i < 256; i += 64) s_lut[wid][i] = list[f].lut[i];
            __builtin_amdgcn_wave_barrier();
            cur = f;
        }
        sgm_pk_path<KP, NF, WIN, SN, false, false>(uniform_sgm_args(list + f), job - rfl(prefix[f]), s_lut[wid], nullptr,
                                            lbuf[wid]);
    }
}

// Launch the two-label kernel for KP label pairs per lane (variant chosen
// at run time).  Instantiated once per KP in k_sgm_inst.hip.
template <int KP>
void sgm_launch_pk(const SgmArgs &a, bool win, bool sn, dim3 grid, hipStream_t s) {
    const size_t lds = a.pg ? (size_t)a.sumG * sizeof(PgPlane) : 0;
#define FMVS_SGMPK(W_, S_, P_)                                                                                 \
    if (win == W_ && sn == S_ && (a.pg != 0) == P_) {                                                         \
        if (a.n_fam == 1 && a.narrow)                                                                         \
            hipLaunchKernelGGL((k_sgm_pk<KP, 1, W_, S_, P_, !P_>), grid, dim3(64 * WAVES), lds, s, a);        \
        else if (a.n_fam == 1)                                                                                \
            hipLaunchKernelGGL((k_sgm_pk<KP, 1, W_, S_, P_, false>), grid, dim3(64 * WAVES), lds, s, a);       \
        else if (a.n_fam <= 4 && a.narrow)                                                                    \
            hipLaunchKernelGGL((k_sgm_pk<KP, 4, W_, S_, P_, !P_>), grid, dim3(64 * WAVES), lds, s, a);        \
        else if (a.n_fam <= 4)                                                                                \
            hipLaunchKernelGGL((k_sgm_pk<KP, 4, W_, S_, P_, false>), grid, dim3(64 * WAVES), lds, s, a);       \
        else                                                                                                  \
            hipLaunchKernelGGL((k_sgm_pk<KP, kMaxFam, W_, S_, P_, false>), grid, dim3(64 * WAVES), lds, s, a); \
        return;                                                                                               \
    }
    FMVS_SGMPK(false, false, false)
    FMVS_SGMPK(true, false, false)
    FMVS_SGMPK(false, true, false)
    FMVS_SGMPK(true, true, false)
    FMVS_SGMPK(false, false, true)
    FMVS_SGMPK(true, false, true)
#undef FMVS_SGMPK
}

// The persistent form over several frames (no path gradient): nf_max bounds
// the families of every frame (1 or up to 4).
template <int KP>
hipError_t sgm_launch_pk_jobs(const SgmArgs *list, const int *prefix, int n, unsigned *counter, bool win, bool sn,
                              int nf_max, int blocks, hipStream_t s) {
#define FMVS_SGMJ(W_, S_)                                                                                        \
    if (win == W_ && sn == S_) {                                                                                \
        if (nf_max == 1)                                                                                        \
            hipLaunchKernelGGL((k_sgm_pk_jobs<KP, 1, W_, S_>), dim3(blocks), dim3(64 * WAVES), 0, s, list, prefix, \
                               n, counter);                                                                     \
        else if (nf_max <= 4)                                                                                   \
            hipLaunchKernelGGL((k_sgm_pk_jobs<KP, 4, W_, S_>), dim3(blocks), dim3(64 * WAVES), 0, s, list, prefix, \
                               n, counter);                                                                     \
        else                                                                                                    \
            return hipErrorInvalidValue;                                                                        \
        return hipGetLastError();                                                                               \
    }
    FMVS_SGMJ(false, false)
    FMVS_SGMJ(true, false)
    FMVS_SGMJ(false, true)
    FMVS_SGMJ(true, true)
#undef FMVS_SGMJ
    return hipErrorInvalidValue;
}

}  // namespace fmvs
