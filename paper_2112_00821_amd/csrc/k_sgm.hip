// Host dispatch of the semi-global aggregation and the winner-takes-all
// kernels (Eq. sgm-path, sgm-aggr, sgm-wta of the paper); the aggregation
// kernels themselves are in k_sgm.hpp (the two-label kernel is instantiated
// per label-pair count in k_sgm_inst.hip so the variants compile in
// parallel).
#include "k_sgm.hpp"

#include <algorithm>
#include <cstdlib>
#include <cstring>

namespace fmvs {

extern template void sgm_launch_pk<1>(const SgmArgs &, bool, bool, dim3, hipStream_t);
extern template void sgm_launch_pk<2>(const SgmArgs &, bool, bool, dim3, hipStream_t);
extern template void sgm_launch_pk<3>(const SgmArgs &, bool, bool, dim3, hipStream_t);
extern template void sgm_launch_pk<4>(const SgmArgs &, bool, bool, dim3, hipStream_t);
extern template hipError_t sgm_launch_pk_jobs<1>(const SgmArgs *, const int *, int, unsigned *, bool, bool, int, int,
                                                 hipStream_t);
extern template hipError_t sgm_launch_pk_jobs<2>(const SgmArgs *, const int *, int, unsigned *, bool, bool, int, int,
                                                 hipStream_t);
extern template hipError_t sgm_launch_pk_jobs<3>(const SgmArgs *, const int *, int, unsigned *, bool, bool, int, int,
                                                 hipStream_t);
extern template hipError_t sgm_launch_pk_jobs<4>(const SgmArgs *, const int *, int, unsigned *, bool, bool, int, int,
                                                 hipStream_t);

int sgm_paths(int dir, int w, int h) {
    int dx = dir_dx(dir), dy = dir_dy(dir);
    if (dy == 0) return h;
    if (dx == 0) return w;
    return w + h - 1;
}

// Winner-takes-all over the summed path costs (Eq. sgm-aggr, sgm-wta) of
// fewer than 8 labels: one thread per pixel, all NB directions' loads in
// flight at once (direction by direction, 100x80 x 7 labels, 8 paths: the stage
// call 45 us, 38 us so; 1280x720 0.44 ms, 0.70 with a wavefront a pixel).
// The packed (cost << 16 | label) minimum gives the smallest label on ties.
// Also records the aggregate at the winner's two neighbours inside its family
// window for the refinement.
template <int NB>
__global__ __launch_bounds__(64) void k_wta_few(const SgmArgs a) {
    const size_t N = (size_t)a.w * a.h;
    const size_t p = (size_t)blockIdx.x * 64 + threadIdx.x;
    if (p >= N) return;
    const int D = a.D;
    uint32_t tot[7] = {0, 0, 0, 0, 0, 0, 0}, key = 0xFFFFFFFFu;
    uint16_t v[7][NB];
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        const size_t at = p * D + min(i, D - 1);
#pragma unroll
        for (int b = 0; b < NB; ++b) v[i][b] = a.in[b][at];
    }
#pragma unroll
    for (int i = 0; i < 7; ++i) {
#pragma unroll
        for (int b = 0; b < NB; ++b) tot[i] += v[i][b];
        const uint32_t k = (tot[i] << 16) | (uint32_t)i;
        key = i < D && k < key ? k : key;
    }
    const int best = (int)(key & 0xFFFFu);
    int f = 0;
    while (f + 1 < a.n_fam && best >= a.foff[f + 1]) ++f;
    const int l = best - a.foff[f];
    uint32_t cm = 0xFFFF, cp = 0xFFFF;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        if (l >= 1 && i == best - 1) cm = tot[i];
        if (l + 1 < a.W[f] && i == best + 1) cp = tot[i];
    }
    a.wta[p] = (uint16_t)best;
    a.c3[3 * p] = (uint16_t)cm;
    a.c3[3 * p + 1] = (uint16_t)(key >> 16);
    a.c3[3 * p + 2] = (uint16_t)cp;
}

// Row-level (16-lane) minimum: every lane of a DPP row ends with its row's
// minimum.
__device__ __forceinline__ uint32_t row_min_u32(uint32_t v) {
    uint32_t t;
    t = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false);
    v = v < t ? v : t;
    t = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false);
    v = v < t ? v : t;
    t = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xF, 0xF, false);
    v = v < t ? v : t;
    t = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xF, 0xF, false);
    return v < t ? v : t;
}

typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

// Winner-takes-all from 8 labels on: a DPP row of 16 lanes owns one pixel (4
// pixels per wavefront, contiguous in memory); each lane reads 8 labels of
// every direction buffer with one 16-byte load and adds them as packed 16-bit
// pairs (the aggregate fits 16 bits by the configuration's bound); argmin and
// the neighbours' aggregates come from row-level DPP reductions.  Bound by
// the path costs' bytes: 16-bit ones are read at 6.1 TB/s (1920x1080 x 128
// labels, 8 paths).  Where the label count is no multiple of 8 the last chunk
// starts 8 before the end, so that every load stays inside its pixel: the
// labels it repeats have the same sums.  Rows then start at 2-byte steps and
// loads are not aligned; all directions' are in flight at once (the stage
// call: 641x479 x 97 labels, 4 paths 308 us with one label a lane, 238 waiting
// for each direction, 232 so; 33x20 x 31, 8 paths 26.4, 28.0 and 25.6 us).
// The narrow forms read 9 bits a label (narrow_sums), at 4.8 TB/s: 0.67 ms
// with 16 bits, 0.55 so.
typedef unsigned short ushort8_t __attribute__((ext_vector_type(8), aligned(2)));
typedef uint32_t uint2_t __attribute__((ext_vector_type(2)));

// Aggregates of 8 labels (chunk c) of pixel p from NB directions' narrow path
// costs: NB costs S plus the heights, a byte each, plus 256 for each 9th bit.
// The bits of 8 labels are a nibble of the even labels' word and one of the
// odd labels'; a product spreads a nibble over four byte counters.
template <int NB, int NCH>
__device__ __forceinline__ void narrow_sums(const SgmArgs &a, size_t p, int c, int j, ushort2_t (&s4)[4]) {
    const size_t N = (size_t)a.w * a.h;
    const int D = a.D;
    const size_t bits = narrow_bits_at(N, D) + (p * NCH + j) * 16 + (size_t)((c & 8) ? 8 : 0);
    const int at = 4 * (c & 7);
    const uint2_t s = *(const uint2_t *)(a.S + p * D + 8 * c);
    uint2_t v[NB], m[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const uint8_t *in = (const uint8_t *)a.in[b];
        v[b] = __builtin_nontemporal_load((const uint2_t *)(in + p * D + 8 * c));
        m[b] = *(const uint2_t *)(in + bits);
    }
    constexpr uint32_t kLow = 0x00FF00FFu;
    uint32_t t[2][2], cnt[2] = {0, 0};   // [word][odd label], the counters [odd label]
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        t[i][0] = (s[i] & kLow) * NB;
        t[i][1] = ((s[i] >> 8) & kLow) * NB;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            t[i][0] += v[b][i] & kLow;
            t[i][1] += (v[b][i] >> 8) & kLow;
            cnt[i] += __umul24(__builtin_amdgcn_ubfe(m[b][i], at, 4), 0x204081u) & 0x01010101u;
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t up = i ? 0x030c020cu : 0x010c000cu;
        const uint32_t e = t[i][0] + __builtin_amdgcn_perm(0u, cnt[0], up);
        const uint32_t o = t[i][1] + __builtin_amdgcn_perm(0u, cnt[1], up);
        s4[2 * i] = __builtin_bit_cast(ushort2_t, __builtin_amdgcn_perm(o, e, 0x05040100u));
        s4[2 * i + 1] = __builtin_bit_cast(ushort2_t, __builtin_amdgcn_perm(o, e, 0x07060302u));
    }
    // the next chunk's loads stay behind this one's sums: the registers of
    // several chunks would leave two wavefronts a SIMD
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t t4 = __builtin_bit_cast(uint32_t, s4[i]);
        asm volatile("" : "+v"(t4) : : "memory");
        s4[i] = __builtin_bit_cast(ushort2_t, t4);
    }
}

enum WtaForm { kWtaAligned, kWtaUnaligned4, kWtaUnaligned8, kWtaNarrow4, kWtaNarrow8 };
template <int NCH, int FORM>
__global__ __launch_bounds__(256) void k_wta16(const SgmArgs a) {
    constexpr int UNALIGNED = FORM == kWtaUnaligned4 ? 4 : FORM == kWtaUnaligned8 ? 8 : 0;   // directions
    constexpr bool ALIGNED = !UNALIGNED;
    constexpr int NARROW = FORM == kWtaNarrow4 ? 4 : FORM == kWtaNarrow8 ? 8 : 0;   // directions
    const int lane = threadIdx.x & 63;
    const int row = lane >> 4, l16 = lane & 15;
    const size_t N = (size_t)a.w * a.h;
    const int D = a.D;
    const int nch = (D + 7) >> 3;
    const size_t waves = (size_t)gridDim.x * 4;
    const size_t wid = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const size_t vol_bytes = N * D * 2;
    const bool rsrc_ok = vol_bytes < ((size_t)1 << 32);
    for (size_t pb = wid * 4; pb < N; pb += waves * 4) {
        const size_t p = pb + row;
        const bool pv = p < N;
        uint32_t key = 0xFFFFFFFFu;
        uint32_t acc[NCH][4];
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            const int c = l16 + 16 * j;
            const bool cv = pv && c < nch;
            const int i0c = ALIGNED ? 8 * c : min(8 * c, D - 8);   // the chunk's first label
            ushort2_t s4[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
            if constexpr (NARROW != 0) narrow_sums<NARROW, NCH>(a, pv ? p : N - 1, min(c, nch - 1), j, s4);
            if constexpr (UNALIGNED != 0) {
                if (cv) {
                    ushort8_t v[UNALIGNED];
#pragma unroll
                    for (int b = 0; b < UNALIGNED; ++b)
                        v[b] = __builtin_nontemporal_load((const ushort8_t *)(a.in[b] + p * D + i0c));
#pragma unroll
                    for (int b = 0; b < UNALIGNED; ++b) {
                        const uint4 u = __builtin_bit_cast(uint4, v[b]);
                        s4[0] = s4[0] + __builtin_bit_cast(ushort2_t, u.x);
                        s4[1] = s4[1] + __builtin_bit_cast(ushort2_t, u.y);
                        s4[2] = s4[2] + __builtin_bit_cast(ushort2_t, u.z);
                        s4[3] = s4[3] + __builtin_bit_cast(ushort2_t, u.w);
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                if (ALIGNED && !NARROW && b < a.n_in && cv) {
                    // each path cost is read once: non-temporal load
                    // through a buffer resource over the whole volume
                    // (32-bit byte offsets), else a plain load
                    uint4 v;
                    if (rsrc_ok) {
                        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
                            const_cast<uint16_t *>(a.in[b]), 0, (int)(uint32_t)vol_bytes, 0x00020000);
                        v = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                                          rb, (uint32_t)((p * D + 8 * c) * 2), 0, kNonTemporal));
                    } else {
                        v = *(const uint4 *)(a.in[b] + p * D + 8 * c);
                    }
                    s4[0] += __builtin_bit_cast(ushort2_t, v.x);
                    s4[1] += __builtin_bit_cast(ushort2_t, v.y);
                    s4[2] += __builtin_bit_cast(ushort2_t, v.z);
                    s4[3] += __builtin_bit_cast(ushort2_t, v.w);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[j][e] = __builtin_bit_cast(uint32_t, s4[e]);
                if (cv) {
                    const uint32_t lo = acc[j][e] & 0xFFFFu, hi = acc[j][e] >> 16;
                    const uint32_t i0 = (uint32_t)(i0c + 2 * e);
                    const uint32_t k0 = (lo << 16) | i0, k1 = (hi << 16) | (i0 + 1);
                    key = k0 < key ? k0 : key;
                    key = k1 < key ? k1 : key;
                }
            }
        }
        key = row_min_u32(key);
        const int best = (int)(key & 0xFFFFu);
        int f = 0;
        while (f + 1 < a.n_fam && best >= a.foff[f + 1]) ++f;
        const int l = best - a.foff[f];
        const bool has_m = l >= 1, has_p = l + 1 < a.W[f];
        uint32_t cm = 0xFFFFu, cp = 0xFFFFu;
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            const int c = l16 + 16 * j;
            const int i0c = ALIGNED || c >= nch ? 8 * c : min(8 * c, D - 8);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int i = i0c + e;
                const uint32_t v = (e & 1) ? (acc[j][e >> 1] >> 16) : (acc[j][e >> 1] & 0xFFFFu);
                if (has_m && i == best - 1) cm = v;
                if (has_p && i == best + 1) cp = v;
            }
        }
        cm = row_min_u32(cm);
        cp = row_min_u32(cp);
        if (pv && l16 == 0) {
            a.wta[p] = (uint16_t)best;
            a.c3[3 * p] = (uint16_t)cm;
            a.c3[3 * p + 1] = (uint16_t)(key >> 16);
            a.c3[3 * p + 2] = (uint16_t)cp;
        }
    }
}

template <int K>
static void launch_k(const SgmArgs &a, bool win, bool sn, dim3 grid, hipStream_t s) {
#define FMVS_SGM(W_, S_, P_)                                                                  \
    if (win == W_ && sn == S_ && (a.pg != 0) == P_) {                                         \
        if (a.n_fam == 1)                                                                     \
            hipLaunchKernelGGL((k_sgm<K, 1, W_, S_, P_>), grid, dim3(64 * WAVES), 0, s, a);   \
        else                                                                                  \
            hipLaunchKernelGGL((k_sgm<K, kMaxFam, W_, S_, P_>), grid, dim3(64 * WAVES), 0, s, a); \
        return;                                                                               \
    }
    FMVS_SGM(false, false, false)
    FMVS_SGM(true, false, false)
    FMVS_SGM(false, true, false)
    FMVS_SGM(true, true, false)
    FMVS_SGM(false, false, true)
    FMVS_SGM(true, false, true)
#undef FMVS_SGM
}


static void launch_wta(const SgmArgs &a, hipStream_t s) {
    const size_t N = (size_t)a.w * a.h;
    const bool four = a.n_in == 4;   // else eight directions
    if (a.D < 8) {
        const dim3 few((unsigned)((N + 63) / 64));
        if (four)
            hipLaunchKernelGGL(k_wta_few<4>, few, dim3(64), 0, s, a);
        else
            hipLaunchKernelGGL(k_wta_few<8>, few, dim3(64), 0, s, a);
        return;
    }
    const dim3 grid((unsigned)std::min<size_t>((N + 15) / 16, 65536)), block(256);
    const int form = a.narrow      ? (four ? kWtaNarrow4 : kWtaNarrow8)
                     : (a.D & 7)   ? (four ? kWtaUnaligned4 : kWtaUnaligned8)
                                   : kWtaAligned;
#define FMVS_WTA(N_)                                                                              \
    switch (form) {                                                                              \
        case kWtaAligned: k_wta16<N_, kWtaAligned><<<grid, block, 0, s>>>(a); return;            \
        case kWtaUnaligned4: k_wta16<N_, kWtaUnaligned4><<<grid, block, 0, s>>>(a); return;      \
        case kWtaUnaligned8: k_wta16<N_, kWtaUnaligned8><<<grid, block, 0, s>>>(a); return;      \
        case kWtaNarrow4: k_wta16<N_, kWtaNarrow4><<<grid, block, 0, s>>>(a); return;            \
        default: k_wta16<N_, kWtaNarrow8><<<grid, block, 0, s>>>(a); return;                     \
    }
    switch ((a.D + 127) / 128) {   // 8-label chunks per lane
        case 1: FMVS_WTA(1)
        case 2: FMVS_WTA(2)
        case 3: FMVS_WTA(3)
        default: FMVS_WTA(4)
    }
#undef FMVS_WTA
}

// One thread per label pair of the n pixels from pixel p0 on.
__global__ __launch_bounds__(256) void k_widen(const uint8_t *__restrict__ S, const uint8_t *__restrict__ in, size_t N,
                                               int D, size_t p0, size_t n, uint16_t *__restrict__ dst) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t q = i / (unsigned)(D / 2);
    if (q >= n) return;
    const size_t p = p0 + q;
    const int pair = (int)(i - q * (unsigned)(D / 2));
    const uint32_t *m = (const uint32_t *)(in + narrow_bits_at(N, D)) +
                        (p * ((D + 127) / 128) + (pair >> 6)) * 4 + 2 * ((pair >> 5) & 1);
    for (int o = 0; o < 2; ++o) {
        const size_t at = p * D + 2 * pair + o;
        dst[q * D + 2 * pair + o] = (uint16_t)(S[at] + in[at] + (((m[o] >> (pair & 31)) & 1u) << 8));
    }
}

hipError_t launch_widen(const uint8_t *S, const void *narrow, size_t N, int D, size_t p0, size_t n, uint16_t *dst,
                        hipStream_t s) {
    const size_t pairs = n * (D / 2);
    hipLaunchKernelGGL(k_widen, dim3((unsigned)((pairs + 255) / 256)), dim3(256), 0, s, S, (const uint8_t *)narrow, N,
                       D, p0, n, dst);
    return hipGetLastError();
}

__global__ void k_zero_u32(unsigned *p) {
    if (threadIdx.x == 0) *p = 0u;
}

// Packed two-label kernel when every family window is even (all variants);
// the one-label kernel otherwise.
static bool use_packed(const SgmArgs &a) {
    if (a.final_mode || (a.D & 1)) return false;
    for (int f = 0; f < a.n_fam; ++f)
        if (a.W[f] & 1) return false;
    // FASSMVS_SGM_UNPACKED=1 selects the one-label kernel (same results);
    // read per launch so a process can run both
    const char *e = std::getenv("FASSMVS_SGM_UNPACKED");
    return !(e && std::atoi(e) != 0);
}

// The path costs of a direction are S plus a height of at most P2, so where
// no P2 exceeds 511 they can be held as a byte a label and a 9th bit.  The
// two-label kernel then writes 9 bits a label and direction and the winner's
// pass reads them, in place of 16 each; on large frames both are bound by
// those bytes (1920x1080 x 128 labels, 3 levels, 8 paths: 1.87 -> 1.60 ms and
// 0.88 -> 0.71 ms; 2704x1520, 4 families: 11.0 -> 9.7 and 5.7 -> 4.6 ms).
// What decides it is measured on one level, aggregation and winner together,
// time of the narrow form over the wide one's:
//  - labels missing of a pixel's last 128: a step's arithmetic is the same
//    without them, its bytes are fewer.  8 paths, 210 million labels, mean of
//    six processes a side (which differ by up to 1.2): 64 labels 1.15, 96 1.28,
//    112 1.21, 120 1.02, 128 0.95; two pairs a lane 136 1.11, 168 1.05, 192
//    1.09, 208 1.02, 216 0.92, 256 0.95; three 264 1.03, 288 1.00, 304 0.94,
//    384 0.87; four 392 0.89, 512 0.78.  4 paths: 64 1.08, 112 1.10, 120 0.92,
//    128 0.96; 136 1.05, 192 1.07, 200 0.92, 216 0.87; 264 0.96.
//  - the level's size: 128 labels, 8 paths 0.99 at 109 million labels, 0.97 at
//    150, 0.82 at 300; 4 paths 1.01 at 150, 0.96 at 210, 0.84 at 300; 384
//    labels 0.87 and 0.90 at 137 million with 8 and 4.
//  - the path gradient's arithmetic beside it: 1.03 -> 1.06 ms at 960x540.
// The winner's pass takes whole chunks of 8 labels, and from 16 labels on the
// bits (a word of 16 bytes per 128 labels) fit behind the bytes in the room of
// the 16-bit form.
bool sgm_narrow(const SgmArgs &a) {
    if ((a.D & 7) || a.D < 16 || a.D > kMaxLabels || a.n_fam > 4 || a.pg || !use_packed(a)) return false;
    const int pairs = (a.D + 127) / 128, missing = 128 * pairs - a.D;
    const int may[2][5] = {{0, 8, 56, 120, 128}, {0, 0, 40, 96, 128}};
    if (missing > may[a.n_dirs == 8][pairs]) return false;
    const size_t large = pairs <= 2 && a.n_dirs < 8 ? (size_t)3 << 26 : (size_t)1 << 27;
    if ((size_t)a.w * a.h * a.D < large) return false;
    return *std::max_element(a.lut, a.lut + 256) <= 511 && *std::min_element(a.lut, a.lut + 256) >= 0;
}

hipError_t launch_sgm(const SgmArgs &a0, hipStream_t s) {
    SgmArgs a = a0;
    a.path_begin[0] = 0;
    for (int i = 0; i < a.n_dirs; ++i) a.path_begin[i + 1] = a.path_begin[i] + sgm_paths(a.dirs[i], a.w, a.h);
    for (int i = a.n_dirs + 1; i < 9; ++i) a.path_begin[i] = a.path_begin[a.n_dirs];
    int paths = a.path_begin[a.n_dirs];
    if (a.final_mode) {
        if (a.D > kMaxLabels) return hipErrorInvalidValue;
        launch_wta(a, s);
        return hipGetLastError();
    }
    if (paths == 0) return hipSuccess;
    dim3 grid((unsigned)((paths + WAVES - 1) / WAVES));
    bool win = a.offs != nullptr, sn = a.dI != nullptr;
    if (a.pg && (sn || a.sumG > kMaxPgPlanes || !a.delta)) return hipErrorInvalidValue;
    if (a.narrow || use_packed(a)) {
        switch ((a.D + 127) / 128) {
            case 1: sgm_launch_pk<1>(a, win, sn, grid, s); break;
            case 2: sgm_launch_pk<2>(a, win, sn, grid, s); break;
            case 3: sgm_launch_pk<3>(a, win, sn, grid, s); break;
            case 4: sgm_launch_pk<4>(a, win, sn, grid, s); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    int K = (a.D + 63) / 64;
    switch (K) {
        case 1: launch_k<1>(a, win, sn, grid, s); break;
        case 2: launch_k<2>(a, win, sn, grid, s); break;
        case 3: launch_k<3>(a, win, sn, grid, s); break;
        case 4: launch_k<4>(a, win, sn, grid, s); break;
        case 5: launch_k<5>(a, win, sn, grid, s); break;
        case 6: launch_k<6>(a, win, sn, grid, s); break;
        case 7: launch_k<7>(a, win, sn, grid, s); break;
        case 8: launch_k<8>(a, win, sn, grid, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Several frames' aggregation in one persistent launch (two steps, as for
// the sweep).  prepare_sgm_batch: host[0..n-1] are the frames' args, each
// with its directions and output buffers set (write mode, no path gradient,
// even label counts and windows so the two-label kernel applies, at most 4
// families, the same windows / surface-normal choice); their path prefix
// per direction is set and they are written with the job prefix (n + 1
// ints) to out (host memory of sgm_batch_bytes(n)).  Returns the job count
// (paths over all frames), or -1 if the frames cannot share a launch; *kp,
// *win, *sn, *nf_max receive the kernel variant.
size_t sgm_batch_bytes(int n) { return sizeof(SgmArgs) * n + sizeof(int) * (n + 1); }

int prepare_sgm_batch(SgmArgs *host, int n, void *out, int *kp, bool *win, bool *sn, int *nf_max) {
    if (n < 1) return -1;
    int *prefix = (int *)((SgmArgs *)out + n);
    prefix[0] = 0;
    *kp = 1;
    *nf_max = 1;
    *win = host[0].offs != nullptr;
    *sn = host[0].dI != nullptr;
    for (int i = 0; i < n; ++i) {
        SgmArgs &a = host[i];
        if (a.pg || a.final_mode || !use_packed(a) || a.n_fam > 4 || (a.offs != nullptr) != *win ||
            (a.dI != nullptr) != *sn)
            return -1;
        a.path_begin[0] = 0;
        for (int d = 0; d < a.n_dirs; ++d) a.path_begin[d + 1] = a.path_begin[d] + sgm_paths(a.dirs[d], a.w, a.h);
        for (int d = a.n_dirs + 1; d < 9; ++d) a.path_begin[d] = a.path_begin[a.n_dirs];
        prefix[i + 1] = prefix[i] + a.path_begin[a.n_dirs];
        *kp = std::max(*kp, (a.D + 127) / 128);
        *nf_max = std::max(*nf_max, a.n_fam);
    }
    if (*kp > 4) return -1;
    std::memcpy(out, host, sizeof(SgmArgs) * n);
    return prefix[n];
}

// launch_sgm_batch: the args block prepared above in device memory at dev;
// counter: a device word the launch takes jobs from, cleared here by a fill
// kernel.  The grid holds up to six workgroups per CU; every wavefront
// leaves when the jobs run out.
hipError_t launch_sgm_batch(const void *dev, int n, int jobs, int kp, bool win, bool sn, int nf_max,
                            unsigned *counter, hipStream_t s) {
    if (jobs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, s, counter);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const SgmArgs *dl = (const SgmArgs *)dev;
    const int *dp = (const int *)((const SgmArgs *)dev + n);
    const int blocks = std::min((jobs + WAVES - 1) / WAVES, 256 * 6);
    switch (kp) {
        case 1: return sgm_launch_pk_jobs<1>(dl, dp, n, counter, win, sn, nf_max, blocks, s);
        case 2: return sgm_launch_pk_jobs<2>(dl, dp, n, counter, win, sn, nf_max, blocks, s);
        case 3: return sgm_launch_pk_jobs<3>(dl, dp, n, counter, win, sn, nf_max, blocks, s);
        case 4: return sgm_launch_pk_jobs<4>(dl, dp, n, counter, win, sn, nf_max, blocks, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fmvs
