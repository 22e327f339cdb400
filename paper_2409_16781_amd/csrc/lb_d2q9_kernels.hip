// Two-dimensional D2Q9 lattices: step, masks, initialisation, macros and
// raw-state repacking.
#include <algorithm>

#include "lb_device.h"

namespace lbm {
namespace {

// ----------------------------------------------------------- D2Q9 (2-D) --
// The paper's own two-dimensional model (D2Q9, Section 2 and Fig. 1) for the
// lid-driven cavity it benchmarks (Section 3.3): the same fused pull update,
// 9 populations, FP32 storage of f - w.  Bounce-back off a wall returns the
// site's own opposite value; off the lid it adds 6 w_i (c_i . u_lid).

constexpr int kQ2 = 9;
constexpr int CX2[kQ2] = {0, 1, -1, 0, 0, 1, 1, -1, -1};
constexpr int CY2[kQ2] = {0, 0, 0, 1, -1, 1, -1, 1, -1};
constexpr int OPP2[kQ2] = {0, 2, 1, 4, 3, 8, 7, 6, 5};
constexpr int kPlusX2[3] = {1, 5, 6};
constexpr int kMinusX2[3] = {2, 7, 8};

// BGK collision of one D2Q9 site (shifted populations, no force), written as
// pair increments like the D3Q19 collision: axis pairs (1,2), (3,4) take the
// remainder of sum_p c_p n_p = 0, the rest population that of the mass.
// Every fused multiply-add is written out, so that all kernels round alike.
__device__ __forceinline__ void collide2(float (&g)[kQ2], const Step2Args &p)
{
#pragma clang fp contract(off)
    const float s1 = g[1] + g[2], d1 = g[1] - g[2];
    const float s3 = g[3] + g[4], d3 = g[3] - g[4];
    const float s5 = g[5] + g[8], d5 = g[5] - g[8];
    const float s6 = g[6] + g[7], d6 = g[6] - g[7];
    const float drho = g[0] + (s1 + s3) + (s5 + s6);
    const float jx = d1 + d5 + d6;
    const float jy = d3 + d5 - d6;
    const float inv = __builtin_amdgcn_rcpf(1.0f + drho);
    const float ux = jx * inv, uy = jy * inv;
    const float t = __builtin_fmaf(-1.5f, __builtin_fmaf(jx, ux, jy * uy), drho);
    const float base1 = p.ow1 * t, base2 = p.ow2 * t;
    const float c5 = jx + jy, c6 = jx - jy;
    constexpr float kSixth = 1.0f / 6.0f;
    const float n5 = __builtin_fmaf(-kSixth, c5, d5), n6 = __builtin_fmaf(-kSixth, c6, d6);
    const float n1 = -(n5 + n6), n3 = -(n5 - n6);
    float sum_hs = 0.0f;
    relax_pair(g[1], g[2], s1, n1, jx, inv, base1, p.q1, 0.0f, 0.0f, p.hom, sum_hs);
    relax_pair(g[3], g[4], s3, n3, jy, inv, base1, p.q1, 0.0f, 0.0f, p.hom, sum_hs);
    relax_pair(g[5], g[8], s5, n5, c5, inv, base2, p.q2, 0.0f, 0.0f, p.hom, sum_hs);
    relax_pair(g[6], g[7], s6, n6, c6, inv, base2, p.q2, 0.0f, 0.0f, p.hom, sum_hs);
    g[0] = __builtin_fmaf(-2.0f, sum_hs, g[0]);
}

// Totals of the V stored sites of a lane: groups of two sites (one, if V = 1)
// are summed in FP64, and each group's mass and momentum are split into two
// parts whose sums are exact in any order (as add_moments for D3Q19), so a
// step's totals do not depend on the launch that took it.  Stored as three
// first parts, then three second parts.
template <int V>
__device__ __forceinline__ void add_totals2(const float (&g)[kQ2][V], double (&acc)[6], const TotalSplit &sp,
                                            bool count = true)
{
    constexpr int U = V >= 2 ? 2 : 1;
#pragma unroll
    for (int e = 0; e < V; e += U) {
        double t[kQ2];
#pragma unroll
        for (int i = 0; i < kQ2; ++i) {
            t[i] = (double)g[i][e];
            if constexpr (U == 2) t[i] += (double)g[i][e + 1];
        }
        const double s5 = t[5] + t[6], s7 = t[7] + t[8], d = t[5] - t[6], d7 = t[7] - t[8];
        const double v[3] = {(t[0] + ((t[1] + t[2]) + (t[3] + t[4]))) + (s5 + s7), (t[1] - t[2]) + (s5 - s7),
                             (t[3] - t[4]) + (d + d7)};
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double x = count ? v[k] : 0.0;
            const double hi = (x + sp.m1) - sp.m1;
            acc[k] += hi;
            acc[3 + k] += ((x - hi) + sp.m2) - sp.m2;
        }
    }
}

template <int NW, bool kSolids>
__global__ __launch_bounds__(kBlock) void step2d(Step2Args a)
{
    using K = Codec<kF32>;
    constexpr int V = NW;
    __shared__ EdgeLds lds;
    const char *src = reinterpret_cast<const char *>(a.src);
    char *dst = reinterpret_cast<char *>(a.dst);
    const uint32_t nx = (uint32_t)a.nx, ny = (uint32_t)a.ny;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int rit = (int)threadIdx.x >> a.lg_row_lanes;
    double acc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const int ntiles = (a.nslots + kBlock - 1) / kBlock;
    if (const int b = blockIdx.x; b < ntiles) {  // one workgroup per tile
        const int slot = b * kBlock + (int)threadIdx.x;
        const bool active = slot < a.nslots;
        const uint32_t s0 = (uint32_t)(active ? slot : a.nslots - 1) * V;
        const uint32_t y = fastdiv(s0, a.div_pitch);
        const uint32_t x0 = s0 - y * nx;
        const uint32_t ym = (y == 0 ? ny : y) - 1, yp = (y + 1 == ny) ? 0 : y + 1;
        const uint64_t own = a.lay.row_base(y) + x0;
        uint64_t rb[kQ2];
#pragma unroll
        for (int i = 0; i < kQ2; ++i)
            rb[i] = a.lay.row_base(CY2[i] > 0 ? ym : (CY2[i] < 0 ? yp : y)) + (uint64_t)i * a.lay.seg;
        bool dirty = false;  // the V sites share one 64-site chunk (V | 64)
        if constexpr (kSolids) dirty = a.chunkdirty[s0 >> 6] != 0;
        Lane<NW> d[kQ2];
#pragma unroll
        for (int i = 0; i < kQ2; ++i) d[i] = ldv<NW>(src + (rb[i] + x0) * 4);
        // Near solids: the masks and the site's own values of every population
        // that may bounce, loaded together with the pulls (not after the
        // masks).  Rows y +- 1 are not the own row, so directions 3..8 load
        // their opposite at the own row; for 1 and 2 it is the unshifted pull.
        uint32_t m[V];
        Lane<NW> ownv[kQ2];
        if constexpr (kSolids) {
            if (dirty) {
                load_masks<V>(a.nbmask + s0, m);
#pragma unroll
                for (int i = 3; i < kQ2; ++i) ownv[i] = ldv<NW>(src + (own + OPP2[i] * a.lay.seg) * 4);
            }
            ownv[1] = d[2];
            ownv[2] = d[1];
        }

        // x-edges: the element beyond a wave comes from the neighbouring
        // wave through LDS when that wave is in this tile and the element is
        // in the same row; the periodic wrap too when tiles hold whole rows;
        // anything else (tile ends of long rows) by a direct load
        const bool left_edge = (lane == 0) || (x0 == 0);
        const bool row_end = x0 + V >= nx;
        const bool right_edge = (lane == 63) || row_end;
        __syncthreads();  // the previous tile's readers of lds are done
        if (a.lds_edges) {
            if (row_end) {
#pragma unroll
                for (int k = 0; k < 3; ++k) lds.row_last[rit][k] = d[kPlusX2[k]].w[NW - 1];
            }
            if (x0 == 0) {
#pragma unroll
                for (int k = 0; k < 3; ++k) lds.row_first[rit][k] = d[kMinusX2[k]].w[0];
            }
        }
        if (lane == 63) {
#pragma unroll
            for (int k = 0; k < 3; ++k) lds.wave_last[wave][k] = d[kPlusX2[k]].w[NW - 1];
        }
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < 3; ++k) lds.wave_first[wave][k] = d[kMinusX2[k]].w[0];
        }
        __syncthreads();
        const uint32_t xl = (x0 == 0 ? nx : x0) - 1;
        const uint32_t xr = row_end ? 0 : x0 + V;
        // the neighbour of a wave seam inside a row is a lane of this tile
        const bool left_lds = x0 == 0 ? a.lds_edges != 0 : wave > 0;
        const bool right_lds = row_end ? a.lds_edges != 0 : wave < kBlock / 64 - 1;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int i = kPlusX2[k];
            uint32_t prev = wave_shr1(d[i].w[NW - 1]);
            if (left_edge) prev = left_lds ? (x0 == 0 ? lds.row_last[rit][k] : lds.wave_last[wave - 1][k])
                                           : ld_elem<kF32>(src, rb[i] + xl);
            d[i] = shift_in_from_left<kF32, NW>(d[i], prev);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int i = kMinusX2[k];
            uint32_t next = wave_shl1(d[i].w[0]);
            if (right_edge) next = right_lds ? (row_end ? lds.row_first[rit][k] : lds.wave_first[wave + 1][k])
                                             : ld_elem<kF32>(src, rb[i] + xr);
            d[i] = shift_in_from_right<kF32, NW>(d[i], next);
        }

        uint32_t dead = 0;
        uint32_t lidsel[kQ2];  // bit e: site e's value of direction i bounced off the lid
#pragma unroll
        for (int i = 0; i < kQ2; ++i) lidsel[i] = 0;
        if constexpr (kSolids) {
            if (dirty) {
#pragma unroll
                for (int e = 0; e < V; ++e) dead |= (m[e] >> 31) << e;
#pragma unroll
                for (int i = 1; i < kQ2; ++i) {
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        if ((m[e] >> i) & 1u) d[i].w[e] = ownv[i].w[e];
                        lidsel[i] |= ((m[e] >> (8 + i)) & 1u) << e;
                    }
                }
            }
        }
#pragma unroll
        for (int e = 0; e < V; ++e) {
            float g[kQ2];
#pragma unroll
            for (int i = 0; i < kQ2; ++i) {
                g[i] = K::dec(d[i].w[e]);
                if constexpr (kSolids)
                    if ((lidsel[i] >> e) & 1u) g[i] += a.lidc[i];
            }
            collide2(g, a);
            const bool live = !((dead >> e) & 1u);
#pragma unroll
            for (int i = 0; i < kQ2; ++i) d[i].w[e] = live ? K::enc(g[i]) : 0u;
        }
        if (active) {
            if (dead != (1u << V) - 1u) {
                const StoreBase sb = store_base(dst, own, 4);
#pragma unroll
                for (int i = 0; i < kQ2; ++i) stv_pop<NW>(sb, (uint32_t)i * a.lay.seg * 4u, d[i]);
            }
            // totals of the stored values (dead sites hold zero)
            float out[kQ2][V];
#pragma unroll
            for (int i = 0; i < kQ2; ++i)
#pragma unroll
                for (int e = 0; e < V; ++e) out[i][e] = K::dec(d[i].w[e]);
            add_totals2<V>(out, acc, a.split);
        }
    }
    const double parts[8] = {acc[0], acc[1], acc[2], 0.0, acc[3], acc[4], acc[5], 0.0};
    store_block_totals<8>(parts, a.partials + 8 * (size_t)blockIdx.x);
    if (a.nprev > 0 && blockIdx.x == 0) append_prev_totals<8>(a.nprev, a.prev);
}

// ------------------------------------------ several steps in one launch --
// A step reads and writes 72 bytes a site and step2d runs near the rate of a
// copy; march2d takes T steps between a load and a store.  A wave marches
// along y over a strip of 64 vectors of V columns, all T steps in its
// registers: row y is loaded, then step 1 of row y - 1 is complete and is
// collided, then step 2 of row y - 2, ... and step T of row y - T is stored.
// Between two rows each step keeps 9 values a site: the pulled values of its
// pending row with c_y = 0 and +1, and the last row's own values with c_y =
// +1 (a bounced value, or the next row's pulled one).  Values move between
// columns by wave shifts, so the outer H lanes of a strip are a halo computed
// twice (and T rows on each side of a chunk), and no wave waits for another.
// The next row is loaded as soon as the first step has taken this one (two
// rows ahead: no faster).
//
// Measured on MI355X, 4096^2, microseconds a step, one / two / four steps a
// launch: 186 / 111 / 66 without walls, 191 / 116 / 80 with (the waves along
// the side walls, whose rows all bounce, end last).  Four steps: 265 us a
// launch, 274 without collisions and totals (memory: 1.4 GB) and as long for
// the 1050 vector instructions a row (two sites a lane) at two waves a SIMD;
// a quarter of them are the totals' FP64 additions.
constexpr int kPY[3] = {3, 5, 7}, kMY[3] = {4, 6, 8};  // c_y = +1 and -1, with c_x = 0, 1, -1
constexpr uint32_t kNoSite2 = 0xfffffffcu;             // byte offset beyond every descriptor: the access is dropped

// Lanes of a strip's halo on each side: T columns, and with two columns a lane
// four lanes, so that a strip is 448 bytes of a row and neighbours share no
// 64-byte sector (4096^2, four steps: 296 us a launch at 480 bytes, 265 at 448).
constexpr int halo_lanes(int V, int T) { return V == 2 ? 4 : T; }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc2(const void *p)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, 0x7fffffff, 0x00020000);
}

// v moved one column to the right (cx = 1), to the left (-1), or as it is
// (zero moves in at the ends of the wave).
template <int V>
__device__ __forceinline__ void shift_x(const float (&v)[V], int cx, float (&r)[V])
{
    if (cx > 0) {
#pragma unroll
        for (int e = V - 1; e > 0; --e) r[e] = v[e - 1];
        r[0] = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v[V - 1]), 0x138, 0xf, 0xf, true));
    } else if (cx < 0) {
#pragma unroll
        for (int e = 0; e < V - 1; ++e) r[e] = v[e + 1];
        r[V - 1] = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v[0]), 0x130, 0xf, 0xf, true));
    } else {
#pragma unroll
        for (int e = 0; e < V; ++e) r[e] = v[e];
    }
}

// Direction i at sites with masks m: own opposite value where x - c_i is solid.
template <int V>
__device__ __forceinline__ void bounce2(float (&f)[V], const float (&own)[V], const uint32_t (&m)[V], int i)
{
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const uint32_t solid = (uint32_t)((int)(m[e] << (31 - i)) >> 31);  // all ones or zero
        f[e] = __builtin_bit_cast(float, (solid & __builtin_bit_cast(uint32_t, own[e])) |
                                             (~solid & __builtin_bit_cast(uint32_t, f[e])));
    }
}

// Direction i: plus the lid's term where x - c_i is the lid.
template <int V>
__device__ __forceinline__ void push2(float (&f)[V], const uint32_t (&m)[V], int i, float lid)
{
#pragma unroll
    for (int e = 0; e < V; ++e) f[e] = ((m[e] >> (8 + i)) & 1u) ? f[e] + lid : f[e];
}

template <int V>
__device__ __forceinline__ void load_vec2(uint32_t (&r)[V], __amdgpu_buffer_rsrc_t d, uint32_t at, uint32_t base)
{
    if constexpr (V == 2) {
        typedef unsigned int v2u __attribute__((ext_vector_type(2)));
        const v2u x = __builtin_amdgcn_raw_buffer_load_b64(d, at, base, 0);
        r[0] = x[0];
        r[1] = x[1];
    } else {
        r[0] = __builtin_amdgcn_raw_buffer_load_b32(d, at, base, 0);
    }
}

template <int V, int T, bool kSolids>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2))) void march2d(March2Args m)
{
    const Step2Args &a = m.s;
    int b = blockIdx.x;
    if (a.nprev > 0 && b-- == 0) {
        append_prev_totals<8>(a.nprev, a.prev);
        return;
    }
    constexpr int H = halo_lanes(V, T);
    const int lane = threadIdx.x & 63;
    const int item = __builtin_amdgcn_readfirstlane(4 * tile_of(b, (m.nitems + 3) / 4, 1) + ((int)threadIdx.x >> 6));
    if (item >= m.nitems) return;
    const int strip = item % m.nstrips, Y0 = item / m.nstrips * m.chunk;
    const int ny = a.ny, nv = a.nx / V, L = min(m.chunk, ny - Y0);
    int c = strip * (64 - 2 * H) + lane - H;
    const bool own = lane >= H && lane < 64 - H && c < nv;
    c %= nv;
    c = c < 0 ? c + nv : c;
    const uint32_t at = (uint32_t)c * V * 4u;
    const uint32_t seg4 = a.lay.seg * 4u;
    const char *src = reinterpret_cast<const char *>(a.src);
    char *dst = reinterpret_cast<char *>(a.dst);

    // pending values of each step: pulled c_y = 0 (0, 1, 2) and +1 (3, 5, 7)
    // of its row, and that row's own values of 3, 5, 7
    float F0[T][3][V], FP[T][3][V], P[T][3][V];
    double acc[T][6];
    uint32_t mk[T + 1][V];  // masks of rows y .. y - T
#pragma unroll
    for (int s = 0; s < T; ++s) {
#pragma unroll
        for (int k = 0; k < 6; ++k) acc[s][k] = 0.0;
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int e = 0; e < V; ++e) F0[s][j][e] = FP[s][j][e] = P[s][j][e] = 0.0f;
    }
#pragma unroll
    for (int s = 0; s <= T; ++s) {
#pragma unroll
        for (int e = 0; e < V; ++e) mk[s][e] = 0;
    }

    // row Y0 - T, and the masks and chunk flags one and two rows ahead
    int y = (Y0 - T) % ny;
    y = y < 0 ? y + ny : y;
    auto next = [&](int r) { return r + 1 == ny ? 0 : r + 1; };
    uint32_t q[kQ2][V], mq[V];
    uint32_t flag = 0;
    auto load = [&](int r) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t d = rsrc2(src + a.lay.row_base((uint32_t)r) * 4u);
#pragma unroll
        for (int i = 0; i < kQ2; ++i) load_vec2<V>(q[i], d, at, i * seg4);
    };
    auto load_flag = [&](int r) __attribute__((always_inline)) {
        return (uint32_t)a.chunkdirty[((uint32_t)r * (uint32_t)a.nx + (uint32_t)c * V) >> 6];
    };
    auto load_mask = [&](int r, uint32_t f) __attribute__((always_inline)) {
        load_vec2<V>(mq, rsrc2(a.nbmask + (size_t)r * a.nx), f != 0 ? at : kNoSite2, 0);
    };
    if constexpr (kSolids) {
        load_mask(y, load_flag(y));
        flag = load_flag(next(y));
    }
    load(y);
    // The stores of a row, of 4 V bytes a lane; lanes at kNoSite2 store nothing.
    auto store = [&](int r, uint32_t to, const float (&g)[kQ2][V]) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t d = rsrc2(dst + a.lay.row_base((uint32_t)r) * 4u);
#pragma unroll
        for (int i = 0; i < kQ2; ++i) {
            if constexpr (V == 2) {
                typedef unsigned int v2u __attribute__((ext_vector_type(2)));
                const v2u x = {__builtin_bit_cast(uint32_t, g[i][0]), __builtin_bit_cast(uint32_t, g[i][1])};
                __builtin_amdgcn_raw_buffer_store_b64(x, d, to, i * seg4, kStoreAux);
            } else {
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, g[i][0]), d, to, i * seg4, kStoreAux);
            }
        }
    };
    {
        // as many dropped stores as a row has: the wait for a row's loads then
        // counts the stores behind them on every path, and waits for none
        float none[kQ2][V] = {};
        store(Y0, kNoSite2, none);
    }
    // Row y of the march, the k-th of the chunk's L + 2 T.  dirty: a site of the
    // rows in flight bounces; lid: off the lid.
    auto row = [&](int k, bool dirty, bool lid) __attribute__((always_inline)) {
        const int y1 = next(y);
        float g[kQ2][V];
#pragma unroll
        for (int i = 0; i < kQ2; ++i)
#pragma unroll
            for (int e = 0; e < V; ++e) g[i][e] = __builtin_bit_cast(float, q[i][e]);
#pragma unroll
        for (int s = 0; s < T; ++s) {
            // g: row y - s after s steps; f: row y - s - 1, pulled
            float f[kQ2][V];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int cx = j == 0 ? 0 : (j == 1 ? 1 : -1);
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    f[j][e] = F0[s][j][e];
                    f[kPY[j]][e] = FP[s][j][e];
                }
                shift_x<V>(g[kMY[j]], cx, f[kMY[j]]);
                shift_x<V>(g[j], cx, F0[s][j]);
                shift_x<V>(P[s][j], cx, FP[s][j]);
            }
            if (kSolids && dirty) {
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    const int i = kMY[j];  // its opposite is 3, 7, 5 for 4, 6, 8
                    bounce2<V>(f[i], P[s][j == 0 ? 0 : 3 - j], mk[s + 1], i);
                    bounce2<V>(FP[s][j], g[OPP2[kPY[j]]], mk[s], kPY[j]);
                }
                bounce2<V>(F0[s][1], g[2], mk[s], 1);
                bounce2<V>(F0[s][2], g[1], mk[s], 2);
                if (lid) {
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        push2<V>(f[kMY[j]], mk[s + 1], kMY[j], a.lidc[kMY[j]]);
                        push2<V>(FP[s][j], mk[s], kPY[j], a.lidc[kPY[j]]);
                    }
                    push2<V>(F0[s][1], mk[s], 1, a.lidc[1]);
                    push2<V>(F0[s][2], mk[s], 2, a.lidc[2]);
                }
            }
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int e = 0; e < V; ++e) P[s][j][e] = g[kPY[j]][e];
            if (s == 0) {
                // the row is taken: load the next one (past the last, a row that is not used)
                load(y1);
                if constexpr (kSolids) {
                    load_mask(y1, flag);
                    flag = load_flag(next(y1));
                }
                __builtin_amdgcn_sched_barrier(0);  // not later: they have this row's time to arrive
            }
#pragma unroll
            for (int e = 0; e < V; ++e) {
                float h[kQ2];
#pragma unroll
                for (int i = 0; i < kQ2; ++i) h[i] = f[i][e];
                collide2(h, a);
#pragma unroll
                for (int i = 0; i < kQ2; ++i) g[i][e] = h[i];
            }
            if (kSolids && dirty) {  // solid sites hold zero
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const uint32_t keep = ~(uint32_t)((int)mk[s + 1][e] >> 31);
#pragma unroll
                    for (int i = 0; i < kQ2; ++i)
                        g[i][e] = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, g[i][e]) & keep);
                }
            }
            const int r = k - s - 1 - T;  // row of the chunk that has taken step s + 1
            add_totals2<V>(g, acc[s], a.split, r >= 0 && r < L);
        }
        // step T of row y - T
        const int r = k - 2 * T;
        store(Y0 + max(r, 0), r >= 0 && own ? at : kNoSite2, g);
        y = y1;
        // no copy of the next row's values before this point: it would wait for them
        __builtin_amdgcn_sched_barrier(0);
    };
    // the masks of the next row become mk[0]; all bits of the rows in flight
    auto take_masks = [&]() __attribute__((always_inline)) {
        uint32_t any = 0;
#pragma unroll
        for (int e = 0; e < V; ++e) {
#pragma unroll
            for (int s = T; s > 0; --s) {
                mk[s][e] = mk[s - 1][e];
                any |= mk[s][e];
            }
            mk[0][e] = mq[e];
            any |= mq[e];
        }
        return any;
    };
    const int rows = L + 2 * T;
    for (int k = 0; k < rows; ++k) {
        bool dirty = false, lid = false;
        if constexpr (kSolids) {
            const uint32_t any = take_masks();
            dirty = __builtin_amdgcn_ballot_w64(any != 0) != 0;
            lid = __builtin_amdgcn_ballot_w64((any & 0x1fe00u) != 0) != 0;
        }
        row(k, dirty, lid);
    }
#pragma unroll
    for (int s = 0; s < T; ++s) {
        double v[8] = {acc[s][0], acc[s][1], acc[s][2], 0.0, acc[s][3], acc[s][4], acc[s][5], 0.0};
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = own ? v[k] : 0.0;
        const double x = wave_reduce<8>(v);
        if (lane % 8 == 0) m.partials[s][8 * (size_t)item + wave_component<8>(lane)] = x;
    }
}

// bit i (1..8): site x - c_i is solid; bit 8 + i: it is the lid; bit 31: the site is solid.
__global__ __launch_bounds__(kBlock) void build_masks2d(const uint8_t *flags, int nx, int ny, uint32_t *nbmask)
{
    const int64_t n = (int64_t)nx * ny;
    for (int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x; s < n; s += (int64_t)gridDim.x * kBlock) {
        const int x = (int)(s % nx), y = (int)(s / nx);
        uint32_t m = flags[s] ? (1u << 31) : 0u;
#pragma unroll
        for (int i = 1; i < kQ2; ++i) {
            int xs = x - CX2[i], ys = y - CY2[i];
            xs = xs < 0 ? xs + nx : (xs >= nx ? xs - nx : xs);
            ys = ys < 0 ? ys + ny : (ys >= ny ? ys - ny : ys);
            const uint8_t f = flags[(int64_t)ys * nx + xs];
            if (f) m |= 1u << i;
            if (f == 2) m |= 1u << (8 + i);
        }
        nbmask[s] = m;
    }
}

// g_i = f_i^eq(rho, u) - w_i in FP64, rounded once (D2Q9 weights).
__global__ __launch_bounds__(kBlock) void init2d(float *dst, Layout lay, int nx, int ny, const double *rho,
                                                 const double *u, const uint8_t *flags)
{
    const int64_t n = (int64_t)nx * ny;
    for (int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x; s < n; s += (int64_t)gridDim.x * kBlock) {
        const bool solid = flags && flags[s];
        const double r = rho ? rho[s] : 1.0;
        const double ux = u ? u[s] : 0.0, uy = u ? u[n + s] : 0.0;
        const double uu = ux * ux + uy * uy;
        const uint32_t y = (uint32_t)(s / nx), x = (uint32_t)(s - (int64_t)y * nx);
        const uint64_t own = lay.row_base(y) + x;
#pragma unroll
        for (int i = 0; i < kQ2; ++i) {
            const double w = i == 0 ? 4.0 / 9.0 : (i < 5 ? 1.0 / 9.0 : 1.0 / 36.0);
            const double cu = CX2[i] * ux + CY2[i] * uy;
            dst[own + i * lay.seg] = solid ? 0.0f : (float)(w * ((r - 1.0) + r * (3.0 * cu + 4.5 * cu * cu - 1.5 * uu)));
        }
    }
}

__global__ __launch_bounds__(kBlock) void macros2d(const float *src, Layout lay, int nx, int ny, const uint8_t *flags,
                                                   float *rho, float *u)
{
    const int64_t n = (int64_t)nx * ny;
    for (int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x; s < n; s += (int64_t)gridDim.x * kBlock) {
        float r = 0.0f, ux = 0.0f, uy = 0.0f;
        if (!(flags && flags[s])) {
            const uint32_t y = (uint32_t)(s / nx), x = (uint32_t)(s - (int64_t)y * nx);
            const uint64_t own = lay.row_base(y) + x;
            float g[kQ2];
#pragma unroll
            for (int i = 0; i < kQ2; ++i) g[i] = src[own + i * lay.seg];
            const float m = g[0] + ((g[1] + g[2]) + (g[3] + g[4])) + ((g[5] + g[6]) + (g[7] + g[8]));
            const float px = (g[1] - g[2]) + (g[5] + g[6]) - (g[7] + g[8]);
            const float py = (g[3] - g[4]) + (g[5] - g[6]) + (g[7] - g[8]);
            r = 1.0f + m;
            ux = px / r;
            uy = py / r;
        }
        if (rho) rho[s] = r;
        if (u) {
            u[s] = ux;
            u[n + s] = uy;
        }
    }
}

// One byte per 64 consecutive sites: 1 if any of them has a mask bit set.
__global__ __launch_bounds__(kBlock) void build_chunkdirty(const uint32_t *nbmask, int64_t n, uint8_t *dirty)
{
    const int64_t nchunks = (n + 63) / 64;
    for (int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x; c < nchunks; c += (int64_t)gridDim.x * kBlock) {
        const int64_t end = (c + 1) * 64 < n ? (c + 1) * 64 : n;
        uint32_t any = 0;
        for (int64_t s = c * 64; s < end; ++s) any |= nbmask[s];
        dirty[c] = any ? 1 : 0;
    }
}

}  // namespace

hipError_t launch_step2d(int variant, bool solids, const Step2Args &a, int grid, hipStream_t s)
{
    void *fn;
    if (variant == 1)
        fn = solids ? reinterpret_cast<void *>(&step2d<4, true>) : reinterpret_cast<void *>(&step2d<4, false>);
    else if (variant == 2)
        fn = solids ? reinterpret_cast<void *>(&step2d<2, true>) : reinterpret_cast<void *>(&step2d<2, false>);
    else
        fn = solids ? reinterpret_cast<void *>(&step2d<1, true>) : reinterpret_cast<void *>(&step2d<1, false>);
    Step2Args arg = a;
    void *params[] = {&arg};
    return hipLaunchKernel(fn, dim3(grid), dim3(kBlock), params, 0, s);
}

// Chunk of rows of a launch of steps steps, and its time in microseconds.  Up
// to one wave a SIMD a row of four steps takes 2.7 us (two columns a lane), up
// to two waves 3.9 us, and more waves are further rounds; a launch takes 9 us
// more.  Two steps: 1.56, 2.6 and 6 us.  Measured, four steps: 512^2 at 3 rows a
// chunk 39 us (855 waves of 11 rows), 1024^2 63 at 12 and 62 at 6 (860 and 1710
// waves), 2048^2 116 at 20, 4096^2 265 without and 319 with walls at 79; two
// steps: 1024^2 29 at 6, 2048^2 70 at 20, 4096^2 223 at 79.
March2Shape march2_shape(int variant, int steps, int nx, int ny, int cus)
{
    const int V = variant == 3 ? 1 : 2, H = halo_lanes(V, steps), nv = nx / V, simds = 4 * cus;
    March2Shape best{};
    best.us = 1e300;
    const int nstrips = (nv + 64 - 2 * H - 1) / (64 - 2 * H);
    best.group = (64 - 2 * H) * V;
    const int fewest = (ny + kMarchChunk - 1) / kMarchChunk;
    for (int chunks = fewest; chunks <= ny; ++chunks) {
        const int chunk = (ny + chunks - 1) / chunks;
        if ((ny + chunk - 1) / chunk != chunks) continue;
        const int64_t waves = (int64_t)nstrips * chunks;
        if (waves > 64 * (int64_t)simds && chunks > fewest) break;
        const double rounds = (double)((waves + 2 * simds - 1) / (2 * simds));
        const double row = (V == 2 ? 1.0 : 0.62) * (waves <= simds ? (steps == 4 ? 2.7 : 1.56) : (steps == 4 ? 3.9 : 2.6));
        const double us = (steps == 4 ? 9.0 : 6.0) + rounds * (chunk + 2 * steps) * row;
        if (us < best.us) {
            best.us = us;
            best.nstrips = nstrips;
            best.chunk = chunk;
            best.nitems = (int)waves;
        }
    }
    best.group *= best.chunk;
    return best;
}

namespace {
template <int V, int T>
void *march2d_fn(bool solids)
{
    return solids ? reinterpret_cast<void *>(&march2d<V, T, true>) : reinterpret_cast<void *>(&march2d<V, T, false>);
}
}  // namespace

hipError_t launch_march2d(int variant, int steps, bool solids, const March2Args &a, hipStream_t s)
{
    void *fn = variant == 3 ? (steps == 4 ? march2d_fn<1, 4>(solids) : march2d_fn<1, 2>(solids))
                            : (steps == 4 ? march2d_fn<2, 4>(solids) : march2d_fn<2, 2>(solids));
    March2Args arg = a;
    void *params[] = {&arg};
    return hipLaunchKernel(fn, dim3((a.nitems + 3) / 4 + (a.s.nprev > 0 ? 1 : 0)), dim3(kBlock), params, 0, s);
}

hipError_t launch_masks2d(const uint8_t *flags, int nx, int ny, uint32_t *nbmask, uint8_t *chunkdirty, hipStream_t s)
{
    const int64_t n = (int64_t)nx * ny;
    build_masks2d<<<grid_for((uint64_t)n), kBlock, 0, s>>>(flags, nx, ny, nbmask);
    build_chunkdirty<<<grid_for((uint64_t)(n + 63) / 64), kBlock, 0, s>>>(nbmask, n, chunkdirty);
    return hipGetLastError();
}

hipError_t launch_init2d(void *dst, const Layout &lay, int nx, int ny, const double *rho, const double *u,
                         const uint8_t *flags, hipStream_t s)
{
    init2d<<<grid_for((uint64_t)nx * ny), kBlock, 0, s>>>(static_cast<float *>(dst), lay, nx, ny, rho, u, flags);
    return hipGetLastError();
}

hipError_t launch_macros2d(const void *src, const Layout &lay, int nx, int ny, const uint8_t *flags, float *rho,
                           float *u, hipStream_t s)
{
    macros2d<<<grid_for((uint64_t)nx * ny), kBlock, 0, s>>>(static_cast<const float *>(src), lay, nx, ny, flags, rho,
                                                            u);
    return hipGetLastError();
}

namespace {
__global__ __launch_bounds__(kBlock) void repack2d_kernel(float *planes, float *state, Layout lay, int64_t n,
                                                          int to_state)
{
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < (int64_t)kQ2 * n; k += (int64_t)gridDim.x * kBlock) {
        const int i = (int)(k / n);
        const int64_t s = k - (int64_t)i * n;
        const uint32_t row = (uint32_t)(s / lay.nx);
        const uint64_t li = lay.row_base(row) + (uint64_t)i * lay.seg + (uint64_t)(s - (int64_t)row * lay.nx);
        if (to_state)
            state[li] = planes[k];
        else
            planes[k] = state[li];
    }
}
}  // namespace

hipError_t launch_repack2d(void *planes, void *state, const Layout &lay, int64_t n, bool to_state, hipStream_t s)
{
    repack2d_kernel<<<grid_for((uint64_t)kQ2 * n), kBlock, 0, s>>>(static_cast<float *>(planes),
                                                                   static_cast<float *>(state), lay, n, to_state ? 1 : 0);
    return hipGetLastError();
}

}  // namespace lbm
