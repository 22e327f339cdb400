// Two steps of a lattice in one pass over memory (column-marching kernel).
//
// A step of the fused update (Section 3.1) is bound by the 19 loads and 19
// stores of every site, and step_vec runs within a few percent of a streaming
// copy.  Doing two steps between a load and a store of the state halves that
// traffic: a workgroup marches along y over a tile of 64 columns (x) and up to
// 13 planes (z), and keeps what the second step needs of the first one on the
// chip.
//
//  - The region of a tile is its own (core) sites and one site around them in
//    x and z.  Per row y of the march, the region's lanes pull and collide the
//    first step (one wave per plane, one lane per column; one more wave for
//    the two halo columns), and put the 16 populations that change column or
//    plane into LDS.  After a barrier the core lanes gather their neighbours'
//    values: those with c_y = -1 belong to the second step of row y - 1, which
//    is complete now and is collided and stored; those with c_y = 0 wait one
//    row and those with c_y = +1 two rows, in registers.
//  - The exchange buffers hold two rows of the twelve populations that are
//    read in their own row and four rows of the other four (154.7 KiB of the
//    CU's 160), so one barrier a row is enough.  1024 threads at 128 VGPRs: 16
//    waves a CU, the largest region the register file holds (19 values in
//    flight, 19 waiting and the collision's temporaries per site).
//  - The loads of the next row are issued between the first step and the
//    barrier and land during the second step.  Lanes and rows without a site
//    load and store through descriptors (or offsets) out of range, which move
//    nothing: no branch around them, so the waits count loads and stores
//    exactly and no wave waits for its stores.
//  - Tiles are dealt to the XCDs in contiguous ranges, x fastest, then z: the
//    halo columns and planes of concurrent tiles are then mostly hits in the
//    XCD's L2.
//
// Both steps round and sum exactly as two step_vec launches (collide, and
// add_moments' order-independent totals): the state and the per-step totals
// are the same bits.
//
// Measured on MI355X, FP32, microseconds a step with its totals, step_vec (its
// default width) -> march2: 512^3 3174 -> 2240, 256^3 400 -> 294, 96^3 27.3 ->
// 23.3, 64^3 9.5 -> 8.9, 48^3 7.3 -> 6.4, 32^3 4.9 -> 5.7, 24^3 5.0 -> 4.7.
// What bounds it on large lattices is memory: without the collisions it runs
// at the same speed (4.9 TB/s over 21.9 GB a launch at 512^3, 10.2 of them
// stores), and issuing the loads earlier (a whole row ahead) or deeper prefetch
// of the halo waves is slower.  On small ones it is the row of the march (0.36
// us per wave of the region).  Marching along z puts consecutive rows of a wave
// 20 MB apart at 512^3 and is 5% slower; one step per launch in this scheme
// loses to step_vec (3.4-4.4 ms at 512^3).
#include <algorithm>

#include "lb_device.h"

namespace lbm {
namespace {

constexpr int kMW = 64;                  // columns of a tile (one per lane)
constexpr int kMRegion = kMarchRows + 2; // planes of a region
constexpr int kMRS = kMW + 2;            // LDS row: halo column, 64 columns, halo column
constexpr int kMPlane = kMRegion * kMRS; // LDS words of one population
constexpr int kMThreads = 64 * (kMRegion + 1);
constexpr uint32_t kNoSite = 0xfffffffcu; // byte offset beyond every descriptor: the access is dropped

// Populations that stay in the row (c_y = 0), move with the march (+1) and
// against it (-1); the first of each list stays in its column and plane and
// needs no exchange.
constexpr int kY0[9] = {0, 1, 2, 5, 6, 11, 12, 13, 14};
constexpr int kYp[5] = {3, 7, 9, 15, 16};
constexpr int kYm[5] = {4, 8, 10, 17, 18};

// Exchange buffers: twelve populations (c_y = 0 and -1) of two rows, which
// are read in the row they are written in, and four (c_y = +1) of four rows,
// read two rows later (a third row would be overwritten by waves one barrier
// ahead).  Word of population i in the buffer of row k.
constexpr int kExA = 12 * kMPlane, kExP = 4 * kMPlane;
constexpr int kSlot[kQ] = {-1, 0, 1, -1, -1, 2, 3, 0, 8, 1, 9, 4, 5, 6, 7, 2, 3, 10, 11};
struct Exchange {
    float a[2 * kExA], p[4 * kExP];
};

// Offsets from the site's own slot minus one plane and one column: of the own
// value of population i, and of the value it brings from its neighbour.
constexpr int own_at(int i) { return kSlot[i] * kMPlane + kMRS + 1; }
constexpr int pulled_at(int i) { return kSlot[i] * kMPlane + (1 - CZ[i]) * kMRS + (1 - CX[i]); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void *p, uint32_t bytes = 0x7fffffffu)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ int wrap1(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// q[i] = population i pulled by the wave's row (y, z) at columns vx (byte
// offsets of x - 1, x, x + 1); on = false: no access.
__device__ __forceinline__ void load_row(float (&q)[kQ], const MarchArgs &a, int y, int z, const uint32_t (&vx)[3],
                                         uint32_t seg4, bool on)
{
    const int ys[3] = {wrap1(y - 1, a.ny), y, wrap1(y + 1, a.ny)}, zs[3] = {wrap1(z - 1, a.nz), z, wrap1(z + 1, a.nz)};
    const uint32_t v[3] = {on ? vx[0] : kNoSite, on ? vx[1] : kNoSite, on ? vx[2] : kNoSite};
    const char *src = reinterpret_cast<const char *>(a.src);
    __amdgpu_buffer_rsrc_t r[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int j = 0; j < 3; ++j) r[k][j] = rsrc_of(src + a.lay.row_base((uint32_t)(zs[k] * a.ny + ys[j])) * 4u);
#pragma unroll
    for (int i = 0; i < kQ; ++i)
        q[i] = __builtin_bit_cast(float,
                                  __builtin_amdgcn_raw_buffer_load_b32(r[1 - CZ[i]][1 - CY[i]], v[1 - CX[i]], i * seg4, 0));
}

// a summed over the lanes l and l ^ 32 in the lower half of the wave, b in
// the upper half (and likewise over l ^ 16 in even and odd rows of 16 lanes).
__device__ __forceinline__ double fold32(double a, double b)
{
    const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    const auto lo = __builtin_amdgcn_permlane32_swap(x.x, y.x, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(x.y, y.y, false, false);
    return __builtin_bit_cast(double, make_uint2(lo[0], hi[0])) + __builtin_bit_cast(double, make_uint2(lo[1], hi[1]));
}

__device__ __forceinline__ double fold16(double a, double b)
{
    const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    const auto lo = __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
    return __builtin_bit_cast(double, make_uint2(lo[0], hi[0])) + __builtin_bit_cast(double, make_uint2(lo[1], hi[1]));
}

// Totals of a row: the split moments of the wave's sites (add_moments; the
// sums are exact in any order), folded over the four rows of 16 lanes so that
// a lane keeps one component: mass in lanes 0..15, then momentum x, y, z.
// Two doubles a lane and step instead of eight.  All 64 lanes take part, those
// without a live site with zeros (all: every lane has one).
__device__ __forceinline__ void row_totals(const float (&g)[kQ], bool live, bool all, double (&acc)[2], const TotalSplit &sp)
{
    double t[kQ], v[4], part[8];
#pragma unroll
    for (int i = 0; i < kQ; ++i) t[i] = (double)g[i];
    moments_of_totals(t, v[0], v[1], v[2], v[3]);
    if (!all) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = live ? v[k] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) part[k] = 0.0;
    add_moments<8>(v[0], v[1], v[2], v[3], part, sp);
#pragma unroll
    for (int h = 0; h < 2; ++h)
        acc[h] += fold16(fold32(part[4 * h], part[4 * h + 2]), fold32(part[4 * h + 1], part[4 * h + 3]));
}

// Hand the first step's values of a region site to the exchange buffers.
__device__ __forceinline__ void hand_out(const float (&q)[kQ], float *a, float *p)
{
#pragma unroll
    for (int j = 1; j < 9; ++j) a[own_at(kY0[j])] = q[kY0[j]];
#pragma unroll
    for (int j = 1; j < 5; ++j) a[own_at(kYm[j])] = q[kYm[j]];
#pragma unroll
    for (int j = 1; j < 5; ++j) p[own_at(kYp[j])] = q[kYp[j]];
}

// kMacros: also the density and velocity of the second step (rho_out, u_out).
template <bool kForce, bool kMacros>
__global__ __launch_bounds__(kMThreads) void march2(MarchArgs a)
{
    __shared__ Exchange ex;
    int t = blockIdx.x;
    if (a.nprev > 0 && t-- == 0) {
        append_split_totals(a.nprev, a.prev, reinterpret_cast<SplitLds<2, kMThreads / 64> &>(ex));
        return;
    }
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    t = tile_of(t, a.ntiles, 1);
    const int tx = t % a.nxt, tz = t / a.nxt % a.nzt, ty = t / (a.nxt * a.nzt);
    const int X0 = tx * kMW, Y0 = ty * a.chunk, Z0 = tz * a.rows;
    const int W = min(kMW, nx - X0), H = min(a.rows, nz - Z0), L = min(a.chunk, ny - Y0);
    uint32_t seg4 = a.lay.seg * 4u;
    const char *src = reinterpret_cast<const char *>(a.src);
    char *dst = reinterpret_cast<char *>(a.dst);
    // An instruction takes one scalar operand: with these in vector registers
    // the per-direction force constants need no moves (18 a collision, which
    // the compiler would also hoist out of the march and spill).
    Coll cp = a.coll;
    if constexpr (kForce) asm volatile("" : "+v"(cp.hom), "+v"(cp.q1), "+v"(cp.q2));
    // rows Y0 - 1 .. Y0 + L take their first step at k = 0 .. last; every wave
    // passes the barrier of each k up to the next odd one
    const int last = L + 1;
    float mom[4];

    if (wave == kMRegion) {
        // the halo columns X0 - 1 (lanes 0..15, one per plane) and X0 + W (16..31)
        const bool in = lane < 32 && (lane & 15) < H + 2;
        const int rz = in ? (lane & 15) : 1, rc = lane < 16 ? 0 : W + 1;
        const int x = wrap1(X0 + rc - 1, nx), z = wrap1(Z0 + rz - 1, nz);
        const uint32_t xo[3] = {(uint32_t)wrap1(x - 1, nx), (uint32_t)x, (uint32_t)wrap1(x + 1, nx)};
        const uint32_t zr[3] = {(uint32_t)(wrap1(z - 1, nz) * ny), (uint32_t)(z * ny), (uint32_t)(wrap1(z + 1, nz) * ny)};
        const int base = (rz - 1) * kMRS + rc - 1;
        float q[kQ];
        auto load = [&](int y) __attribute__((always_inline)) {
            const uint32_t ys[3] = {(uint32_t)wrap1(y - 1, ny), (uint32_t)y, (uint32_t)wrap1(y + 1, ny)};
#pragma unroll
            for (int i = 0; i < kQ; ++i) {
                const uint64_t at = a.lay.row_base(zr[1 - CZ[i]] + ys[1 - CY[i]]) + (uint64_t)i * a.lay.seg + xo[1 - CX[i]];
                q[i] = *reinterpret_cast<const float *>(src + at * 4u);
            }
        };
        load(wrap1(Y0 - 1, ny));
        for (int k = 0; k <= last; ++k) {
            collide<kForce>(q, cp, mom[0], mom[1], mom[2], mom[3]);
            if (in) hand_out(q, ex.a + (k & 1) * kExA + base, ex.p + (k & 3) * kExP + base);
            if (k < last) load(wrap1(Y0 + k, ny));
            __syncthreads();
        }
        if (!(last & 1)) __syncthreads();
        return;
    }
    if (wave >= H + 2) {
        for (int k = 0; k <= (last | 1); ++k) __syncthreads();
        return;
    }
    const bool in = lane < W;
    const int x = X0 + lane, z = wrap1(Z0 + wave - 1, nz);
    const uint32_t vx[3] = {in ? (uint32_t)wrap1(x - 1, nx) * 4u : kNoSite, in ? (uint32_t)x * 4u : kNoSite,
                            in ? (uint32_t)wrap1(x + 1, nx) * 4u : kNoSite};
    const int base = (wave - 1) * kMRS + lane;  // of the site's own slot, one plane and one column back
    float q[kQ];
    load_row(q, a, wrap1(Y0 - 1, ny), z, vx, seg4, true);
    if (wave == 0 || wave == H + 1) {
        for (int k = 0; k <= last; ++k) {
            collide<kForce>(q, cp, mom[0], mom[1], mom[2], mom[3]);
            if (in) hand_out(q, ex.a + (k & 1) * kExA + base, ex.p + (k & 3) * kExP + base);
            load_row(q, a, wrap1(Y0 + k, ny), z, vx, seg4, k < last);
            __syncthreads();
        }
        if (!(last & 1)) __syncthreads();
        return;
    }
    // a core plane
    double acc1[2] = {0.0, 0.0}, acc2[2] = {0.0, 0.0};
    float d0[9];                           // c_y = 0 values of the second step that wait for one row
    float up1 = 0.0f, up2 = 0.0f;          // population 3 of the last row and the one before
#pragma unroll
    for (int k = 0; k < 9; ++k) d0[k] = 0.0f;
    const bool all = W == kMW;
    // first step of row Y0 + k - 1, second step of row Y0 + k - 2; A: the
    // two-row buffer of this row
    auto row = [&](int k, float *A) __attribute__((always_inline)) {
        float *P = ex.p + base + (k & 3) * kExP;
        collide<kForce>(q, cp, mom[0], mom[1], mom[2], mom[3]);
        if (k >= 1 && k < last) row_totals(q, in, all, acc1, a.split);
        if (in) hand_out(q, A + base, P);
        const float own0 = q[0], up0 = q[3], down0 = q[4];
        asm volatile("" : "+s"(seg4));  // the populations' offsets are formed anew: kept, they spill other scalars
        load_row(q, a, wrap1(Y0 + k, ny), z, vx, seg4, k < last);
        __builtin_amdgcn_sched_barrier(0);  // the loads stay here: earlier they cost registers, later time
        __syncthreads();
        // the second step of the last row
        const float *Pbb = ex.p + base + ((k + 2) & 3) * kExP;
        const float *Ao = A + base;
        float f[kQ];
#pragma unroll
        for (int j = 0; j < 9; ++j) f[kY0[j]] = d0[j];
        f[3] = up2;
        f[4] = down0;
#pragma unroll
        for (int j = 1; j < 5; ++j) f[kYp[j]] = Pbb[pulled_at(kYp[j])];
#pragma unroll
        for (int j = 1; j < 5; ++j) f[kYm[j]] = Ao[pulled_at(kYm[j])];
        d0[0] = own0;
#pragma unroll
        for (int j = 1; j < 9; ++j) d0[j] = Ao[pulled_at(kY0[j])];
        const bool second = k >= 2 && k <= last;
        if (second) collide<kForce>(f, cp, mom[0], mom[1], mom[2], mom[3]);
        asm volatile("" : "+s"(seg4));
        const uint32_t r2 = (uint32_t)(z * ny + (second ? Y0 + k - 2 : Y0));
        const __amdgpu_buffer_rsrc_t rd = rsrc_of(dst + a.lay.row_base(r2) * 4u);
        const uint32_t vs = second ? vx[1] : kNoSite;
#pragma unroll
        for (int i = 0; i < kQ; ++i)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, f[i]), rd, vs, i * seg4, kStoreAux);
        if constexpr (kMacros) {
            const size_t n = (size_t)nx * ny * nz, s0 = (size_t)r2 * nx;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                __builtin_amdgcn_raw_buffer_store_b32(
                    __builtin_bit_cast(uint32_t, mom[c]), rsrc_of(c == 0 ? a.rho_out + s0 : a.u_out + (c - 1) * n + s0), vs, 0, 0);
        }
        if (second) row_totals(f, in, all, acc2, a.split);
        up2 = up1;
        up1 = up0;
    };
    {
        // as many dropped stores as a row has, so that the loop's first wait
        // counts the same accesses as its others
        const __amdgpu_buffer_rsrc_t rd = rsrc_of(src);
#pragma unroll
        for (int i = 0; i < kQ + (kMacros ? 4 : 0); ++i)
            __builtin_amdgcn_raw_buffer_store_b32(0u, rd, kNoSite, i * seg4, kStoreAux);
    }
    for (int k = 0; k <= last; k += 2) {
        // The 9.6 KB of this loop start 16 bytes into a 32-byte block of code,
        // wherever the code before it ends: 512^3 in 2233 us a step, at 0, 8 and
        // 24 bytes 2356, 2337 and 2292 (other sizes and a force: within 1%).
        asm volatile(".p2align 5\ns_nop 0\ns_nop 0\ns_nop 0\ns_nop 0");
        row(k, ex.a);
        row(k + 1, ex.a + kExA);
    }
    const size_t part = ((size_t)ty * nz + (Z0 + wave - 1)) * a.nxt + tx;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int off = 8; off >= 1; off /= 2) {
            acc1[h] += __shfl_xor(acc1[h], off, 64);
            acc2[h] += __shfl_xor(acc2[h], off, 64);
        }
        if (lane % 16 == 0) {
            a.partials[0][8 * part + 4 * h + lane / 16] = acc1[h];
            a.partials[1][8 * part + 4 * h + lane / 16] = acc2[h];
        }
    }
}

}  // namespace

// Tile shape of two-step launches for an nx x ny x nz lattice on cus compute
// units, and whether they beat two one-step launches.  Fitted to sweeps of
// rows and chunk for thirteen lattices of 32^3 to 384^3 (the shape it picks is
// within 13% of the best): a launch takes rounds x (chunk + 2) rows of the
// march, of 0.36 us per wave; when the tiles are whole rounds of the CUs, the
// workgroup that appends totals delays one of them (6 us).  Where rows do not
// start on 64-byte sectors neighbouring tiles share the sectors at their edges
// and store them in parts: little lost while the state fits the L2s, 1.25x in
// the memory-side cache, 1.4x to 1.8x beyond (200^3: 440 us against 414 of two
// one-step launches; 192^3: 260 against 361).  A one-step launch takes 6.3 us
// and its bytes at 6.4 TB/s: that is its time with 16-byte vectors.  With the
// widths of default_variant the estimate is off by a little on both sides: it
// keeps pairs at 32^3 (5.7 us a step against 4.9) and one step a launch at
// 125^3 (55.0 against 51.8 in pairs) and 101x75x47 (15.4 against 14.4).
MarchShape march_shape(int nx, int ny, int nz, int cus)
{
    MarchShape best{};
    const double sites = (double)nx * ny * nz;
    const double two_steps = 2.0 * (6.3 + sites * 152.0 / 6.4e6);
    const double sectors = nx % 16 == 0 ? 1.0 : (sites * 152.0 <= 32e6 ? 1.05 : (sites * 152.0 <= 256e6 ? 1.25 : 1.65));
    best.nxt = (nx + kMW - 1) / kMW;
    double best_us = 1e300;
    for (int rows = 1; rows <= kMarchRows && rows <= nz; ++rows) {
        const int nzt = (nz + rows - 1) / rows;
        if (rows < kMarchRows && rows < nz && (nz + rows) / (rows + 1) == nzt) continue;  // one more plane costs no tile
        const int fewest = (ny + kMarchChunk - 1) / kMarchChunk;
        for (int chunks = fewest; chunks <= ny; ++chunks) {
            const int chunk = (ny + chunks - 1) / chunks;
            if ((ny + chunk - 1) / chunk != chunks) continue;
            const int64_t tiles = (int64_t)best.nxt * nzt * chunks;
            if (tiles > 64 * (int64_t)cus && chunks > fewest) break;  // shorter chunks only add halos
            const double rounds = (double)((tiles + cus - 1) / cus);
            const double us = (tiles % cus == 0 ? 9.5 : 3.5) + rounds * (chunk + 2) * (0.07 + 0.36 * (rows + 3)) * sectors;
            if (us < best_us) {
                best_us = us;
                best.rows = rows;
                best.chunk = chunk;
                best.nzt = nzt;
                best.nyt = chunks;
            }
        }
    }
    best.use = best_us * 1.05 < two_steps;
    return best;
}

hipError_t launch_march2(const MarchArgs &a, hipStream_t s)
{
    const bool force = a.coll.fx != 0.0f || a.coll.fy != 0.0f || a.coll.fz != 0.0f;
    auto *fn = a.rho_out ? (force ? &march2<true, true> : &march2<false, true>)
                         : (force ? &march2<true, false> : &march2<false, false>);
    MarchArgs arg = a;
    void *params[] = {&arg};
    return hipLaunchKernel(reinterpret_cast<void *>(fn), dim3(a.ntiles + (a.nprev > 0 ? 1 : 0)), dim3(kMThreads), params, 0, s);
}

}  // namespace lbm
