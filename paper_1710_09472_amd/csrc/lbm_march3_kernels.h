// lbm_march3_kernels.h -- two time steps of the two-buffer D3V19 scheme in one launch.
//
// A single step moves every population through memory once (152 B per node in FP32) and is
// bound by that. k_march3 takes two steps in one pass: a block owns a column of 64 x 13 nodes
// and walks it along z. Fifteen waves hold one x row each of the plane (the column's rows
// and one on each side), the sixteenth the two nodes beside every row. Per plane each node is
// pulled and collided (step 1) from memory as the single step does; its post-collision
// populations go through LDS (two halves in turn, one barrier per plane) to the nodes they
// stream to, which keep those of the planes below in registers until the plane above has
// come, collide again (step 2) and are written. The next plane's loads are in flight
// meanwhile.
//
// Node arithmetic, rounding of 16-bit storage between the steps and bits are those of single
// steps. Between the steps bounced populations come from the node's own registers.
// What bounds it: memory and the VALU in turn, held together by the barrier (FP32 duct
// 256 x 128 x 128: 726 MB and 46 % VALU issue in 172 us per launch; the column's outer rows,
// one in 6.5, and two planes per segment are computed twice). One block of 16 waves per CU is what
// its registers allow (100 - 128 VGPRs: four waves per SIMD), whatever its LDS. Measured on MI355X, us per
// step against single steps, FP32: Hall duct 87 (109), periodic 256^3 300 (480), 128^3
// porous 43.7 (60.8), 300 x 200 x 100 with obstacles 162 (304); FP16 periodic 256^3 191
// (239). Two blocks of 7 rows per CU instead of one of 15 measured 10 - 20 % slower (a third
// of their rows are outer ones).
#pragma once

#include "lbm_device.h"

#include <algorithm>

namespace lbm {
namespace {

constexpr int kM3Rows = 15, kM3Cols = 64;        // rows and columns a block holds in its row waves
constexpr int kM3Threads = 64 * (kM3Rows + 1);
constexpr int kM3Stride = kM3Cols + 2;           // LDS row: the columns and one on each side
constexpr int kM3Plane = kM3Rows * kM3Stride;

// D3V19 by motion along z: neither, up (e_z = +1), down (kM3Down[j] opposite of ... kM3Up)
constexpr int kM3Flat[9] = {0, 1, 2, 3, 4, 7, 8, 9, 10};
constexpr int kM3Up[5] = {5, 11, 14, 15, 18};
constexpr int kM3Down[5] = {6, 13, 12, 17, 16};  // kM3Up reflected in z
// index in kM3Up of the opposite of kM3Down[j]
constexpr int kM3DownOpp[5] = {0, 2, 1, 4, 3};

// LDS slot of a population that leaves its column of nodes, -1 for q = 0, 5, 6
constexpr int m3_slot(int q) { return q == 0 || q == 5 || q == 6 ? -1 : (q < 5 ? q - 1 : q - 3); }

struct March3Args {
    StepArgs a;
    int ntx, nty, planes;  // tiles along x and y, planes a segment writes
    FastDiv div_ntx, div_nty;
    uint32_t key[2];       // sr_key of the two steps
};

template <int ST, bool MASK, bool SOFT, int FORCE, bool SLIP, bool SR>
__global__ __launch_bounds__(kM3Threads, 4) void k_march3(March3Args ma)
{
    constexpr int LAT = LBM_D3V19;
    using L = Lat<LAT>;
    using T = typename Codec<ST>::T;
    using LT = typename LinkMask<LAT>::T;
    __shared__ float sh[2][16][kM3Plane];
    StepArgs &a = ma.a;
    if constexpr (!SLIP) a.g.slip = 0;
    const Geometry &g = a.g;
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const int bid = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const int col = fast_div(bid, ma.div_ntx), txi = bid - col * ma.ntx;
    const int seg = fast_div(col, ma.div_nty), tyi = col - seg * ma.nty;
    const int x0 = txi * kM3Cols, y0 = tyi * (kM3Rows - 2), z0 = seg * ma.planes;
    const int cols = min(kM3Cols, nx - x0), rows = min(kM3Rows - 2, ny - y0), planes = min(ma.planes, nz - z0);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
    const bool edge = wave == kM3Rows;  // the wave of the two outer columns: lanes 0.. left, 32.. right
    const int lrow = edge ? (lane & 31) : wave, lcol = edge ? (lane < 32 ? 0 : cols + 1) : lane + 1;
    const bool in = lrow < rows + 2 && (edge || lane < cols);
    const bool inner = !edge && wave >= 1 && wave <= rows;  // rows that are written
    auto wrap = [](int v, int n) {
        v %= n;
        return v < 0 ? v + n : v;
    };
    const int xi = wrap(x0 + lcol - 1, nx);
    const int yv = wrap(y0 + lrow - 1, ny);                 // per lane
    const int ys = wrap(y0 + (edge ? 0 : wave) - 1, ny);    // of a row wave
    const unsigned x = (unsigned)xi;
    PullRows r{};
    r.xl = x == 0u ? (unsigned)(nx - 1) : x - 1u;
    r.xr = x + 1u == (unsigned)nx ? 0u : x + 1u;
    auto is_wall_y = [&](int y) { return SLIP && (g.slip & LBM_SLIP_Y) && (y == 0 || y == ny - 1); };
    auto is_wall_z = [&](int z) { return SLIP && (g.slip & LBM_SLIP_Z) && (z == 0 || z == nz - 1); };

    const T *src = static_cast<const T *>(a.src);
    T c[L::Q];  // stored codes of the plane to come
    float sv = 0.f;
    auto load_lk = [&](int z) -> LT {
        return MASK ? *at32(static_cast<const LT *>(a.links), x + (unsigned)nx * (unsigned)(yv + ny * z)) : (LT)0;
    };
    // the pull of plane z for step 1 into c (rows by a scalar base, the outer columns per lane)
    auto load = [&](int z, LT lk) {
        Tile t{};
        t.x0 = xi;
        t.z = z;
        r.zm = wrapm(z, nz);
        r.zp = wrapp(z, nz);
        // own slot: a bounced link reads slot qbar of the node itself, the address chosen per
        // lane (32-bit offsets: the state is below 4 GiB there); waves without a link, most of
        // them where solids are walls, keep the scalar row addresses
        const bool bounced = MASK && !kSolidSlotBB<ST> && __builtin_amdgcn_ballot_w64((lk & (LT)~LinkMask<LAT>::solid) != 0) != 0;
        auto pull = [&](int y, auto sel) {
            t.y = y;
            r.ym = wrapm(y, ny);
            r.yp = wrapp(y, ny);
            const unsigned xc = lane_offset(x), xl = lane_offset(r.xl), xr = lane_offset(r.xr);
            for_q<L::Q>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                const size_t off = pull_row<LAT, q>(g, t, r);
                const unsigned xq = L::ex[q] > 0 ? xl : (L::ex[q] < 0 ? xr : xc);
                if constexpr (sel.value && q != 0) {
                    const unsigned own = (unsigned)L::opp[q] * (unsigned)g.stride + x + (unsigned)nx * (unsigned)(y + ny * z);
                    c[q] = *at32(src, (lk >> q) & 1u ? own : (unsigned)off + xq);
                } else {
                    c[q] = *at32(src + off, xq);
                }
            });
        };
        constexpr std::bool_constant<MASK && !kSolidSlotBB<ST>> select{};
        if (edge || bounced)
            pull(yv, select);
        else
            pull(ys, std::false_type{});
        if (SOFT) sv = *at32(g.s, x + (unsigned)nx * (unsigned)(yv + ny * z));
    };

    // step 2's incoming populations of the plane z - 1 below plane z of step 1
    float flat[9], up[5], next[5], own[5];
    unsigned lk_prev = 0;
    float s_prev = 0.f;
#pragma unroll
    for (int j = 0; j < 5; ++j) up[j] = next[j] = own[j] = 0.f;
#pragma unroll
    for (int j = 0; j < 9; ++j) flat[j] = 0.f;

    int z = wrap(z0 - 1, nz);
    LT lk = 0, lk_next = 0;
    if (in) {
        lk = load_lk(z);
        lk_next = load_lk(wrapp(z, nz));
        load(z, lk);
    }
    for (int it = 0; it < planes + 2; ++it) {
        float(&buf)[16][kM3Plane] = sh[it & 1];
        const int zn = wrapp(z, nz);
        float o[L::Q], s = sv;
        if (in) {
            float d[L::Q];
#pragma unroll
            for (int q = 0; q < L::Q; ++q) d[q] = Codec<ST>::dec(c[q], 1.f);
            collide<LAT, SOFT, FORCE, true>(a.ph, d, s, o);
            if constexpr (ST != LBM_F32) {  // what step 1 stores
                const uint32_t h = SR ? sr_node((uint32_t)(xi + nx * (yv + ny * z)), ma.key[0]) : 0u;
#pragma unroll
                for (int q = 0; q < L::Q; ++q) o[q] = Codec<ST>::dec(enc_store<ST, SR>(o[q], h, q), 1.f);
            }
#pragma unroll
            for (int q = 1; q < L::Q; ++q)
                if (m3_slot(q) >= 0) buf[m3_slot(q)][lrow * kM3Stride + lcol] = o[q];
            load(zn, lk_next);  // (past the segment's end: a plane of the grid all the same)
        }
        LT lk_far = in ? load_lk(wrapp(zn, nz)) : (LT)0;
        __syncthreads();
        if (inner && in) {
            // population q of plane z at the node it streams to within the plane; beside a
            // free-slip wall row the reflected one of the node's own row
            auto read = [&](auto qc) -> float {
                constexpr int q = decltype(qc)::value;
                if constexpr (m3_slot(q) < 0) {
                    return o[q];
                } else {
                    int rr = lrow - L::ey[q], p = m3_slot(q);
                    if constexpr (SLIP && L::ey[q] != 0) {
                        if (is_wall_y(L::ey[q] > 0 ? wrapm(ys, ny) : wrapp(ys, ny))) {
                            rr = lrow;
                            p = m3_slot(reflected<LAT>(q, true, false));
                        }
                    }
                    return buf[p][rr * kM3Stride + lcol - L::ex[q]];
                }
            };
            float down[5], fl[9], nx5[5];
            for_q<5>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                down[j] = read(std::integral_constant<int, kM3Down[j]>{});
                nx5[j] = read(std::integral_constant<int, kM3Up[j]>{});
            });
            for_q<9>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                fl[j] = read(std::integral_constant<int, kM3Flat[j]>{});
            });
            if constexpr (MASK) {  // (opaque: the reads stay one batch instead of a branch per link)
#pragma unroll
                for (int j = 0; j < 5; ++j) asm volatile("" : "+v"(down[j]), "+v"(nx5[j]));
#pragma unroll
                for (int j = 0; j < 9; ++j) asm volatile("" : "+v"(fl[j]));
            }
            float e[L::Q];
            for_q<5>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                e[kM3Up[j]] = up[j];
                // into plane z - 1 from above, or, where plane z is a wall, reflected from itself
                e[kM3Down[j]] = is_wall_z(z) ? next[j] : down[j];
                // into plane z from below, or, where plane z - 1 is a wall, reflected from itself
                up[j] = is_wall_z(wrapm(z, nz)) ? down[j] : next[j];
            });
#pragma unroll
            for (int j = 0; j < 9; ++j) {
                e[kM3Flat[j]] = flat[j];
                flat[j] = fl[j];
            }
            if (MASK && __builtin_amdgcn_ballot_w64(((lk_prev | (unsigned)lk) & ~(unsigned)LinkMask<LAT>::solid) != 0) != 0) {
                for_q<5>([&](auto jc) {
                    constexpr int j = decltype(jc)::value, qd = kM3Down[j], qu = kM3Up[j];
                    e[qd] = link_select<qd>(lk_prev, own[kM3DownOpp[j]], e[qd]);
                    up[j] = link_select<qu>((unsigned)lk, o[L::opp[qu]], up[j]);
                });
                for_q<9>([&](auto jc) {
                    constexpr int j = decltype(jc)::value, q = kM3Flat[j];
                    if constexpr (q != 0) flat[j] = link_select<q>((unsigned)lk, o[L::opp[q]], flat[j]);
                });
            }
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                next[j] = nx5[j];
                own[j] = o[kM3Up[j]];
            }
            const unsigned lk2 = lk_prev;
            const float s2 = s_prev;
            lk_prev = (unsigned)lk;
            s_prev = s;
            if (it >= 2) {
                float o2[1][L::Q];
                collide<LAT, SOFT, FORCE, true>(a.ph, e, s2, o2[0]);
                Tile t{};
                t.x0 = xi;
                t.y = ys;
                t.z = z0 + it - 2;
                t.own = (int)lane_offset((unsigned)(xi + nx * (ys + ny * t.z)));
                t.valid = true;
                const LT lo[1] = {(LT)lk2};
                const uint32_t h[1] = {SR ? sr_node((uint32_t)t.own, ma.key[1]) : 0u};
                // the next plane's loads are waited for before the stores are issued: one
                // in-order counter serves both
#pragma unroll
                for (int q = 0; q < L::Q; ++q) asm volatile("" : "+v"(c[q]));
                store_tile<LAT, ST, MASK, 1, SR, false, true>(g, static_cast<T *>(a.dst), t, lo, o2, h);
            }
        }
        z = zn;
        lk = lk_next;
        lk_next = lk_far;
    }
}

// Two time steps from a.src into a.dst with the step keys `keys`.
template <int ST, bool SR>
hipError_t march3_st(int force, const StepArgs &a, const March3Plan &p, const uint32_t *keys, hipStream_t st)
{
    const bool mask = a.links != nullptr, soft = a.g.s != nullptr, slip = a.g.slip != 0;
    March3Args ma{};
    ma.a = a;
    ma.ntx = p.ntx;
    ma.nty = p.nty;
    ma.planes = p.planes;
    ma.div_ntx = make_fastdiv(ma.ntx);
    ma.div_nty = make_fastdiv(ma.nty);
    ma.key[0] = keys[0];
    ma.key[1] = keys[1];
    const dim3 grid(ma.ntx * ma.nty * ((a.g.nz + ma.planes - 1) / ma.planes)), block(kM3Threads);
#define LBM_M3_K(M, S, F, SL) hipLaunchKernelGGL((k_march3<ST, M, S, F, SL, SR>), grid, block, 0, st, ma)
    // 16-bit states without solids come here only where this kernel beats single steps: rounded
    // to nearest, without a source term
#define LBM_M3(M, S, F)                                                    \
    do {                                                                   \
        if constexpr (ST == LBM_F32 || M || (!SR && (F == 0 || F == 3))) { \
            if (M && slip)                                                 \
                LBM_M3_K(M, S, F, M);                                      \
            else                                                           \
                LBM_M3_K(M, S, F, false);                                  \
        } else {                                                           \
            return hipErrorInvalidValue;                                   \
        }                                                                  \
    } while (0)
#define LBM_M3_F(M, S)   \
    if (force == 0)      \
        LBM_M3(M, S, 0); \
    else if (force == 1) \
        LBM_M3(M, S, 1); \
    else if (force == 2) \
        LBM_M3(M, S, 2); \
    else                 \
        LBM_M3(M, S, 3)
    if (mask) {
        if (soft) LBM_M3_F(true, true); else LBM_M3_F(true, false);
    } else {
        if (soft) LBM_M3_F(false, true); else LBM_M3_F(false, false);
    }
#undef LBM_M3_F
#undef LBM_M3
#undef LBM_M3_K
    return hipGetLastError();
}

}  // namespace
}  // namespace lbm
