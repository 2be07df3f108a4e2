// lbm_march_kernels.h -- several time steps of the two-buffer D2V9 scheme in one launch.
//
// A single step moves every population through memory once (72 B per node in FP32) and is
// bound by that. k_march takes up to five steps in one pass over memory: a wave owns a strip
// of columns (its 64 lanes are 64 consecutive nodes of a row) and walks it upwards along y.
// Per row it pulls and collides step 1 from memory as the single step does; the
// post-collision row then stays in registers, where step 2 of the row below, step 3 of the
// row below that, ... take it up, and only the last step's row is written. Populations that
// move along y wait in registers for the row they move to, those that move along x go to
// the neighbouring lane by a DPP wave shift: no LDS, no barriers, waves independent of each
// other. The four outermost nodes of a strip on each side, and the steps - 1 rows before and
// after its segment of rows, only feed their neighbours (they are computed by two waves).
//
// Every node goes through the same arithmetic as in the single step (collide, and the
// rounding of 16-bit storage between steps), so the bits are the same. Between the steps of
// a launch a bounced population is taken from the node's own registers (f_q = g_qbar of the
// same node where the link mask has bit q) for every storage format; in memory each format
// keeps its own convention (kSolidSlotBB).
//
// What bounds it: the VALU at five steps per launch (about 500 instructions per row of 64
// lanes, of which 56 are written; FP32 4096^2 issues VALU in 89 % of its cycles), no longer memory:
// on that grid a launch of two steps took 320 us, of three 330 us, of five 350 us, against
// 190 us for one single step. Measured on MI355X, us per step against single steps: periodic
// 4096^2 FP32 70 (190), FP16 63 (101); with disks FP32 82, FP16 86. Two nodes per lane (fewer lanes lost
// at the strips' edges) measured the same in FP32 and 20 % slower in 16 bits (twice the
// registers, half the waves); streamed stores 5 % slower (neighbouring waves complete the
// lines at the strips' edges in the cache).
#pragma once

#include "lbm_device.h"

#include <algorithm>

namespace lbm {
namespace {

// D2V9 by motion along y: q = 2, 5, 6 up (e_y = +1), 4, 7, 8 down, 0, 1, 3 neither.
constexpr int kUp[3] = {2, 5, 6}, kDown[3] = {4, 7, 8}, kFlat[3] = {0, 1, 3};

constexpr int kMarchBlock = 256;  // threads per block: four strips side by side
constexpr int kMarchHalo = kMarchSteps - 1;          // lanes on each side that only feed their neighbours
constexpr int kMarchWidth = 64 - 2 * kMarchHalo;     // columns a wave writes

// What a later step of a launch keeps between two rows, r being the row of the step before
// it that came last.
struct Carry {
    float flat[3];  // incoming q = 0, 1, 3 of row r
    float up[3];    // incoming q = 2, 5, 6 of row r (from row r - 1)
    float next[3];  // q = 2, 5, 6 on their way from row r to row r + 1
    float own[3];   // solids: post-collision q = 2, 5, 6 of row r at their own nodes
    unsigned lk;    // solids: link mask of row r
    float s;        // porosity of row r
};

struct MarchArgs {
    StepArgs a;
    int steps;       // steps of this launch, 3 or 5
    int nbx;         // blocks side by side
    int rows;        // rows a segment writes
    FastDiv div_nbx;
    uint32_t keys[kMarchSteps];  // sr_key of the steps but the last
    uint32_t last_key;           // sr_key of the last step
};

template <int ST, bool MASK, bool SOFT, int FORCE, bool SLIP, bool SR>
__global__ __launch_bounds__(kMarchBlock, 4) void k_march(MarchArgs ma)
{
    constexpr int LAT = LBM_D2V9;
    using L = Lat<LAT>;
    using T = typename Codec<ST>::T;
    using LT = typename LinkMask<LAT>::T;
    StepArgs &a = ma.a;
    if constexpr (!SLIP) a.g.slip = 0;
    const Geometry &g = a.g;
    const int nx = g.nx, ny = g.ny;
    // blocks in contiguous slabs per XCD: neighbouring strips share the lines at their edges
    // in one L2 (measured: FP32 4096^2 352 us per launch against 363 in the hardware order)
    const int bid = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const int seg = fast_div(bid, ma.div_nbx);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int xs = ((bid - seg * ma.nbx) * (kMarchBlock / 64) + wave) * kMarchWidth;
    if (xs >= nx) return;
    const int y0 = seg * ma.rows, steps = ma.steps;
    const int nrows = min(ma.rows, ny - y0);
    const int lane = (int)(threadIdx.x & 63);
    const bool writes = lane >= kMarchHalo && lane < 64 - kMarchHalo && xs + lane - kMarchHalo < nx;
    int xi = (xs + lane - kMarchHalo) % nx;  // the lane's node, wrapped into the row
    if (xi < 0) xi += nx;
    const unsigned x = (unsigned)xi;
    PullRows r{};
    r.xl = x == 0u ? (unsigned)(nx - 1) : x - 1u;
    r.xr = x + 1u == (unsigned)nx ? 0u : x + 1u;
    Tile t{};
    t.x0 = xi;
    t.valid = true;
    auto to_row = [&](int y) {
        t.y = y;
        t.own = xi + nx * y;
        r.ym = wrapm(y, ny);
        r.yp = wrapp(y, ny);
    };
    auto is_wall = [&](int y) { return SLIP && (g.slip & LBM_SLIP_Y) && (y == 0 || y == ny - 1); };

    const T *src = static_cast<const T *>(a.src);
    struct Row {  // stored codes as loaded: decoded where they are used, so that no load is waited for earlier
        T c[L::Q];
        float s;
    };
    auto load_lk = [&](int y) -> LT {
        return MASK ? *at32(static_cast<const LT *>(a.links), x + (unsigned)nx * (unsigned)y) : (LT)0;
    };
    // The pull of row y (link mask lk) for step 1. Own slot: a bounced link reads slot qbar of
    // the node itself; the address is chosen per lane (the link mask came a row earlier), so
    // that no load waits for another (32-bit offsets: the state is below 4 GiB there).
    auto load_row = [&](int y, LT lk, Row &row) {
        to_row(y);
        // (with a mask, FP32 1531 x 1117 disks: 12.0 -> 11.8 us per step with the unrolling below;
        // without one the widened offsets cost nothing and pinning them cost 1-2 %)
        const unsigned xc = MASK ? lane_offset(x) : x;
        const unsigned xl = MASK ? lane_offset(r.xl) : r.xl, xr = MASK ? lane_offset(r.xr) : r.xr;
        for_q<L::Q>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const size_t off = pull_row<LAT, q>(g, t, r);
            const unsigned xq = L::ex[q] > 0 ? xl : (L::ex[q] < 0 ? xr : xc);
            if constexpr (MASK && !kSolidSlotBB<ST> && q != 0) {
                const unsigned own = (unsigned)L::opp[q] * (unsigned)g.stride + (unsigned)t.own;
                row.c[q] = *at32(src, (lk >> q) & 1u ? own : (unsigned)off + xq);
            } else {
                row.c[q] = *at32(src + off, xq);
            }
        });
        row.s = SOFT ? *at32(g.s, (unsigned)t.own) : 0.f;
    };

    Carry c[kMarchSteps - 1] = {};

    // Step l >= 2 of the row below y, the row of step l - 1 whose post-collision values, link
    // mask and porosity are o, lk, s; on return they are those of its own row. `live`: that
    // row's inputs are complete.
    auto advance = [&](auto lc, int y, bool live, float(&o)[L::Q], unsigned &lk, float &s) {
        constexpr int l = decltype(lc)::value;
        Carry &k = c[l - 2];
        if constexpr (ST != LBM_F32) {  // what step l - 1 stores
            const uint32_t h = SR ? sr_node((uint32_t)(xi + nx * y), ma.keys[l - 2]) : 0u;
#pragma unroll
            for (int q = 0; q < L::Q; ++q) o[q] = Codec<ST>::dec(enc_store<ST, SR>(o[q], h, q), 1.f);
        }
        // every population at the column it streams to
        float sh[L::Q];
        for_q<L::Q>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            sh[q] = L::ex[q] > 0 ? lane_prev(o[q]) : (L::ex[q] < 0 ? lane_next(o[q]) : o[q]);
        });
        // q = 4, 7, 8 into row y - 1: from row y, or, where that is a wall plane, the reflected
        // q = 2, 6, 5 of row y - 1 itself
        float dn[3] = {sh[4], sh[7], sh[8]};
        if (is_wall(y)) {
            dn[0] = k.next[0];
            dn[1] = k.next[2];
            dn[2] = k.next[1];
        }
        // what row y keeps: q = 2, 5, 6 from row y - 1 (from a wall plane there the reflected
        // q = 4, 8, 7 of row y), q = 0, 1, 3 of its own
        float up[3] = {k.next[0], k.next[1], k.next[2]};
        if (is_wall(wrapm(y, ny))) {
            up[0] = sh[4];
            up[1] = sh[8];
            up[2] = sh[7];
        }
        float fl[3] = {o[0], sh[1], sh[3]};
        if constexpr (MASK) {
            dn[0] = link_select<4>(k.lk, k.own[0], dn[0]);
            dn[1] = link_select<7>(k.lk, k.own[1], dn[1]);
            dn[2] = link_select<8>(k.lk, k.own[2], dn[2]);
            up[0] = link_select<2>(lk, o[4], up[0]);
            up[1] = link_select<5>(lk, o[7], up[1]);
            up[2] = link_select<6>(lk, o[8], up[2]);
            fl[1] = link_select<1>(lk, o[3], fl[1]);
            fl[2] = link_select<3>(lk, o[1], fl[2]);
        }
        float d[L::Q];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            d[kFlat[j]] = k.flat[j];
            d[kUp[j]] = k.up[j];
            d[kDown[j]] = dn[j];
            k.flat[j] = fl[j];
            k.up[j] = up[j];
            k.next[j] = sh[kUp[j]];
            k.own[j] = o[kUp[j]];
        }
        const unsigned lk_row = k.lk;
        const float s_row = k.s;
        k.lk = lk;
        k.s = s;
        lk = lk_row;
        s = s_row;
        if (live) collide<LAT, SOFT, FORCE>(a.ph, d, s, o);
    };

    // rows of step 1: y0 - (steps - 1) .. y0 + nrows - 1 + (steps - 1), wrapped; in iteration
    // `it` the last step reaches row y0 + it - first
    int y = (y0 - (steps - 1)) % ny;
    if (y < 0) y += ny;
    const int first = 2 * (steps - 1), nit = nrows + first;
    LT lk0 = load_lk(y), lk1 = load_lk(wrapp(y, ny));
    Row row0, row1;
    load_row(y, lk0, row0);
    auto iteration = [&](int it, Row &cur, Row &nxt) {
        const int yn = wrapp(y, ny);
        load_row(yn, lk1, nxt);  // (past the segment's end: rows of the grid all the same)
        LT lk2 = load_lk(wrapp(yn, ny));
        float d[L::Q], o[L::Q], s = cur.s;
        unsigned lk = lk0;
#pragma unroll
        for (int q = 0; q < L::Q; ++q) d[q] = Codec<ST>::dec(cur.c[q], 1.f);
        collide<LAT, SOFT, FORCE>(a.ph, d, s, o);
        // the later steps, each a row further down, as far as their first row has come
        auto later = [&](auto self, auto lc, int yl) -> void {
            constexpr int l = decltype(lc)::value;
            const bool live = it >= 2 * (l - 1);
            advance(lc, yl, live, o, lk, s);
            if constexpr (l < kMarchSteps)
                if (live && l < steps) self(self, std::integral_constant<int, l + 1>{}, wrapm(yl, ny));
        };
        later(later, std::integral_constant<int, 2>{}, y);
        // The next row's loads are waited for before this row's stores are issued: loads and
        // stores share one in-order counter, and a wait after the stores would be one for them.
#pragma unroll
        for (int q = 0; q < L::Q; ++q) asm volatile("" : "+v"(nxt.c[q]));
        if (SOFT) asm volatile("" : "+v"(nxt.s));
        if (MASK) asm volatile("" : "+v"(lk2));
        if (it >= first && writes) {
            to_row(y0 + it - first);
            if (MASK) t.own = (int)lane_offset((unsigned)t.own);
            const LT lo[1] = {(LT)lk};
            float(&o1)[1][L::Q] = reinterpret_cast<float(&)[1][L::Q]>(o);
            const uint32_t h[1] = {SR ? sr_node((uint32_t)t.own, ma.last_key) : 0u};
            store_tile<LAT, ST, MASK, 1, SR, false, false>(g, static_cast<T *>(a.dst), t, lo, o1, h);
        }
        y = yn;
        lk0 = lk1;
        lk1 = lk2;
    };
    if constexpr (MASK) {
        // two at a time, so that the row buffers change roles without moves (without a mask that
        // costs registers and with them a block per CU: FP32 4096^2, 50 steps 3.71 -> 3.82 ms)
        for (int it = 0; it < nit; it += 2) {
            iteration(it, row0, row1);
            if (it + 1 < nit) iteration(it + 1, row1, row0);
        }
    } else {
        for (int it = 0; it < nit; ++it) {
            iteration(it, row0, row1);
            row0 = row1;
        }
    }
}

// Rows per segment: the segments fill every CU once with one block fewer than it can hold
// (longer segments recompute fewer rows; a second round of blocks would leave CUs idle at its
// end. FP32 2048^2 with disks, us per launch at 3 / 4 / 5 blocks per CU: 142 / 147 / 151); at
// least 16 rows, below which the recomputed ones weigh more than idle CUs (FP32 1531 x 1117
// disks: 16 rows 12.8 us per step, 8 rows 13.3 us, 24 rows 16.9 us).
template <class Kernel>
int march_rows(Kernel kernel, int nbx, int ny, int cus)
{
    static const int per_cu = [&] {  // a property of the kernel, the same on every gfx950
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, kMarchBlock, 0) != hipSuccess || n < 1) n = 4;
        return std::max(1, n - 1);
    }();
    const int segs = std::max(1, per_cu * cus / nbx);
    return std::max(16, (ny + segs - 1) / segs);
}

template <int ST, bool MASK, bool SOFT, int FORCE, bool SLIP, bool SR>
hipError_t march_launch(MarchArgs &ma, int cus, hipStream_t st)
{
    constexpr int W = kMarchWidth * (kMarchBlock / 64);
    const Geometry &g = ma.a.g;
    const auto kernel = k_march<ST, MASK, SOFT, FORCE, SLIP, SR>;
    ma.nbx = (g.nx + W - 1) / W;
    ma.rows = march_rows(kernel, ma.nbx, g.ny, cus);
    ma.div_nbx = make_fastdiv(ma.nbx);
    const int nseg = (g.ny + ma.rows - 1) / ma.rows;
    hipLaunchKernelGGL(kernel, dim3(ma.nbx * nseg), dim3(kMarchBlock), 0, st, ma);
    return hipGetLastError();
}

// `steps` time steps (3 or 5) from a.src into a.dst with the step keys `keys`.
template <int ST, bool SR>
hipError_t march_st(int force, const StepArgs &a, int cus, int steps, const uint32_t *keys, hipStream_t st)
{
    const bool mask = a.links != nullptr, soft = a.g.s != nullptr, slip = a.g.slip != 0;
    MarchArgs ma{};
    ma.a = a;
    ma.steps = steps;
    for (int k = 0; k < steps; ++k) ma.keys[k] = ma.last_key = keys[k];
#define LBM_MARCH(M, S, F) \
    return M && slip ? march_launch<ST, M, S, F, M, SR>(ma, cus, st) : march_launch<ST, M, S, F, false, SR>(ma, cus, st)
#define LBM_MARCH_F(M, S)                   \
    do {                                    \
        if (force == 0) LBM_MARCH(M, S, 0); \
        if (force == 1) LBM_MARCH(M, S, 1); \
        if (force == 2) LBM_MARCH(M, S, 2); \
        LBM_MARCH(M, S, 3);                 \
    } while (0)
    if (mask) {
        if (soft) LBM_MARCH_F(true, true); else LBM_MARCH_F(true, false);
    } else {
        if (soft) LBM_MARCH_F(false, true); else LBM_MARCH_F(false, false);
    }
#undef LBM_MARCH_F
#undef LBM_MARCH
}

}  // namespace
}  // namespace lbm
