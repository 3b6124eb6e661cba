// Host-side bounds check of the index schemes of the balanced-tile kernels of 2D and 3D (tile_kernel.hpp) and of the
// wave tiles of 1D (line_kernel.hpp) (no GPU use).
//
// For every tile the kernels are instantiated with, enumerate what they compute: the LDS slots a thread stages its
// cells to, the packed address and stride of every face's upwind stencil on either side (and of a face that takes cell
// values), the flux slots a cell reads back; and for the wave tiles, on grids of every kind of end, the staged slots and
// the cells behind them.  Exit status 0 only if every index is in bounds and stands for the intended cell.
#include <cstdio>
#include <map>
#include <tuple>

#include "line_kernel.hpp"
#include "tile_kernel.hpp"

using namespace bub;

static int failures = 0;
#define CHECK(cond, ...)                                 \
    do {                                                 \
        if (!(cond)) {                                   \
            if (failures < 20) std::printf(__VA_ARGS__); \
            ++failures;                                  \
        }                                                \
    } while (0)

using Cell = std::tuple<int, int, int>;

template <int D, int TX, int TY, int TZ, int BLOCK>
void check_tile()
{
    using G = Geo<D, TX, TY, TZ>;
    using S = TileLds<D, TX, TY, TZ>;
    constexpr int CPT = (G::C + BLOCK - 1) / BLOCK;
    std::map<int, Cell> staged;   // LDS slot -> cell
    for (int tid = 0; tid < BLOCK; ++tid)
        for (int r = 0; r < CPT; ++r) {
            const int ci = tid + r * BLOCK;
            if (ci >= G::C) continue;   // (a thread without a cell stages cell 0 to the slot past the arrays)
            int i, j, k;
            const int h = G::cdecode(ci, i, j, k);
            if (ci < G::T) CHECK(r == 0 || ci >= BLOCK, "owned cell %d is not its thread's first\n", ci);
            int l[3] = {S::CELLS, S::CELLS, S::CELLS};
            if (D == 2) l[0] = S::template slot<0>(i, j, k);
            else {
                if (h == 0 || h < 0) l[0] = S::template slot<0>(i, j, k);
                if (h == 1 || h < 0) l[1] = S::template slot<1>(i, j, k);
                if (h == 2 || h < 0) l[2] = S::template slot<(D > 2 ? 2 : 0)>(i, j, k);
            }
            for (int e = 0; e < S::NL; ++e) {
                if (l[e] == S::CELLS) continue;
                CHECK(l[e] >= 0 && l[e] < S::CELLS, "%dD cell %d: slot %d of %d\n", D, ci, l[e], S::CELLS);
                CHECK(!staged.count(l[e]), "%dD cell %d: slot %d taken\n", D, ci, l[e]);
                staged[l[e]] = Cell(i, j, k);
            }
        }
    auto faces = [&](auto dtag) {
        constexpr int d = decltype(dtag)::value;
        constexpr int BX = G::template BX<d>(), BY = G::template BY<d>();
        constexpr int FD = d == 0 ? G::FX : (d == 1 ? G::FY : G::FZ), st = S::template stride<d>();
        CHECK(FD <= BLOCK, "faces\n");
        for (int t = 0; t < FD; ++t) {
            const int f[3] = {t % BX, (t / BX) % BY, t / (BX * BY)};
            for (int right = 0; right < 2; ++right)
                for (int ok = 0; ok < 2; ++ok) {
                    int p[3] = {f[0], f[1], f[2]};
                    p[d] -= 3;
                    int at = S::template slot<d>(p[0], p[1], p[2]) + (right ? 5 * st : 0), sd = right ? -st : st;
                    if (!ok) at += 2 * sd, sd = 0;
                    const int packed = (int)((unsigned)sd << 16) | at, at2 = packed & 0xffff, sd2 = packed >> 16;
                    CHECK(at2 == at && sd2 == sd, "%dD dir %d face %d: %d %d unpack to %d %d\n", D, d, t, at, sd, at2, sd2);
                    for (int o = 0; o < 5; ++o) {
                        const int l = at2 + o * sd2, off = ok ? o : 2;
                        Cell want(f[0], f[1], f[2]);
                        const int at_d = right ? 2 - off : off - 3;   // from the far end of its own side
                        if (d == 0) std::get<0>(want) += at_d;
                        if (d == 1) std::get<1>(want) += at_d;
                        if (d == 2) std::get<2>(want) += at_d;
                        CHECK(staged.count(l) && staged[l] == want, "%dD dir %d face %d side %d: entry %d at slot %d\n", D, d, t,
                              right, o, l);
                    }
                }
        }
        // an owned cell's low and high face are its threads' flux slots
        for (int oc = 0; oc < G::T; ++oc) {
            const int li = oc % TX, lj = (oc / TX) % G::TY, lk = oc / (TX * G::TY);
            const int lo = d == 0 ? li + (TX + 1) * (lj + G::TY * lk)
                                  : (d == 1 ? li + TX * (lj + (G::TY + 1) * lk) : li + TX * (lj + G::TY * lk));
            const int hi = lo + (d == 0 ? 1 : (d == 1 ? TX : TX * G::TY));
            const Cell me(li, lj, lk);
            Cell up = me;
            if (d == 0) std::get<0>(up) += 1;
            if (d == 1) std::get<1>(up) += 1;
            if (d == 2) std::get<2>(up) += 1;
            auto face = [&](int t) { return Cell(t % BX, (t / BX) % BY, t / (BX * BY)); };
            CHECK(lo >= 0 && hi < FD && face(lo) == me && face(hi) == up, "%dD dir %d cell %d: faces %d %d\n", D, d, oc, lo, hi);
        }
    };
    faces(std::integral_constant<int, 0>{});
    faces(std::integral_constant<int, 1>{});
    if (D > 2) faces(std::integral_constant<int, (D > 2 ? 2 : 0)>{});
}

void check_line(int nx, int bc)
{
    for (int tile = 0; tile * LINE_TX < nx; ++tile) {
        const int x0 = tile * LINE_TX;
        std::map<int, long long> staged;
        bool dum = false;
        for (int lane = 0; lane < 64; ++lane) {
            const long long c = map_coord(x0 + lane, nx, bc, dum);
            const int hx = lane < 3 ? lane - 3 : 61 + lane;
            const long long ch = lane < 5 ? map_coord(x0 + hx, nx, bc, dum) : c;
            const int hslot = lane < 5 ? hx + 3 : LINE_SLOTS - 1;
            CHECK(c >= 0 && c < nx && ch >= 0 && ch < nx, "line %d: cells %lld %lld\n", nx, c, ch);
            CHECK(lane + 3 < LINE_SLOTS - 1 && hslot >= 0 && hslot < LINE_SLOTS, "line slot\n");
            CHECK(!staged.count(lane + 3), "line slot %d taken\n", lane + 3);
            staged[lane + 3] = c;
            if (lane < 5) {
                CHECK(!staged.count(hslot), "line slot %d taken\n", hslot);
                staged[hslot] = ch;
            }
        }
        for (int lane = 0; lane < 64; ++lane)   // the face at the low side of x0 + lane
            for (int right = 0; right < 2; ++right)
                for (int ok = 0; ok < 2; ++ok) {
                    int st = lane + (right ? 5 : 0), sd = right ? -1 : 1;
                    if (!ok) st += 2 * sd, sd = 0;
                    for (int o = 0; o < 5; ++o) {
                        const int off = ok ? o : 2, x = x0 + lane + (right ? 2 - off : off - 3);
                        CHECK(staged.count(st + o * sd) && staged[st + o * sd] == map_coord(x, nx, bc, dum),
                              "line %d lane %d side %d entry %d\n", nx, lane, right, o);
                    }
                }
    }
}

int main()
{
    // the tiles of tile.hip
    check_tile<2, 16, 15, 1, 256>();
    check_tile<2, 32, 15, 1, 512>();
    check_tile<3, 8, 8, 3, 256>();
    check_tile<3, 8, 8, 7, 512>();
    for (int bc = 0; bc < 3; ++bc)
        for (int nx : {1, 2, 3, 5, 62, 63, 64, 65, 126, 127, 400})
            if (bc != 1 || nx >= 3) check_line(nx, bc);
    std::printf("%s (%d failures)\n", failures ? "FAIL" : "OK", failures);
    return failures ? 1 : 0;
}
