// Host emulation of the half transforms of negacyclic_fft.h (N = 1024, four points per lane): the 64 lanes are looped
// over, the lane swaps and the LDS exchanges are arrays, and the stages, table entries and slot rules are the header's
// own.  Checks, for both halves:
//   1. the slots of an exchange are distinct, inside the buffer, and what is read is what the partner lane stored;
//   2. forward against the definition X_k = sum_j u_j exp(2 pi i j (4k+1) / (4M)), in the layout of the key rows:
//      lane t, register m <-> the k whose place in a Plan<3, 3> row is key_lane + key_reg;
//   3. inverse(forward(u)) = u after the last stage that joins the halves.
#include <cmath>
#include <complex>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "largest.h"
#include "negacyclic_fft.h"

using namespace she;
using HP = HalfPlan;
constexpr int L = 64, M = HP::M;

static std::vector<double> g_tw(2 * HP::COUNT);
static int failures = 0;
#define CHECK(c, ...) do { if (!(c)) { failures++; std::printf(__VA_ARGS__); } } while (0)

struct Lanes { double r[L][4], i[L][4]; };

static void entries(int pass, int h, int t, CosTan (&e)[2])
{
    for (int q = 0; q < 2; q++) {
        if (pass == 0) { e[q] = HP::first_entry(h, q); continue; }
        e[q].c = g_tw[2 * HP::entry(pass, h, q, t)];
        e[q].t = g_tw[2 * HP::entry(pass, h, q, t) + 1];
    }
}

// lane bit `bit` <-> register bit: lanes with the bit set give register `a` and take register `b` of their partner
static void swap_bit(double (&x)[L][4], int bit, int a, int b)
{
    for (int t = 0; t < L; t++)
        if (!(t & bit)) std::swap(x[t | bit][a], x[t][b]);
}
static void swap54(double (&x)[L][4])
{
    swap_bit(x, 32, 0, 2); swap_bit(x, 32, 1, 3);
    swap_bit(x, 16, 0, 1); swap_bit(x, 16, 2, 3);
}

static void exchange(Lanes &x, int (*from)(int, int), int (*to)(int, int))
{
    static double br[HP::XSLOTS], bi[HP::XSLOTS];
    for (int t = 0; t < L; t++) for (int m = 0; m < 4; m++) { br[from(m, t)] = x.r[t][m]; bi[from(m, t)] = x.i[t][m]; }
    for (int t = 0; t < L; t++) for (int m = 0; m < 4; m++) { x.r[t][m] = br[to(m, t)]; x.i[t][m] = bi[to(m, t)]; }
}
static int store1(int m, int t) { return HP::store1(m, t); }
static int load1(int m, int t) { return HP::load1(m, t); }
static int store2(int m, int t) { return HP::store2(m, t); }
static int load2(int m, int t) { return HP::load2(m, t); }

static void passes(Lanes &x, int pass, int h, bool inverse)
{
    for (int t = 0; t < L; t++) {
        CosTan e[2];
        entries(pass, h, t, e);
        if (inverse) node_pass_inverse<4>(x.r[t], x.i[t], e); else node_pass<4>(x.r[t], x.i[t], e);
    }
}

int main()
{
    make_half_twiddles(g_tw.data());
    for (int which = 0; which < 2; which++) {
        std::vector<int> seen(HP::XSLOTS, 0), read(HP::XSLOTS, 0);
        for (int t = 0; t < L; t++)
            for (int m = 0; m < 4; m++) {
                const int s = which ? store2(m, t) : store1(m, t), r = which ? load2(m, t) : load1(m, t);
                CHECK(s >= 0 && s < HP::XSLOTS && r >= 0 && r < HP::XSLOTS, "slot outside the buffer\n");
                seen[s]++; read[r]++;
            }
        for (int s = 0; s < HP::XSLOTS; s++) CHECK(seen[s] <= 1 && seen[s] == read[s], "exchange %d slot %d: %d stores, %d loads\n", which, s, seen[s], read[s]);
        for (int m = 0; m < 4; m++)
            for (int t0 = 0; t0 < L; t0 += 16) {
                int mask = 0;
                for (int t = t0; t < t0 + 16; t++) mask |= 1 << ((which ? load2(m, t) : load1(m, t)) % 16);
                CHECK(mask == 0xFFFF, "exchange %d: sixteen lanes share a slot modulo 16\n", which);
            }
    }
    std::vector<double> ur(M), ui(M);
    uint64_t s = 1;
    for (int j = 0; j < M; j++) {
        s = s * 6364136223846793005ull + 1442695040888963407ull; ur[j] = (double)(int)((s >> 40) & 127) - 64;
        s = s * 6364136223846793005ull + 1442695040888963407ull; ui[j] = (double)(int)((s >> 40) & 127) - 64;
    }
    const long double pi = 3.14159265358979323846264338327950288L;
    Lanes half[2];
    long double worst = 0;
    for (int h = 0; h < 2; h++) {
        Lanes &x = half[h];
        const double c = h ? -std::sqrt(0.5) : std::sqrt(0.5);
        for (int t = 0; t < L; t++)
            for (int m = 0; m < 4; m++) {
                const int a = 64 * m + t, b = a + 256;
                x.r[t][m] = ur[a] + c * (ur[b] - ui[b]);
                x.i[t][m] = ui[a] + c * (ur[b] + ui[b]);
            }
        passes(x, 0, h, false); swap54(x.r); swap54(x.i);
        passes(x, 1, h, false); exchange(x, store1, load1);
        passes(x, 2, h, false); exchange(x, store2, load2);
        passes(x, 3, h, false);
        for (int t = 0; t < L; t++)
            for (int m = 0; m < 4; m++) {
                const int place = HP::key_lane(h, t) + HP::key_reg(m);
                const int k = 64 * (place >> 6) + ((place >> 3) & 7) + 8 * (place & 7);
                CHECK((k & 1) == h, "a place of the other half\n");
                long double re = 0, im = 0;
                for (int j = 0; j < M; j++) {
                    const long double ang = 2 * pi * (long double)(((long long)j * (4 * k + 1)) % (4 * M)) / (4 * M);
                    re += ur[j] * cosl(ang) - ui[j] * sinl(ang);
                    im += ur[j] * sinl(ang) + ui[j] * cosl(ang);
                }
                keep_largest(worst, fabsl(re - x.r[t][m]));
                keep_largest(worst, fabsl(im - x.i[t][m]));
            }
    }
    // 512 points of magnitude 64: a few hundred rounding errors of 2^-53 relative to sums of at most 2^15
    CHECK(worst < 1e-9L, "forward differs from the definition by %Lg\n", worst);
    for (int h = 0; h < 2; h++) {
        Lanes &x = half[h];
        passes(x, 3, h, true); exchange(x, load2, store2);
        passes(x, 2, h, true); exchange(x, load1, store1);
        passes(x, 1, h, true); swap54(x.r); swap54(x.i);
        passes(x, 0, h, true);
    }
    long double back = 0;
    for (int t = 0; t < L; t++)
        for (int m = 0; m < 4; m++) {
            const int a = 64 * m + t, b = a + 256;
            const double y0r = half[0].r[t][m], y0i = half[0].i[t][m], y1r = half[1].r[t][m], y1i = half[1].i[t][m];
            const double dr = y0r - y1r, di = y0i - y1i, f = std::sqrt(0.5) / 512;
            for (long double e : {fabsl((y0r + y1r) / 512 - ur[a]), fabsl((y0i + y1i) / 512 - ui[a]),
                                  fabsl((dr + di) * f - ur[b]), fabsl((di - dr) * f - ui[b])})
                keep_largest(back, e);
        }
    CHECK(back < 1e-10L, "inverse(forward(u)) differs from u by %Lg\n", back);
    std::printf("forward %Lg inverse %Lg failures %d\n", worst, back, failures);
    return failures != 0;
}
