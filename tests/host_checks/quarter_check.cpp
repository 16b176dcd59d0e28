// Host emulation of the transforms of k_blind_rotate_wide (negacyclic_fft.h: HalfLanes, QuarterInverse): lane swaps and
// exchanges are loops over arrays; stages, table entries, slot and lane rules are the header's own.  Checks
//   1. HalfLanes' LDS exchange: slots distinct and inside the buffer, sixteen lanes reading sixteen slots modulo 16;
//   2. forward against the definition X_k = sum_j u_j exp(2 pi i j (4k+1) / (4M)), in the layout of the key rows;
//   3. QuarterInverse reads every value of a half's spectrum once, in the layout of the key rows, and with the last two
//      stages gives back u.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "largest.h"
#include "negacyclic_fft.h"

using namespace she;
using HP = HalfPlan;
using HL = HalfLanes;
using QI = QuarterInverse;
constexpr int L = 64, M = HP::M;
static int failures = 0;
#define CHECK(c, ...) do { if (!(c)) { failures++; std::printf(__VA_ARGS__); } } while (0)
static std::vector<double> g_tw(2 * HP::COUNT), g_q(2 * QI::COUNT);

template <int P> struct Lanes { double r[L][P], i[L][P]; };

// lane bit <-> register bit: lanes with the bit set give register `a` and take register `b` of their partner
template <int P> static void swap_bit(Lanes<P> &x, int bit, int a, int b)
{
    for (int t = 0; t < L; t++)
        if (!(t & bit)) { std::swap(x.r[t | bit][a], x.r[t][b]); std::swap(x.i[t | bit][a], x.i[t][b]); }
}
static void swap_bits(Lanes<4> &x, int hi, int lo)
{
    swap_bit(x, hi, 0, 2); swap_bit(x, hi, 1, 3); swap_bit(x, lo, 0, 1); swap_bit(x, lo, 2, 3);
}
static void pass(Lanes<4> &x, int which, int h)
{
    for (int t = 0; t < L; t++) {
        CosTan e[2];
        const int lane = which == 2 ? HL::plan_lane_c(t) : which == 3 ? HL::plan_lane_d(t) : t;
        for (int q = 0; q < 2; q++) {
            const int at = which ? HP::entry(which, h, q, lane) : 0;
            e[q] = which ? CosTan{g_tw[2 * at], g_tw[2 * at + 1]} : HP::first_entry(h, q);
        }
        node_pass<4>(x.r[t], x.i[t], e);
    }
}
static int frequency(int place) { return 64 * (place >> 6) + ((place >> 3) & 7) + 8 * (place & 7); }

int main()
{
    make_half_twiddles(g_tw.data());
    make_quarter_twiddles(g_q.data());
    std::vector<int> seen(HL::XSLOTS, 0);
    for (int t = 0; t < L; t++)
        for (int m = 0; m < 4; m++) { const int r = HL::load(m, t); CHECK(r >= 0 && r < HL::XSLOTS, "slot\n"); seen[r]++; }
    for (int t = 0; t < L; t++)
        for (int m = 0; m < 4; m++) {
            const int w = HL::store(m, t);
            CHECK(w >= 0 && w < HL::XSLOTS && seen[w] == 1, "not stored and read once\n");
            seen[w] = 2;
        }
    for (int m = 0; m < 4; m++)
        for (int t0 = 0; t0 < L; t0 += 16) {
            int mask = 0;
            for (int t = t0; t < t0 + 16; t++) {
                mask |= 1 << (HL::load(m, t) % 16);
            }
            CHECK(mask == 0xFFFF, "sixteen lanes share a slot modulo 16\n");
        }
    std::vector<double> ur(M), ui(M);
    uint64_t s = 1;
    for (int j = 0; j < M; j++) {
        s = s * 6364136223846793005ull + 1442695040888963407ull; ur[j] = (double)(int)((s >> 40) & 127) - 64;
        s = s * 6364136223846793005ull + 1442695040888963407ull; ui[j] = (double)(int)((s >> 40) & 127) - 64;
    }
    const long double pi = 3.14159265358979323846264338327950288L;
    long double worst = 0;
    double spec_r[2][256], spec_i[2][256];
    for (int h = 0; h < 2; h++) {
        Lanes<4> x;
        const double c = h ? -std::sqrt(0.5) : std::sqrt(0.5);
        for (int t = 0; t < L; t++)
            for (int m = 0; m < 4; m++) {
                const int a = 64 * m + HL::position(t), b = a + 256;
                x.r[t][m] = ur[a] + c * (ur[b] - ui[b]);
                x.i[t][m] = ui[a] + c * (ur[b] + ui[b]);
            }
        pass(x, 0, h); swap_bits(x, 32, 16);
        pass(x, 1, h);
        std::vector<double> br(HL::XSLOTS), bi(HL::XSLOTS);
        for (int t = 0; t < L; t++) for (int m = 0; m < 4; m++) { br[HL::store(m, t)] = x.r[t][m]; bi[HL::store(m, t)] = x.i[t][m]; }
        for (int t = 0; t < L; t++) for (int m = 0; m < 4; m++) { x.r[t][m] = br[HL::load(m, t)]; x.i[t][m] = bi[HL::load(m, t)]; }
        pass(x, 2, h); swap_bits(x, 4, 8);
        pass(x, 3, h);
        for (int t = 0; t < L; t++)
            for (int m = 0; m < 4; m++) {
                const int k = frequency(HP::key_lane(h, HL::plan_lane_d(t)) + HP::key_reg(m));
                CHECK((k & 1) == h, "a place of the other half\n");
                long double re = 0, im = 0;
                for (int j = 0; j < M; j++) {
                    const long double ang = 2 * pi * (long double)(((long long)j * (4 * k + 1)) % (4 * M)) / (4 * M);
                    re += ur[j] * cosl(ang) - ui[j] * sinl(ang);
                    im += ur[j] * sinl(ang) + ui[j] * cosl(ang);
                }
                keep_largest(worst, fabsl(re - x.r[t][m]));
                keep_largest(worst, fabsl(im - x.i[t][m]));
                spec_r[h][m * 64 + t] = x.r[t][m]; spec_i[h][m * 64 + t] = x.i[t][m];
            }
    }
    // 512 points of magnitude 64: a few hundred rounding errors of 2^-53 relative to sums of at most 2^15
    CHECK(worst < 1e-9L, "forward differs from the definition by %Lg\n", worst);

    double yr[2][2][128], yi[2][2][128];
    std::vector<int> used(512, 0);
    for (int h = 0; h < 2; h++)
        for (int k1 = 0; k1 < 2; k1++) {
            Lanes<2> x;
            for (int t = 0; t < L; t++)
                for (int m = 0; m < 2; m++) {
                    const int slot = QI::spectrum_slot(k1, t) + 64 * m;
                    x.r[t][m] = spec_r[h][slot]; x.i[t][m] = spec_i[h][slot];
                    used[256 * h + slot]++;
                    CHECK(QI::key_place(h, k1, t) + 256 * m == HP::key_lane(h, HL::plan_lane_d(slot & 63)) + HP::key_reg(slot >> 6),
                          "key place of lane %d\n", t);
                }
            const int bits[6] = {32, 8, 4, 2, 1, 16};
            for (int st = 8; st >= 2; st--) {
                for (int t = 0; t < L; t++) {
                    const int at = (1 << st) - 4 + (QI::node(h, k1, t) & ((1 << st) - 1));
                    CHECK(at >= 0 && at < QI::COUNT, "entry\n");
                    node_butterfly_inverse<false>(x.r[t][0], x.i[t][0], x.r[t][1], x.i[t][1], g_q[2 * at], g_q[2 * at + 1]);
                }
                if (st > 2) swap_bit(x, bits[8 - st], 0, 1);
            }
            for (int t = 0; t < L; t++)
                for (int m = 0; m < 2; m++) { yr[h][k1][QI::position(t) + 64 * m] = x.r[t][m]; yi[h][k1][QI::position(t) + 64 * m] = x.i[t][m]; }
        }
    for (int q = 0; q < 512; q++) CHECK(used[q] == 1, "slot %d read %d times\n", q, used[q]);
    long double back = 0;
    for (int j = 0; j < 128; j++) {
        double ar[2], ai[2], br[2], bi[2];
        for (int h = 0; h < 2; h++) {
            const CosTan w = HP::first_entry(h, 0);
            ar[h] = yr[h][0][j]; ai[h] = yi[h][0][j]; br[h] = yr[h][1][j]; bi[h] = yi[h][1][j];
            node_butterfly_inverse<false>(ar[h], ai[h], br[h], bi[h], w.c, w.t);
        }
        for (int m = 0; m < 2; m++) {
            const double *zr = m ? br : ar, *zi = m ? bi : ai;
            const double dr = zr[0] - zr[1], di = zi[0] - zi[1], f = std::sqrt(0.5) / 512;
            const int a = j + 128 * m, b = a + 256;
            for (long double e : {fabsl((zr[0] + zr[1]) / 512 - ur[a]), fabsl((zi[0] + zi[1]) / 512 - ui[a]),
                                  fabsl((dr + di) * f - ur[b]), fabsl((di - dr) * f - ui[b])})
                keep_largest(back, e);
        }
    }
    CHECK(back < 1e-10L, "inverse(forward(u)) differs from u by %Lg\n", back);
    std::printf("forward %Lg inverse %Lg failures %d\n", worst, back, failures);
    return failures != 0;
}
