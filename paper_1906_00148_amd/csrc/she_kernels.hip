// HIP kernels of the bootstrapped-gate path for gfx950 (MI355X).
//
// One circuit level of G independent gates runs as three launches:
//   k_lincomb       gate-specific TLWE linear combination + modulus switch to Z_2N
//   k_blind_rotate  n CMux steps per gate (decompose, forward transforms, pointwise
//                   products with the streamed spectral bootstrapping key, inverse
//                   transforms), then sample extraction and key-switch digit rounding
//   k_key_switch    subtraction of the selected key-switching rows
// (SHE, arXiv 1906.00148: Section 3.1 for the gates, Section 2 for bootstrapping; the
// construction itself is the cited TFHE gate bootstrapping.)
#include "negacyclic_fft.h"
#include "she_internal.h"
#include <algorithm>
#include <mutex>
#pragma clang fp contract(fast)

namespace she {

__device__ __forceinline__ uint32_t *ct_ptr(const CtSpace &cs, uint32_t id)
{
    return id < cs.cap ? cs.pool + (size_t)id * cs.stride : cs.temp + (size_t)(id - cs.cap) * cs.stride;
}

// ------------------------------------------------------------------------------------------
// Linear combination and modulus switch.  One block per gate.
// Pre-bootstrap sample = (0, off) + sa*ca + sb*cb, doubled for XOR/XNOR; every word is then
// rounded to the nearest multiple of 1/2N.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(128) void k_lincomb(CtSpace cs, const uint8_t *__restrict__ type,
                                                 const uint32_t *__restrict__ in0, const uint32_t *__restrict__ in1,
                                                 const uint32_t *__restrict__ in2, uint32_t n, uint32_t log2_2N,
                                                 uint16_t *__restrict__ bar, uint32_t bar_stride)
{
    const uint32_t g = blockIdx.x;
    const uint32_t ty = type[g];
    const uint32_t e = 1u << 29;
    const uint32_t rnd = 1u << (31 - log2_2N), sh = 32 - log2_2N;
    uint16_t *dst = bar + (size_t)g * bar_stride;
    if (ty >= SHE_MAJ3) {
        // three-input gate: s = +-ca +- cb +- cc has phase (2k-3)/8 for k true inputs; majority is the sign of s,
        // parity the sign of -2s (phase +1/4 for odd k, -1/4 for even k); no offset (in2 is non-null for these)
        const uint32_t m = ty - SHE_MAJ3;
        const bool parity = (m >> 3) != 0;
        const uint32_t *ca = ct_ptr(cs, in0[g]), *cb = ct_ptr(cs, in1[g]), *cc = ct_ptr(cs, in2[g]);
        for (uint32_t i = threadIdx.x; i <= n; i += blockDim.x) {
            const uint32_t a = ca[i], b = cb[i], c = cc[i];
            uint32_t x = ((m & 1) ? 0u - a : a) + ((m & 2) ? 0u - b : b) + ((m & 4) ? 0u - c : c);
            if (parity) x = 0u - 2u * x;
            dst[i] = (uint16_t)((x + rnd) >> sh);
        }
        return;
    }
    // sign of ca, sign of cb, offset, doubling
    uint32_t off = e; bool na = false, nb = false, dbl = false;
    switch (ty) {
    case SHE_AND:   off = 0u - e; break;
    case SHE_NAND:  off = e; na = nb = true; break;
    case SHE_OR:    off = e; break;
    case SHE_NOR:   off = 0u - e; na = nb = true; break;
    case SHE_XOR:   off = 2 * e; dbl = true; break;
    case SHE_XNOR:  off = 0u - 2 * e; na = nb = true; dbl = true; break;
    case SHE_ANDNY: off = 0u - e; na = true; break;
    case SHE_ANDYN: off = 0u - e; nb = true; break;
    case SHE_ORNY:  off = e; na = true; break;
    default:        off = e; nb = true; break;     // SHE_ORYN
    }
    const uint32_t *ca = ct_ptr(cs, in0[g]);
    const uint32_t *cb = ct_ptr(cs, in1[g]);
    for (uint32_t i = threadIdx.x; i <= n; i += blockDim.x) {
        uint32_t a = ca[i], b = cb[i];
        uint32_t x = (na ? 0u - a : a) + (nb ? 0u - b : b);
        if (dbl) x += x;
        if (i == n) x += off;
        dst[i] = (uint16_t)((x + rnd) >> sh);
    }
}

// ------------------------------------------------------------------------------------------
// Blind rotation.  One gate per L lanes; a wavefront never talks to another one.
// ------------------------------------------------------------------------------------------
constexpr int BR_WAVES = 4;     // measured: 2 and 8 wavefronts per workgroup are slower

// Where the rotations of MUXes leave their samples: those of a launch from `first` on, if it has any.
struct RawSamples {
    uint32_t *ext, first;
    __device__ __forceinline__ bool takes(uint32_t g) const { return ext && g >= first; }
    __device__ __forceinline__ uint32_t *row(uint32_t g, uint32_t N) const { return ext + (size_t)(g - first) * (N + 1); }
};

// LC: the gadget length when it is known at compile time (the loops over the 2 LC rows of a step are then unrolled:
// shifts and row offsets become constants, measured 1.2 % faster at l = 3 on alternating runs), 0 for any length.
template <class PL> struct WaveShared {               // the LDS arrays of one workgroup
    uint32_t acc[BR_WAVES * PL::GPW][2][PL::N];
    double2 xch[BR_WAVES * PL::GPW][PL::XSLOTS];
    double2 tw[TwTable<PL>::COUNT];
};

template <class PL, bool TRACK, int LC>
__device__ __forceinline__ void rotate_by_wavefront(
    uint32_t (*s_acc)[2][PL::N], double2 (*s_xch)[PL::XSLOTS], double2 *s_tw, uint32_t block,
    const uint16_t *__restrict__ bar, uint32_t bar_stride, uint32_t n, uint32_t l_arg, uint32_t bg_bit,
    const double2 *__restrict__ bk_hat, const double2 *__restrict__ tw_table, uint32_t ks_bits,
    uint32_t *__restrict__ ext_b, uint16_t *__restrict__ ksd, uint32_t gates, unsigned *round_err, const CtSpace &cs,
    const uint32_t *__restrict__ out_ids, RawSamples raw)
{
    constexpr int P = PL::P, L = PL::L, M = PL::M, N = PL::N, GPW = PL::GPW;
    const uint32_t l = LC ? (uint32_t)LC : l_arg;

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int sub = lane / L, t = lane % L;
    const int slot = wave * GPW + sub;
    const uint32_t g_raw = (block * BR_WAVES + wave) * GPW + sub;
    load_twiddles<PL>(s_tw, tw_table);                                    // the only workgroup barrier
    if ((block * BR_WAVES + wave) * GPW >= gates) return;               // whole wavefront idle
    const bool live = g_raw < gates;
    const uint32_t g = live ? g_raw : gates - 1;                          // idle lanes shadow the last gate

    LaneCtx<PL> lc;
    lc.init(t, s_xch[slot], s_tw);
    uint32_t(*acc)[N] = s_acc[slot];
    const uint16_t *mybar = bar + (size_t)g * bar_stride;

    // ACC = (0, X^(-bbar) * testv), testv = 1/8 on every coefficient
    {
        const uint32_t bbar = mybar[n];
        for (int j = t; j < N; j += L) {
            acc[0][j] = 0;
            acc[1][j] = (((uint32_t)j + bbar) & N) ? 0u - (1u << 29) : (1u << 29);
        }
    }
    wave_lds_fence();

    const uint32_t Bg = 1u << bg_bit, half_bg = Bg >> 1;
    uint32_t dec_off = 1u << (31 - l * bg_bit);
    uint32_t flip = 0;      // top bit of every digit field: field ^ top, read as signed, is field - Bg/2
    for (uint32_t p = 1; p <= l; p++) { dec_off += half_bg << (32 - p * bg_bit); flip |= half_bg << (32 - p * bg_bit); }
    float worst = 0.f;

    uint32_t abar_next = mybar[0];
    // spectra of the key row in use; row 0 of the next step is requested before the inverse transforms
    double2 bv[2][P];
    {
        const double2 *row = bk_hat + t;
#pragma unroll
        for (int o = 0; o < 2; o++)
#pragma unroll
            for (int k = 0; k < P; k++) bv[o][k] = row[(o * P + k) * L];
    }
    for (uint32_t i = 0; i < n; i++) {
        const uint32_t abar = abar_next;
        abar_next = mybar[i + 1];                                          // i+1 == n reads bbar: harmless

        double sr[2][P], si[2][P];                                         // spectra of the two output components
#pragma unroll
        for (int k = 0; k < P; k++) { sr[0][k] = si[0][k] = sr[1][k] = si[1][k] = 0.0; }

#pragma unroll(LC ? 2 : 1)
        for (int c = 0; c < 2; c++) {
            // D_c = X^abar * ACC_c - ACC_c at this lane's 2P coefficients
            uint32_t dlo[P], dhi[P];
#pragma unroll
            for (int m = 0; m < P; m++) {
                const uint32_t j0 = t + L * m, j1 = j0 + M;
                const uint32_t s0 = (j0 - abar) & (2 * N - 1), s1 = (j1 - abar) & (2 * N - 1);
                uint32_t v0 = acc[c][s0 & (N - 1)], v1 = acc[c][s1 & (N - 1)];
                v0 = (s0 & N) ? 0u - v0 : v0;
                v1 = (s1 & N) ? 0u - v1 : v1;
                // + dec_off: rounding and digit centring; ^ flip: turns each field into its signed digit
                dlo[m] = (v0 - acc[c][j0] + dec_off) ^ flip;
                dhi[m] = (v1 - acc[c][j1] + dec_off) ^ flip;
            }
#pragma unroll(LC ? LC : 1)
            for (uint32_t p = 0; p < l; p++) {
                const uint32_t sh = 32 - (p + 1) * bg_bit;
                const uint32_t r = c * l + p;
                double xr[P], xi[P];
#pragma unroll
                for (int m = 0; m < P; m++) {
                    // the builtin returns unsigned: go through int so that the conversion is signed
                    xr[m] = (double)(int)__builtin_amdgcn_sbfe(dlo[m], sh, bg_bit);
                    xi[m] = (double)(int)__builtin_amdgcn_sbfe(dhi[m], sh, bg_bit);
                }
                // a wavefront inside a transform issues ahead of one in the products or the decomposition: its LDS
                // round trips start sooner and the other wavefront's arithmetic fills them (measured: 1-2 %)
                __builtin_amdgcn_s_setprio(3);
                forward<PL>(lc, xr, xi);
                __builtin_amdgcn_s_setprio(0);
                __builtin_amdgcn_sched_barrier(0);     // keeps the products out of the transform's schedule (measured: +4%)
                // request the next row (of this step, or row 0 of the next one) register by register as the products
                // free them; after the last step this reads the last row once more, which is harmless
                const size_t nxt = std::min<size_t>((size_t)i * 2 * l + r + 1, (size_t)n * 2 * l - 1);
                const double2 *row = bk_hat + nxt * 2 * P * L + t;
#pragma unroll
                for (int o = 0; o < 2; o++) {
#pragma unroll
                    for (int k = 0; k < P; k++) {
                        const double2 b = bv[o][k];
                        // two fused multiply-adds per part (a += x*y - z*w would cost a multiply, an fma and an add)
                        sr[o][k] = __builtin_fma(-xi[k], b.y, __builtin_fma(xr[k], b.x, sr[o][k]));
                        si[o][k] = __builtin_fma(xi[k], b.x, __builtin_fma(xr[k], b.y, si[o][k]));
                        bv[o][k] = row[(o * P + k) * L];
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        {
            // both inverse transforms side by side through the one exchange buffer (measured: 21.0 -> 20.7 ms)
            double2 *const xch2[2] = {lc.xch, lc.xch};
            inverse_n<PL, 2, true>(lc, xch2, sr, si);
        }
#pragma unroll
        for (int o = 0; o < 2; o++) {
#pragma unroll
            for (int m = 0; m < P; m++) {
                const double vr = sr[o][m], vi = si[o][m];
                if (TRACK) {
                    worst = fmaxf(worst, (float)fabs(vr - rint(vr)));
                    worst = fmaxf(worst, (float)fabs(vi - rint(vi)));
                }
                // |v| < 2^51: adding 1.5*2^52 leaves round(v) mod 2^32 in the low word
                const uint32_t ir = (uint32_t)__double2loint(vr + 6755399441055744.0);
                const uint32_t ii = (uint32_t)__double2loint(vi + 6755399441055744.0);
                acc[o][t + L * m] += ir;
                acc[o][t + L * m + M] += ii;
            }
        }
        wave_lds_fence();
    }

    if (TRACK && round_err) atomicMax(round_err, __float_as_uint(worst));

    // sample extraction: a''_0 = A_0, a''_j = -A_{N-j}, b'' = B_0
    if (live && raw.takes(g)) {
        // a rotation of a MUX: the sample itself is kept, two of them are summed before the key switch
        uint32_t *dst = raw.row(g, N);
        for (int j = t; j < N; j += L) dst[j] = (j == 0) ? acc[0][0] : 0u - acc[0][N - j];
        if (t == 0) dst[N] = acc[1][0];
    } else if (live) {
        // keep the top ks_bits of each a'' rounded
        const uint32_t rnd = 1u << (31 - ks_bits), sh = 32 - ks_bits;
        uint16_t *dst = ksd + ((size_t)(g / KS_GROUP) * N) * KS_GROUP + (g % KS_GROUP);
        for (int j = t; j < N; j += L) {
            const uint32_t a = (j == 0) ? acc[0][0] : 0u - acc[0][N - j];
            dst[(size_t)j * KS_GROUP] = (uint16_t)((a + rnd) >> sh);
        }
        if (t == 0) ext_b[g] = acc[1][0];
        // the key switch subtracts its rows from (0, b''): leave that in the output slot
        if (out_ids) {
            uint32_t *o = ct_ptr(cs, out_ids[g]);
            const uint32_t body = acc[1][0];
            for (uint32_t c = t; c <= n; c += L) o[c] = (c == n) ? body : 0u;
        }
    }
}

template <class PL, bool TRACK, int LC>
__global__ __launch_bounds__(64 * BR_WAVES, 2) void k_blind_rotate(
    const uint16_t *__restrict__ bar, uint32_t bar_stride, uint32_t n, uint32_t l, uint32_t bg_bit,
    const double2 *__restrict__ bk_hat, const double2 *__restrict__ tw_table, uint32_t ks_bits,
    uint32_t *__restrict__ ext_b, uint16_t *__restrict__ ksd, uint32_t gates, unsigned *round_err, CtSpace cs,
    const uint32_t *__restrict__ out_ids, RawSamples raw)
{
    __shared__ uint32_t s_acc[BR_WAVES * PL::GPW][2][PL::N];
    __shared__ double2 s_xch[BR_WAVES * PL::GPW][PL::XSLOTS];
    __shared__ double2 s_tw[TwTable<PL>::COUNT];
    rotate_by_wavefront<PL, TRACK, LC>(s_acc, s_xch, s_tw, blockIdx.x, bar, bar_stride, n, l, bg_bit, bk_hat, tw_table,
                                       ks_bits, ext_b, ksd, gates, round_err, cs, out_ids, raw);
}

// ------------------------------------------------------------------------------------------
// Blind rotation of a small level on two wavefronts per gate, one or two gates per workgroup: at N = 1024 with l = 3 levels
// of more than three and at most four gates per compute unit, and two gates at a time k_blind_rotate_mixed's pairs
// (k_blind_rotate_wide and k_blind_rotate_quad have the smaller levels, k_blind_rotate_mixed the others), at other parameters
// levels of up to six (SHE_OPT_SPLIT_BELOW's default).
// A level of a few hundred gates leaves most SIMDs with one wavefront or none, and the time of
// the kernel above is then the latency of one wavefront's serial chain of 6 forward and 2
// inverse transforms per CMux.  Here wavefront c of a gate owns accumulator component c: it
// decomposes ACC_c, transforms its l digit polynomials, multiplies them with rows c*l..c*l+l-1
// of the key for both output components, hands the partial spectrum of the other component to
// its partner through LDS, and inverse-transforms its own component.  The chain per CMux is
// l forward transforms, one exchange and one inverse transform.  Results are bit-identical to
// k_blind_rotate's only up to FP64 summation order; both are exact after rounding.
// ------------------------------------------------------------------------------------------
// Workgroup barrier for LDS traffic only: earlier LDS operations of this wavefront are complete
// (they finish in issue order, the counter reaches zero when the last one has), global loads
// stay in flight.  The wait is written out: the one that the fence stands for has been seen to
// disappear where the barrier opens a loop whose entry has nothing outstanding, though the way
// round the loop has (stores of one step read by another wavefront before they had landed).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_waitcnt(0xC07F);                                     // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int largest_divisor_up_to(int v, int cap) { int d = cap < v ? cap : v; while (d > 1 && v % d) d--; return d < 1 ? 1 : d; }
// Key values in flight per wavefront of the split kernel.  With 16 it spills 21 registers at N = 1024 (36 in the mixed kernel),
// with 12 none: 700 / 900 / 1400 gates 4.45 / 5.78 / 7.85 ms with 16, 3.96 / 5.65 / 7.40 with 12, 4.00 / 5.68 / 7.47 with 8.
constexpr int SPLIT_KD = 12;
// LR > 0: the gadget has LR levels (l == LR) and a wavefront transforms its LR digit polynomials side by side
// (forward_pipelined), streaming the key rows through SPLIT_KD values in flight; LR == 0: any l, one at a time.
template <class PL, int GB> struct SplitShared {       // the LDS arrays of one workgroup
    uint32_t acc[2 * GB][PL::N];
    double2 xch[2 * GB][PL::XSLOTS];
    double2 tw[TwTable<PL>::COUNT];
};

template <class PL, bool TRACK, int GB, int LR>
__device__ __forceinline__ void rotate_by_component(
    SplitShared<PL, GB> &sh, uint32_t first_gate,
    const uint16_t *__restrict__ bar, uint32_t bar_stride, uint32_t n, uint32_t l, uint32_t bg_bit,
    const double2 *__restrict__ bk_hat, const double2 *__restrict__ tw_table, uint32_t ks_bits,
    uint32_t *__restrict__ ext_b, uint16_t *__restrict__ ksd, uint32_t gates, unsigned *round_err, const CtSpace &cs,
    const uint32_t *__restrict__ out_ids, RawSamples raw)
{
    constexpr int P = PL::P, L = PL::L, M = PL::M, N = PL::N;
    static_assert(PL::GPW == 1, "one transform per wavefront");
    auto &s_acc = sh.acc; auto &s_xch = sh.xch; auto &s_tw = sh.tw;

    const int wave = threadIdx.x >> 6, t = threadIdx.x & 63;
    const int c = wave & 1;                                               // component owned
    // a wavefront pair past the end shadows the last gate and stores nothing: it still meets every barrier
    const uint32_t g_raw = first_gate + (wave >> 1);
    const bool live = g_raw < gates;
    const uint32_t g = live ? g_raw : gates - 1;
    load_twiddles<PL>(s_tw, tw_table);

    LaneCtx<PL> lc;
    lc.init(t, s_xch[wave], s_tw);
    uint32_t *acc = s_acc[wave];
    const double2 *theirs = s_xch[wave ^ 1];
    const uint16_t *mybar = bar + (size_t)g * bar_stride;

    // ACC = (0, X^(-bbar) * testv), testv = 1/8 on every coefficient
    {
        const uint32_t bbar = mybar[n];
        for (int j = t; j < N; j += L) acc[j] = c == 0 ? 0u : ((((uint32_t)j + bbar) & N) ? 0u - (1u << 29) : (1u << 29));
    }
    wave_lds_fence();

    const uint32_t Bg = 1u << bg_bit, half_bg = Bg >> 1;
    uint32_t dec_off = 1u << (31 - l * bg_bit);
    uint32_t flip = 0;
    for (uint32_t p = 1; p <= l; p++) { dec_off += half_bg << (32 - p * bg_bit); flip |= half_bg << (32 - p * bg_bit); }
    float worst = 0.f;

    // spectra of the key row in use, own output component first
    const size_t row_elems = (size_t)2 * P * L;
    const int mine_off = c * P * L + t, other_off = (c ^ 1) * P * L + t;
    double2 bm[P], bo[P];
    if constexpr (LR == 0) {
        const double2 *row = bk_hat + (size_t)(c * l) * row_elems;
#pragma unroll
        for (int k = 0; k < P; k++) { bm[k] = row[mine_off + k * L]; bo[k] = row[other_off + k * L]; }
    }
    // LR > 0: key value j = (p*2 + o)*P + k of this component's LR rows sits at rows[j*L]
    // (KD divides NV, so that a value keeps its place in the ring from one step to the next)
    constexpr int NV = LR * 2 * P, KD = LR > 0 ? largest_divisor_up_to(NV, SPLIT_KD) : 1;
    double2 kv[KD];
    if constexpr (LR > 0) {
        const double2 *rows = bk_hat + (size_t)(c * LR) * row_elems + t;
#pragma unroll
        for (int j = 0; j < KD; j++) kv[j] = rows[j * L];
    }
    uint32_t abar_next = mybar[0];
    for (uint32_t i = 0; i < n; i++) {
        const uint32_t abar = abar_next;
        abar_next = mybar[i + 1];                                          // i+1 == n reads bbar: harmless

        double mr[P], mi[P], orr[P], oi[P];                                // partial spectra: own component, the other one
        if constexpr (LR == 0) {
#pragma unroll
            for (int k = 0; k < P; k++) { mr[k] = mi[k] = orr[k] = oi[k] = 0.0; }
        }

        // D_c = X^abar * ACC_c - ACC_c at this lane's 2P coefficients
        uint32_t dlo[P], dhi[P];
#pragma unroll
        for (int m = 0; m < P; m++) {
            const uint32_t j0 = t + L * m, j1 = j0 + M;
            const uint32_t s0 = (j0 - abar) & (2 * N - 1), s1 = (j1 - abar) & (2 * N - 1);
            uint32_t v0 = acc[s0 & (N - 1)], v1 = acc[s1 & (N - 1)];
            v0 = (s0 & N) ? 0u - v0 : v0;
            v1 = (s1 & N) ? 0u - v1 : v1;
            dlo[m] = (v0 - acc[j0] + dec_off) ^ flip;
            dhi[m] = (v1 - acc[j1] + dec_off) ^ flip;
        }
        if constexpr (LR > 0) {
            double xr[LR][P], xi[LR][P];
#pragma unroll
            for (int p = 0; p < LR; p++)
#pragma unroll
                for (int m = 0; m < P; m++) {
                    xr[p][m] = (double)(int)__builtin_amdgcn_sbfe(dlo[m], 32 - (p + 1) * bg_bit, bg_bit);
                    xi[p][m] = (double)(int)__builtin_amdgcn_sbfe(dhi[m], 32 - (p + 1) * bg_bit, bg_bit);
                }
            forward_pipelined<PL, LR>(lc, xr, xi);
            __builtin_amdgcn_sched_barrier(0);
            // this step's remaining key values, then the first KD of the next step (the last step's again at the end)
            const double2 *rows = bk_hat + ((size_t)i * 2 * LR + c * LR) * row_elems + t;
            const double2 *rows_next = bk_hat + ((size_t)std::min(i + 1, n - 1) * 2 * LR + c * LR) * row_elems + t;
#pragma unroll
            for (int j = 0; j < NV; j++) {
                const int p = j / (2 * P), o = (j / P) % 2, k = j % P;
                const double2 b = kv[j % KD];
                // output component o of the key row; o == c is this wavefront's own
                double &ar = (o == c) ? mr[k] : orr[k];
                double &ai = (o == c) ? mi[k] : oi[k];
                if (p == 0) {
                    ar = __builtin_fma(-xi[p][k], b.y, xr[p][k] * b.x);
                    ai = __builtin_fma(xi[p][k], b.x, xr[p][k] * b.y);
                } else {
                    ar = __builtin_fma(-xi[p][k], b.y, __builtin_fma(xr[p][k], b.x, ar));
                    ai = __builtin_fma(xi[p][k], b.x, __builtin_fma(xr[p][k], b.y, ai));
                }
                kv[j % KD] = (j + KD < NV) ? rows[(j + KD) * L] : rows_next[(j + KD - NV) * L];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        for (uint32_t p = 0; LR == 0 && p < l; p++) {
            const uint32_t sh = 32 - (p + 1) * bg_bit;
            double xr[P], xi[P];
#pragma unroll
            for (int m = 0; m < P; m++) {
                xr[m] = (double)(int)__builtin_amdgcn_sbfe(dlo[m], sh, bg_bit);
                xi[m] = (double)(int)__builtin_amdgcn_sbfe(dhi[m], sh, bg_bit);
            }
            forward<PL>(lc, xr, xi);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < P; k++) {
                mr[k] = __builtin_fma(-xi[k], bm[k].y, __builtin_fma(xr[k], bm[k].x, mr[k]));
                mi[k] = __builtin_fma(xi[k], bm[k].x, __builtin_fma(xr[k], bm[k].y, mi[k]));
                orr[k] = __builtin_fma(-xi[k], bo[k].y, __builtin_fma(xr[k], bo[k].x, orr[k]));
                oi[k] = __builtin_fma(xi[k], bo[k].x, __builtin_fma(xr[k], bo[k].y, oi[k]));
            }
            // next row of this component: same step, or the first of the next step (the last row again at the end)
            {
                const uint32_t ni = (p + 1 < l) ? i : std::min(i + 1, n - 1), np = (p + 1 < l) ? p + 1 : 0;
                const double2 *row = bk_hat + ((size_t)ni * 2 * l + c * l + np) * row_elems;
#pragma unroll
                for (int k = 0; k < P; k++) { bm[k] = row[mine_off + k * L]; bo[k] = row[other_off + k * L]; }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // hand the other component's partial spectrum to the partner, take the partner's for this one
        wave_lds_fence();
#pragma unroll
        for (int k = 0; k < P; k++) lc.xch[k * PL::XROW + t] = make_double2(orr[k], oi[k]);
        lds_barrier();
#pragma unroll
        for (int k = 0; k < P; k++) {
            const double2 v = theirs[k * PL::XROW + t];
            mr[k] += v.x; mi[k] += v.y;
        }
        lds_barrier();                                                      // the partner has read this buffer: free for the inverse
        inverse<PL>(lc, mr, mi);
#pragma unroll
        for (int m = 0; m < P; m++) {
            const double vr = mr[m], vi = mi[m];
            if (TRACK) {
                worst = fmaxf(worst, (float)fabs(vr - rint(vr)));
                worst = fmaxf(worst, (float)fabs(vi - rint(vi)));
            }
            acc[t + L * m] += (uint32_t)__double2loint(vr + 6755399441055744.0);
            acc[t + L * m + M] += (uint32_t)__double2loint(vi + 6755399441055744.0);
        }
        wave_lds_fence();
    }

    if (TRACK && round_err) atomicMax(round_err, __float_as_uint(worst));

    // sample extraction: wavefront 0 holds A (mask a''_0 = A_0, a''_j = -A_{N-j}), wavefront 1 holds B (body b'' = B_0)
    if (!live) return;
    if (raw.takes(g)) {
        uint32_t *dst = raw.row(g, N);
        if (c == 0) {
            for (int j = t; j < N; j += L) dst[j] = (j == 0) ? acc[0] : 0u - acc[N - j];
        } else if (t == 0) {
            dst[N] = acc[0];
        }
    } else if (c == 0) {
        const uint32_t rnd = 1u << (31 - ks_bits), sh = 32 - ks_bits;
        uint16_t *dst = ksd + ((size_t)(g / KS_GROUP) * N) * KS_GROUP + (g % KS_GROUP);
        for (int j = t; j < N; j += L) {
            const uint32_t a = (j == 0) ? acc[0] : 0u - acc[N - j];
            dst[(size_t)j * KS_GROUP] = (uint16_t)((a + rnd) >> sh);
        }
    } else {
        const uint32_t body = acc[0];
        if (t == 0) ext_b[g] = body;
        if (out_ids) {                       // the key switch subtracts its rows from (0, b'')
            uint32_t *o = ct_ptr(cs, out_ids[g]);
            for (uint32_t w = t; w <= n; w += L) o[w] = (w == n) ? body : 0u;
        }
    }
}

template <class PL, bool TRACK, int GB, int LR>
__global__ __launch_bounds__(128 * GB, 2) void k_blind_rotate_split(
    const uint16_t *__restrict__ bar, uint32_t bar_stride, uint32_t n, uint32_t l, uint32_t bg_bit,
    const double2 *__restrict__ bk_hat, const double2 *__restrict__ tw_table, uint32_t ks_bits,
    uint32_t *__restrict__ ext_b, uint16_t *__restrict__ ksd, uint32_t gates, unsigned *round_err, CtSpace cs,
    const uint32_t *__restrict__ out_ids, RawSamples raw)
{
    __shared__ SplitShared<PL, GB> sh;
    rotate_by_component<PL, TRACK, GB, LR>(sh, blockIdx.x * GB, bar, bar_stride, n, l, bg_bit, bk_hat, tw_table, ks_bits,
                                           ext_b, ksd, gates, round_err, cs, out_ids, raw);
}

// ------------------------------------------------------------------------------------------
// Blind rotation of a level of more than one and at most two gates per compute unit, and of parts of larger ones (in
// k_blind_rotate_mixed: a rest of at most one gate per compute unit beyond full rounds, and one gate per compute unit beside
// pairs): one gate per workgroup of four wavefronts (N = 1024, l = LR).  What bounds such a level
// is the length of one gate's chain of n CMuxes, so the chain is cut as far as the transforms allow without a wavefront
// waiting for another inside one.
// Wavefront (c, h) owns accumulator component c and half h of the spectrum (HalfLanes): it cuts the digits of all of
// D_c = X^abar ACC_c - ACC_c, runs the first stage of its LR transforms for half h only and then LR transforms of 256
// points, multiplies with rows c*LR.. of the key for both outputs, hands the other component's partial half spectrum to
// wavefront (c^1, h), transforms its own component's half back, swaps the result with wavefront (c, h^1) and finishes
// the last stage for the coefficients that it keeps in registers: those of the 256-blocks h and h + 2.
// Nobody reads the accumulator with computed addresses: its owner writes ACC - (decomposition offset) in place and
// X^abar ACC already rotated (8 computed addresses and signs per lane instead of 16), so D_c is one subtraction of two
// words at fixed offsets.
// A CMux takes a gate alone 3.5 us (8300 cycles): 600 FP64 instructions per wavefront at the 2.5 ns that a wavefront alone
// on its SIMD issues them, 190 integer ones, 260 for exchanges through the registers, and LDS traffic of the four
// wavefronts (24 stores and 33 loads of 1 KB each); they overlap little, since the wavefronts run in step.  Two gates on a
// compute unit take 5.4 us: the vector ALU is busy 72 % of it, and wavefronts wait to issue LDS instructions a tenth of it (a
// fifth with the last exchange through LDS as well).
// Measured at n = 630, ms per launch of 300 / 512 gates: 3.4 / 3.65 (3.45 / 3.85 with the last exchange through LDS as well)
// against 3.9 / 4.0 of k_blind_rotate_split; with a third gate per compute unit quads alone are slower (700 gates: 5.2 ms, three
// to a compute unit on 168 registers 5.1) than that kernel (4.9) and than k_blind_rotate_mixed's pair and quad (4.0).
// ------------------------------------------------------------------------------------------
struct QuadShared {
    uint32_t rot[2][HalfPlan::N], base[2][HalfPlan::N];
    double2 xch[4][HalfLanes::XSLOTS], hand[4][4 * HalfPlan::ROW];
    double2 tw[HalfPlan::COUNT];
};

template <bool TRACK, int LR>
__device__ __forceinline__ void rotate_by_quad(
    QuadShared &sh, uint32_t g,
    const uint16_t *__restrict__ bar, uint32_t bar_stride, uint32_t n, uint32_t bg_bit,
    const double2 *__restrict__ bk_hat, const double2 *__restrict__ half_table, uint32_t ks_bits,
    uint32_t *__restrict__ ext_b, uint16_t *__restrict__ ksd, unsigned *round_err, const CtSpace &cs,
    const uint32_t *__restrict__ out_ids, RawSamples raw)
{
    using HP = HalfPlan;
    constexpr int N = HP::N, L = HP::L;
    auto &s_rot = sh.rot; auto &s_base = sh.base; auto &s_xch = sh.xch; auto &s_hand = sh.hand; auto &s_tw = sh.tw;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t = threadIdx.x & 63;
    const int c = wave >> 1, h = wave & 1;
    for (int e = threadIdx.x; e < HP::COUNT; e += 256) s_tw[e] = half_table[e];
    __syncthreads();
    HalfLanes hl;
    hl.init(t, h, s_tw);
    double2 *const xch = s_xch[wave];
    const double2 *from_other = s_hand[wave ^ 2], *from_half = s_xch[wave ^ 1];
    const uint16_t *mybar = bar + (size_t)g * bar_stride;

    const uint32_t half_bg = 1u << (bg_bit - 1);
    uint32_t dec_off = 1u << (31 - LR * bg_bit);
    uint32_t flip = 0;      // top bit of every digit field: field ^ top, read as signed, is field - Bg/2
#pragma unroll
    for (int p = 1; p <= LR; p++) { dec_off += half_bg << (32 - p * bg_bit); flip |= half_bg << (32 - p * bg_bit); }
    float worst = 0.f;

    // own coefficients: v[m] at pos + 64 (4h + m), v[4 + m] at 512 more; ACC = (0, X^(-bbar) * testv)
    uint32_t v[8];
    const int pos = HalfLanes::position(t), own = pos + 256 * h;
    {
        const uint32_t bbar = mybar[n];
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const uint32_t j = own + 64 * (q & 3) + 512 * (q >> 2);
            v[q] = c == 0 ? 0u : (((j + bbar) & N) ? 0u - (1u << 29) : (1u << 29));
        }
    }
    auto publish = [&](uint32_t abar) {
        const uint32_t x0 = 4 * ((uint32_t)own + abar);
        char *const rot = reinterpret_cast<char *>(s_rot[c]);
#pragma unroll
        for (int q = 0; q < 8; q++) {
            s_base[c][own + 64 * (q & 3) + 512 * (q >> 2)] = v[q] - dec_off;
            const uint32_t x = x0 + 256 * (q & 3) + 2048 * (q >> 2);          // 4 * (j + abar): bit 12 is the sign
            const uint32_t neg = (uint32_t)__builtin_amdgcn_sbfe((int)x, 12, 1);
            *reinterpret_cast<uint32_t *>(rot + (x & (4 * N - 1))) = (v[q] ^ neg) - neg;
        }
    };

    // Key values of one output component (o = 0: the other one, o = 1: the own one) of a step, requested as the products
    // of the component before them free their registers.  (All 24 of a step held at once, requested at other points of
    // the step, is no faster: 2.2 to 2.4 ms.)
    const size_t row_elems = (size_t)2 * HP::M;
    const int key_lane = HP::key_lane(h, HalfLanes::plan_lane_d(t));
    double2 kv[LR][4];
    auto request = [&](uint32_t step, int o, int p) {
        const double2 *row = bk_hat + ((size_t)step * 2 * LR + c * LR + p) * row_elems + (o ? c : c ^ 1) * HP::M;
#pragma unroll
        for (int m = 0; m < 4; m++) kv[p][m] = row[HP::key_reg(m) + key_lane];
    };
#pragma unroll
    for (int p = 0; p < LR; p++) request(0, 0, p);
    publish(mybar[0]);
    uint32_t abar_next = mybar[1];                                            // n == 1 reads bbar: harmless
    const double cs1 = h ? -0.70710678118654752440 : 0.70710678118654752440; // +-cos(pi/4) of the first stage
    CosTan eb[2], ec[2], ed[2];
    hl.entries<1>(eb); hl.entries<2>(ec); hl.entries<3>(ed);
    for (uint32_t i = 0; i < n; i++) {
        lds_barrier();                                                        // both arrays of both components are written
        uint32_t dlo[8], dhi[8];
#pragma unroll
        for (int m = 0; m < 8; m++) {
            dlo[m] = (s_rot[c][pos + L * m] - s_base[c][pos + L * m]) ^ flip;
            dhi[m] = (s_rot[c][pos + L * m + 512] - s_base[c][pos + L * m + 512]) ^ flip;
        }
        double xr[LR][4], xi[LR][4];
        double mr[4], mi[4], orr[4], oi[4];                                   // half spectra: own component, the other one
        // first stage: a +- exp(i pi/4) b with a, b the positions 64 m + pos and 64 m + pos + 256; (1 + i) b in integers
        auto head = [&](int p) {
#pragma unroll
            for (int m = 0; m < 4; m++) {
                const uint32_t sh = 32 - (p + 1) * bg_bit;
                const int ar = (int)__builtin_amdgcn_sbfe((int)dlo[m], sh, bg_bit), ai = (int)__builtin_amdgcn_sbfe((int)dhi[m], sh, bg_bit);
                const int br = (int)__builtin_amdgcn_sbfe((int)dlo[m + 4], sh, bg_bit), bi = (int)__builtin_amdgcn_sbfe((int)dhi[m + 4], sh, bg_bit);
                xr[p][m] = __builtin_fma(cs1, (double)(br - bi), (double)ar);
                xi[p][m] = __builtin_fma(cs1, (double)(br + bi), (double)ai);
            }
            hl.pass_a(xr[p], xi[p]);
        };
        auto products = [&](int p, double (&ar)[4], double (&ai)[4]) {
#pragma unroll
            for (int m = 0; m < 4; m++) {
                const double2 b = kv[p][m];
                if (p == 0) {
                    ar[m] = __builtin_fma(-xi[p][m], b.y, xr[p][m] * b.x);
                    ai[m] = __builtin_fma(xi[p][m], b.x, xr[p][m] * b.y);
                } else {
                    ar[m] = __builtin_fma(-xi[p][m], b.y, __builtin_fma(xr[p][m], b.x, ar[m]));
                    ai[m] = __builtin_fma(xi[p][m], b.x, __builtin_fma(xr[p][m], b.y, ai[m]));
                }
            }
        };
        // The exchanges of one polynomial run beside the arithmetic of the others: with the passes of all of them side by
        // side the four wavefronts, which run in step, wait for the LDS pipe together (2.59 against 2.49 ms).
#pragma unroll
        for (int s = 0; s < LR + 2; s++) {
            if (s < LR) { head(s); hl.pass_b(xch, xr[s], xi[s], eb); }
            if (s >= 1 && s - 1 < LR) hl.pass_c(xr[s - 1], xi[s - 1], ec);
            if (s >= 2) {
                node_pass<4>(xr[s - 2], xi[s - 2], ed);
                products(s - 2, orr, oi);
                request(i, 1, s - 2);
            }
        }
#pragma unroll
        for (int m = 0; m < 4; m++) s_hand[wave][m * HP::ROW + t] = make_double2(orr[m], oi[m]);
        // the own component's products run while the hand-over is under way; then the next step's first values are
        // requested (the last step's again at the end)
#pragma unroll
        for (int p = 0; p < LR; p++) { products(p, mr, mi); request(std::min(i + 1, n - 1), 0, p); }
        lds_barrier();
#pragma unroll
        for (int m = 0; m < 4; m++) { const double2 w = from_other[m * HP::ROW + t]; mr[m] += w.x; mi[m] += w.y; }
        hl.inverse(xch, mr, mi, eb, ec, ed);
        // the exchange buffer is free again; the partner has read it before it meets the barrier at the loop's top
        wave_lds_fence();
#pragma unroll
        for (int m = 0; m < 4; m++) xch[m * HP::ROW + t] = make_double2(mr[m], mi[m]);
        lds_barrier();
        // last stage: (y0 + y1) / 512 for half 0, conj(w) (y0 - y1) / 512 for half 1; adding 1.5*2^52 leaves the rounded
        // value modulo 2^32 in the low word
        constexpr double magic = 6755399441055744.0, scale = 1.0 / 512, rot = 0.70710678118654752440 / 512;
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const double2 w = from_half[m * HP::ROW + t];
            double re, im, f;
            if (h == 0) {
                re = mr[m] + w.x; im = mi[m] + w.y; f = scale;
            } else {
                const double dr = w.x - mr[m], di = w.y - mi[m];
                re = dr + di; im = di - dr; f = rot;
            }
            if (TRACK) {
                worst = fmaxf(worst, (float)fabs(re * f - rint(re * f)));
                worst = fmaxf(worst, (float)fabs(im * f - rint(im * f)));
            }
            v[m] += (uint32_t)__double2loint(__builtin_fma(re, f, magic));
            v[4 + m] += (uint32_t)__double2loint(__builtin_fma(im, f, magic));
        }
        publish(abar_next);
        abar_next = mybar[std::min(i + 2, n)];
    }
    if (TRACK && round_err) atomicMax(round_err, __float_as_uint(worst));

    // sample extraction by the whole workgroup: a''_0 = A_0, a''_j = -A_{N-j}, b'' = B_0
    lds_barrier();
    const uint32_t body = s_base[1][0] + dec_off;
    if (raw.takes(g)) {
        uint32_t *dst = raw.row(g, N);
        for (int j = threadIdx.x; j < N; j += 256) dst[j] = (j == 0) ? s_base[0][0] + dec_off : 0u - (s_base[0][N - j] + dec_off);
        if (threadIdx.x == 0) dst[N] = body;
    } else {
        const uint32_t rnd = 1u << (31 - ks_bits), sh = 32 - ks_bits;
        uint16_t *dst = ksd + ((size_t)(g / KS_GROUP) * N) * KS_GROUP + (g % KS_GROUP);
        for (int j = threadIdx.x; j < N; j += 256) {
            const uint32_t a = (j == 0) ? s_base[0][0] + dec_off : 0u - (s_base[0][N - j] + dec_off);
            dst[(size_t)j * KS_GROUP] = (uint16_t)((a + rnd) >> sh);
        }
        if (threadIdx.x == 0) ext_b[g] = body;
        if (out_ids) {                       // the key switch subtracts its rows from (0, b'')
            uint32_t *o = ct_ptr(cs, out_ids[g]);
            for (uint32_t w = threadIdx.x; w <= n; w += 256) o[w] = (w == n) ? body : 0u;
        }
    }
}

template <bool TRACK, int LR>
__global__ __launch_bounds__(256, 2) void k_blind_rotate_quad(
    const uint16_t *__restrict__ bar, uint32_t bar_stride, uint32_t n, uint32_t bg_bit,
    const double2 *__restrict__ bk_hat, const double2 *__restrict__ half_table, uint32_t ks_bits,
    uint32_t *__restrict__ ext_b, uint16_t *__restrict__ ksd, unsigned *round_err, CtSpace cs,
    const uint32_t *__restrict__ out_ids, RawSamples raw)
{
    __shared__ QuadShared sh;
    rotate_by_quad<TRACK, LR>(sh, blockIdx.x, bar, bar_stride, n, bg_bit, bk_hat, half_table, ks_bits, ext_b, ksd, round_err,
                              cs, out_ids, raw);
}

// ------------------------------------------------------------------------------------------
// Blind rotation of a level of at most one gate per compute unit: one gate per workgroup of twelve wavefronts (N = 1024,
// l = 3), three on a SIMD, so that one's LDS round trips and dependent FP64 instructions are filled by the others.
// Wavefront (p, c, h) transforms digit p of D_c = X^abar ACC_c - ACC_c for half h of the spectrum and leaves it in LDS.
// After a barrier the eight with p < 2 form output component c's quarter (h, k1 = p) from all 2 l rows, read a few values
// ahead of the products, and transform it back (QuarterInverse); after a second barrier the eight with p > 0 join the
// quarters, keep the accumulator (four coefficients per lane) and publish ACC and X^abar ACC for the next step.
// The key: 96 KB per step and compute unit enter through its one path of 64 bytes a clock, 1500 cycles of a step's 6000,
// and a wavefront that issues loads faster than that stands still.  So a step's twelve values per multiplying wavefront wait
// in registers, requested by one half of them while the others publish and by the other half at the head of the next
// transform; it matters less so, too, whether the key comes from HBM or from the Infinity Cache.
// Cycles of a step, 6300 in all: transforms 3300 (three wavefronts on a SIMD with 270 vector instructions each, 120 of them
// FP64, 48 exchanges through the registers), products 700, inverse 700, joining and publishing 850, barriers.  The vector
// ALU is busy 80 % of them, the LDS pipe 43 %; a sixth of the LDS cycles are bank conflicts (the store to y puts sixteen
// neighbouring lanes on eight slots modulo 16, and the 8-byte halves of base lie 16 bytes apart).
// Measured at n = 630, ms per rotation of 1 / 83 / 250 / 256 gates: 1.66 / 1.68 / 1.72 / 1.74 with the key in the Infinity
// Cache, 1.66 / 1.69 / 1.75 / 1.83 with the key in HBM; k_blind_rotate_quad takes 2.26 / 2.26 / 2.30 / 2.27 and 2.60 / 2.42 /
// 2.41 / 2.41.  (That is at 2.4 GHz; where the card lowers its clock to 2.0, 250 gates take 2.0 to 2.1 ms.)  With the inverse
// transforms in four wavefronts, a half each, it was 6 % slower; eight wavefronts in all, four of them with two digits, take
// as long as the four of k_blind_rotate_quad.  A register more than there are costs 500 cycles of every step where the wait
// for it is on the way; another order of the wavefronts' priorities, or the second half of the key requested any later, 2 to
// 12 %.
// With more than one gate per compute unit a second workgroup does not fit (162 registers x 12), two rounds take longer
// than k_blind_rotate_quad's one (3.7 against 3.5 ms), and so do pairs of gates that share the key values (3.8).
// ------------------------------------------------------------------------------------------
// (What is addressed by lane alone first: an LDS instruction's own offset reaches 64 KB, so all but the last of the twelve
// exchange buffers.  Those with exclusive-or slots of 256 in place of k_blind_rotate_quad's rows of 65: 83 / 160 / 250 gates
// 1.671 / 1.674 / 1.729 ms against 1.679 / 1.684 / 1.730.)
struct WideShared {
    uint32_t rot[2][HalfPlan::N];                               // X^abar ACC, plain order
    uint4 base[2][2][2][64];                                       // ACC - offset: [component][block of 256][upper 512][lane], word 2u + m: + 64u + 128m
    double2 y[2][2][2][128];                                       // [component][half][quarter]: transformed back
    double2 xch[2][3][2][HalfLanes::XSLOTS];                       // [component][digit][half]: exchange, then the half spectrum
};

// A launch fills the compute units that its gates leave idle with workgroups that read the key once, side by side from its
// beginning, so that the gates, which have room for one step's values only, find them in the Infinity Cache.  A reader takes
// 64 bytes a clock, 150 GB/s, four times the 37 GB/s (96 KB per 2.6 us) at which the gates go through the key, so that a few
// are enough, and with a gate on every compute unit there is none.  Key in HBM, ms for 1 / 83 / 250 gates with no reader, one,
// four, and all: 1.91 / 1.82 / 1.82, 1.73 / 1.71 / 1.73, 1.66 / 1.69 / 1.71, 1.66 / 1.69 / 1.70; 255 gates 1.82 and with their
// one reader 1.73; 256 gates 1.83.  Key in the Infinity Cache: no difference.  A key larger than that cache (402 MB, n = 4096):
// 12.4 / 11.7 / 11.8, 12.0 / 11.5 / 11.6, 12.1 / 11.6 / 11.6, 12.3 / 11.7 / 11.7 ms, so it needs no rule of its own.  Work of
// other streams on the chip is held up no longer than by the gates alone (0 and 255 readers measured alike).
// Touching lines some steps ahead from the gates' own workgroups is no substitute: a compute unit's loads return in order, so
// that the touches hold up the values behind them (one gate: 2.28 ms).
__device__ __forceinline__ void read_ahead(const double2 *__restrict__ key, size_t elems, uint32_t worker, uint32_t workers)
{
    constexpr int IN_FLIGHT = 8;
    const size_t stride = (size_t)workers * blockDim.x;
    for (size_t at = (size_t)worker * blockDim.x + threadIdx.x; at < elems; at += IN_FLIGHT * stride) {
        double2 v[IN_FLIGHT];
#pragma unroll
        for (int q = 0; q < IN_FLIGHT; q++) v[q] = key[std::min(at + q * stride, elems - 1)];
#pragma unroll
        for (int q = 0; q < IN_FLIGHT; q++) asm volatile("" ::"v"(v[q].x), "v"(v[q].y));
    }
}

template <bool TRACK>
__global__ __launch_bounds__(768, 3) void k_blind_rotate_wide(
    const uint16_t *__restrict__ bar, uint32_t bar_stride, uint32_t n, uint32_t bg_bit,
    const double2 *__restrict__ bk_hat, const double2 *__restrict__ half_table, uint32_t ks_bits,
    uint32_t *__restrict__ ext_b, uint16_t *__restrict__ ksd, uint32_t gates, unsigned *round_err, CtSpace cs,
    const uint32_t *__restrict__ out_ids, RawSamples raw)
{
    using HP = HalfPlan;
    constexpr int N = HP::N, L = HP::L, LR = 3, THREADS = 768;
    __shared__ WideShared sh;
    const uint32_t g = blockIdx.x;
    if (g >= gates) {
        read_ahead(bk_hat, (size_t)n * 2 * LR * 2 * HP::M, g - gates, gridDim.x - gates);
        return;
    }
    uint32_t *const raw_row = raw.takes(g) ? raw.row(g, N) : nullptr;         // (decided at the end: + 0.5 % for one gate)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t = threadIdx.x & 63;
    const int p = wave >> 2, c = (wave >> 1) & 1, h = wave & 1;
    HalfLanes hl;
    hl.init(t, h, half_table);
    const uint16_t *mybar = bar + (size_t)g * bar_stride;

    const uint32_t half_bg = 1u << (bg_bit - 1);
    uint32_t dec_off = 1u << (31 - LR * bg_bit);
    uint32_t flip = 0;      // top bit of every digit field: field ^ top, read as signed, is field - Bg/2
#pragma unroll
    for (int q = 1; q <= LR; q++) { dec_off += half_bg << (32 - q * bg_bit); flip |= half_bg << (32 - q * bg_bit); }
    const uint32_t digit_sh = 32 - (p + 1) * bg_bit;
    float worst = 0.f;
    const double cs1 = h ? -0.70710678118654752440 : 0.70710678118654752440; // +-cos(pi/4) of the first stage
    CosTan eb[2], ec[2], ed[2];
    hl.entries<1>(eb); hl.entries<2>(ec); hl.entries<3>(ed);

    // Coefficients kept by a wavefront with p > 0: v[m] at pos + 64u + 128m + 256h, u = p - 1, v[2 + m] at 512 more.
    uint32_t v[4];
    const int u = p - 1, pos = HalfLanes::position(t), own = pos + 64 * u + 256 * h;
    auto publish = [&](uint32_t abar) {
        const uint32_t x0 = 4 * ((uint32_t)own + abar);
        char *const rot = reinterpret_cast<char *>(sh.rot[c]);
#pragma unroll
        for (int q = 0; q < 2; q++)
            reinterpret_cast<uint2 *>(&sh.base[c][h][q][t])[u] = make_uint2(v[2 * q] - dec_off, v[2 * q + 1] - dec_off);
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const uint32_t x = x0 + 512 * (q & 1) + 2048 * (q >> 1);          // 4 * (j + abar): bit 12 is the sign
            const uint32_t neg = (uint32_t)__builtin_amdgcn_sbfe((int)x, 12, 1);
            *reinterpret_cast<uint32_t *>(rot + (x & (4 * N - 1))) = (v[q] ^ neg) - neg;
        }
    };
    // digit p of D_c, transformed for half h
    auto transform = [&]() {
        uint32_t dlo[8], dhi[8];
#pragma unroll
        for (int b = 0; b < 2; b++) {
            const uint4 lo = sh.base[c][b][0][t], hi = sh.base[c][b][1][t];
            const uint32_t l4[4] = {lo.x, lo.z, lo.y, lo.w}, h4[4] = {hi.x, hi.z, hi.y, hi.w};
#pragma unroll
            for (int m = 0; m < 4; m++) {
                dlo[4 * b + m] = (sh.rot[c][pos + L * (4 * b + m)] - l4[m]) ^ flip;
                dhi[4 * b + m] = (sh.rot[c][pos + L * (4 * b + m) + 512] - h4[m]) ^ flip;
            }
        }
        double xr[4], xi[4];
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const int ar = (int)__builtin_amdgcn_sbfe((int)dlo[m], digit_sh, bg_bit), ai = (int)__builtin_amdgcn_sbfe((int)dhi[m], digit_sh, bg_bit);
            const int br = (int)__builtin_amdgcn_sbfe((int)dlo[m + 4], digit_sh, bg_bit), bi = (int)__builtin_amdgcn_sbfe((int)dhi[m + 4], digit_sh, bg_bit);
            xr[m] = __builtin_fma(cs1, (double)(br - bi), (double)ar);
            xi[m] = __builtin_fma(cs1, (double)(br + bi), (double)ai);
        }
        double2 *const xch = sh.xch[c][p][h];
        hl.pass_a(xr, xi);
        hl.pass_b(xch, xr, xi, eb);
        hl.pass_c(xr, xi, ec);
        node_pass<4>(xr, xi, ed);
        wave_lds_fence();
#pragma unroll
        for (int m = 0; m < 4; m++) xch[L * m + t] = make_double2(xr[m], xi[m]);
    };
    // The last two stages for the positions pos + 64u and 128 more of block h; adding 1.5*2^52 leaves the rounded value
    // modulo 2^32 in the low word.
    auto finish = [&]() {
        constexpr double magic = 6755399441055744.0, scale = 1.0 / 512, rot = 0.70710678118654752440 / 512;
        const double sign = h ? -1.0 : 1.0, turn = h ? 1.0 : 0.0, f = h ? rot : scale;
        double ar[2], ai[2], br[2], bi[2];                                      // of half 0 and half 1: positions without and with 128
#pragma unroll
        for (int e = 0; e < 2; e++) {
            const double2 y0 = sh.y[c][e][0][64 * u + pos], y1 = sh.y[c][e][1][64 * u + pos];
            const CosTan w = HP::first_entry(e, 0);
            ar[e] = y0.x; ai[e] = y0.y; br[e] = y1.x; bi[e] = y1.y;
            node_butterfly_inverse<false>(ar[e], ai[e], br[e], bi[e], w.c, w.t);
        }
#pragma unroll
        for (int m = 0; m < 2; m++) {
            const double(&zr)[2] = m ? br : ar, (&zi)[2] = m ? bi : ai;
            const double sr = __builtin_fma(sign, zr[1], zr[0]), si = __builtin_fma(sign, zi[1], zi[0]);
            const double re = __builtin_fma(turn, si, sr), im = __builtin_fma(-turn, sr, si);
            if (TRACK) {
                worst = fmaxf(worst, (float)fabs(re * f - rint(re * f)));
                worst = fmaxf(worst, (float)fabs(im * f - rint(im * f)));
            }
            v[m] += (uint32_t)__double2loint(__builtin_fma(re, f, magic));
            v[2 + m] += (uint32_t)__double2loint(__builtin_fma(im, f, magic));
        }
    };

    // The key values of output component c at this wavefront's quarter, all 2 LR rows.
    double2 kv[2 * LR][2];
    const double2 *key = bk_hat + c * HP::M + QuarterInverse::key_place(h, p & 1, t);
    auto request = [&](uint32_t step) {
#pragma unroll
        for (int r = 0; r < 2 * LR; r++) {
            const double2 *row = key + ((size_t)step * 2 * LR + r) * 2 * HP::M;
#pragma unroll
            for (int m = 0; m < 2; m++) kv[r][m] = row[256 * m];
        }
    };
    QuarterInverse qi;
    const int slot = QuarterInverse::spectrum_slot(p & 1, t);
    if (p < 2) qi.init(h, p, t, half_table + HP::COUNT);
    if (p == 0) request(0);
    if (p > 0) {
        // ACC = (0, X^(-bbar) * testv)
        const uint32_t bbar = mybar[n];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const uint32_t j = own + 128 * (q & 1) + 512 * (q >> 1);
            v[q] = c == 0 ? 0u : (((j + bbar) & N) ? 0u - (1u << 29) : (1u << 29));
        }
        publish(mybar[0]);
    }
    for (uint32_t i = 0; i < n; i++) {
        const uint32_t abar_next = mybar[i + 1];                                  // i + 1 == n reads bbar: harmless
        lds_barrier();
        if (p == 1) request(i);
        __builtin_amdgcn_sched_barrier(0);
        transform();
        lds_barrier();
        if (p < 2) {
            // the rows' spectra are read AHEAD values ahead of the products
            constexpr int AHEAD = 6, VALUES = 4 * LR;
            double2 x[AHEAD];
            double mr[2], mi[2];
            auto value = [&](int q) { return sh.xch[q / 2 / LR][q / 2 % LR][h][slot + 64 * (q % 2)]; };
#pragma unroll
            for (int q = 0; q < AHEAD; q++) x[q] = value(q);
#pragma unroll
            for (int q = 0; q < VALUES; q++) {
                const int m = q % 2;
                const double2 w = x[q % AHEAD], b = kv[q / 2][m];
                if (q + AHEAD < VALUES) x[q % AHEAD] = value(q + AHEAD);
                if (q < 2) {
                    mr[m] = __builtin_fma(-w.y, b.y, w.x * b.x);
                    mi[m] = __builtin_fma(w.y, b.x, w.x * b.y);
                } else {
                    mr[m] = __builtin_fma(-w.y, b.y, __builtin_fma(w.x, b.x, mr[m]));
                    mi[m] = __builtin_fma(w.y, b.x, __builtin_fma(w.x, b.y, mi[m]));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            qi.run(mr, mi);
#pragma unroll
            for (int m = 0; m < 2; m++) sh.y[c][h][p][QuarterInverse::position(t) + 64 * m] = make_double2(mr[m], mi[m]);
        }
        lds_barrier();
        if (p == 0) {
            request(std::min(i + 1, n - 1));                                      // the last step's again at the end
        } else {
            finish();
            publish(abar_next);
        }
    }
    if (TRACK && p && round_err) atomicMax(round_err, __float_as_uint(worst));
    lds_barrier();

    // sample extraction by the whole workgroup: a''_0 = A_0, a''_j = -A_{N-j}, b'' = B_0
    auto word = [&](int comp, int j) {
        const uint32_t *w = reinterpret_cast<const uint32_t *>(sh.base[comp]);
        return w[((((j >> 8) & 1) * 2 + (j >> 9)) * 64 + HalfLanes::position(j & 63)) * 4 + 2 * ((j >> 6) & 1) + ((j >> 7) & 1)] + dec_off;
    };
    const uint32_t body = word(1, 0);
    if (raw_row) {
        uint32_t *dst = raw_row;
        for (int j = threadIdx.x; j < N; j += THREADS) dst[j] = (j == 0) ? word(0, 0) : 0u - word(0, N - j);
        if (threadIdx.x == 0) dst[N] = body;
    } else {
        const uint32_t rnd = 1u << (31 - ks_bits), sft = 32 - ks_bits;
        uint16_t *dst = ksd + ((size_t)(g / KS_GROUP) * N) * KS_GROUP + (g % KS_GROUP);
        for (int j = threadIdx.x; j < N; j += THREADS) {
            const uint32_t a = (j == 0) ? word(0, 0) : 0u - word(0, N - j);
            dst[(size_t)j * KS_GROUP] = (uint16_t)((a + rnd) >> sft);
        }
        if (threadIdx.x == 0) ext_b[g] = body;
        if (out_ids) {                       // the key switch subtracts its rows from (0, b'')
            uint32_t *o = ct_ptr(cs, out_ids[g]);
            for (uint32_t w = threadIdx.x; w <= n; w += THREADS) o[w] = (w == n) ? body : 0u;
        }
    }
}

// Three forms in one launch, in the order of mixed_blocks: workgroups of four gates on a wavefront each, of two gates on two
// wavefronts each, of a single gate on four.
// A level of gates on a wavefront each takes whole rounds: with one gate more than a multiple of four per compute unit, one
// more workgroup sits on a few compute units for as long as a full round does (its wavefronts run 630 CMuxes of 10 us alone,
// whatever else is idle).  Here the rest beyond full rounds runs its 630 CMuxes in 3.6 us (quad) or 6 us (pair) each, beside
// the wavefronts of the last round that the hardware let fall behind (of two on a SIMD the older one goes first: 6.9 ms
// against 10.7).  A level of more than two and at most three gates per compute unit has a pair and a quad on each: eight
// wavefronts, two on every SIMD, where k_blind_rotate_split's six leave two SIMDs with one.
// Measured at n = 630 on 256 compute units, ms, on one box per line:
//   gates on a wavefront each, or k_blind_rotate_split up to 1536, against rounds and quads: 1100 gates 8.4 / 6.2, 1280 8.4 /
//   7.0, 2100 16.1 / 12.3, 2304 16.1 / 12.1, 3300 20.2 / 16.0, 4352 25.3 / 21.0;
//   a rest of up to two gates per compute unit, quads against pairs: 1300 gates 8.8 / 7.2, 1536 8.5 / 7.65, 2400 13.9 / 13.8,
//   2560 13.8 / 13.7, 3584 19.4 / 17.7, 4608 22.8 / 22.6, 5600 28.0 / 27.0;
//   up to three, as before (k_blind_rotate_split, or wavefronts) against a pair and a quad each: 514 gates 4.94 / 3.95, 768
//   4.93 / 4.00, 2700 16.0 / 14.5, 3840 20.1 / 19.4, 4700 24.9 / 23.6, 13001 65.2 / 64.4.
// A rest of more than three gates per compute unit gains nothing (3900: 20.1 / 21.5).
template <bool TRACK, int LR, bool PAIRS>
__global__ __launch_bounds__(256, 2) void k_blind_rotate_mixed(
    const uint16_t *__restrict__ bar, uint32_t bar_stride, uint32_t n, uint32_t bg_bit,
    const double2 *__restrict__ bk_hat, const double2 *__restrict__ tw_table, const double2 *__restrict__ half_table,
    uint32_t ks_bits, uint32_t *__restrict__ ext_b, uint16_t *__restrict__ ksd, uint32_t gates, MixedBlocks blocks,
    unsigned *round_err, CtSpace cs, const uint32_t *__restrict__ out_ids, RawSamples raw)
{
    using PL = Plan<3, 3>;
    static_assert(PL::N == HalfPlan::N && PL::GPW == 1 && BR_WAVES == 4, "all forms on 256 threads at the same ring degree");
    __shared__ union { WaveShared<PL> wave; SplitShared<PL, 2> pair; QuadShared quad; } sh;
    const uint32_t first_pair = blocks.waves * BR_WAVES, first_quad = gates - blocks.quads, b = blockIdx.x;
    if (b < blocks.waves)
        rotate_by_wavefront<PL, TRACK, LR>(sh.wave.acc, sh.wave.xch, sh.wave.tw, b, bar, bar_stride, n, LR, bg_bit, bk_hat,
                                           tw_table, ks_bits, ext_b, ksd, first_pair, round_err, cs, out_ids, raw);
    else if (PAIRS && b < blocks.waves + blocks.pairs)
        rotate_by_component<PL, TRACK, 2, LR>(sh.pair, first_pair + 2 * (b - blocks.waves), bar, bar_stride, n, LR, bg_bit,
                                              bk_hat, tw_table, ks_bits, ext_b, ksd, first_quad, round_err, cs, out_ids, raw);
    else
        rotate_by_quad<TRACK, LR>(sh.quad, first_quad + (b - blocks.waves - blocks.pairs), bar, bar_stride, n, bg_bit, bk_hat,
                                  half_table, ks_bits, ext_b, ksd, round_err, cs, out_ids, raw);
}

// Second half of a native MUX: the two rotations' samples are added, 1/8 goes on the body, and the
// sum is prepared for the key switch exactly as the blind rotation's epilogue prepares a gate.
__global__ __launch_bounds__(256) void k_mux_combine(const uint32_t *__restrict__ raw_ext, uint32_t N, uint32_t n,
                                                     uint32_t ks_bits, uint32_t *__restrict__ ext_b,
                                                     uint16_t *__restrict__ ksd, CtSpace cs,
                                                     const uint32_t *__restrict__ out_ids, uint32_t first)
{
    const uint32_t *e1 = raw_ext + (size_t)(2 * blockIdx.x) * (N + 1), *e0 = e1 + (N + 1);
    const uint32_t g = first + blockIdx.x;                       // its place in the level, behind the `first` gates
    const uint32_t rnd = 1u << (31 - ks_bits), sh = 32 - ks_bits;
    uint16_t *dst = ksd + ((size_t)(g / KS_GROUP) * N) * KS_GROUP + (g % KS_GROUP);
    for (uint32_t j = threadIdx.x; j < N; j += blockDim.x)
        dst[(size_t)j * KS_GROUP] = (uint16_t)((e1[j] + e0[j] + rnd) >> sh);
    const uint32_t body = e1[N] + e0[N] + (1u << 29);
    if (threadIdx.x == 0) ext_b[g] = body;
    if (out_ids) {
        uint32_t *o = ct_ptr(cs, out_ids[g]);
        for (uint32_t c = threadIdx.x; c <= n; c += blockDim.x) o[c] = (c == n) ? body : 0u;
    }
}

// Spectra of the bootstrapping key: one transform per (i, row, component) polynomial.
template <class PL>
__global__ __launch_bounds__(64 * BR_WAVES) void k_bk_transform(const uint32_t *__restrict__ bk_int,
                                                                const double2 *__restrict__ tw_table,
                                                                double2 *__restrict__ bk_hat, uint32_t polys,
                                                                const uint32_t *__restrict__ dst_ids,
                                                                uint32_t polys_per_sample)
{
    constexpr int P = PL::P, L = PL::L, M = PL::M, N = PL::N, GPW = PL::GPW;
    __shared__ double2 s_xch[BR_WAVES * GPW][PL::XSLOTS];
    __shared__ double2 s_tw[TwTable<PL>::COUNT];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int sub = lane / L, t = lane % L;
    const uint32_t first = (blockIdx.x * BR_WAVES + wave) * GPW;
    load_twiddles<PL>(s_tw, tw_table);
    if (first >= polys) return;
    const bool live = first + sub < polys;
    const uint32_t q = live ? first + sub : polys - 1;
    LaneCtx<PL> lc;
    lc.init(t, s_xch[wave * GPW + sub], s_tw);
    const uint32_t *src = bk_int + (size_t)q * N;
    double xr[P], xi[P];
#pragma unroll
    for (int m = 0; m < P; m++) {
        xr[m] = (double)(int)src[t + L * m];                 // torus words taken as signed: centred, |x| <= 2^31
        xi[m] = (double)(int)src[t + L * m + M];
    }
    forward<PL>(lc, xr, xi);
    if (live) {
        // sample s of the source goes to sample dst_ids[s] of the destination (in place when there is no list)
        const size_t qo = dst_ids ? (size_t)dst_ids[q / polys_per_sample] * polys_per_sample + q % polys_per_sample : q;
        double2 *dst = bk_hat + qo * P * L + t;
#pragma unroll
        for (int k = 0; k < P; k++) dst[k * L] = make_double2(xr[k], xi[k]);
    }
}

// ------------------------------------------------------------------------------------------
// Leveled CMux: out = d0 + C [.] (d1 - d0) for a TRGSW selector C in spectral form and TRLWE
// samples in HBM.  One CMux per wavefront; the same decomposition, transforms and products as
// one step of the blind rotation, with the operands streamed from memory instead of LDS.
// ------------------------------------------------------------------------------------------
// With 16 points per lane (N = 2048) the two output spectra and one transform fill the register file (192 of 256), so
// no selector row and no operand is requested ahead there.  What keeps that version at two wavefronts per SIMD and off
// the scratch memory: the words that the digits are cut from wait in LDS between the rows (32 registers), and the
// selector's values run through a ring of four points' worth of loads inside the products.  Per 4096 CMuxes: one
// wavefront per SIMD 282 us; two, every selector value loaded and waited for singly 162 us; the ring 149 us (45
// registers spilled); the words in LDS as well 101 us (12 spilled).
// (Both halves of a transform through one LDS round trip, in a buffer of twice the size, spills 31 registers: 214 us.)

// Sixteen bytes per lane from global memory straight into LDS (lane t's word lands at dst_wave + t): no register is
// held while the load is in flight.  dst_wave is the same for the whole wavefront.
__device__ __forceinline__ void load_to_lds16(const uint4 *src_lane, uint4 *dst_wave)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src_lane,
                                     (__attribute__((address_space(3))) void *)dst_wave, 16, 0, 0);
}

// LC: the gadget length when it is known at compile time (both loops over the rows are then unrolled, and a wait for
// memory sits at the first use of what was loaded instead of at a loop's entry), 0 for a length read at run time.
template <class PL, bool TRACK, int LC>
__global__ __launch_bounds__(64 * BR_WAVES, 2) void k_cmux(const double2 *__restrict__ trgsw_hat,
                                                           uint32_t *trlwe, const uint32_t *__restrict__ sel,
                                                           const uint32_t *__restrict__ in1, const uint32_t *__restrict__ in0,
                                                           const uint32_t *__restrict__ out, uint32_t count, uint32_t l_arg,
                                                           uint32_t bg_bit, const double2 *__restrict__ tw_table,
                                                           unsigned *round_err)
{
    constexpr int P = PL::P, L = PL::L, N = PL::N;
    const uint32_t l = LC ? (uint32_t)LC : l_arg;
    static_assert(PL::GPW == 1, "one transform per wavefront");
    __shared__ double2 s_xch[BR_WAVES][PL::XSLOTS];
    __shared__ double2 s_tw[TwTable<PL>::COUNT];
    constexpr bool STAGE = P <= 8;                                        // component 1's operands wait in LDS
    __shared__ uint4 s_stage[STAGE ? BR_WAVES : 1][STAGE ? P * L : 1];    // [d1 | d0] x P/2 words x 64 lanes
    // With 16 points per lane the words that the digits are cut from wait in LDS between the rows (each lane reads
    // back what it wrote): 32 registers that the transform and the products need.
    constexpr bool WORDS_IN_LDS = P > 8;
    __shared__ uint4 s_words[WORDS_IN_LDS ? BR_WAVES : 1][WORDS_IN_LDS ? (P / 2) * L : 1];
    const int wave = threadIdx.x >> 6, t = threadIdx.x & 63;
    load_twiddles<PL>(s_tw, tw_table);                                    // once per workgroup: the grid is persistent

    LaneCtx<PL> lc;
    lc.init(t, s_xch[wave], s_tw);
    const uint32_t Bg = 1u << bg_bit, half_bg = Bg >> 1;
    uint32_t dec_off = 1u << (31 - l * bg_bit);
    uint32_t flip = 0;
    for (uint32_t p = 1; p <= l; p++) { dec_off += half_bg << (32 - p * bg_bit); flip |= half_bg << (32 - p * bg_bit); }
    float worst = 0.f;

    // a wavefront takes CMux g, g + (wavefronts in the grid), ...; g is uniform, so the four ids are scalar loads.
    // Operands are requested ahead, before the inverse transforms: the words of d0 that the result is added to and
    // component 0 of the NEXT CMux into registers (the selector row's are idle then), component 1 of the next CMux
    // into LDS, which costs no register.  (Component 1 requested into registers during component 0's last transform
    // spills 86 of them: 73 us per 4096 CMuxes against 55 with nothing ahead, 53 without component 1, 47 with LDS.)
    const uint32_t stride = gridDim.x * BR_WAVES;
    constexpr int Q = P / 2;
    constexpr bool AHEAD = P <= 8;                                         // 16 points per lane leave no idle registers
    uint4 pu[Q], pv[Q];                                                    // requested TRLWE words of d1 and d0
    uint32_t g = __builtin_amdgcn_readfirstlane(blockIdx.x * BR_WAVES + wave);
    if (AHEAD && g < count) {
        const uint4 *a1 = reinterpret_cast<const uint4 *>(trlwe + (size_t)in1[g] * 2 * N) + t;
        const uint4 *a0 = reinterpret_cast<const uint4 *>(trlwe + (size_t)in0[g] * 2 * N) + t;
        if constexpr (STAGE) {
#pragma unroll
            for (int q = 0; q < Q; q++) {
                load_to_lds16(a1 + N / 4 + q * L, &s_stage[wave][q * L]);
                load_to_lds16(a0 + N / 4 + q * L, &s_stage[wave][(Q + q) * L]);
            }
        }
#pragma unroll
        for (int q = 0; q < Q; q++) { pu[q] = a1[q * L]; pv[q] = a0[q * L]; }
    }
    for (; g < count; g += stride) {
    const uint32_t *d1 = trlwe + (size_t)in1[g] * 2 * N, *d0 = trlwe + (size_t)in0[g] * 2 * N;
    uint32_t *dst = trlwe + (size_t)out[g] * 2 * N;
    const double2 *rows = trgsw_hat + (size_t)sel[g] * 2 * l * 2 * P * L + t;

    constexpr bool ROW_AHEAD = P <= 8;
    double2 bv[2][ROW_AHEAD ? P : 1];
    if constexpr (ROW_AHEAD) {
#pragma unroll
        for (int o = 0; o < 2; o++)
#pragma unroll
            for (int k = 0; k < P; k++) bv[o][k] = rows[(o * P + k) * L];
    }

    double sr[2][P], si[2][P];
#pragma unroll
    for (int k = 0; k < P; k++) { sr[0][k] = si[0][k] = sr[1][k] = si[1][k] = 0.0; }

#pragma unroll(LC ? 2 : 1)
    for (int c = 0; c < 2; c++) {
        // TRLWE samples are stored in transform order: the 16-byte word (q, t) of a component holds the coefficients
        // t + L*2q, t + L*2q + M, t + L*(2q+1), t + L*(2q+1) + M, the ones lane t works on
        uint32_t dlo[WORDS_IN_LDS ? 1 : P], dhi[WORDS_IN_LDS ? 1 : P];
        if (STAGE && c == 1) {
#pragma unroll
            for (int q = 0; q < Q; q++) { pu[q] = s_stage[wave][q * L + t]; pv[q] = s_stage[wave][(Q + q) * L + t]; }
        } else if (c == 1 || !AHEAD) {
            const uint4 *a1 = reinterpret_cast<const uint4 *>(d1 + c * N) + t, *a0 = reinterpret_cast<const uint4 *>(d0 + c * N) + t;
#pragma unroll
            for (int q = 0; q < Q; q++) { pu[q] = a1[q * L]; pv[q] = a0[q * L]; }
        }
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const uint4 u = pu[q], v = pv[q];
            const uint4 w = make_uint4((u.x - v.x + dec_off) ^ flip, (u.y - v.y + dec_off) ^ flip,
                                       (u.z - v.z + dec_off) ^ flip, (u.w - v.w + dec_off) ^ flip);
            if constexpr (WORDS_IN_LDS) {
                s_words[wave][q * L + t] = w;
            } else {
                dlo[2 * q] = w.x; dhi[2 * q] = w.y; dlo[2 * q + 1] = w.z; dhi[2 * q + 1] = w.w;
            }
        }
#pragma unroll(LC ? LC : 1)
        for (uint32_t p = 0; p < l; p++) {
            const uint32_t sh = 32 - (p + 1) * bg_bit;
            const uint32_t r = c * l + p;
            double xr[P], xi[P];
            if constexpr (WORDS_IN_LDS) {
#pragma unroll
                for (int q = 0; q < Q; q++) {
                    const uint4 w = s_words[wave][q * L + t];
                    xr[2 * q] = (double)(int)__builtin_amdgcn_sbfe(w.x, sh, bg_bit);
                    xi[2 * q] = (double)(int)__builtin_amdgcn_sbfe(w.y, sh, bg_bit);
                    xr[2 * q + 1] = (double)(int)__builtin_amdgcn_sbfe(w.z, sh, bg_bit);
                    xi[2 * q + 1] = (double)(int)__builtin_amdgcn_sbfe(w.w, sh, bg_bit);
                }
            } else {
#pragma unroll
                for (int m = 0; m < P; m++) {
                    xr[m] = (double)(int)__builtin_amdgcn_sbfe(dlo[m], sh, bg_bit);
                    xi[m] = (double)(int)__builtin_amdgcn_sbfe(dhi[m], sh, bg_bit);
                }
            }
            forward<PL>(lc, xr, xi);
            if constexpr (ROW_AHEAD) {
#pragma unroll
                for (int o = 0; o < 2; o++)
#pragma unroll
                    for (int k = 0; k < P; k++) {
                        const double2 b = bv[o][k];
                        sr[o][k] = __builtin_fma(-xi[k], b.y, __builtin_fma(xr[k], b.x, sr[o][k]));
                        si[o][k] = __builtin_fma(xi[k], b.x, __builtin_fma(xr[k], b.y, si[o][k]));
                    }
            } else {
                // no room for a row: the selector's values for RING points are in flight while the products of the
                // points before them run (a transformed value's registers are free once both outputs have used it)
                constexpr int RING = 4;
                const double2 *row = rows + (size_t)r * 2 * P * L;
                double2 ring[RING][2];
                __builtin_amdgcn_sched_barrier(0);                        // not into the transform: no register is free there
#pragma unroll
                for (int k = 0; k < RING; k++) { ring[k][0] = row[k * L]; ring[k][1] = row[(P + k) * L]; }
#pragma unroll
                for (int k = 0; k < P; k++) {
                    const double2 b0 = ring[k % RING][0], b1 = ring[k % RING][1];
                    if (k + RING < P) { ring[k % RING][0] = row[(k + RING) * L]; ring[k % RING][1] = row[(P + k + RING) * L]; }
                    sr[0][k] = __builtin_fma(-xi[k], b0.y, __builtin_fma(xr[k], b0.x, sr[0][k]));
                    si[0][k] = __builtin_fma(xi[k], b0.x, __builtin_fma(xr[k], b0.y, si[0][k]));
                    sr[1][k] = __builtin_fma(-xi[k], b1.y, __builtin_fma(xr[k], b1.x, sr[1][k]));
                    si[1][k] = __builtin_fma(xi[k], b1.x, __builtin_fma(xr[k], b1.y, si[1][k]));
                }
            }
            if (ROW_AHEAD && r + 1 < 2 * l) {
                const double2 *row = rows + (size_t)(r + 1) * 2 * P * L;
#pragma unroll
                for (int o = 0; o < 2; o++)
#pragma unroll
                    for (int k = 0; k < (ROW_AHEAD ? P : 0); k++) bv[o][k] = row[(o * P + k) * L];
            }
        }
    }
    // the words of d0 that the products are added to, and the next CMux's first component (this one's again after the
    // last: harmless), requested ahead of the inverse transforms
    uint4 base[2][AHEAD ? Q : 1];
    if constexpr (AHEAD) {
        const uint32_t gn = g + stride < count ? g + stride : g;
        const uint4 *a1 = reinterpret_cast<const uint4 *>(trlwe + (size_t)in1[gn] * 2 * N) + t;
        const uint4 *a0 = reinterpret_cast<const uint4 *>(trlwe + (size_t)in0[gn] * 2 * N) + t;
        // the next CMux's second component goes to LDS (this one's was consumed before its transforms).  After a
        // wavefront's last CMux this loads its own words once more: loads return in order, and the result's stores
        // wait for `base`, requested after it, so no wavefront leaves with such a load in flight.
        if constexpr (STAGE) {
#pragma unroll
            for (int q = 0; q < Q; q++) {
                load_to_lds16(a1 + N / 4 + q * L, &s_stage[wave][q * L]);
                load_to_lds16(a0 + N / 4 + q * L, &s_stage[wave][(Q + q) * L]);
            }
        }
#pragma unroll
        for (int o = 0; o < 2; o++) {
            const uint4 *b0 = reinterpret_cast<const uint4 *>(d0 + o * N) + t;
#pragma unroll
            for (int q = 0; q < Q; q++) base[o][q] = b0[q * L];
        }
#pragma unroll
        for (int q = 0; q < Q; q++) { pu[q] = a1[q * L]; pv[q] = a0[q * L]; }
    }
    {
        double2 *const xch2[2] = {lc.xch, lc.xch};
        inverse_n<PL, 2, true>(lc, xch2, sr, si);
    }
#pragma unroll
    for (int o = 0; o < 2; o++) {
        uint4 *ao = reinterpret_cast<uint4 *>(dst + o * N) + t;
#pragma unroll
        for (int q = 0; q < Q; q++) {
            if (TRACK) {
#pragma unroll
                for (int m = 2 * q; m < 2 * q + 2; m++) {
                    worst = fmaxf(worst, (float)fabs(sr[o][m] - rint(sr[o][m])));
                    worst = fmaxf(worst, (float)fabs(si[o][m] - rint(si[o][m])));
                }
            }
            uint4 v = AHEAD ? base[o][AHEAD ? q : 0] : (reinterpret_cast<const uint4 *>(d0 + o * N) + t)[q * L];
            v.x += (uint32_t)__double2loint(sr[o][2 * q] + 6755399441055744.0);
            v.y += (uint32_t)__double2loint(si[o][2 * q] + 6755399441055744.0);
            v.z += (uint32_t)__double2loint(sr[o][2 * q + 1] + 6755399441055744.0);
            v.w += (uint32_t)__double2loint(si[o][2 * q + 1] + 6755399441055744.0);
            ao[q * L] = v;
        }
    }
    wave_lds_fence();                                                     // the exchange buffer is reused by the next CMux
    }
    if (TRACK && round_err) atomicMax(round_err, __float_as_uint(worst));
}

// ------------------------------------------------------------------------------------------
// Leveled CMux of small levels: one CMux per workgroup of four wavefronts, (component c, half h of the spectrum) as in
// k_blind_rotate_quad.  Such a level takes as long as one CMux does, operands and selector rows fetched from memory: a
// wavefront's chain of 2l + 2 transforms becomes l + 1 transforms of half the length.  Measured, us per launch of 1 / 33 /
// 256 / 512 CMuxes, one wavefront against four: N = 1024 12.4 / 16.0 / 16.8 / 17.8 against 7.5 / 8.0 / 9.2 / 14.2, N =
// 2048 21.9 / 28.0 / 33.4 / 36.4 against 14.0 / 14.8 / 19.9 / 29.4 (by HIP events; 5.2 / 6.1 / 7.0 / 12.1 and 11.4 / 12.6 /
// 17.6 / 26.9 in the kernel trace; levels of up to 192 have their ids in the arguments, k_cmux_quad_args); with more than two
// CMuxes per compute unit a second round of workgroups starts and k_cmux is as fast or faster (768: 18.7 against 17.9, 37.6
// against 40.2).
// ------------------------------------------------------------------------------------------
template <int N, bool TRACK>
__device__ __forceinline__ void cmux_by_quad(const double2 *__restrict__ trgsw_hat, uint32_t *trlwe, uint32_t sel, uint32_t in1,
                                             uint32_t in0, uint32_t out, uint32_t l, uint32_t bg_bit,
                                             const double2 *__restrict__ table, unsigned *round_err)
{
    using HT = HalfTransform<N>;
    constexpr int P = HT::POINTS, M = N / 2, L = 64;
    __shared__ double2 s_xch[4][HT::XSLOTS], s_hand[4][P * L];
    // with four points per lane a lane's entries go straight to registers, with no copy and no barrier (8.2 -> 7.6 us)
    constexpr bool TABLE_IN_LDS = P > 4;
    __shared__ double2 s_tw[TABLE_IN_LDS ? HT::COUNT : 1];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t = threadIdx.x & 63;
    const int c = wave >> 1, h = wave & 1;
    const uint32_t *d1 = trlwe + (size_t)in1 * 2 * N, *d0 = trlwe + (size_t)in0 * 2 * N;
    const double2 *rows = trgsw_hat + ((size_t)sel * 2 + c) * l * 2 * M;        // rows of this component, [l][2][M]
    // every word of d1 - d0's component c, before the table is waited for (16-byte words as in k_cmux)
    uint4 u[P], v[P];
#pragma unroll
    for (int q = 0; q < P; q++) {
        u[q] = (reinterpret_cast<const uint4 *>(d1 + c * N) + t)[q * L];
        v[q] = (reinterpret_cast<const uint4 *>(d0 + c * N) + t)[q * L];
    }
    HT ht;
    if constexpr (TABLE_IN_LDS) {
        for (int e = threadIdx.x; e < HT::COUNT; e += 256) s_tw[e] = table[e];
        __syncthreads();
        ht.init(t, h, s_xch[wave], s_tw);
    } else {
        ht.init(t, h, s_xch[wave], table);
    }

    const uint32_t half_bg = 1u << (bg_bit - 1);
    uint32_t dec_off = 1u << (31 - l * bg_bit);
    uint32_t flip = 0;      // top bit of every digit field: field ^ top, read as signed, is field - Bg/2
    for (uint32_t p = 1; p <= l; p++) { dec_off += half_bg << (32 - p * bg_bit); flip |= half_bg << (32 - p * bg_bit); }
    float worst = 0.f;

    uint32_t dlo[2 * P], dhi[2 * P];                                         // positions t + 64 m
#pragma unroll
    for (int q = 0; q < P; q++) {
        dlo[2 * q] = (u[q].x - v[q].x + dec_off) ^ flip;     dhi[2 * q] = (u[q].y - v[q].y + dec_off) ^ flip;
        dlo[2 * q + 1] = (u[q].z - v[q].z + dec_off) ^ flip; dhi[2 * q + 1] = (u[q].w - v[q].w + dec_off) ^ flip;
    }
    // Selector values of a row: output c ^ 1 is requested a row ahead, output c as well where registers allow (four points
    // per lane), else once the transform has run (held through it with eight points, 55 registers are spilled;
    // as it is, 24: 100 bytes of scratch per lane).
    constexpr bool BOTH_AHEAD = P <= 4;
    double2 km[P], ko[P];
    auto request = [&](double2 (&k)[P], uint32_t p, int o) {
        const double2 *row = rows + ((size_t)p * 2 + o) * M;
#pragma unroll
        for (int m = 0; m < P; m++) k[m] = row[ht.key(m)];
    };
    request(ko, 0, c ^ 1);
    if (BOTH_AHEAD) request(km, 0, c);
    const double cs1 = h ? -0.70710678118654752440 : 0.70710678118654752440; // +-cos(pi/4) of the first stage
    double mr[P], mi[P], orr[P], oi[P];                                      // partial half spectra: own component, the other one
#pragma unroll
    for (int m = 0; m < P; m++) mr[m] = mi[m] = orr[m] = oi[m] = 0.0;
    for (uint32_t p = 0; p < l; p++) {
        const uint32_t sh = 32 - (p + 1) * bg_bit;
        double xr[P], xi[P];
#pragma unroll
        for (int m = 0; m < P; m++) {
            const int ar = (int)__builtin_amdgcn_sbfe((int)dlo[m], sh, bg_bit), ai = (int)__builtin_amdgcn_sbfe((int)dhi[m], sh, bg_bit);
            const int br = (int)__builtin_amdgcn_sbfe((int)dlo[m + P], sh, bg_bit), bi = (int)__builtin_amdgcn_sbfe((int)dhi[m + P], sh, bg_bit);
            xr[m] = __builtin_fma(cs1, (double)(br - bi), (double)ar);
            xi[m] = __builtin_fma(cs1, (double)(br + bi), (double)ai);
        }
        ht.forward(xr, xi);
        if (!BOTH_AHEAD) {
            __builtin_amdgcn_sched_barrier(0);
            request(km, p, c);
        }
#pragma unroll
        for (int m = 0; m < P; m++) {
            orr[m] = __builtin_fma(-xi[m], ko[m].y, __builtin_fma(xr[m], ko[m].x, orr[m]));
            oi[m] = __builtin_fma(xi[m], ko[m].x, __builtin_fma(xr[m], ko[m].y, oi[m]));
        }
#pragma unroll
        for (int m = 0; m < P; m++) {
            mr[m] = __builtin_fma(-xi[m], km[m].y, __builtin_fma(xr[m], km[m].x, mr[m]));
            mi[m] = __builtin_fma(xi[m], km[m].x, __builtin_fma(xr[m], km[m].y, mi[m]));
        }
        if (p + 1 < l) {
            request(ko, p + 1, c ^ 1);
            if (BOTH_AHEAD) request(km, p + 1, c);
        }
    }
    // the words of d0 that this wavefront's result is added to: 16-byte words P/2 h .. P/2 h + P/2 - 1
    uint4 base[P / 2];
#pragma unroll
    for (int q = 0; q < P / 2; q++) base[q] = (reinterpret_cast<const uint4 *>(d0 + c * N) + t)[(P / 2 * h + q) * L];
#pragma unroll
    for (int m = 0; m < P; m++) s_hand[wave][m * L + t] = make_double2(orr[m], oi[m]);
    lds_barrier();
#pragma unroll
    for (int m = 0; m < P; m++) { const double2 w = s_hand[wave ^ 2][m * L + t]; mr[m] += w.x; mi[m] += w.y; }
    ht.inverse(mr, mi);
    wave_lds_fence();
#pragma unroll
    for (int m = 0; m < P; m++) s_xch[wave][m * L + t] = make_double2(mr[m], mi[m]);
    lds_barrier();
    // last stage: (y0 + y1) / M for half 0, conj(w) (y0 - y1) / M for half 1; adding 1.5*2^52 leaves the rounded value
    // modulo 2^32 in the low word
    constexpr double magic = 6755399441055744.0, scale = 1.0 / M, rot = 0.70710678118654752440 / M;
    uint32_t lo[P], hi[P];
#pragma unroll
    for (int m = 0; m < P; m++) {
        const double2 w = s_xch[wave ^ 1][m * L + t];
        double re, im, f;
        if (h == 0) {
            re = mr[m] + w.x; im = mi[m] + w.y; f = scale;
        } else {
            const double dr = w.x - mr[m], di = w.y - mi[m];
            re = dr + di; im = di - dr; f = rot;
        }
        if (TRACK) {
            worst = fmaxf(worst, (float)fabs(re * f - rint(re * f)));
            worst = fmaxf(worst, (float)fabs(im * f - rint(im * f)));
        }
        lo[m] = (uint32_t)__double2loint(__builtin_fma(re, f, magic));
        hi[m] = (uint32_t)__double2loint(__builtin_fma(im, f, magic));
    }
    uint4 *dst = reinterpret_cast<uint4 *>(trlwe + (size_t)out * 2 * N + c * N) + t;
#pragma unroll
    for (int q = 0; q < P / 2; q++)
        dst[(P / 2 * h + q) * L] = make_uint4(base[q].x + lo[2 * q], base[q].y + hi[2 * q], base[q].z + lo[2 * q + 1], base[q].w + hi[2 * q + 1]);
    if (TRACK && round_err) atomicMax(round_err, __float_as_uint(worst));
}

template <int N, bool TRACK>
__global__ __launch_bounds__(256, 2) void k_cmux_quad(const double2 *__restrict__ trgsw_hat, uint32_t *trlwe,
                                                      const uint32_t *__restrict__ sel, const uint32_t *__restrict__ in1,
                                                      const uint32_t *__restrict__ in0, const uint32_t *__restrict__ out,
                                                      uint32_t l, uint32_t bg_bit, const double2 *__restrict__ table,
                                                      unsigned *round_err)
{
    const uint32_t g = blockIdx.x;
    cmux_by_quad<N, TRACK>(trgsw_hat, trlwe, sel[g], in1[g], in0[g], out[g], l, bg_bit, table, round_err);
}

// The same with the level's ids in the kernel's arguments: no copy to the device precedes the launch (a call of 1 / 33 / 132
// CMuxes 23.9 / 25.0 / 25.8 -> 20.2 / 20.5 / 21.0 us at N = 1024, 29.4 / 31.4 / 34.0 -> 25.8 / 26.8 / 29.5 at N = 2048), and
// the ids are not read behind a pointer (0.5 us of the kernel's 9).
template <int N, bool TRACK>
__global__ __launch_bounds__(256, 2) void k_cmux_quad_args(CmuxIds, const double2 *__restrict__ trgsw_hat, uint32_t *trlwe,
                                                           uint32_t l, uint32_t bg_bit, const double2 *__restrict__ table,
                                                           unsigned *round_err)
{
    // the ids are the first argument; read where they lie, since an array among the arguments that is indexed at run time
    // would be copied to scratch memory first
    const __attribute__((address_space(4))) uint32_t *ids =
        (const __attribute__((address_space(4))) uint32_t *)__builtin_amdgcn_kernarg_segment_ptr() + blockIdx.x;
    cmux_by_quad<N, TRACK>(trgsw_hat, trlwe, ids[0], ids[CMUX_ARG_IDS], ids[2 * CMUX_ARG_IDS], ids[3 * CMUX_ARG_IDS], l, bg_bit,
                           table, round_err);
}

// TRLWE samples from the pool into consecutive places, in the order of their coefficients, for one copy to the host (33
// samples of N = 1024 read back: 40 us; a copy for each and the reordering on the host 510).  The 16-byte word (q, t) of
// a component holds the coefficients t + 128 q, t + 128 q + N/2, t + 128 q + 64, t + 128 q + 64 + N/2.
__device__ __forceinline__ void gather_trlwe(const uint32_t *__restrict__ trlwe, uint32_t *__restrict__ dst, uint32_t id, uint32_t N)
{
    const uint4 *src = reinterpret_cast<const uint4 *>(trlwe + (size_t)id * 2 * N);
    uint32_t *d = dst + (size_t)blockIdx.x * 2 * N;
    for (uint32_t w = threadIdx.x; w < N / 2; w += 256) {
        const uint32_t c = w / (N / 4), q = w % (N / 4) / 64, j = c * N + 128 * q + w % 64;
        const uint4 v = src[w];
        d[j] = v.x; d[j + N / 2] = v.y; d[j + 64] = v.z; d[j + 64 + N / 2] = v.w;
    }
}
__global__ __launch_bounds__(256) void k_trlwe_gather(const uint32_t *__restrict__ trlwe, uint32_t *__restrict__ dst,
                                                      const uint32_t *__restrict__ ids, uint32_t N)
{
    gather_trlwe(trlwe, dst, ids[blockIdx.x], N);
}
// With the ids in the arguments, read where they lie as in k_cmux_quad_args: no copy to the device precedes the launch
// (a read of 1 / 8 samples 27.6 / 29.0 -> 24.0 / 27.0 us).
__global__ __launch_bounds__(256) void k_trlwe_gather_args(GatherIds, const uint32_t *__restrict__ trlwe,
                                                           uint32_t *__restrict__ dst, uint32_t N)
{
    const __attribute__((address_space(4))) uint32_t *ids =
        (const __attribute__((address_space(4))) uint32_t *)__builtin_amdgcn_kernarg_segment_ptr();
    gather_trlwe(trlwe, dst, ids[blockIdx.x], N);
}

// ------------------------------------------------------------------------------------------
// Key switch.  Block = KS_GROUP gates x KS_COLS output words; every thread owns one output
// word of all the gates, so each key row that is loaded serves KS_GROUP gates.
// ------------------------------------------------------------------------------------------
constexpr int KS_COLS = 128;

__global__ __launch_bounds__(KS_COLS) void k_key_switch(CtSpace cs, const uint32_t *__restrict__ ks,
                                                        uint32_t ks_stride, const uint16_t *__restrict__ ksd,
                                                        const uint32_t *__restrict__ ext_b,
                                                        const uint32_t *__restrict__ out_ids, uint32_t N, uint32_t t,
                                                        uint32_t bb, uint32_t n, uint32_t gates)
{
    const uint32_t grp = blockIdx.x;
    const uint32_t col = blockIdx.y * KS_COLS + threadIdx.x;
    const uint32_t colc = col <= n ? col : n;
    const uint32_t nrows = (1u << bb) - 1;
    uint32_t acc[KS_GROUP];
#pragma unroll
    for (int g = 0; g < KS_GROUP; g++) acc[g] = 0;

    const uint32_t *dg = (const uint32_t *)(ksd + (size_t)grp * N * KS_GROUP);
    for (uint32_t i = 0; i < N; i++) {
        uint32_t yw[KS_GROUP / 2];
#pragma unroll
        for (int q = 0; q < KS_GROUP / 2; q++) yw[q] = dg[(size_t)i * (KS_GROUP / 2) + q];
        for (uint32_t j = 0; j < t; j++) {
            const uint32_t sh = (t - 1 - j) * bb;
            const uint32_t *rows = ks + ((size_t)(i * t + j) * nrows) * ks_stride + colc;
            for (uint32_t v = 1; v <= nrows; v++) {
                const uint32_t r = rows[(size_t)(v - 1) * ks_stride];
#pragma unroll
                for (int g = 0; g < KS_GROUP; g++) {
                    const uint32_t y = (yw[g >> 1] >> (16 * (g & 1))) & 0xffffu;
                    const uint32_t d = (y >> sh) & nrows;
                    acc[g] -= (d == v) ? r : 0u;
                }
            }
        }
    }
    if (col > n) return;
#pragma unroll
    for (int g = 0; g < KS_GROUP; g++) {
        const uint32_t gi = grp * KS_GROUP + g;
        if (gi < gates) {
            uint32_t v = acc[g];
            if (col == n) v += ext_b[gi];
            ct_ptr(cs, out_ids[gi])[col] = v;
        }
    }
}

// ------------------------------------------------------------------------------------------
// Key switch as an int8 matrix product on the MFMA units (base 4, 8 digits).
//   out[g][c] = (0, b'')[c] - sum_{i,j} KS[i][j][d_gij][c]
// is sum_k A[g][k] * KS[k][c] with A the one-hot encoding of the digits, k = (i, j, v).  A is
// 0/1 and every KS word is split into four signed bytes, so four i32 += i8*i8 products
// (|sum| <= 2^20) recombined with shifts give the exact result modulo 2^32.
// One v_mfma_i32_32x32x32_i8 consumes the 32 k of one i (8 digits x 4 values; the v = 0
// column of A is always 0).  A wavefront owns 64 gates x 32 output words; a block of four
// wavefronts shares the key bytes through LDS; blockIdx.z splits the i range and partial
// sums are subtracted atomically from the slot that the blind rotation initialised.
// ------------------------------------------------------------------------------------------
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
constexpr int KSM_WAVES = 4, KSM_TILES = 2;   // measured: 1 tile (4 or 6 waves per SIMD), 3 and 4 tiles are slower

__device__ __forceinline__ int onehot_byte(uint32_t d) { return (int)((1u << (d << 3)) & 0xFFFFFF00u); }

// The four wavefronts of a workgroup work on the same 32 output words, so the 4 KiB of key bytes of a step (four byte
// planes x 64 lanes x 16 bytes) are fetched once per workgroup, wavefront w bringing plane w straight into LDS
// (global_load_lds), and every wavefront reads them from there.  (Each wavefront loading them for itself through the
// vector L1 kept that cache's pending-request stall at 60 % of the kernel's time: 0.375 against 0.278 ms per 4096 gates.)
// Two stages: a step's bytes are requested during the step before; requesting two steps ahead through four stages is
// no faster (0.284 ms).  Every wavefront of a workgroup meets every barrier: one with no gates of its own still brings
// its plane.  i_per_block must be even.
__global__ __launch_bounds__(64 * KSM_WAVES, 3) void k_key_switch_mfma(CtSpace cs, const int8_t *__restrict__ ksb,
                                                                     uint32_t cols_p, const uint16_t *__restrict__ ksd,
                                                                     const uint32_t *__restrict__ out_ids, uint32_t N,
                                                                     uint32_t n, uint32_t gates, uint32_t i_per_block)
{
    __shared__ uint4 s_b0[4 * 64], s_b1[4 * 64];                           // [plane][lane], one array per stage
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5, c32 = lane & 31;
    const uint32_t tile_first = blockIdx.x * KSM_WAVES * KSM_TILES;              // live: the workgroup exists for it
    const uint32_t tile0 = tile_first + wave * KSM_TILES;                        // in units of 32 gates
    const uint32_t col = blockIdx.y * 32 + c32;
    const uint32_t i0 = blockIdx.z * i_per_block, i1 = min(N, i0 + i_per_block);

    v16i acc[KSM_TILES][4];
#pragma unroll
    for (int t = 0; t < KSM_TILES; t++)
#pragma unroll
        for (int p = 0; p < 4; p++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[t][p][r] = 0;

    const uint16_t *yp[KSM_TILES];
    bool tile_live[KSM_TILES];
#pragma unroll
    for (int t = 0; t < KSM_TILES; t++) {
        tile_live[t] = (tile0 + t) * 32 < gates;
        yp[t] = ksd + ((size_t)(tile_live[t] ? tile0 + t : tile_first) * N) * KS_GROUP + c32;
    }
    // this wavefront's plane of a step: 1 KiB, lane (half, c32) takes the 16 bytes of column c32, half `half`
    const uint4 *mine = reinterpret_cast<const uint4 *>(ksb + ((size_t)wave * cols_p + col) * 32 + 16 * half);
    const size_t step_u4 = (size_t)4 * cols_p * 2;                          // one i further, in 16-byte units
    const uint32_t ysh = 8 * (1 - half);

    uint32_t y_next[KSM_TILES];
    load_to_lds16(mine + (size_t)i0 * step_u4, s_b0 + wave * 64);
#pragma unroll
    for (int t = 0; t < KSM_TILES; t++) y_next[t] = yp[t][(size_t)i0 * KS_GROUP];

    auto step = [&](uint32_t i, const uint4 *cur, uint4 *other) {
        // this step's bytes have landed (every wavefront waits for its own plane, then all meet), and nobody still
        // reads the other stage (its readers waited for their values before their products, a step ago)
        __builtin_amdgcn_s_waitcnt(0x0F70);                                 // vmcnt(0)
        __builtin_amdgcn_s_barrier();
        uint32_t yv[KSM_TILES];
#pragma unroll
        for (int t = 0; t < KSM_TILES; t++) yv[t] = y_next[t];
        const uint32_t in = min(i + 1, i1 - 1);                             // past the end: the last step again, unused
        load_to_lds16(mine + (size_t)in * step_u4, other + wave * 64);
#pragma unroll
        for (int t = 0; t < KSM_TILES; t++) y_next[t] = yp[t][(size_t)in * KS_GROUP];
        __builtin_amdgcn_sched_barrier(0);                                  // the requests stay ahead of the products
        v4i b[4];
#pragma unroll
        for (int p = 0; p < 4; p++) {
            const uint4 w = cur[p * 64 + lane];
            b[p] = v4i{(int)w.x, (int)w.y, (int)w.z, (int)w.w};
        }
#pragma unroll
        for (int t = 0; t < KSM_TILES; t++) {
            const uint32_t y = (yv[t] >> ysh) & 0xffu;                                    // this half's four digits
            v4i a;
            a.x = onehot_byte((y >> 6) & 3);
            a.y = onehot_byte((y >> 4) & 3);
            a.z = onehot_byte((y >> 2) & 3);
            a.w = onehot_byte(y & 3);
#pragma unroll
            for (int p = 0; p < 4; p++) acc[t][p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b[p], acc[t][p], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);                                  // the next step's wait stays behind the products
    };
    for (uint32_t i = i0; i < i1; i += 2) {
        step(i, s_b0, s_b1);
        step(i + 1, s_b1, s_b0);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                                     // no load into LDS is in flight at the end

    if (col > n) return;
#pragma unroll
    for (int t = 0; t < KSM_TILES; t++) {
        if (!tile_live[t]) continue;
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const uint32_t row = 8 * (r / 4) + 4 * half + (r % 4);
            const uint32_t g = (tile0 + t) * 32 + row;
            if (g >= gates) continue;
            const uint32_t v = (uint32_t)acc[t][0][r] + ((uint32_t)acc[t][1][r] << 8) + ((uint32_t)acc[t][2][r] << 16) +
                               ((uint32_t)acc[t][3][r] << 24);
            atomicAdd(ct_ptr(cs, out_ids[g]) + col, 0u - v);
        }
    }
}

// The same for a few gates, one workgroup of them, and at most KSF_STEPS coefficients a workgroup.  Such a level is bound by
// how much of the key is under way: k_key_switch_mfma has one step's 4 KiB per workgroup, waits for them 0.4 to 0.8 us a step,
// and cannot have more, since a wait for its digits is a wait for everything.  Here all digits are in LDS before the first step
// and three steps' bytes are under way; wavefronts without a gate only bring their plane.  us by HIP events at n = 630 for 1 /
// 31 / 64 / 83 / 130 / 200 / 256 gates: 27 / 32 / 38 / 38 / 38 / 38.5 / 39 -> 17.7 / 22.4 / 28 / 30.5 / 33.5 / 36.5 / 37.5 to 41:
// what is left grows with the sums that 32 splits add atomically.  (Half as many splits 24 / 29 / 34 / 38 / 39 / 40 / 41, seven
// steps under way 21 / 26 / 31.5 / 35 / 38 / 41 / 43.)  So it has the levels of up to KSF_GATES.
constexpr int KSF_STEPS = 32, KSF_GATES = 192;
__global__ __launch_bounds__(64 * KSM_WAVES, 3) void k_key_switch_few(CtSpace cs, const int8_t *__restrict__ ksb,
                                                                    uint32_t cols_p, const uint16_t *__restrict__ ksd,
                                                                    const uint32_t *__restrict__ out_ids, uint32_t N,
                                                                    uint32_t n, uint32_t gates, uint32_t i_per_block)
{
    constexpr int GROUPS = KSF_GATES / KS_GROUP;
    static_assert(KSF_GATES <= 32 * KSM_WAVES * KSM_TILES && KSF_GATES % (32 * KSM_TILES) == 0, "whole wavefronts of gates");
    __shared__ uint4 s_b0[4 * 64], s_b1[4 * 64], s_b2[4 * 64], s_b3[4 * 64];     // [plane][lane], one array per stage
    __shared__ uint4 s_digits[GROUPS][KSF_STEPS * KS_GROUP / 8];
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5, c32 = lane & 31;
    const uint32_t tile0 = wave * KSM_TILES, col = blockIdx.x * 32 + c32;
    const uint32_t i0 = blockIdx.y * i_per_block, i1 = i0 + i_per_block;

    // the digits of all gates for these coefficients
    const uint32_t words = i_per_block * KS_GROUP / 8, live_groups = (gates + KS_GROUP - 1) / KS_GROUP;
    for (uint32_t e = threadIdx.x; e < live_groups * words; e += 64 * KSM_WAVES) {
        const uint32_t grp = e / words, w = e % words;
        s_digits[grp][w] = reinterpret_cast<const uint4 *>(ksd + ((size_t)grp * N + i0) * KS_GROUP)[w];
    }
    __syncthreads();

    v16i acc[KSM_TILES][4];
#pragma unroll
    for (int t = 0; t < KSM_TILES; t++)
#pragma unroll
        for (int p = 0; p < 4; p++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[t][p][r] = 0;
    const uint4 *mine = reinterpret_cast<const uint4 *>(ksb + ((size_t)wave * cols_p + col) * 32 + 16 * half);
    const size_t step_u4 = (size_t)4 * cols_p * 2;                          // one i further, in 16-byte units
    const uint32_t ysh = 8 * (1 - half);
    const bool live = tile0 * KS_GROUP < gates;                             // the same for the wavefront
    auto fetch = [&](uint32_t i, uint4 *stage) { load_to_lds16(mine + (size_t)min(i, i1 - 1) * step_u4, stage + wave * 64); };

    auto step = [&](uint32_t i, const uint4 *cur, uint4 *free_stage) {
        // this step's bytes have landed, those of the two steps behind it may be on their way; nobody reads the free stage
        __builtin_amdgcn_s_waitcnt(0x0F72);                                 // vmcnt(2)
        __builtin_amdgcn_s_barrier();
        fetch(i + 3, free_stage);                                           // past the end: the last step again, unused
        __builtin_amdgcn_sched_barrier(0);
        if (live) {
            v4i b[4];
#pragma unroll
            for (int p = 0; p < 4; p++) {
                const uint4 w = cur[p * 64 + lane];
                b[p] = v4i{(int)w.x, (int)w.y, (int)w.z, (int)w.w};
            }
#pragma unroll
            for (int t = 0; t < KSM_TILES; t++) {
                const uint32_t yv = reinterpret_cast<const uint16_t *>(s_digits[tile0 + t])[(i - i0) * KS_GROUP + c32];
                const uint32_t y = (yv >> ysh) & 0xffu;                     // this half's four digits
                v4i a;
                a.x = onehot_byte((y >> 6) & 3);
                a.y = onehot_byte((y >> 4) & 3);
                a.z = onehot_byte((y >> 2) & 3);
                a.w = onehot_byte(y & 3);
#pragma unroll
                for (int p = 0; p < 4; p++) acc[t][p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b[p], acc[t][p], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch(i0, s_b0); fetch(i0 + 1, s_b1); fetch(i0 + 2, s_b2);
    for (uint32_t i = i0; i < i1; i += 4) {
        step(i, s_b0, s_b3);
        step(i + 1, s_b1, s_b0);
        step(i + 2, s_b2, s_b1);
        step(i + 3, s_b3, s_b2);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                                     // no load into LDS is in flight at the end

    if (col > n || !live) return;
#pragma unroll
    for (int t = 0; t < KSM_TILES; t++) {
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const uint32_t row = 8 * (r / 4) + 4 * half + (r % 4);
            const uint32_t g = (tile0 + t) * 32 + row;
            if (g >= gates) continue;
            const uint32_t v = (uint32_t)acc[t][0][r] + ((uint32_t)acc[t][1][r] << 8) + ((uint32_t)acc[t][2][r] << 16) +
                               ((uint32_t)acc[t][3][r] << 24);
            atomicAdd(ct_ptr(cs, out_ids[g]) + col, 0u - v);
        }
    }
}

// ------------------------------------------------------------------------------------------
// Pool plumbing
// ------------------------------------------------------------------------------------------
// dst <- src, or its complement (word-wise negation) when the source id carries WIRE_NEG
__global__ void k_copy_ct(CtSpace cs, const uint32_t *__restrict__ src_ids, const uint32_t *__restrict__ dst_ids,
                          uint32_t n)
{
    const uint32_t ref = src_ids[blockIdx.x];
    const bool neg = (ref & WIRE_NEG) != 0;
    const uint32_t *s = ct_ptr(cs, ref & ~WIRE_NEG);
    uint32_t *d = ct_ptr(cs, dst_ids[blockIdx.x]);
    for (uint32_t i = threadIdx.x; i <= n; i += blockDim.x) d[i] = neg ? 0u - s[i] : s[i];
}

// ------------------------------------------------------------------------------------------
// Client side: fresh encryptions and phases of samples in the pool, one wavefront per sample.  The random words of a
// sample's stream are addressed (she_host.cpp has the definition), so every lane makes its own.  Bound by the pool's
// memory and the call itself (42 and 37 us for 6272 samples of n = 630, the key bits uploaded with each call and cleared
// again at its end, 2 to 3 us of that); on the host's threads, with the pool filled from and read into a staged copy, 1.4
// and 1.5 ms.
// ------------------------------------------------------------------------------------------
constexpr int FRESH_WAVES = 7, PHASE_WAVES = 4, KEY_BATCH = 10;      // ten words per lane: a whole sample at n = 630

__device__ __forceinline__ uint64_t stream_mix(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
constexpr uint64_t STREAM_STEP = 0x9E3779B97F4A7C15ull;
__device__ __forceinline__ uint64_t stream_word(uint64_t key, uint64_t c) { return stream_mix(key + (c + 1) * STREAM_STEP); }

// sum over the wavefront's lanes
__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += (uint32_t)__shfl_xor((int)v, d, 64);
    return v;
}

// Seven wavefronts make the mask and its sum of a sample each while the eighth computes the seven errors, a logarithm and a
// cosine in 64 bits, on a lane each; the key's bits are requested side by side.  Bound by the random words, three 32-bit
// multiplications and two more for every one, and by the launch.  Calls for 100 / 1000 / 2500 / 6272 bits: 29.6 / 30.0 / 33.3
// / 41.5 us; with the errors on the first lane of every sample's own wavefront, and the key bits one after the other, 32.1 /
// 32.8 / 35.8 / 45.7; with 3, 11 or 15 samples a workgroup up to 1 us more.
// The error is computed as she_host.cpp computes it, with this card's log and cos.  Both sides' functions are accurate to
// a few units in the last place, so that the unrounded values differ by less than 2^-48 of their size: where the value is
// further than 2^-44 of its size (and 2^-40) from halfway between two integers, both round to the same one.  Where it is
// not, the sample's number goes into `retry` (its first word counts them), no error is added, and the host adds its own.
__global__ __launch_bounds__(64 * (FRESH_WAVES + 1)) void k_fresh_samples(CtSpace cs, const uint32_t *__restrict__ ids,
                                                                          const uint8_t *__restrict__ bits,
                                                                          const uint8_t *__restrict__ lwe_key, uint32_t n,
                                                                          uint64_t stream_base, double sigma, uint32_t count,
                                                                          uint32_t *retry_count, uint32_t *__restrict__ retry)
{
#pragma clang fp contract(off)
    __shared__ uint32_t s_sum[FRESH_WAVES];
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63, first = blockIdx.x * FRESH_WAVES;
    const uint32_t k = first + (wave < FRESH_WAVES ? wave : lane);
    const bool live = k < count && (wave < FRESH_WAVES || lane < FRESH_WAVES);
    uint32_t body = 0;
    if (live && wave < FRESH_WAVES) {
        const uint64_t key = stream_mix(stream_base + k);
        uint32_t *dst = ct_ptr(cs, ids[k]);
        uint32_t sum = 0;
        for (uint32_t i0 = lane; i0 < n; i0 += 64 * KEY_BATCH) {
            uint32_t bit[KEY_BATCH];
#pragma unroll
            for (int q = 0; q < KEY_BATCH; q++) bit[q] = lwe_key[std::min(i0 + 64 * q, n - 1)];
            uint64_t at = key + (uint64_t)(i0 + 1) * STREAM_STEP;                  // stream_word's argument, one addition a word
#pragma unroll
            for (int q = 0; q < KEY_BATCH; q++, at += 64 * STREAM_STEP) {
                const uint32_t i = i0 + 64 * q;
                if (i < n) {
                    const uint32_t a = (uint32_t)(stream_mix(at) >> 32);
                    dst[i] = a;
                    sum += bit[q] ? a : 0u;
                }
            }
        }
        sum = wave_sum(sum);
        if (lane == 0) s_sum[wave] = sum;
    } else if (live) {
        const uint64_t key = stream_mix(stream_base + k);
        const double unit = 1.0 / 9007199254740992.0;                         // 2^-53
        const double u1 = (double)((stream_word(key, n) >> 11) + 1) * unit;
        const double u2 = (double)(stream_word(key, (uint64_t)n + 1) >> 11) * unit;
        const double radius = sqrt(-2.0 * log(u1));
        const double normal = radius * cos(6.283185307179586476925286766559 * u2);
        const double scaled = normal * sigma * 4294967296.0, rounded = rint(scaled);
        const double to_half = 0.5 - fabs(scaled - rounded);
        body = (bits[k] ? (1u << 29) : 0u - (1u << 29)) + (uint32_t)(int64_t)rounded;
        if (!(to_half > fabs(scaled) * 0x1p-44 + 0x1p-40)) {
            retry[atomicAdd(retry_count, 1u)] = k;
            body = bits[k] ? (1u << 29) : 0u - (1u << 29);
        }
    }
    __syncthreads();
    if (live && wave == FRESH_WAVES) ct_ptr(cs, ids[k])[n] = body + s_sum[lane];
}

// A lane's words and key bits are requested side by side, not one after the other: calls for 100 / 2500 / 6272 bits
// 29.6 / 30.5 / 36.8 us against 31.7 / 32.4 / 38.6 (3.0 / 3.3 / 5.8 in the kernel against 5.4 / 5.6 / 9.1).
__global__ __launch_bounds__(64 * PHASE_WAVES) void k_phase_bits(CtSpace cs, const uint32_t *__restrict__ ids,
                                                                 const uint8_t *__restrict__ lwe_key, uint32_t n,
                                                                 uint32_t count, uint8_t *__restrict__ bits)
{
    const uint32_t k = blockIdx.x * PHASE_WAVES + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (k >= count) return;
    const uint32_t *ct = ct_ptr(cs, ids[k]);
    const uint32_t body = ct[n];
    uint32_t sum = 0;
    for (uint32_t i0 = lane; i0 < n; i0 += 64 * KEY_BATCH) {
        uint32_t word[KEY_BATCH], bit[KEY_BATCH];
#pragma unroll
        for (int q = 0; q < KEY_BATCH; q++) {
            const uint32_t i = std::min(i0 + 64 * q, n - 1);                   // past the end: the last word, not added
            word[q] = ct[i]; bit[q] = lwe_key[i];
        }
#pragma unroll
        for (int q = 0; q < KEY_BATCH; q++) sum += bit[q] && i0 + 64 * q < n ? word[q] : 0u;
    }
    sum = wave_sum(sum);
    if (lane == 0) bits[k] = (int32_t)(body - sum) > 0;
}

// The words of the staging buffer that held the key's bits and plaintext bits, cleared at the end of a client call.  The
// launch is all it costs (hipMemsetAsync in its place: 5 to 8 us of the call instead of 1 to 3).
__global__ __launch_bounds__(256) void k_clear_words(uint32_t *__restrict__ dst, uint32_t words)
{
    for (uint32_t w = blockIdx.x * 256 + threadIdx.x; w < words; w += gridDim.x * 256) dst[w] = 0;
}

// ------------------------------------------------------------------------------------------
// Host launchers
// ------------------------------------------------------------------------------------------
using Plan256 = Plan<1, 7>;
using Plan512 = Plan<2, 4>;
using Plan1024 = Plan<3, 3>;

// N = 2048 has transforms, key spectra and the leveled CMux; the blind rotation is built for N <= 1024
bool plan_supported(uint32_t N) { return N == 256 || N == 512 || N == 1024 || N == 2048; }

template <class PL> static size_t tw_doubles() { return 2 * (size_t)TwTable<PL>::COUNT; }

size_t twiddle_doubles(uint32_t N)
{
    switch (N) {
    case 256: return tw_doubles<Plan256>();
    case 512: return tw_doubles<Plan512>();
    case 1024: return tw_doubles<Plan1024>();
    case 2048: return tw_doubles<Plan2048>();
    }
    return 0;
}

void fill_twiddles(uint32_t N, double *out)
{
    switch (N) {
    case 256: make_twiddles<Plan256>(out); break;
    case 512: make_twiddles<Plan512>(out); break;
    case 1024: make_twiddles<Plan1024>(out); break;
    case 2048: make_twiddles<Plan2048>(out); break;
    }
}

size_t half_twiddle_doubles(uint32_t N) { return N == HalfPlan::N ? 2 * (size_t)(HalfPlan::COUNT + QuarterInverse::COUNT) : 0; }
void fill_half_twiddles(double *out)
{
    make_half_twiddles(out);
    make_quarter_twiddles(out + 2 * HalfPlan::COUNT);
}

size_t bk_hat_elems(const she_params &P) { return (size_t)P.n * 2 * P.l * 2 * (P.N / 2); }

template <class PL>
static hipError_t bk_transform_t(const she_params &P, const uint32_t *d_bk_int, const DeviceKeys &K, hipStream_t st)
{
    const uint32_t polys = P.n * 2 * P.l * 2;
    const uint32_t per_block = BR_WAVES * PL::GPW;
    hipLaunchKernelGGL((k_bk_transform<PL>), dim3((polys + per_block - 1) / per_block), dim3(64 * BR_WAVES), 0, st,
                       d_bk_int, K.twiddles, K.bk_hat, polys, (const uint32_t *)nullptr, 1u);
    return hipGetLastError();
}

template <class PL>
static hipError_t trgsw_transform_t(const she_params &P, const DeviceKeys &K, const uint32_t *d_int, double2 *trgsw_hat,
                                    const uint32_t *d_ids, size_t samples, hipStream_t st)
{
    const uint32_t pps = 2 * P.l * 2, polys = (uint32_t)(samples * pps);
    const uint32_t per_block = BR_WAVES * PL::GPW;
    hipLaunchKernelGGL((k_bk_transform<PL>), dim3((polys + per_block - 1) / per_block), dim3(64 * BR_WAVES), 0, st,
                       d_int, K.twiddles, trgsw_hat, polys, d_ids, pps);
    return hipGetLastError();
}

// Levels with their ids in the kernel's arguments; the lists are host memory.
template <int N>
static hipError_t cmux_args_t(const she_params &P, const DeviceKeys &K, const double2 *trgsw_hat, uint32_t *trlwe,
                              const uint32_t *sel, const uint32_t *in1, const uint32_t *in0, const uint32_t *out, size_t count,
                              unsigned *d_round_err, hipStream_t st)
{
    const double2 *table = N == HalfPlan::N ? K.half_twiddles : K.twiddles;
    CmuxIds ids;
    fill_cmux_ids(ids, sel, in1, in0, out, count);
#define SHE_LAUNCH_CMUX_QUAD(TRACK)                                                                                       \
    hipLaunchKernelGGL((k_cmux_quad_args<N, TRACK>), dim3((unsigned)count), dim3(256), 0, st, ids, trgsw_hat, trlwe, P.l, \
                       P.bg_bit, table, d_round_err)
    if (d_round_err) SHE_LAUNCH_CMUX_QUAD(true); else SHE_LAUNCH_CMUX_QUAD(false);
#undef SHE_LAUNCH_CMUX_QUAD
    return hipGetLastError();
}

template <class PL>
static hipError_t cmux_t(const she_params &P, const DeviceKeys &K, const double2 *trgsw_hat, uint32_t *trlwe,
                         const uint32_t *d_sel, const uint32_t *d_in1, const uint32_t *d_in0, const uint32_t *d_out,
                         size_t count, unsigned *d_round_err, hipStream_t st)
{
    if constexpr (PL::N == 1024 || PL::N == 2048) {
        // up to two CMuxes per compute unit: four wavefronts each (measured beside the kernel)
        if (count <= 2 * (size_t)K.cus) {
            const double2 *table = PL::N == HalfPlan::N ? K.half_twiddles : K.twiddles;
#define SHE_LAUNCH_CMUX_QUAD(TRACK)                                                                                   \
    hipLaunchKernelGGL((k_cmux_quad<PL::N, TRACK>), dim3((unsigned)count), dim3(256), 0, st, trgsw_hat, trlwe, d_sel, \
                       d_in1, d_in0, d_out, P.l, P.bg_bit, table, d_round_err)
            if (d_round_err) SHE_LAUNCH_CMUX_QUAD(true); else SHE_LAUNCH_CMUX_QUAD(false);
#undef SHE_LAUNCH_CMUX_QUAD
            return hipGetLastError();
        }
    }
    // persistent: at most the workgroups per compute unit that fit (two), each wavefront loops over its share
    const size_t wgs = (count + BR_WAVES - 1) / BR_WAVES;
    const size_t per_cu = 2;
    const dim3 grid((unsigned)std::min<size_t>(wgs, per_cu * std::max<uint32_t>(K.cus, 1))), block(64 * BR_WAVES);
    if (d_round_err)
        hipLaunchKernelGGL((k_cmux<PL, true, 0>), grid, block, 0, st, trgsw_hat, trlwe, d_sel, d_in1, d_in0, d_out,
                           (uint32_t)count, P.l, P.bg_bit, K.twiddles, d_round_err);
    else if (P.l == 3 && PL::P <= 8)
        hipLaunchKernelGGL((k_cmux<PL, false, 3>), grid, block, 0, st, trgsw_hat, trlwe, d_sel, d_in1, d_in0, d_out,
                           (uint32_t)count, P.l, P.bg_bit, K.twiddles, d_round_err);
    else
        hipLaunchKernelGGL((k_cmux<PL, false, 0>), grid, block, 0, st, trgsw_hat, trlwe, d_sel, d_in1, d_in0, d_out,
                           (uint32_t)count, P.l, P.bg_bit, K.twiddles, d_round_err);
    return hipGetLastError();
}

hipError_t launch_trgsw_transform(const she_params &P, const DeviceKeys &K, const uint32_t *d_int, double2 *trgsw_hat,
                                  const uint32_t *d_ids, size_t samples, hipStream_t st)
{
    if (!samples) return hipSuccess;
    switch (P.N) {
    case 256: return trgsw_transform_t<Plan256>(P, K, d_int, trgsw_hat, d_ids, samples, st);
    case 512: return trgsw_transform_t<Plan512>(P, K, d_int, trgsw_hat, d_ids, samples, st);
    case 1024: return trgsw_transform_t<Plan1024>(P, K, d_int, trgsw_hat, d_ids, samples, st);
    case 2048: return trgsw_transform_t<Plan2048>(P, K, d_int, trgsw_hat, d_ids, samples, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_cmux(const she_params &P, const DeviceKeys &K, const double2 *trgsw_hat, uint32_t *trlwe,
                       const uint32_t *sel, const uint32_t *in1, const uint32_t *in0, const uint32_t *out, size_t count,
                       unsigned *d_round_err, hipStream_t st)
{
    if (!count) return hipSuccess;
    if (cmux_ids_in_arguments(P.N, count, K.cus))
        return P.N == 1024 ? cmux_args_t<1024>(P, K, trgsw_hat, trlwe, sel, in1, in0, out, count, d_round_err, st)
                           : cmux_args_t<2048>(P, K, trgsw_hat, trlwe, sel, in1, in0, out, count, d_round_err, st);
    switch (P.N) {
    case 256: return cmux_t<Plan256>(P, K, trgsw_hat, trlwe, sel, in1, in0, out, count, d_round_err, st);
    case 512: return cmux_t<Plan512>(P, K, trgsw_hat, trlwe, sel, in1, in0, out, count, d_round_err, st);
    case 1024: return cmux_t<Plan1024>(P, K, trgsw_hat, trlwe, sel, in1, in0, out, count, d_round_err, st);
    case 2048: return cmux_t<Plan2048>(P, K, trgsw_hat, trlwe, sel, in1, in0, out, count, d_round_err, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_trlwe_gather(const uint32_t *trlwe, uint32_t *d_dst, const uint32_t *ids, size_t count, uint32_t N,
                               hipStream_t st)
{
    if (!count) return hipSuccess;
    if (gather_ids_in_arguments(count)) {
        GatherIds a;
        for (size_t k = 0; k < GATHER_ARG_IDS; k++) a.id[k] = k < count ? ids[k] : 0;
        hipLaunchKernelGGL(k_trlwe_gather_args, dim3((unsigned)count), dim3(256), 0, st, a, trlwe, d_dst, N);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_trlwe_gather, dim3((unsigned)count), dim3(256), 0, st, trlwe, d_dst, ids, N);
    return hipGetLastError();
}

hipError_t launch_bk_transform(const she_params &P, const uint32_t *d_bk_int, const DeviceKeys &K, hipStream_t st)
{
    switch (P.N) {
    case 256: return bk_transform_t<Plan256>(P, d_bk_int, K, st);
    case 512: return bk_transform_t<Plan512>(P, d_bk_int, K, st);
    case 1024: return bk_transform_t<Plan1024>(P, d_bk_int, K, st);
    case 2048: return bk_transform_t<Plan2048>(P, d_bk_int, K, st);
    }
    return hipErrorInvalidValue;
}

static uint32_t ilog2(uint32_t v) { uint32_t r = 0; while ((1u << r) < v) r++; return r; }

hipError_t launch_lincomb(const she_params &P, const CtSpace &cs, const uint8_t *d_type, const uint32_t *d_in0,
                          const uint32_t *d_in1, const uint32_t *d_in2, size_t gates, const LevelWork &W, hipStream_t st)
{
    if (!gates) return hipSuccess;
    hipLaunchKernelGGL(k_lincomb, dim3((unsigned)gates), dim3(128), 0, st, cs, d_type, d_in0, d_in1, d_in2, P.n,
                       ilog2(2 * P.N), W.bar, W.bar_stride);
    return hipGetLastError();
}

template <class PL>
static hipError_t blind_rotate_t(const she_params &P, const DeviceKeys &K, size_t gates, const LevelWork &W,
                                 unsigned *d_round_err, const CtSpace &cs, const uint32_t *d_out, hipStream_t st,
                                 RawSamples raw, size_t split_below)
{
    const uint32_t ks_bits = P.ks_t * P.ks_basebit;
    const bool split = gates <= split_below;
    if constexpr (PL::N == HalfPlan::N) {
        // these three kernels are built for three digits per coefficient only
        const RotationKernel kernel = P.l == 3 ? rotation_kernel(gates, K.cus, split_below) : RotationKernel::WAVES;
        if (kernel == RotationKernel::MIXED) {
            const MixedBlocks blocks = mixed_blocks(gates, K.cus, split_below);
            const dim3 grid(blocks.waves + blocks.pairs + blocks.quads);
#define SHE_LAUNCH_MIXED(TRACK, PAIRS)                                                                                \
    hipLaunchKernelGGL((k_blind_rotate_mixed<TRACK, 3, PAIRS>), grid, dim3(64 * BR_WAVES), 0, st, W.bar, W.bar_stride, \
                       P.n, P.bg_bit, K.bk_hat, K.twiddles, K.half_twiddles, ks_bits, W.ext_b, W.ksd, (uint32_t)gates, \
                       blocks, d_round_err, cs, d_out, raw)
            if (blocks.pairs) { if (d_round_err) SHE_LAUNCH_MIXED(true, true); else SHE_LAUNCH_MIXED(false, true); }
            else if (d_round_err) SHE_LAUNCH_MIXED(true, false);
            else SHE_LAUNCH_MIXED(false, false);
#undef SHE_LAUNCH_MIXED
            return hipGetLastError();
        }
        // up to one gate per compute unit: twelve wavefronts per gate (measured beside the kernel)
        if (kernel == RotationKernel::WIDE) {
#define SHE_LAUNCH_WIDE(TRACK)                                                                                        \
    hipLaunchKernelGGL((k_blind_rotate_wide<TRACK>), dim3(K.cus), dim3(768), 0, st, W.bar, W.bar_stride, P.n,         \
                       P.bg_bit, K.bk_hat, K.half_twiddles, ks_bits, W.ext_b, W.ksd, (uint32_t)gates, d_round_err,    \
                       cs, d_out, raw)
            if (d_round_err) SHE_LAUNCH_WIDE(true); else SHE_LAUNCH_WIDE(false);
#undef SHE_LAUNCH_WIDE
            return hipGetLastError();
        }
        // up to two gates per compute unit: four wavefronts per gate (measured beside the kernel)
        if (kernel == RotationKernel::QUAD) {
#define SHE_LAUNCH_QUAD(TRACK)                                                                                        \
    hipLaunchKernelGGL((k_blind_rotate_quad<TRACK, 3>), dim3((unsigned)gates), dim3(256), 0, st, W.bar, W.bar_stride, \
                       P.n, P.bg_bit, K.bk_hat, K.half_twiddles, ks_bits, W.ext_b, W.ksd, d_round_err, cs, d_out, raw)
            if (d_round_err) SHE_LAUNCH_QUAD(true); else SHE_LAUNCH_QUAD(false);
#undef SHE_LAUNCH_QUAD
            return hipGetLastError();
        }
    }
    if (split) {
        // One gate (two wavefronts) or two gates per workgroup.  What counts is the wavefronts on the fullest compute unit;
        // two workgroups of one gate share a SIMD pair badly.  Measured at n=630 on 256 compute units, in ms for 256 / 512
        // / 768 / 1024 / 1280 / 1536 gates, one per workgroup, two per workgroup, and one wavefront per gate:
        //   N=1024, l=2  2.6 / 3.8 / 4.0 / 4.6 / 6.6 / 8.8   3.2 / 3.2 / 5.0 / 5.0 / 7.5 / 7.4   4.7 to 1024, then 7.2 / 7.3
        //   N=512, l=3   1.9 / 2.6 / 2.8 / 3.3 / 4.6 / 6.2   2.3 / 2.3 / 3.7 / 3.7 / 5.5 / 5.5   3.8 to 1024, then 5.9
        //   N=256, l=3   1.4 / 1.8 / 2.1 / 2.5 / 3.1 / 3.7   1.6 / 1.6 / 2.5 / 2.6 / 3.6 / 3.6   3.4 to 1024, then 4.8
        // (at N=512, l=2 one per workgroup stays ahead at 1536: 3.8 against 4.0).  At N=1024 with l=3 launches of up to two
        // gates per compute unit run on twelve or four wavefronts each, those of up to three and of five to six go to the
        // mixed kernel, and one per workgroup is the only form: 769 to 1024 gates (900: 5.65 ms, two per workgroup 6.2), and
        // above them, with SHE_OPT_SPLIT_BELOW raised, what the mixed kernel does not take.
        const size_t per_cu = (gates + K.cus - 1) / std::max<uint32_t>(K.cus, 1);
        const bool triple = P.l == 3;
        constexpr bool quads = PL::N == HalfPlan::N;
        const bool two = (per_cu == 2 || per_cu == 6) && !(quads && triple);
        const dim3 grid((unsigned)(two ? (gates + 1) / 2 : gates)), block(two ? 256 : 128);
#define SHE_LAUNCH_SPLIT(TRACK, GB, LR)                                                                               \
    hipLaunchKernelGGL((k_blind_rotate_split<PL, TRACK, GB, LR>), grid, block, 0, st, W.bar, W.bar_stride, P.n, P.l,  \
                       P.bg_bit, K.bk_hat, K.twiddles, ks_bits, W.ext_b, W.ksd, (uint32_t)gates, d_round_err, cs,     \
                       d_out, raw)
        if (triple) {
            if constexpr (quads) {
                if (d_round_err) SHE_LAUNCH_SPLIT(true, 1, 3); else SHE_LAUNCH_SPLIT(false, 1, 3);
            } else if (d_round_err) { if (two) SHE_LAUNCH_SPLIT(true, 2, 3); else SHE_LAUNCH_SPLIT(true, 1, 3); }
            else { if (two) SHE_LAUNCH_SPLIT(false, 2, 3); else SHE_LAUNCH_SPLIT(false, 1, 3); }
        } else {
            if (d_round_err) { if (two) SHE_LAUNCH_SPLIT(true, 2, 0); else SHE_LAUNCH_SPLIT(true, 1, 0); }
            else { if (two) SHE_LAUNCH_SPLIT(false, 2, 0); else SHE_LAUNCH_SPLIT(false, 1, 0); }
        }
#undef SHE_LAUNCH_SPLIT
        return hipGetLastError();
    }
    const uint32_t per_block = BR_WAVES * PL::GPW;
    const dim3 grid((unsigned)((gates + per_block - 1) / per_block)), block(64 * BR_WAVES);
    if (d_round_err)
        hipLaunchKernelGGL((k_blind_rotate<PL, true, 0>), grid, block, 0, st, W.bar, W.bar_stride, P.n, P.l, P.bg_bit,
                           K.bk_hat, K.twiddles, ks_bits, W.ext_b, W.ksd, (uint32_t)gates, d_round_err, cs, d_out, raw);
    else if (P.l == 3)
        hipLaunchKernelGGL((k_blind_rotate<PL, false, 3>), grid, block, 0, st, W.bar, W.bar_stride, P.n, P.l, P.bg_bit,
                           K.bk_hat, K.twiddles, ks_bits, W.ext_b, W.ksd, (uint32_t)gates, d_round_err, cs, d_out, raw);
    else
        hipLaunchKernelGGL((k_blind_rotate<PL, false, 0>), grid, block, 0, st, W.bar, W.bar_stride, P.n, P.l, P.bg_bit,
                           K.bk_hat, K.twiddles, ks_bits, W.ext_b, W.ksd, (uint32_t)gates, d_round_err, cs, d_out, raw);
    return hipGetLastError();
}

hipError_t launch_blind_rotate(const she_params &P, const DeviceKeys &K, const CtSpace &cs, const uint32_t *d_out,
                               size_t gates, const LevelWork &W, unsigned *d_round_err, hipStream_t st, bool mux,
                               size_t split_below)
{
    if (!gates) return hipSuccess;
    if (!K.ks_bytes) d_out = nullptr;      // the generic key switch writes the slot itself
    const RawSamples raw{mux ? W.raw_ext : nullptr, (uint32_t)W.direct};
    switch (P.N) {
    case 256: return blind_rotate_t<Plan256>(P, K, gates, W, d_round_err, cs, d_out, st, raw, split_below);
    case 512: return blind_rotate_t<Plan512>(P, K, gates, W, d_round_err, cs, d_out, st, raw, split_below);
    case 1024: return blind_rotate_t<Plan1024>(P, K, gates, W, d_round_err, cs, d_out, st, raw, split_below);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_mux_combine(const she_params &P, const DeviceKeys &K, const CtSpace &cs, const uint32_t *d_out,
                              size_t muxes, const LevelWork &W, hipStream_t st)
{
    if (!muxes) return hipSuccess;
    hipLaunchKernelGGL(k_mux_combine, dim3((unsigned)muxes), dim3(256), 0, st, W.raw_ext, P.N, P.n,
                       P.ks_t * P.ks_basebit, W.ext_b, W.ksd, cs, K.ks_bytes ? d_out : nullptr, (uint32_t)W.direct);
    return hipGetLastError();
}

hipError_t launch_key_switch(const she_params &P, const DeviceKeys &K, const CtSpace &cs, const uint32_t *d_out,
                             size_t gates, const LevelWork &W, hipStream_t st)
{
    if (!gates) return hipSuccess;
    if (K.ks_bytes) {
        const unsigned per_block = 32 * KSM_TILES * KSM_WAVES;                 // gates per workgroup
        const unsigned gate_blocks = (unsigned)((gates + per_block - 1) / per_block);
        const unsigned col_tiles = K.ks_cols / 32;
        const unsigned split = key_switch_split(P.N, gates, gate_blocks, col_tiles, K.cus);
        if (gates <= KSF_GATES && P.N / split <= KSF_STEPS) {
            hipLaunchKernelGGL(k_key_switch_few, dim3(col_tiles, split), dim3(64 * KSM_WAVES), 0, st, cs, K.ks_bytes, K.ks_cols,
                               W.ksd, d_out, P.N, P.n, (uint32_t)gates, P.N / split);
            return hipGetLastError();
        }
        const dim3 grid(gate_blocks, col_tiles, split);
        hipLaunchKernelGGL(k_key_switch_mfma, grid, dim3(64 * KSM_WAVES), 0, st, cs, K.ks_bytes, K.ks_cols, W.ksd, d_out,
                           P.N, P.n, (uint32_t)gates, P.N / split);              // N / split: a power of two >= 8
        return hipGetLastError();
    }
    const dim3 grid((unsigned)((gates + KS_GROUP - 1) / KS_GROUP), (P.n + 1 + KS_COLS - 1) / KS_COLS);
    hipLaunchKernelGGL(k_key_switch, grid, dim3(KS_COLS), 0, st, cs, K.ks, K.ks_stride, W.ksd, W.ext_b, d_out, P.N,
                       P.ks_t, P.ks_basebit, P.n, (uint32_t)gates);
    return hipGetLastError();
}

hipError_t launch_fresh_samples(const CtSpace &cs, const uint32_t *d_ids, const uint8_t *d_bits, const uint8_t *d_key,
                                uint32_t n, uint64_t stream_base, double sigma, size_t count, uint32_t *d_retry_count,
                                uint32_t *d_retry, hipStream_t st)
{
    if (!count) return hipSuccess;
    hipLaunchKernelGGL(k_fresh_samples, dim3((unsigned)((count + FRESH_WAVES - 1) / FRESH_WAVES)), dim3(64 * (FRESH_WAVES + 1)),
                       0, st, cs, d_ids, d_bits, d_key, n, stream_base, sigma, (uint32_t)count, d_retry_count, d_retry);
    return hipGetLastError();
}
hipError_t launch_phase_bits(const CtSpace &cs, const uint32_t *d_ids, const uint8_t *d_key, uint32_t n, size_t count,
                             uint8_t *d_bits, hipStream_t st)
{
    if (!count) return hipSuccess;
    hipLaunchKernelGGL(k_phase_bits, dim3((unsigned)((count + PHASE_WAVES - 1) / PHASE_WAVES)), dim3(64 * PHASE_WAVES), 0,
                       st, cs, d_ids, d_key, n, (uint32_t)count, d_bits);
    return hipGetLastError();
}
hipError_t launch_clear_words(uint32_t *d_dst, size_t words, hipStream_t st)
{
    if (!words) return hipSuccess;
    const size_t blocks = std::min<size_t>((words + 255) / 256, 1024);
    hipLaunchKernelGGL(k_clear_words, dim3((unsigned)blocks), dim3(256), 0, st, d_dst, (uint32_t)words);
    return hipGetLastError();
}
hipError_t launch_copy_ct(const CtSpace &cs, const uint32_t *d_src_ids, const uint32_t *d_dst_ids, size_t count,
                          uint32_t n, hipStream_t st)
{
    if (!count) return hipSuccess;
    hipLaunchKernelGGL(k_copy_ct, dim3((unsigned)count), dim3(128), 0, st, cs, d_src_ids, d_dst_ids, n);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Scratch of the entry point that allocates nothing (she_eval_gates_device_noalloc): the level's rounded
// samples, extracted bodies and key-switch digits live in this file-scope array instead of allocated
// buffers.  Every GPU that loads the library holds its own 16 MiB copy until the process ends.  In host code
// the array's name is only a stand-in: the device address comes from hipGetSymbolAddress, once per device
// with that device current, and only that pointer is handed to kernels.
// ------------------------------------------------------------------------------------------
constexpr size_t NOALLOC_SCRATCH_BYTES = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

hipError_t noalloc_scratch(int device, void **ptr, size_t *bytes)
{
    constexpr int MAX_DEVICES = 64;
    static void *address[MAX_DEVICES] = {};
    static std::mutex guard;
    if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(guard);
    if (!address[device]) {
        int current = -1;
        hipError_t rc = hipGetDevice(&current);
        if (rc != hipSuccess) return rc;
        if (current != device) return hipErrorInvalidDevice;
        void *p = nullptr;
        rc = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (rc != hipSuccess) return rc;
        if (!p) return hipErrorInvalidSymbol;
        address[device] = p;
    }
    *ptr = address[device];
    *bytes = NOALLOC_SCRATCH_BYTES;
    return hipSuccess;
}

// ------------------------------------------------------------------------------------------
// FP64 issue-rate probe (diagnostic): independent chains of one instruction form, 2 wavefronts per SIMD
// like the blind rotation.  form 0: fma with scalar multiplier and addend (the best case), 1: fma with
// three vector-register operands (the form of the pointwise products), 2: add of two vector registers
// (the butterflies).  form 3: the add stream of form 2 with the blind rotation's memory instructions
// beside it, per 64 additions 6 LDS reads and 3 LDS writes of 16 bytes per lane in the exchange buffer's
// layout and 2 global loads of 16 bytes per lane that stream `src` the way the key rows are streamed
// (the kernel has 6.5, 3.3 and 2.5 per 64 FP64 instructions); every loaded value is consumed by one of
// the 64 additions.  out receives one value per thread so that the chains stay alive.
// ------------------------------------------------------------------------------------------
template <int FORM> __global__ __launch_bounds__(256) void k_fp64_probe(double *out, int iters, double mul, double add,
                                                                        const double2 *__restrict__ src, uint32_t src_rows)
{
    double a[8], b = mul + threadIdx.x * 1e-12, c = add + threadIdx.x * 1e-15;
#pragma unroll
    for (int k = 0; k < 8; k++) a[k] = threadIdx.x * 1e-3 + k;
    if (FORM == 3) {
        __shared__ double2 s_buf[4][8 * 65];
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
        double2 *buf = s_buf[wave];
        for (int e = lane; e < 8 * 65; e += 64) buf[e] = make_double2(0.0, 0.0);
        wave_lds_fence();
        const int rd = (lane & 7) * 65 + (lane >> 3);                      // the transposing read of an exchange
        uint32_t row = (blockIdx.x * 4 + wave) % src_rows;                  // rows of 64 x 16 bytes
        // global loads run four iterations (256 additions) ahead, about as far as the kernel requests its key rows
        double2 g[4][2];
#pragma unroll
        for (int j = 0; j < 4; j++) { g[j][0] = src[(size_t)row * 64 + lane]; g[j][1] = g[j][0]; }
        for (int it = 0; it < iters; it += 4) {
#pragma unroll
            for (int j = 0; j < 4; j++) {
                // 3 stores, 6 loads, 64 additions; loaded values replace c in 16 of the additions
                buf[0 * 65 + lane] = make_double2(a[0], a[1]);
                buf[3 * 65 + lane] = make_double2(a[2], a[3]);
                buf[6 * 65 + lane] = make_double2(a[4], a[5]);
                wave_lds_fence();
                double2 v[6];
#pragma unroll
                for (int q = 0; q < 6; q++) v[q] = buf[rd + q * 8];
#pragma unroll
                for (int rep = 0; rep < 6; rep++)
#pragma unroll
                    for (int k = 0; k < 8; k++) a[k] = a[k] + c;
                wave_lds_fence();
#pragma unroll
                for (int q = 0; q < 6; q++) { a[q] = a[q] + v[q].x; a[q + 2] = a[q + 2] + v[q].y; }
                a[0] = a[0] + g[j][0].x; a[1] = a[1] + g[j][0].y; a[2] = a[2] + g[j][1].x; a[3] = a[3] + g[j][1].y;
                row = row + 2 < src_rows ? row + 2 : 0;
                g[j][0] = src[(size_t)row * 64 + lane];
                g[j][1] = src[(size_t)(row + 1) * 64 + lane];
            }
        }
    } else {
        for (int it = 0; it < iters; it++) {
#pragma unroll
            for (int rep = 0; rep < 8; rep++)
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    if (FORM == 0) a[k] = __builtin_fma(a[k], mul, add);
                    if (FORM == 1) a[k] = __builtin_fma(a[k], b, c);
                    if (FORM == 2) a[k] = a[k] + c;
                }
        }
    }
    double sum = 0;
#pragma unroll
    for (int k = 0; k < 8; k++) sum += a[k];
    out[blockIdx.x * blockDim.x + threadIdx.x] = sum;
}

// LDS throughput probe: every lane moves 16 bytes per operation, eight operations per iteration, in the exchange
// buffer's layout; ROW = slots per row.  PATTERN 0: loads of consecutive slots, 1: stores of consecutive slots,
// 2: loads at a*ROW + b + 8m for lane 8a + b, 3: loads at b*ROW + 8a + m.
template <int PATTERN, int ROW> __global__ __launch_bounds__(256) void k_lds_probe(uint32_t *out, int iters)
{
    __shared__ uint4 buf[4][8 * ROW];
    const int wave = threadIdx.x >> 6, t = threadIdx.x & 63, a = t >> 3, b8 = t & 7;
    uint4 acc = make_uint4(t, 1, 2, 3);
    uint4 *b = buf[wave];
    for (int k = t; k < 8 * ROW; k += 64) b[k] = acc;
    wave_lds_fence();
    for (int i = 0; i < iters; i++) {
#pragma unroll
        for (int m = 0; m < 8; m++) {
            if (PATTERN == 1) { acc.x += i; b[m * ROW + t] = acc; continue; }
            const uint4 v = PATTERN == 0 ? b[m * ROW + t] : PATTERN == 2 ? b[a * ROW + b8 + 8 * m] : b[b8 * ROW + 8 * a + m];
            acc.x += v.x; acc.y ^= v.y; acc.z += v.z; acc.w ^= v.w;
        }
        wave_lds_fence();
    }
    out[blockIdx.x * 256 + threadIdx.x] = acc.x ^ acc.y ^ acc.z ^ acc.w;
}

hipError_t launch_lds_probe(int form, uint32_t *d_out, uint32_t blocks, int iters, hipStream_t st)
{
    constexpr int ROW0 = Plan1024::xrow(0), ROW1 = Plan1024::xrow(1);
    switch (form) {
    case 0: hipLaunchKernelGGL((k_lds_probe<0, ROW1>), dim3(blocks), dim3(256), 0, st, d_out, iters); break;
    case 1: hipLaunchKernelGGL((k_lds_probe<1, ROW1>), dim3(blocks), dim3(256), 0, st, d_out, iters); break;
    case 2: hipLaunchKernelGGL((k_lds_probe<2, ROW0>), dim3(blocks), dim3(256), 0, st, d_out, iters); break;
    case 3: hipLaunchKernelGGL((k_lds_probe<2, 65>), dim3(blocks), dim3(256), 0, st, d_out, iters); break;
    case 4: hipLaunchKernelGGL((k_lds_probe<3, ROW1>), dim3(blocks), dim3(256), 0, st, d_out, iters); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_fp64_probe(int form, double *d_out, uint32_t blocks, int iters, const double2 *src, uint32_t src_rows,
                             hipStream_t st)
{
#define SHE_LAUNCH_PROBE(F) hipLaunchKernelGGL(k_fp64_probe<F>, dim3(blocks), dim3(256), 0, st, d_out, iters, 1.0000001, 1e-9, src, src_rows)
    switch (form) {
    case 0: SHE_LAUNCH_PROBE(0); break;
    case 1: SHE_LAUNCH_PROBE(1); break;
    case 2: SHE_LAUNCH_PROBE(2); break;
    case 3: if (!src || src_rows < 4) return hipErrorInvalidValue; SHE_LAUNCH_PROBE(3); break;
    default: return hipErrorInvalidValue;
    }
#undef SHE_LAUNCH_PROBE
    return hipGetLastError();
}

}  // namespace she
