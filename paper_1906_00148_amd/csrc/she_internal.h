// Internal declarations shared by the host files and the kernel file of the library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string>
#include <vector>

#include "../../include/she.h"

namespace she {

constexpr int KS_GROUP = 32;        // gates whose key-switch digits are stored together / share one key-switch block
constexpr int MAX_LEVEL_CHUNK = 32768;  // gates per kernel launch; larger levels are cut into chunks

inline uint32_t round_up(uint32_t v, uint32_t m) { return (v + m - 1) / m * m; }

// Everything a kernel needs to find ciphertexts: ids below `cap` are pool slots, ids from
// `cap` on are slots of the internal temporary buffer (slot 0 = trivial 0, slot 1 = trivial 1).
struct CtSpace {
    uint32_t *pool;
    uint32_t *temp;
    uint32_t cap;
    uint32_t stride;   // words per slot (n+1 rounded up to 32)
};

struct DeviceKeys {
    double2 *bk_hat = nullptr;    // [n][2l][2][P][L] spectra of the bootstrapping key
    uint32_t *ks = nullptr;       // [N][t][base-1][ks_stride]; only for key-switch shapes without an MFMA kernel
    int8_t *ks_bytes = nullptr;   // [N][4 byte planes][ks_cols][32 = 8 digits x 4 values] signed bytes (base 4, t = 8)
    uint32_t ks_cols = 0;         // n+1 rounded up to 32
    double2 *twiddles = nullptr;  // [K-1][P][L]
    double2 *half_twiddles = nullptr;   // table of the half transforms (N = 1024)
    uint32_t ks_stride = 0;
    uint32_t cus = 1;             // compute units of the device (launch shaping)
};

struct LevelWork {                // scratch of one level launch, sized for `gates` gates
    uint16_t *bar = nullptr;      // [gates][bar_stride]: abar_0..abar_{n-1}, bbar
    uint32_t *ext_b = nullptr;    // [gates] body of the extracted sample
    uint16_t *ksd = nullptr;      // [gates/KS_GROUP][N][KS_GROUP] rounded top bits of the extracted mask
    uint32_t bar_stride = 0;
    size_t gates = 0;
    uint32_t *raw_ext = nullptr;  // [jobs][N+1] extracted samples of MUX rotations (not yet key-switched)
    size_t raw_jobs = 0;
    size_t direct = 0;            // gates of a launch; its rotations from there on belong to MUXes, two each
};

// ---- kernel launchers (she_kernels.hip); each returns a hipError_t and never synchronises ----
bool plan_supported(uint32_t N);
size_t twiddle_doubles(uint32_t N);
void fill_twiddles(uint32_t N, double *host_out);
size_t half_twiddle_doubles(uint32_t N);    // 0: no half transforms at this ring degree
void fill_half_twiddles(double *host_out);
size_t bk_hat_elems(const she_params &P);   // number of double2 in DeviceKeys::bk_hat

hipError_t launch_bk_transform(const she_params &P, const uint32_t *d_bk_int, const DeviceKeys &K, hipStream_t st);
// leveled mode: spectra of `samples` TRGSW samples d_int[s][2l][2][N] into slots d_ids[s] of trgsw_hat; CMux batch
hipError_t launch_trgsw_transform(const she_params &P, const DeviceKeys &K, const uint32_t *d_int, double2 *trgsw_hat,
                                  const uint32_t *d_ids, size_t samples, hipStream_t st);
// Levels of so few CMuxes have their id lists in the kernel's arguments: 3 KB of the 4 that HIP takes, a round number and not
// where the gain ends (a call of 192 / 193 entries takes 21.4 / 25.0 us at N = 1024, 32.1 / 36.0 at N = 2048; four lists of
// about 240 entries would still fit).
constexpr size_t CMUX_ARG_IDS = 192;
inline bool cmux_ids_in_arguments(uint32_t N, size_t count, uint32_t cus)
{
    return (N == 1024 || N == 2048) && count <= CMUX_ARG_IDS && count <= 2 * (size_t)cus;
}
struct CmuxIds { uint32_t id[4][CMUX_ARG_IDS]; };                   // sel, in1, in0, out
// The whole block is handed to the device: places without an entry are cleared, since what the host's memory held there,
// key bits perhaps, is nothing that a kernel's arguments should keep.
inline void fill_cmux_ids(CmuxIds &ids, const uint32_t *sel, const uint32_t *in1, const uint32_t *in0, const uint32_t *out,
                          size_t count)
{
    const uint32_t *const lists[4] = {sel, in1, in0, out};
    for (int q = 0; q < 4; q++)
        for (size_t k = 0; k < CMUX_ARG_IDS; k++) ids.id[q][k] = k < count ? lists[q][k] : 0;
}
// The four lists: host memory, read before the call returns, if cmux_ids_in_arguments(P.N, count, K.cus); device memory if not.
hipError_t launch_cmux(const she_params &P, const DeviceKeys &K, const double2 *trgsw_hat, uint32_t *trlwe,
                       const uint32_t *sel, const uint32_t *in1, const uint32_t *in0, const uint32_t *out, size_t count,
                       unsigned *d_round_err, hipStream_t st);
// Reads of so few samples have their ids in the kernel's arguments: 1 KB of the 4 that HIP takes.
constexpr size_t GATHER_ARG_IDS = 256;
struct GatherIds { uint32_t id[GATHER_ARG_IDS]; };
inline bool gather_ids_in_arguments(size_t count) { return count <= GATHER_ARG_IDS; }
// samples ids[0 .. count) of the pool -> d_dst [count][2][N] in the order of their coefficients; the list: host memory, read
// before the call returns, if gather_ids_in_arguments(count); device memory if not
hipError_t launch_trlwe_gather(const uint32_t *trlwe, uint32_t *d_dst, const uint32_t *ids, size_t count, uint32_t N,
                               hipStream_t st);
// d_in2 may be null when no type is a three-input gate
hipError_t launch_lincomb(const she_params &P, const CtSpace &cs, const uint8_t *d_type, const uint32_t *d_in0,
                          const uint32_t *d_in1, const uint32_t *d_in2, size_t gates, const LevelWork &W, hipStream_t st);
// Workgroups of 256 threads that k_blind_rotate_mixed runs a launch with, in this order: four gates on a wavefront each, two
// gates on two wavefronts each (the last pair may have one), one gate on four; none at all: not a launch for that kernel.  Two
// workgroups are resident on a compute unit.  Whole rounds of four gates per compute unit go to wavefronts; of the rest, up to
// one gate per compute unit goes to quads and up to two to pairs, one workgroup per compute unit either way, and up to three
// to a pair and a quad per compute unit, which beyond ONE round would leave most compute units three workgroups of different
// length (1700 gates: 11.1 ms against 10.0).  The two sides of the other lines are measured beside the kernel.
struct MixedBlocks { uint32_t waves = 0, pairs = 0, quads = 0; };
inline MixedBlocks mixed_blocks(size_t gates, uint32_t cus, size_t split_below)
{
    const size_t rounds = gates / (4 * (size_t)cus), rest = gates % (4 * (size_t)cus);
    MixedBlocks b;
    if (!rest || rest > split_below) return b;
    if (rounds && rest <= cus) b.quads = (uint32_t)rest;
    else if (rounds && rest <= 2 * (size_t)cus) b.pairs = (uint32_t)((rest + 1) / 2);
    else if (rounds != 1 && rest > 2 * (size_t)cus && rest <= 3 * (size_t)cus) {
        b.pairs = (uint32_t)((rest - cus + 1) / 2);
        b.quads = (uint32_t)rest - 2 * b.pairs;
    } else return b;
    b.waves = (uint32_t)(rounds * cus);
    return b;
}
// Which kernel a launch of that many rotations gets at N = 1024 with l = 3 (measured beside each of them).
enum class RotationKernel { WIDE, QUAD, SPLIT, MIXED, WAVES };
inline RotationKernel rotation_kernel(size_t gates, uint32_t cus, size_t split_below)
{
    const MixedBlocks b = mixed_blocks(gates, cus, split_below);
    if (b.pairs + b.quads) return RotationKernel::MIXED;
    if (gates > split_below) return RotationKernel::WAVES;
    return gates <= cus ? RotationKernel::WIDE : gates <= 2 * (size_t)cus ? RotationKernel::QUAD : RotationKernel::SPLIT;
}
hipError_t launch_blind_rotate(const she_params &P, const DeviceKeys &K, const CtSpace &cs, const uint32_t *d_out,
                               size_t gates, const LevelWork &W, unsigned *d_round_err /* nullptr = no tracking */,
                               hipStream_t st, bool mux = false /* rotations from W.direct on write W.raw_ext instead of digits
                                                                   and slots */,
                               size_t split_below = 0 /* levels, and rests beyond full rounds, of at most this many
                                                        gates may run on several wavefronts per gate */);
// MUX m: sample = raw_ext[2m] + raw_ext[2m+1] + (0, 1/8) -> key-switch digits, body and slot initialisation of the level's
// entry W.direct + m (d_out: the ids of all the level's entries)
hipError_t launch_mux_combine(const she_params &P, const DeviceKeys &K, const CtSpace &cs, const uint32_t *d_out,
                              size_t muxes, const LevelWork &W, hipStream_t st);
// Workgroups among which k_key_switch_mfma splits the range of N coefficients (`gate_blocks` x `col_tiles` of them for every
// split): the power of two with the least estimated time.  Three workgroups fit a compute unit; a step (one coefficient)
// takes one alone 0.33 us with the key in the caches and 0.52 with the key from memory, two 0.41 / 0.57 and three 0.6 / 0.62,
// hence 75 and 81 % of a full compute unit's; a round of workgroups costs about four steps more to start and to end; and
// every split adds its sums to the slots atomically, about a step for 9000 gates x column tiles.
// The other sides measured, us, the mean of both places of the key, at n = 630 for 512 / 700 / 1100 / 2048 / 2304 / 4096
// gates: so 64 / 86 / 140 / 175 / 181 / 298, about a thousand workgroups at all sizes 80 / 109 / 150 / 175 / 192 / 298, no
// more than are resident at once 64 / 86 / 140 / 181 / 181 / 319; at n = 1024 for 1 / 513 / 2048: 49 / 132 / 278, 49 / 132 /
// 295, 51 / 148 / 319; at n = 4096 for 1 / 513 / 1536: 135 / 400 / 775, 161 / 438 / 864, 170 / 543 / 1077.
inline uint32_t key_switch_split(uint32_t N, size_t gates, uint32_t gate_blocks, uint32_t col_tiles, uint32_t cus)
{
    constexpr uint64_t RESIDENT = 3, STEP[RESIDENT] = {0, 75, 81}, FULL = 100, ROUND = 4 * FULL, PER_ADDED = 9000 / FULL;
    uint64_t least = ~(uint64_t)0;
    uint32_t best = 1;
    for (uint32_t split = 1; split <= 32 && N / split >= 8; split *= 2) {
        const uint64_t per_cu = ((uint64_t)gate_blocks * col_tiles * split + cus - 1) / (cus ? cus : 1);
        const uint64_t full = per_cu / RESIDENT, rest = per_cu % RESIDENT;
        const uint64_t time = N / split * (full * FULL + STEP[rest]) + (full + (rest > 0)) * ROUND + split * gates * col_tiles / PER_ADDED;
        if (time < least) { least = time; best = split; }
    }
    return best;
}
hipError_t launch_key_switch(const she_params &P, const DeviceKeys &K, const CtSpace &cs, const uint32_t *d_out,
                             size_t gates, const LevelWork &W, hipStream_t st);
// fresh encryptions of d_bits under the key bits d_key into the slots d_ids (stream_base: fresh_stream_base); samples whose
// error the host has to add (fresh_error) are listed in d_retry, *d_retry_count of them (zeroed by the caller)
hipError_t launch_fresh_samples(const CtSpace &cs, const uint32_t *d_ids, const uint8_t *d_bits, const uint8_t *d_key,
                                uint32_t n, uint64_t stream_base, double sigma, size_t count, uint32_t *d_retry_count,
                                uint32_t *d_retry, hipStream_t st);
// decryptions: d_bits[k] = sign of the phase of slot d_ids[k]
hipError_t launch_phase_bits(const CtSpace &cs, const uint32_t *d_ids, const uint8_t *d_key, uint32_t n, size_t count,
                             uint8_t *d_bits, hipStream_t st);
// zeroes `words` (< 2^32 - 2^18) words
hipError_t launch_clear_words(uint32_t *d_dst, size_t words, hipStream_t st);
// diagnostic: `blocks` workgroups of 256 threads, each thread 64*iters dependent-free FP64 instructions of one form
hipError_t launch_fp64_probe(int form, double *d_out, uint32_t blocks, int iters, const double2 *src, uint32_t src_rows,
                             hipStream_t st);
hipError_t launch_lds_probe(int form, uint32_t *d_out, uint32_t blocks, int iters, hipStream_t st);
hipError_t launch_copy_ct(const CtSpace &cs, const uint32_t *d_src_ids, const uint32_t *d_dst_ids, size_t count,
                          uint32_t n, hipStream_t st);

// Device address and size of the static scratch buffer on `device` (which must be the current device); looked up
// once per device and kept.  The buffer belongs to the loaded code object: it is never freed.
hipError_t noalloc_scratch(int device, void **ptr, size_t *bytes);

// ---- host-side key material and samples (she_host.cpp) ----
struct HostKeys {
    std::vector<uint8_t> lwe_key, ring_key;
    std::vector<uint32_t> bk;    // [n][2][l][2][N]
    std::vector<uint32_t> ks;    // [N][t][base-1][n+1]
};
void generate_keys(const she_params &P, uint64_t seed, HostKeys &out);
// fresh encryptions: sample k's stream has the key finalise(fresh_stream_base + k); fresh_error is its rounded error
uint64_t fresh_stream_base(uint64_t enc_seed);
uint32_t fresh_error(const she_params &P, uint64_t enc_seed, uint64_t k);
// key-switching key as signed byte planes for the MFMA kernel: out[i][plane][col][j*4+v]
void pack_ks_bytes(const she_params &P, const std::vector<uint32_t> &ks, uint32_t cols_p, std::vector<int8_t> &out);
// leveled mode: fresh TRGSW samples of bits [count][2][l][2][N], fresh TRLWE samples of mu[count][N] as [count][2][N]
// (noise bk_std, or none), phases B - A*s' of TRLWE samples
void fresh_trgsw(const she_params &P, const std::vector<uint8_t> &ring_key, const uint8_t *bits, size_t count,
                 uint64_t seed, uint32_t *out);
void fresh_trlwe(const she_params &P, const std::vector<uint8_t> &ring_key, const uint32_t *mu, size_t count,
                 uint64_t seed, uint32_t *out);
void trlwe_phases(const she_params &P, const std::vector<uint8_t> &ring_key, const uint32_t *cts, size_t count,
                  uint32_t *phases);

// ---- netlists of the layer operators (she_circuits.cpp) ----
constexpr uint32_t WIRE_NEG = 0x80000000u;   // flag on a wire reference: the complement of that wire
constexpr int MUX_BASE = SHE_NUM_GATES;       // netlist type of a native MUX entry: MUX_BASE + 16*code1 + code0 (< SHE_MAJ3)
inline bool is_mux_type(uint8_t t) { return t >= MUX_BASE && t < SHE_MAJ3; }
inline bool has_third_operand(uint8_t t) { return t >= MUX_BASE; }     // MUX entries and three-input gates

// Estimated time of a level, in microseconds at N = 1024 and l = 3, from its rotations per compute unit: the steps of the
// kernels that launch_blind_rotate chooses, as measured at n = 630 on 256 compute units (a launch of 256 / 512 / 768 / 1024 /
// 1536 / 2048 / 3072 / 4096 rotations takes 1.85 / 3.5 / 4.05 / 5.85 / 7.65 / 10.35 / 16.05 / 20.05 ms, one rotation more 3.35 /
// 3.95 / 5.5 / 6.1 / 9.75 / 11.95 / 16.05 / 20.95), with 0.1 ms for its other kernels.  Only ratios count, so that other key
// lengths are served as well.
double level_time(uint64_t rotations, uint32_t cus);
double level_time(uint64_t gates, uint64_t mux_rotations, uint32_t cus);       // in one launch or two: see launches_apart
bool level_time_holds(const she_params &P, uint32_t cus, size_t split_below);  // the kernels are the ones that it knows
// Whether the rotations of a level's gates and those of its MUXes run in two launches, one after the other, because together
// they would take longer: where the sum just exceeds what runs on several wavefronts per rotation, or a number of full rounds.
// Measured at n = 630 on 256 compute units, ms, one launch / two: N = 1024, l = 3: 1030 gates and 255 MUXes 9.45 / 9.30,
// 1157 and 579 13.8 / 12.5, but 600 and 400 7.3 / 9.3; l = 2: 2048 and 64 12.4 / 11.0, 250 and 128 3.1 / 5.1; N = 512, l = 3:
// 3000 and 40 12.3 / 11.0; N = 256, l = 3: 800 and 370 4.85 / 4.55, 2048 and 64 6.9 / 6.1, 250 and 128 1.55 / 2.6.
bool launches_apart(const she_params &P, uint64_t gates, uint64_t mux_rotations, uint32_t cus, size_t split_below);
struct Netlist {
    // wire ids: [0, cap) pool slots, cap = trivial 0, cap+1 = trivial 1, cap+2.. temporaries.
    // With `fold` set, a gate fixed by constant or repeated operands is not emitted: gate()
    // returns a constant, an operand, or an operand with WIRE_NEG (complementing a ciphertext
    // is a free negation of its words), and complemented operands of a real gate are absorbed
    // into the gate code.
    uint32_t cap = 0;
    uint32_t next_temp = 0;
    bool fold = false;
    bool native_mux = false;                    // mux() emits one three-input entry instead of three gates
    bool cells3 = false;                        // adders use cells of two three-input gates (parity, majority)
    bool columns = false;                       // shift-accumulate sums by column compression (nl_columns)
    bool overflow = false;                      // more wires than 31-bit ids can name
    std::vector<uint8_t> type;
    std::vector<uint32_t> in0, in1, in2, out;   // in2: third operand of MUX entries and three-input gates (0 otherwise)
    std::vector<uint32_t> copy_src, copy_dst;   // executed after all gates; copy_src may carry WIRE_NEG

    explicit Netlist(uint32_t capacity, bool fold_constants = false, bool mux_native = false, bool cells3 = false,
                     bool columns = false)
        : cap(capacity), next_temp(capacity + 2), fold(fold_constants), native_mux(mux_native), cells3(cells3),
          columns(columns) {}
    uint64_t rotations() const;                 // blind rotations: one per gate, two per MUX entry
    uint32_t zero() const { return cap; }
    uint32_t one() const { return cap + 1; }
    uint32_t gate(int code, uint32_t a, uint32_t b);
    uint32_t mux(uint32_t s, uint32_t u, uint32_t v);
    // majority (base SHE_MAJ3) or parity (base SHE_XOR3) of three wires with one bootstrap
    uint32_t gate3(int base, uint32_t a, uint32_t b, uint32_t c);
    // route the wires in `wires` to the caller's ids `dst`: gate outputs are renamed,
    // anything else (inputs, constants, a wire used twice) is copied at the end
    void bind_outputs(const std::vector<uint32_t> &wires, const uint32_t *dst);
    // stable sort of the entries by (depth, gates before MUX entries); returns the first index of each
    // level (+ end); mux_start[lv] receives the index of level lv's first MUX entry.  With cus > 0 the levels, no more of them,
    // are evened out for a device of that many compute units (see even_levels); if they are, *unsorted receives the netlist as
    // it was, for a caller that may have to fall back on the earliest levels.
    std::vector<size_t> levelize(std::vector<size_t> *mux_start = nullptr, uint32_t cus = 0, Netlist *unsorted = nullptr);
    // Levels that move entries for which later ones have time out of levels that they only just push over a step of level_time;
    // empty where the estimate gains nothing.  `lev`: the earliest level of every entry, 1 .. deepest, the entries still in
    // topological order.
    std::vector<uint32_t> even_levels(const std::vector<uint32_t> &lev, uint32_t deepest, uint32_t cus) const;
    // after levelize and bind_outputs: re-numbers the remaining temporaries so that slots are reused once their last
    // reader's level has run; `bounds` are levelize's.  Returns the slots needed (constants included), 0 on an
    // internal inconsistency.
    size_t compact_temporaries(const std::vector<size_t> &bounds);
};
std::vector<uint32_t> nl_add(Netlist &nl, const std::vector<uint32_t> &a, const std::vector<uint32_t> &b, uint32_t cap_bits);
std::vector<uint32_t> nl_sub(Netlist &nl, const std::vector<uint32_t> &p, const std::vector<uint32_t> &q);
std::vector<uint32_t> nl_tree(Netlist &nl, std::vector<std::vector<uint32_t>> terms, uint32_t in_bits, uint32_t acc_bits);
std::vector<uint32_t> nl_max(Netlist &nl, const std::vector<uint32_t> &x, const std::vector<uint32_t> &y);
// signed sum of unsigned terms (wires LSB first, no padding; sign +1 / -1) mod 2^acc_bits by column compression;
// the netlist must fold constants and use three-input cells
struct SignedTerm { std::vector<uint32_t> bits; int sign; };
std::vector<uint32_t> nl_columns(Netlist &nl, const std::vector<SignedTerm> &terms, uint32_t acc_bits, int64_t bias = 0);
std::vector<uint32_t> nl_constant(Netlist &nl, int64_t value, uint32_t bits);   // trivial wires of a plaintext integer

}  // namespace she
