// Size dispatch: picks the kernel whose register arrays fit n.
#include "bed.h"
#include "bed_kernel.h"

namespace bed {

hipError_t launch_lane(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_packed(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_pair(const KernelArgs&, hipStream_t);
hipError_t launch_packed_rows(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_wave_n4(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_wave_n8(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_wave_n12(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_wave_n16(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_wave_n20(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_wave_n24(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_wave_n28(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_wave_n32(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_wave_n40(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_wave_n48(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_wave_n56(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_wave_n64(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_block(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_dc_wave(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_dc_block(const KernelArgs&, int, bool, hipStream_t);
hipError_t launch_spectral(const KernelArgs&, hipStream_t);

namespace {

constexpr int kPackedFromBatch = 2560;
constexpr int kPackedRowsFromBatch = 4096;
constexpr int kPackedRowsValuesFromBatch = 3072;   // eigenvalues only
constexpr int kPairUpToBatch = 512;
constexpr int kLane4FromBatch = 20480;
constexpr int kLane8FromBatch = 32768;
constexpr int kLane3BeatsJacobi = 147456;
constexpr int kLane4BeatsJacobi = 196608;

enum Family { kLaneFamily, kPackedFamily, kWaveFamily, kPairFamily, kBlockFamily, kPackedRowsFamily };
struct Choice {
    Family family;
    int N;               // register-array size of the instantiation (0 for the block kernel)
    const char* name;
};

Choice wave_choice(int n);

// Which kernel of Givens rotations serves a problem.  `forced` (kFamilyAuto unless a test
// or a measurement asks for one family) must be able to serve n: the caller has checked.
Choice choose(int batch, int n, int stage, bool want_v, int forced) {
    if (forced == kFamilyLane) return n <= 4 ? Choice{kLaneFamily, 4, "lane_kernel<4>"} : Choice{kLaneFamily, 8, "lane_kernel<8>"};
    if (forced == kFamilyPacked) {
        if (n <= 4) return {kPackedFamily, 4, "packed_kernel<4>"};
        if (n <= 8) return {kPackedFamily, 8, "packed_kernel<8>"};
        if (n <= 12) return {kPackedFamily, 12, "packed_kernel<12>"};
        if (n <= 16) return {kPackedFamily, 16, "packed_kernel<16>"};
        if (n <= 24) return {kPackedFamily, 24, "packed_kernel<24>"};
        return {kPackedFamily, 32, "packed_kernel<32>"};
    }
    if (forced == kFamilyWave) return wave_choice(n);
    if (forced == kFamilyPair) return {kPairFamily, 0, n <= 40 ? "pair_kernel<40>" : n <= 48 ? "pair_kernel<48>" : n <= 56 ? "pair_kernel<56>" : "pair_kernel<64>"};
    if (forced == kFamilyBlock) return {kBlockFamily, 0, "block_kernel"};
    if (forced == kFamilyPackedRows) {
        if (n <= 20) return {kPackedRowsFamily, 20, "packed_rows_kernel<20>"};
        if (n <= 24) return {kPackedRowsFamily, 24, "packed_rows_kernel<24>"};
        if (n <= 28) return {kPackedRowsFamily, 28, "packed_rows_kernel<28>"};
        return {kPackedRowsFamily, 32, "packed_rows_kernel<32>"};
    }
    // Measured crossovers on MI355X (us per launch, eigenvectors on; wave / packed / lane):
    //   n = 4:  batch 2048: 8.4 / 8.6 / 13.0   4096: 11.5 / 9.1 / 13.7   16384: 27.7 / 13.2 / 14.2   32768: 49 / 21.7 / 14.9
    //   n = 8:  batch 2048: 17.2 / 17.8 / 49.5  4096: 25.3 / 18.0 / 49.4  32768: 127 / 58.1 / 56.6    65536: 231 / 96.9 / 57.6
    //   n = 16: batch 2048: 34.1 / 36.3         3072: 42.6 / 35.4         4096: 51.6 / 35.5           16384: 152 / 76.7
    //   n = 24: batch 2048: 73.4 / 80.4         3072: 93.7 / 97.0         4096: 112 / 100             16384: 356 / 289
    //   n = 32: batch 2048: 115 / 123           3072: 145 / 161           4096: 179 / 163             16384: 571 / 496
    // Below kPackedFromBatch the chip is not full and one wavefront per matrix, whose per-matrix
    // latency is lowest, finishes first.  Then four matrices per wavefront (n <= 16) share the
    // instructions of the scalar recurrence.  For tiny matrices in very large batches one matrix per
    // lane (64 per wavefront) has no redundant work at all, but a latency several times higher.
    // The fused spectral function follows the same choice; the stage hooks stay with one wavefront
    // per matrix.
    const bool whole = (stage == kFull || stage == kSpectral);
    if (whole && n <= 4 && batch >= kLane4FromBatch) return {kLaneFamily, 4, "lane_kernel<4>"};
    if (whole && n <= 8 && batch >= kLane8FromBatch) return {kLaneFamily, 8, "lane_kernel<8>"};
    if (whole && n <= 16 && batch >= kPackedFromBatch) return choose(batch, n, stage, want_v, kFamilyPacked);
    // 16 < n <= 32, from batch 4096 (us per launch, wave / two per wavefront / four per wavefront with
    // two rows per lane:
    //   n = 20: batch 3072: 72.8 / 80.5 / 75.3   4096: 87.5 / 80.6 / 74.7   8192: 146 / 124 / 97    16384: 264 / 220 / 195
    //   n = 24: batch 3072: 93.6 / 97.5 / 96.3   4096: 115 / 101 / 95       8192: 193 / 163 / 129   16384: 355 / 288 / 238
    //   n = 28: batch 3072: 119 / 130 / 125      4096: 145 / 131 / 124      8192: 247 / 232 / 165   16384: 456 / 400 / 309
    //   n = 32: batch 3072: 148 / 162 / 152      4096: 180 / 163 / 152      8192: 309 / 275 / 205   16384: 571 / 488 / 379):
    // four matrices per wavefront, also for the fused spectral function up to the 26 rows for which the rotations
    // give it (divide and conquer beyond); two per wavefront remains for forced-family runs
    // (eigenvalues only, n = 32: batch 3072: 125 / 109 / 95   4096: 149 / 108 / 94   16384: 479 / 379 / 230)
    if (whole && n > 16 && n <= 32 && batch >= (want_v ? kPackedRowsFromBatch : kPackedRowsValuesFromBatch))
        return choose(batch, n, stage, want_v, kFamilyPackedRows);
    // 32 < n <= 64 with eigenvectors while the chip is mostly idle: two wavefronts per matrix
    // (us per launch, wave / pair: n = 48: batch 256: 175 / 165, 512: 179 / 168, 768: 179 / 203;
    //  n = 64: batch 256: 285 / 274, 512: 293 / 274, 768: 290 / 327)
    if (stage == kFull && want_v && n > 32 && n <= 64 && batch <= kPairUpToBatch) return choose(batch, n, stage, want_v, kFamilyPair);
    if (n <= 64) return wave_choice(n);
    return {kBlockFamily, 0, "block_kernel"};     // 64 < n <= 128: four wavefronts per matrix
}

Choice wave_choice(int n) {
    if (n <= 4) return {kWaveFamily, 4, "wave_kernel<4>"};
    if (n <= 8) return {kWaveFamily, 8, "wave_kernel<8>"};
    if (n <= 12) return {kWaveFamily, 12, "wave_kernel<12>"};
    if (n <= 16) return {kWaveFamily, 16, "wave_kernel<16>"};
    if (n <= 20) return {kWaveFamily, 20, "wave_kernel<20>"};
    if (n <= 24) return {kWaveFamily, 24, "wave_kernel<24>"};
    if (n <= 28) return {kWaveFamily, 28, "wave_kernel<28>"};
    if (n <= 32) return {kWaveFamily, 32, "wave_kernel<32>"};
    if (n <= 40) return {kWaveFamily, 40, "wave_kernel<40>"};
    if (n <= 48) return {kWaveFamily, 48, "wave_kernel<48>"};
    if (n <= 56) return {kWaveFamily, 56, "wave_kernel<56>"};
    return {kWaveFamily, 64, "wave_kernel<64>"};
}

// Divide and conquer serves the calls that want a decomposition and nothing of the rotations: no
// rotation counts, no threshold or sweep cap of the caller, no forced family, no stage hook.
// What it takes hardly depends on the spectrum; the rotations take fewer sweeps for decaying and
// rank-deficient ones.  So the lines lie where the geometric mean over full-rank, decaying and rank-deficient (3 n / 4)
// covariances, in shares of 56, 19 and 25 %, turns.  Measured, time over that of the rotations as chosen
// above, for the three and their mean (eigenvectors on, and the spectral function within 5 % of it):
//   n = 10: batch 16: 1.06 1.26 1.29 = 1.15   512: 0.97 1.20 1.32 = 1.09   2048: 0.93 1.12 1.21 = 1.03
//   n = 11: batch 16: 1.00 1.11 1.32 = 1.09   64: 1.02  256: 0.98  2048: 0.95   (eigenvalues 16: 1.19, 256: 1.07, 2048: 1.04)
//   n = 12: batch 16: 0.86 1.04 1.13 = 0.95   512: 0.77 0.96 1.10 = 0.88   (eigenvalues 16: 1.03, 512: 0.96)
//   n = 16: batch 512: 0.61 0.77 0.87 = 0.70  (us at full rank 31.6 / 19.2)
//   n = 17: batch 512: 0.82 1.03 1.11 = 0.93  2559: 0.81 0.96 1.06 = 0.89  3072: 1.08 1.29 1.41 = 1.19  4095: 1.03 1.25 1.35 = 1.14
//   n = 18: batch 3072: 1.12  3584: 0.96  4095: 1.09   n = 19: 3072: 1.08  3584: 0.92  4095: 1.03   n = 20: batch 2559: 0.75  3072: 1.02  4095: 0.97  4096: 1.11
//   n = 22: batch 2559: 0.72  4095: 0.90  4096: 1.04                       n = 24: batch 2559: 0.65  4096: 0.95
//   n = 25: batch 512: 0.65   6144: 0.98  8192: 1.18  12288: 1.10          n = 27: batch 6144: 0.89  8192: 1.08  12288: 1.00
//   n = 28: batch 8192: 1.03  16384: 1.01                                  n = 32: batch 512: 0.50   8192: 0.90  16384: 0.88
// Eigenvalues only, where four matrices share a wavefront from batch 3072 on:
//   n = 17: batch 3072: 1.01  3584: 1.27   n = 20: 3072: 0.90  3584: 1.10   n = 22: 3072: 0.89  3584: 1.08   n = 24: 4096: 0.97
//   batch 8192 / 16384: n = 25: 1.34 / 1.15   27: 1.25 / 1.05   28: 1.19 / 1.00   29: 1.23 / 1.23   31: 1.14 / 1.13   32: 1.09 / 1.09
//   batch 6144 / 10000: n = 25: 1.09 / 0.97   27: 0.99 / 0.89   28: 0.95 / 0.85   29: 0.98 / 0.98   31: 0.91 / 0.90   32: 0.87 / 0.86
// (its arrays have 28 or 32 rows, so that what n lacks to them counts against it).  Beyond 32 rows one workgroup per
// matrix, three of them on a compute unit for n <= 64 (768 on the chip; five for eigenvalues only):
//   n = 36: batch 512: 0.67 0.86 0.94 = 0.76   768: 0.73 0.90 0.97 = 0.82   2048 (full rank, us): 157 / 221
//   n = 41: batch 768: 0.70  900: 1.11 (eigenvalues 0.83)    n = 44: 768: 0.65  1024: 1.04, the function 1.00 (0.79)    n = 48: 768: 0.62  1024: 0.98
//   n = 48: 4096 (full rank, us): 445 / 495   n = 52: batch 1024: 0.89   n = 53: batch 1536: 0.85  2048: 1.13  2559: 0.93   n = 56: 2048: 1.06
//   n = 64: batch 256: 0.37  2048: 0.62       us at full rank: n = 100, batch 64: 784 / 211   n = 128, batch 256: 1195 / 239
// By these figures the lines were drawn.  Since then divide and conquer has got leaves of four rows, a reduction without P and products
// by blocks, and the rotations have not changed; the lines have not been drawn again, so most lie below where the two sides would
// turn today.  At and below them, for the same three spectra (us at full rank, rotations / divide and conquer):
//   n = 12: batch 16: 0.76 0.87 0.99 (18.1 / 13.7)   256: 0.70 0.85 0.89   n = 16: batch 512: 0.53 0.66 0.78 (32.0 / 17.1)   2559: 0.54 0.68 0.76
//   n = 17: batch 512: 0.76 0.93 1.01   2560: 0.77 0.92 0.97 (58.5 / 45.3)   n = 20: batch 2560: 0.64 0.81 0.84   n = 22: batch 4095: 0.65 0.79 0.86
//   n = 24: batch 4096: 0.68 0.84 0.86 (95.9 / 65.2)   n = 25: batch 6144: 0.74 0.88 0.95   n = 28: batch 16384: 0.82 0.99 1.05
//   n = 32: batch 512: 0.40 0.53 0.55 (84.7 / 34.3)   16384: 0.71 0.88 0.93 (381 / 271)   n = 36: batch 512: 0.53 0.65 0.71   768: 0.56 0.69 0.77 (116 / 65)
//   n = 43: batch 768: 0.42 0.55 0.60   n = 48: batch 1024: 0.64 0.83 0.94 (184 / 117)   n = 52: batch 1024: 0.60 0.78 0.84   n = 53: batch 1536: 0.55 0.74 0.82
//   n = 56: batch 2048: 0.69 0.90 1.01   n = 64: batch 256: 0.24 0.32 0.35 (277 / 65)   2048: 0.39 0.51 0.56   n = 100: batch 64: 0.17 0.22 0.25 (761 / 133)
//   n = 128: batch 256: 0.13 0.17 0.19 (1172 / 153)
// With roots of third order, the reduction's factors as DPP operands and the tiles of the reduction shared, beyond the lines (event-bracketed loops):
//   n = 12: batch 2560: 0.78 0.96 0.99   4096: 0.95 1.15 1.20   n = 14: batch 4096: 0.86 1.05 1.13   n = 16: batch 2560: 0.59 0.73 0.77 (41.3 / 24.5)
//   4096: 0.70 0.90 0.95   6144: 0.78 0.96 1.07   16384: 1.07 1.36 1.42   n = 18: batch 4096: 0.84 1.00 1.07   n = 20: batch 4096: 0.74 0.91 0.93
//   n = 24: batch 6144: 0.62 0.78 0.82   8192: 0.79 0.99 1.04   n = 26: batch 16384: 0.82 0.99 1.06   n = 40: batch 1536: 0.75 0.96 1.06
//   n = 48: batch 1536: 0.58 0.78 0.84   2048: 0.78 1.01 1.13   n = 8 (registers for 8 rows): batch 512: 0.77 0.95 1.00   2560: 0.89 1.06 1.09
// Their means are below one, but for n = 12 at 4096 (1.04) and n = 16 at 16384 (1.20): the two sides turn beyond the lines, above batch 6144 for
// 16 rows, 8192 for 24, 2048 for 48.  The lines below are those of the first figures and have not been moved.
bool divide_and_conquer(const KernelArgs& args, int stage, bool want_v, int forced) {
    if (forced != kFamilyAuto || (stage != kFull && stage != kSpectral)) return false;
    if (args.rotations || args.abs_eps > 0.f || args.sweep_cap) return false;
    const int n = args.n, batch = args.batch;
    if (n <= 10 || (n == 11 && (!want_v || batch < 256)) || (n == 12 && batch < 16)) return false;
    if (n <= 16) return batch < kPackedFromBatch;
    if (n <= 22 && !want_v) return batch <= kPackedRowsValuesFromBatch;
    if (n <= 18) return batch <= kPackedFromBatch;
    if (n <= 22) return batch < kPackedRowsFromBatch;
    if (n <= 24) return batch <= kPackedRowsFromBatch;
    if (n <= 32) return batch <= 6144 || (want_v ? n > 26 : n % 4 == 0);
    if (n <= 40) return batch <= 768;
    if (n <= 52) return batch <= (want_v && n <= 43 ? 768 : 1024);
    return true;
}

// Up to 4 rows the same calls take the Jacobi form of the kernel that choose() names, in one launch also for the spectral function
// with its decomposition.  In very large batches one matrix per lane needs fewer instructions, and for two rows it
// has a single rotation to do.  n = 3 turns at its line; n = 4 and n <= 2 would a little above theirs (us per launch, rotations / Jacobi:
// eigenvectors, eigenvalues only, spectral function):
//   n = 4: batch 65536: 15.6 / 8.5, 11.4 / 5.7, 15.0 / 9.0   196607: 21.2 / 19.8, 15.0 / 12.9, 20.7 / 20.2   262144: 26.0 / 25.3, 18.2 / 16.5,
//          25.2 / 25.8   393216: 37.2 / 38.2, 25.4 / 24.9
//   n = 3: batch 65536: 11.7 / 8.0, 9.3 / 5.8, 11.4 / 8.5   147456: 14.9 / 14.2, 11.1 / 9.5, 14.5 / 14.5   196607: 15.8 / 17.5, 11.8 / 11.7, 15.4 / 18.1
//   n = 2: batch 20479: 5.6 / 4.0, 5.0 / 3.9, 5.8 / 4.0   65536: 5.1 / 4.1, 4.0 / 4.0, 4.7 / 4.2   98304: 5.5 / 5.1, 4.2 / 4.0, 5.3 / 5.4
//          131072: 5.8 / 6.2, 4.4 / 4.3, 5.5 / 6.6   (n = 1: 65536: 4.1 / 4.0   98304: 4.4 / 4.9)
bool jacobi_form(const KernelArgs& args, int stage, int forced) {
    if (args.n > 4 || forced != kFamilyAuto || (stage != kFull && stage != kSpectral)) return false;
    if (args.rotations || args.abs_eps > 0.f || args.sweep_cap) return false;
    if (stage == kSpectral && args.evecs) return true;
    return args.batch < (args.n == 4 ? kLane4BeatsJacobi : args.n == 3 ? kLane3BeatsJacobi : kLane4FromBatch);
}

}  // namespace

const char* kernel_variant(int batch, int n, bool want_v) { return choose(batch, n, kFull, want_v, kFamilyAuto).name; }

// Name of the divide-and-conquer kernel for n: the instantiations of launch_dc_wave and launch_dc_block.
static const char* divide_and_conquer_name(int n) {
    static const char* const wave[] = {"dc_wave_kernel<12>", "dc_wave_kernel<16>", "dc_wave_kernel<20>",
                                       "dc_wave_kernel<24>", "dc_wave_kernel<28>", "dc_wave_kernel<32>"};
    if (n <= 32) return wave[n <= 12 ? 0 : (n + 3) / 4 - 3];
    return n <= 64 ? "dc_block_kernel<64>" : "dc_block_kernel<128>";
}

bool family_serves(int family, int n) {
    switch (family) {
        case kFamilyAuto: return n >= 1 && n <= 128;
        case kFamilyWave: return n >= 1 && n <= 64;
        case kFamilyPacked: return n >= 1 && n <= 32;
        case kFamilyLane: return n >= 1 && n <= 8;
        case kFamilyBlock: return n > 64 && n <= 128;
        case kFamilyPair: return n > 32 && n <= 64;
        case kFamilyPackedRows: return n >= 1 && n <= 32;
        default: return false;
    }
}

hipError_t launch(const KernelArgs& args, int stage, bool want_v, hipStream_t stream, int forced) {
    if (args.batch == 0) return hipSuccess;
    // the parts are larger than any batch at which a rule turns
    if (args.batch > kMostPerLaunch)
        return in_parts(args, [&](const KernelArgs& part) { return launch(part, stage, want_v, stream, forced); });
    if (divide_and_conquer(args, stage, want_v, forced))
        return args.n <= 32 ? launch_dc_wave(args, stage, want_v, stream) : launch_dc_block(args, stage, want_v, stream);
    if (stage == kSpectral && args.evecs && !jacobi_form(args, stage, forced)) {
        // the spectral function and the decomposition it comes from: the rotation kernels keep V on chip
        // for the former or write it for the latter, so a second kernel forms the function
        const hipError_t err = launch(args, kFull, true, stream, forced);
        return err == hipSuccess ? launch_spectral(args, stream) : err;
    }
    const Choice c = choose(args.batch, args.n, stage, want_v, forced);
    if (jacobi_form(args, stage, forced)) stage = stage == kSpectral ? kJacobiSpectral : kJacobi;
    if (c.family == kPairFamily) {
        if (!want_v || stage != kFull) return hipErrorInvalidValue;     // the pair kernels always form eigenvectors
        return launch_pair(args, stream);
    }
    if (c.family == kPackedRowsFamily) {
        if (stage != kFull && stage != kSpectral) return hipErrorInvalidValue;     // no stage hooks
        return launch_packed_rows(args, stage, want_v, stream);
    }
    if (c.family == kLaneFamily) return launch_lane(args, stage, want_v, stream);
    if (c.family == kPackedFamily) return launch_packed(args, stage, want_v, stream);
    if (c.family == kBlockFamily) return launch_block(args, stage, want_v, stream);
    switch (c.N) {
        case 4: return launch_wave_n4(args, stage, want_v, stream);
        case 8: return launch_wave_n8(args, stage, want_v, stream);
        case 12: return launch_wave_n12(args, stage, want_v, stream);
        case 16: return launch_wave_n16(args, stage, want_v, stream);
        case 20: return launch_wave_n20(args, stage, want_v, stream);
        case 24: return launch_wave_n24(args, stage, want_v, stream);
        case 28: return launch_wave_n28(args, stage, want_v, stream);
        case 32: return launch_wave_n32(args, stage, want_v, stream);
        case 40: return launch_wave_n40(args, stage, want_v, stream);
        case 48: return launch_wave_n48(args, stage, want_v, stream);
        case 56: return launch_wave_n56(args, stage, want_v, stream);
        default: return launch_wave_n64(args, stage, want_v, stream);
    }
}

}  // namespace bed

extern "C" const char* bed_syevd_kernel(int batch, int n, int want_vectors) {
    if (batch < 0 || n < 1 || n > BED_MAX_N) return nullptr;
    bed::KernelArgs args{};
    args.batch = batch;
    args.n = n;
    const bool want_v = want_vectors != 0;
    return bed::divide_and_conquer(args, bed::kFull, want_v, bed::kFamilyAuto) ? bed::divide_and_conquer_name(n)
                                                                               : bed::kernel_variant(batch, n, want_v);
}
