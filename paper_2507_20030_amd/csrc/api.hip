// C ABI of libiwdft: descriptor validation, buffer layout, call ordering, error reporting.
// All arithmetic lives in the kernels; this file only decides what to launch.
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <numeric>
#include <new>
#include <vector>

#include "../../include/iwdft.h"
#include "common.h"
#include "fft_core.h"
#include "fft_tab.h"
#include "tables.h"

using namespace iwdft;

// Library-owned scratch of compressed_decode_attn_static: one copy per GPU, allocated by the loader with the
// code object and held until the process ends.  Host code never uses this name as an address (it is a host-side
// stand-in); the per-device address comes from hipGetSymbolAddress, see static_scratch().
constexpr size_t kStaticScratchBytes = (size_t)IWDFT_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
// Token, query and output tensors are read and written with 16-byte accesses.
bool misaligned16(const void* p) { return ((uintptr_t)p & 15u) != 0; }
const char kAlignMsg[] = "a device tensor is not 16-byte aligned";

struct Plan {  // byte offsets inside the two caller buffers, derived from a descriptor
  std::vector<LayerInfo> layers;
  std::vector<uint16_t> fold;  // see Params::fold
  int64_t n_bins_total = 0;
  int64_t coef_total = 0;  // float2 per tensor
  int64_t ws_total = 0;    // float2 per workspace array
  int32_t G = 1, max_nb = 0, max_Bp = 0;
  bool use_fft = false;          // decode attention through power-of-two FFTs
  bool use_any_prefill = false;  // prefill through interpolated transforms
  int pf_logN = 0;               // ... grid of so many points (log2)
  int64_t pf_Pb = 1, pf_A = 0, pf_period = 0;  // blocks, samples of the longest one, frequencies with taps of their own
  bool use_chirp = false;        // ... through chirp-z transforms (any M up to kChirpMaxM when use_fft is false)
  int chirp_logN = 0;            // length of its circular convolutions
  int chirp_logS = 0;            // length of a table that the state buffer used to hold: its bytes stay, for copies of the buffer
  int64_t chirp_Q = 0;           // points per chirp-z transform: M / Pb (M itself up to 8192)
  size_t off_chirp = 0, off_chirpW = 0;
  size_t off_dec = 0, off_taps = 0;  // in the workspace
  int64_t tw_Q = 0;              // length of the transforms whose twiddle octant is at off_tw
  size_t off_tw = 0;
  int64_t reach = 0;             // largest |frequency| kept
  int dec_logN = 0;              // FFT prefill of a decimated grid of so many points (log2; 0: of the tokens themselves)
  int64_t dec_slices = 0;        // slices whose grids the workspace holds at a time
  int low_logN = 0;              // decode attention on a grid of so many points (log2; 0: on the tokens themselves)
  size_t off_dec_w = 0, off_dec_tw = 0, off_dec_gain = 0, off_low = 0, off_low_gain = 0, off_grid = 0;
  bool use_fft_prefill = false;  // prefill through FFTs (else the dense MFMA contraction)
  bool scale_pairs = false;      // ... with the channels of a pair scaled to one size
  int write_every = 1;           // fused decode step: coefficients written back every this many tokens
  size_t off_layers = 0, off_bins = 0, off_weights = 0, off_fold = 0, off_FK = 0, off_FV = 0, state_bytes = 0;
  size_t off_sinkK = 0, off_sinkV = 0, off_ringK = 0, off_ringV = 0;
  int parts = 1, part_room = 1;  // workgroups per pair of query heads in the softmax (attn_parts.hip), as many as the workspace has room for
  size_t off_parts = 0, off_stats = 0;
  size_t off_qc = 0, off_Pn = 0, off_pe = 0, off_pendK = 0, off_pendV = 0, off_ps = 0, off_direct = 0, ws_bytes = 0;
};

// Most kept bins per layer of the deferred write-back on FFT contexts.
constexpr int kFftMaxBins = 4096;
// Prefill without a flag, M = 2^m: FFTs from this many kept bins in some layer, or from 1 / kFftPrefillMinShare of all bins.
constexpr int kFftPrefillMinBins = 128, kFftPrefillMinShare = 32;
// Most slices per round of the contraction at which the FFT is still ahead: bf16 at 4096 and from 8192 points, fp32 from 8192.
constexpr int kFftPrefillRound16Mid = 208, kFftPrefillRound16 = 144, kFftPrefillRound32 = 168;
constexpr int kMaxExact = 1024;  // most sink + recent tokens (their scores sit in LDS)
constexpr uint32_t kFftMinM = 256;
constexpr int64_t kFftMaxQ = 8192;  // longest transform the FFT attention kernel holds in LDS
constexpr int64_t kChirpMinM = 32, kChirpMaxM = 8192;  // chirp-z transforms: 2 Q - 1 <= 16384 points fit in LDS
// grid points that take as long as one token of the contraction: bf16, fp32, grids of up to 4096 points and longer ones
constexpr int64_t kAnyPrefillPoints[2][2] = {{180, 160}, {250, 185}};
constexpr int64_t kAnyUnevenPoints = 140;  // bf16, longer grids, blocks that do not divide M
constexpr int64_t kAnyMaxPeriod = 65536;  // ... most frequencies with taps of their own (48 bytes each) where the blocks do not divide M
constexpr int64_t kDeferMinRows = 49152;  // fewest coefficient rows (slices x padded bins) of a deferred write-back, chirp-z
constexpr int64_t kChirpMaxBlocks = 256;  // most decimated blocks M / Q of the chirp-z attention
constexpr int kLowMinLogN = 12, kLowMaxLogN = 14;  // grids of prefill and decode attention on low frequencies, M = 2^m
constexpr int64_t kLowMinD = 4, kLowMaxD = 16;     // ... tokens per grid point
constexpr int64_t kGridMinM = 2048;
constexpr int64_t kDecScratch = (int64_t)128 << 20;  // bytes of the grids of a group of slices: they fit the memory-side cache
constexpr int kCus = 256;
constexpr int64_t kPartBytes = (int64_t)64 << 20;  // most bytes of the rows that the parts of a softmax leave
constexpr uint64_t kDirectMaxTerms = 1ull << 30;  // most M * |B| the direct sums are chosen for without being asked

constexpr int64_t tap_floats(int taps) { return taps > 8 ? 12 : 10; }  // of one point (interp.h, load_taps)

// Workgroups per pair of query heads in the softmax: where one each leaves the chip idle they share the blocks of a long context (low
// frequencies: the tokens behind every grid point), as many as the device holds at a time.  What they save in blocks they pay with the launch of
// attn_merge_kernel and its trip over their rows.  Decode step, 16 deferred, one workgroup / shared, us: two blocks (M = 16384), 16 pairs of heads
// 48.7 / 45.8, 64 63.8 / 62.1, 128 132.8 / 138.2; more blocks, M = 65536, 4096 bins, 32 pairs (16 slices of 4 heads) 136 / 86, (32 of 2) 150 / 99, 128 283 / 252; M = 131072, 1500 bins, 64 pairs
// 199 / 93, 256 242 / 215; chirp-z, M = 32708, 2040 bins, 32 pairs 160 / 83, 96 219 / 164; M = 25419 (37 blocks of 687), 20 pairs 3882 / 1183.
// Low frequencies repeat the two transforms in every part: grids of 16384 points, M = 131072, 16 pairs 109 / 95, 64 134 / 120, two parts for 128
// pairs 268 / 268; shorter grids slow down beside each other: 8192 points, M = 65536, 8 pairs 59 / 53, 504 workgroups for 72 pairs 106 / 111;
// 4096 points, M = 65536, 8 pairs 49 / 39; four tokens per grid point gain on 16384 points only (M = 32768, 8 pairs 50 / 50, 32 64 / 64).
int64_t parts_of(int64_t units, int64_t slots, int64_t blocks, int64_t room, int64_t least) {
  const int64_t n = std::min(std::min(units, room), slots / blocks);
  if (n < least) return 1;
  const int64_t share = (units + n - 1) / n;
  return (units + share - 1) / share;  // no more than the longest share asks for
}
// M = 2^m > kFftMaxQ, on a grid of 2^low_logN points or (0) in blocks of kFftMaxQ.
int64_t fft_parts(const Plan& pl, int64_t M, int low_logN, int64_t blocks, int64_t room) {
  if (!low_logN) {
    const int per_thread = (pl.max_Bp + fft_threads(kFftMaxLogQ) - 1) / fft_threads(kFftMaxLogQ);
    return parts_of(M / kFftMaxQ, M / kFftMaxQ == 2 ? kCus / 2 : per_thread > 4 && per_thread <= 8 ? kCus : 2 * kCus, blocks, room, 2);
  }
  const int64_t units = M >> low_logN;  // tokens behind a grid point
  if (units < 8 && low_logN < kLowMaxLogN) return 1;
  return parts_of(units, low_logN < kLowMaxLogN || units < 8 ? kCus / 2 : kCus, blocks, room, 3);
}
int softmax_parts(const Plan& pl, int64_t M, int64_t slices, int64_t ws, int* reserve) {
  *reserve = 1;
  const int64_t blocks = slices * ((pl.G + 1) / 2);
  const int64_t room = std::min<int64_t>(kPartBytes / (int64_t)(sizeof(float2) * (size_t)ws), kMaxParts);
  if (pl.use_fft && M > kFftMaxQ) {
    // the same room whichever bins are kept, as long as the rows are: what the most parts of the grids that could carry rows this long take
    int64_t most = fft_parts(pl, M, 0, blocks, room);
    for (int logN = kLowMinLogN; logN <= kLowMaxLogN; ++logN)
      if ((M >> logN) >= kLowMinD && (M >> logN) <= kLowMaxD && 4 * (int64_t)(pl.max_nb - 1) <= ((int64_t)1 << logN))
        most = std::max(most, fft_parts(pl, M, logN, blocks, room));
    *reserve = (int)most;
    return (int)fft_parts(pl, M, pl.low_logN, blocks, room);
  }
  if (pl.use_chirp && M > pl.chirp_Q)
    *reserve = (int)parts_of(M / pl.chirp_Q, (int64_t)kCus << std::min(kTabMaxLogQ - pl.chirp_logN, 4), blocks, room, 2);
  return *reserve;
}
size_t stats_bytes(const Plan& pl, int64_t slices, int parts) { return sizeof(float4) * (size_t)(slices * ((pl.G + 1) / 2) * parts); }
// The parts' buffers at `rows` and `stats`.
Parts parts_at(const Plan& pl, char* rows, char* stats) {
  Parts p;
  p.n = pl.parts;
  p.stride = pl.ws_total;
  p.rows = (float2*)rows;
  p.stats = (float4*)stats;
  return p;
}

// What decides whether decode attention runs as one launch (attn_slice_fits).
void set_attn_shape(const iwdft_desc& d, const Plan& pl, Params* P) {
  P->n_slices = d.n_layers * d.batch * d.n_kv_heads;
  P->G = pl.G;
  P->M = (uint32_t)d.M;
  P->max_Bp = pl.max_Bp;
  P->S = d.n_sink;
  P->R = d.n_recent;
  P->serial_phases = (d.flags & IWDFT_FLAG_SERIAL_PHASES) ? 1 : 0;
  P->one_fold = pl.use_fft && 4 * (int64_t)pl.max_Bp <= d.M ? 1 : 0;
  for (const LayerInfo& L : pl.layers) P->one_fold &= L.fold_rounds == 1;
}

int make_plan(const iwdft_desc* d, Plan* pl) {
  if (!d) return fail(IWDFT_ERR_ARG, "desc is NULL");
  if (d->n_layers <= 0 || d->batch <= 0 || d->n_kv_heads <= 0 || d->n_q_heads <= 0)
    return fail(IWDFT_ERR_ARG, "n_layers, batch, n_kv_heads, n_q_heads must be positive");
  if (d->n_q_heads % d->n_kv_heads != 0)
    return fail(IWDFT_ERR_ARG, "n_q_heads (%d) is not a multiple of n_kv_heads (%d)", d->n_q_heads,
                d->n_kv_heads);
  if (d->kv_dtype != IWDFT_F32 && d->kv_dtype != IWDFT_BF16)
    return fail(IWDFT_ERR_ARG, "kv_dtype %d is neither IWDFT_F32 nor IWDFT_BF16", d->kv_dtype);
  if (d->write_every > (uint32_t)kMaxPend)
    return fail(IWDFT_ERR_ARG, "write_every = %u exceeds %d", d->write_every, kMaxPend);
  if (d->flags & ~(uint32_t)(IWDFT_FLAG_DIRECT_SYNTHESIS | IWDFT_FLAG_DENSE_PREFILL | IWDFT_FLAG_FFT_PREFILL |
                             IWDFT_FLAG_SHORTCUT | IWDFT_FLAG_SERIAL_PHASES))
    return fail(IWDFT_ERR_ARG, "unknown bits in flags: 0x%x", d->flags);
  if ((d->flags & IWDFT_FLAG_DENSE_PREFILL) && (d->flags & IWDFT_FLAG_FFT_PREFILL))
    return fail(IWDFT_ERR_ARG, "flags ask for both the dense and the FFT prefill");
  if (d->M < 1 || d->M > ((int64_t)1 << 30))
    return fail(IWDFT_ERR_ARG, "M = %lld outside [1, 2^30]", (long long)d->M);
  if (d->n_sink < 0 || d->n_recent < 0) return fail(IWDFT_ERR_ARG, "n_sink / n_recent is negative");
  if ((int64_t)d->n_sink + d->n_recent > kMaxExact)
    return fail(IWDFT_ERR_UNSUPPORTED, "n_sink + n_recent = %lld exceeds %d", (long long)d->n_sink + d->n_recent,
                kMaxExact);
  if (d->head_dim <= 0) return fail(IWDFT_ERR_ARG, "head_dim must be positive");
  if (d->head_dim != kHeadDim)
    return fail(IWDFT_ERR_UNSUPPORTED, "head_dim %d: this build has kernels for head_dim 128 only",
                d->head_dim);
  pl->G = d->n_q_heads / d->n_kv_heads;
  if (pl->G > 64) return fail(IWDFT_ERR_UNSUPPORTED, "more than 64 query heads per KV head");
  if ((int64_t)d->n_layers * d->batch * d->n_kv_heads > ((int64_t)1 << 24))
    return fail(IWDFT_ERR_UNSUPPORTED, "more than 2^24 slices");
  if (!d->bin_offsets || !d->bins) return fail(IWDFT_ERR_ARG, "bin_offsets / bins is NULL");
  if (d->bin_offsets[0] != 0) return fail(IWDFT_ERR_BINS, "bin_offsets[0] must be 0");

  const int64_t slices_per_layer = (int64_t)d->batch * d->n_kv_heads;
  pl->layers.resize(d->n_layers);
  int64_t coef = 0, ws = 0;
  for (int l = 0; l < d->n_layers; ++l) {
    int64_t b0 = d->bin_offsets[l], b1 = d->bin_offsets[l + 1];
    if (b1 <= b0) return fail(IWDFT_ERR_BINS, "layer %d keeps no bins (or offsets decrease)", l);
    if (b1 - b0 > d->M) return fail(IWDFT_ERR_BINS, "layer %d keeps more than M bins", l);
    if (b1 > ((int64_t)1 << 30)) return fail(IWDFT_ERR_UNSUPPORTED, "more than 2^30 bins in total");
    int64_t prev = -1;
    for (int64_t i = b0; i < b1; ++i) {
      int64_t k = d->bins[i];
      if (k < 0 || k >= d->M)
        return fail(IWDFT_ERR_BINS, "layer %d: bin %lld outside [0, M)", l, (long long)k);
      if (k <= prev)
        return fail(IWDFT_ERR_BINS, "layer %d: bins not strictly increasing at entry %lld", l,
                    (long long)(i - b0));
      prev = k;
      if (d->bin_weights && !std::isfinite(d->bin_weights[i]))
        return fail(IWDFT_ERR_BINS, "layer %d: non-finite bin weight", l);
    }
    LayerInfo& L = pl->layers[l];
    L.bin_off = (int32_t)b0;
    L.nb = (int32_t)(b1 - b0);
    L.Bp = (L.nb + kRowPad - 1) / kRowPad * kRowPad;
    L.fold_rounds = 0;
    L.coef_off = coef;
    L.ws_off = ws;
    coef += slices_per_layer * kHeadDim * L.Bp;
    ws += slices_per_layer * pl->G * L.Bp;
    if (L.nb > pl->max_nb) pl->max_nb = L.nb;
    if (L.Bp > pl->max_Bp) pl->max_Bp = L.Bp;
  }
  pl->n_bins_total = d->bin_offsets[d->n_layers];
  pl->coef_total = coef;
  pl->ws_total = ws;

  const bool pow2 = (d->M & (d->M - 1)) == 0;
  pl->use_fft = pow2 && (uint64_t)d->M >= kFftMinM && !(d->flags & IWDFT_FLAG_DIRECT_SYNTHESIS);
  // Prefill: the FFT costs about the same whatever the number of kept bins and in proportion to the slices; the dense contraction
  // grows with the bins in steps of 128 and walks the tokens once per round of 256 workgroups (slices x steps), whether or not
  // the last round is full.  Measured (bf16, dense / FFT, us): 128 slices, M = 1024, 64 bins 52 / 30; M = 4096, 256 bins
  // 235 / 134; M = 8192, 128 bins 336 / 282; one layer of 8, M = 1024, 64 bins, fp32: 78 / 7.3.  256 slices, 128 bins, one full
  // round: M = 2048 125 / 123, M = 4096 238 / 253, M = 8192 466 / 622, M = 16384 930 / 1220 (fp32 222 / 151, 422 / 336, 838 / 876,
  // 1664 / 2185); 200 slices, M = 4096 209 / 203; 160 slices, M = 8192 357 / 396, M = 16384 713 / 761 (fp32 703 / 548, 1391 /
  // 1326); 64 slices, M = 65536: 2594 / 1081.  So the contraction stays where a round has more than kFftPrefillRound.. slices.
  // Below kFftPrefillMinBins and kFftPrefillMinShare it stays as well, though not for speed (M = 4096, 64 bins, 128 slices:
  // 177 / 116): such contexts keep its result.
  const int64_t S = slices_per_layer * d->n_layers, rounds = (S * ((pl->max_nb + 127) / 128) + 255) / 256;
  const bool b16 = d->kv_dtype == IWDFT_BF16;
  const int64_t round_slices = d->M >= 8192            ? (b16 ? kFftPrefillRound16 : kFftPrefillRound32)
                               : b16 && d->M >= 4096 ? kFftPrefillRound16Mid
                                                     : S;  // short contexts: the FFT
  const bool fft_pf_ok = pow2 && (uint64_t)d->M >= kFftMinM;
  if (d->flags & IWDFT_FLAG_FFT_PREFILL) {
    if (!fft_pf_ok)
      return fail(IWDFT_ERR_UNSUPPORTED, "FFT prefill needs M = 2^m >= %d", (int)kFftMinM);
    pl->use_fft_prefill = true;
  } else {
    pl->use_fft_prefill = fft_pf_ok && !(d->flags & IWDFT_FLAG_DENSE_PREFILL) &&
                          (pl->max_nb >= kFftAloneBins ||
                           (d->M <= (int64_t)kStreamMaxM && S <= round_slices * rounds &&
                            (pl->max_nb >= kFftPrefillMinBins || (int64_t)pl->max_nb * kFftPrefillMinShare >= d->M)));
  }
  // Contexts that take the FFT for its speed only, where the contraction would keep every channel alone; see prefill_fft.hip.
  pl->scale_pairs = pl->use_fft_prefill && !(d->flags & IWDFT_FLAG_FFT_PREFILL) && pl->max_nb < kFftAloneBins;
  // Chirp-z attention for M that is not a power of two: M itself up to 8192 points; longer M in Pb decimated blocks
  // of M / Pb points, Pb the smallest divisor of M that brings the block down to 8192 (none: the direct sums).
  pl->use_chirp = false;
  if (!pl->use_fft && !(d->flags & IWDFT_FLAG_DIRECT_SYNTHESIS) && d->M >= kChirpMinM) {
    for (int64_t pb = (d->M + kChirpMaxM - 1) / kChirpMaxM; pb <= kChirpMaxBlocks && d->M / pb >= kChirpMinM; ++pb) {
      if (d->M % pb == 0) {
        pl->use_chirp = true;
        pl->chirp_Q = d->M / pb;
        break;
      }
    }
  }
  if (pl->use_chirp) {
    pl->chirp_logN = pl->chirp_logS = 8;
    while (((int64_t)1 << pl->chirp_logN) < 2 * pl->chirp_Q - 1) ++pl->chirp_logN;
    while (((int64_t)1 << pl->chirp_logS) < 2 * pl->chirp_Q - 1) pl->chirp_logS += 2;
  }
  pl->fold.assign((size_t)pl->n_bins_total, 0);
  if (pl->use_fft || pl->use_chirp) {
    // The FFT attention kernels place the sparse spectrum (each bin k and its mirror -k) into an LDS array:
    // folded modulo the transform length Q (power-of-two kernel) or at k and M - k (chirp-z kernel).  Entries that
    // land on the same slot are added in separate rounds, so the kernels need no atomics and sum in a fixed order:
    // round = how many earlier entries of the layer already use that slot.
    const int64_t Q = pl->use_chirp ? pl->chirp_Q : (d->M < kFftMaxQ ? d->M : kFftMaxQ);
    std::vector<uint16_t> cnt((size_t)Q);
    for (int l = 0; l < d->n_layers && (pl->use_fft || pl->use_chirp); ++l) {
      std::fill(cnt.begin(), cnt.end(), 0);
      LayerInfo& L = pl->layers[l];
      int rounds = 0;
      for (int i = 0; i < L.nb; ++i) {
        const int64_t k = d->bins[L.bin_off + i];
        const int64_t r = k % Q, rm = (Q - r) % Q;
        const int fd = cnt[r]++;
        // a bin whose mirror falls on its own slot (k = 0 or Q/2 mod Q) adds both halves in one write:
        // its mirror byte is 0xff, "no round"
        const int fm = r == rm ? 0xff : cnt[rm]++;
        if (fd > 254 || (r != rm && fm > 254)) { pl->use_fft = pl->use_chirp = false; break; }
        pl->fold[L.bin_off + i] = (uint16_t)(fd | (fm << 8));
        if (fd + 1 > rounds) rounds = fd + 1;
        if (r != rm && fm + 1 > rounds) rounds = fm + 1;
      }
      L.fold_rounds = rounds;
    }
  }

  // Prefill through interpolated transforms where they are faster than the dense contraction.  The transforms cost in proportion to
  // slices and grid points, and 1.5 points per kept bin where blocks are summed in the output rows; the contraction walks the M
  // tokens with 256 workgroups (slices x tiles of 128 bins) at a time, whether or not the last round is full.  The line keeps every call that
  // the transforms do not make slower over 15 lengths from 300 to 32708, 8 to 512 slices and 32 to 2000 bins.  Dense / transforms in us,
  // points per token and round: bf16 M = 3000, 64 slices, 128 bins (175) 140 / 127, 128 slices, 384 bins (175) 277 / 287;
  // M = 4036, 256 slices, 384 bins (173) 569 / 641; M = 8132, 64 slices, 512 bins (129) 462 / 348, 256 slices, 384 bins (172) 1111 / 1350;
  // fp32 M = 5000, 64 slices, 128 bins (210) 399 / 377; M = 6000, 256 slices, 384 bins (233) 1418 / 1619; M = 24573, 96 slices, 256 bins (197)
  // 1915 / 2300; M = 8132, 96 slices, 128 bins (193) 646 / 723.  Blocks of a few points only stay with the contraction.
  // The number of blocks of a longer M need not divide it: the frequencies lie anywhere on the grid, and M is cut into the blocks that cost
  // least (70 x 8 slices, M = 14473 = 41 x 353, 1978 bins: 41 blocks 27.0 ms, 2 7.1; 4 x 8, fp32, M = 25419 = 37 x 687, 4096 bins: 37 6.4, 7 1.4).  Costs in per cent of a
  // point of the longest grid, fitted to 2300 sets of times (190 lengths from 8200 to 65500, 8 to 384 slices, 64 to 4096 bins): a point of a grid of 2^10 .. 2^14 (kPointCost: full device;
  // fewer slices, bf16 and fp32), a bin per block (kBinCost: blocks that divide M; that do not, where the phase takes 64 bits and the taps are those of `period` frequencies, more by
  // 1.2 period / 65536).  Next to the blocks that divide M three sets of a thousand lose 3 % or more, none 7 %; all in all 1.21 times as fast.
  // M = 62811, bf16, 96 slices, 4096 bins 9 even blocks 6.57 ms, 8 uneven 9.64, 1024 bins 4.79, 5.03, 512 bins 4.50, 4.27; fp32, M = 14473, 64
  // bins, 32 slices 2 blocks 384 us, 4 342, 8 265, 15 262, 8 slices 105, 94, 98, 102.
  if (pl->use_chirp && pl->chirp_Q > kFftMinM && !(d->flags & IWDFT_FLAG_DENSE_PREFILL)) {
    static constexpr int kPointCost[3][5] = {{85, 78, 80, 88, 100}, {160, 140, 125, 140, 100}, {175, 120, 105, 90, 100}};
    static constexpr int kBinCost[2][2] = {{300, 325}, {225, 225}};
    const int *point = kPointCost[S >= 16 ? 0 : b16 ? 1 : 2], *bin = kBinCost[b16 ? 0 : 1];
    int64_t least = 0, points = 0;
    for (int64_t pb = (d->M + kChirpMaxM - 1) / kChirpMaxM; pb <= d->M / pl->chirp_Q; ++pb) {
      const int64_t A = (d->M + pb - 1) / pb, g = std::gcd(d->M, pb);
      if (A <= kFftMinM) break;
      const int64_t bins = pb > 1 ? pl->max_nb : 0, period = d->M / g;
      if (g != pb && period > kAnyMaxPeriod) continue;
      int logN = 10;
      while (((int64_t)1 << logN) < 2 * A) ++logN;
      const int64_t cost = pb * (((int64_t)point[logN - 10] << logN) + bins * (g == pb ? bin[0] : bin[1] + bin[1] * period * 6 / (5 * 65536)));
      if (least && cost >= least) continue;
      least = cost;
      points = pb * (((int64_t)1 << logN) + bins * (g == pb ? 3 : 5) / 2);
      pl->pf_logN = logN, pl->pf_Pb = pb, pl->pf_A = A, pl->pf_period = period;
    }
    // uneven blocks on long grids in bf16 lose earlier (points per token and round: M = 37492, 64 slices, 92 bins (142) 1610 / 1709; M = 13827, 87 bins (154) 604 / 643;
    // M = 31870, 200 bins (136) 1.01 times as fast; fp32 M = 24582, 128 slices, 384 bins (181) 1.27)
    const int64_t line = b16 && pl->pf_logN > 12 && d->M % pl->pf_Pb ? kAnyUnevenPoints : kAnyPrefillPoints[b16 ? 0 : 1][pl->pf_logN > 12 ? 1 : 0];
    pl->use_any_prefill = S * points <= line * d->M * rounds;
  }

  // Decode attention of low frequencies (attn_low_kernel) on the smallest grid that carries them, from four tokens per point on (read-only
  // step of 8 .. 1024 slices, 1 to 8 heads, M = 16384 .. 262144: 0.42 to 1.0 of the time; two tokens: M = 16384 1.00 .. 1.08, M = 32768 0.95 .. 1.0) and with 4096 points at least: what few threads
  // save in transforms they lose in the chain over the tokens of each (M = 16384, 256 bins, 8 slices, one head: 31 us without, 41 with
  // 1024 points).  Bins that are each other's mirror would share a slot.
  bool mirrored = false;
  for (int l = 0; l < d->n_layers; ++l) {  // ascending: the bins next to M / 2 on either side are the highest
    const int32_t *b0 = d->bins + d->bin_offsets[l], *b1 = d->bins + d->bin_offsets[l + 1];
    const int32_t* up = std::upper_bound(b0, b1, (int32_t)(d->M / 2));
    if (up > b0) pl->reach = std::max<int64_t>(pl->reach, up[-1]);
    if (up < b1) {
      pl->reach = std::max<int64_t>(pl->reach, d->M - *up);
      mirrored = true;
    }
  }
  if (pow2 && d->M > kFftMaxQ) {
    int logN = kLowMinLogN;
    while (((int64_t)1 << logN) < 4 * pl->reach || (kLowMaxD << logN) < d->M) ++logN;
    if (logN <= kLowMaxLogN && (d->M >> logN) >= kLowMinD) {
      if (pl->use_fft && !mirrored) pl->low_logN = logN;
    }
    // Prefill through that grid (decimate.hip) where it is faster than the transforms of the tokens.  us without / with, 64 slices: 16 tokens
    // per grid point, M = 131072, 2048 bins bf16 2131 / 1564, fp32 3816 / 2274; 8, M = 131072, 4096 bins 4163 / 2123, 4145 / 2884; 8,
    // M = 65536, 2048 bins 1145 / 997, 1857 / 1452; 4, M = 65536, 4096 bins 2147 / 1629, 2095 / 1985; M = 32768, 2048 bins 608 / 787,
    // 937 / 988.  Grids of 4096 points have too few waves below 16 slices (M = 32768, 1024 bins, 8 slices 67 / 85, 120 / 101; 64
    // slices 581 / 493, 930 / 715); there four tokens per point gain in fp32 only (M = 16384, 1024 bins, 64 slices 308 / 385, 494 / 482).
    const int64_t D = d->M >> logN;
    const bool dec = D >= 8 ? logN > kLowMinLogN || S >= 16 : D == 4 && (logN == kLowMaxLogN || (logN == kLowMinLogN && !b16 && S >= 32));
    if (logN <= kLowMaxLogN && dec && pl->use_fft_prefill) {
      pl->dec_logN = logN;
      pl->dec_slices = std::min<int64_t>(S, kDecScratch / ((int64_t)2 * kHeadDim * sizeof(double) << logN));
    }
  }
  // M that is not a power of two, one block: interpolated transforms in place of the chirp-z ones (attn_chirp.hip) where the grid is half as
  // long as the chirp's convolution and the transforms are long enough to matter.  Attention, us, chirp-z / grid: M = 8132, 64 slices, 4 heads, 508 bins
  // 52 / 43, 2033 bins 83 / 75; 512 slices, 8 heads 346 / 228, 647 / 520; M = 3000, 64 slices, 4 heads, 750 bins 44 / 42.  Up to 2048 tokens
  // 0.91 .. 1.14 of the time (M = 2040, 64 slices, 510 bins 33 / 38), with a grid as long as the convolution 0.95 .. 1.14.
  if (pl->use_chirp && pl->chirp_Q == d->M && d->M > kGridMinM) {
    const int logN = pl->chirp_logN - 1;
    if (((int64_t)1 << logN) >= d->M && ((int64_t)1 << logN) > 4 * pl->reach) pl->low_logN = logN;
  }

  // What is left takes the direct O(M |B|) sums: fine for short or sparse states, useless beyond -- refuse instead of
  // running for minutes per step (a prime M of 2^20 with 4096 kept bins is 2^32 sine / cosine pairs per query head).
  if (!pl->use_fft && !pl->use_chirp && !(d->flags & IWDFT_FLAG_DIRECT_SYNTHESIS) &&
      (uint64_t)d->M * (uint64_t)pl->max_nb > kDirectMaxTerms)
    return fail(IWDFT_ERR_UNSUPPORTED,
                "M = %lld with %d kept bins in a layer has no O(M log M) decode attention (M is neither a power of two nor "
                "has a divisor Pb <= %d with 32 <= M / Pb <= %d) and is too large for the direct sums; pick M with such a "
                "divisor (e.g. move tokens to the sink / recent windows) or pass IWDFT_FLAG_DIRECT_SYNTHESIS to insist",
                (long long)d->M, pl->max_nb, (int)kChirpMaxBlocks, (int)kChirpMaxM);

  if (!(d->flags & IWDFT_FLAG_SERIAL_PHASES)) pl->parts = softmax_parts(*pl, d->M, S, ws, &pl->part_room);

  size_t o = 0;
  pl->off_layers = o;  o = align256(o + sizeof(LayerInfo) * (size_t)d->n_layers);
  pl->off_bins = o;    o = align256(o + sizeof(int32_t) * (size_t)pl->n_bins_total);
  pl->off_weights = o; o = align256(o + sizeof(float) * (size_t)pl->n_bins_total);
  pl->off_fold = o;    o = align256(o + sizeof(uint16_t) * (size_t)pl->n_bins_total);
  pl->off_chirp = o;   o = align256(o + (pl->use_chirp ? sizeof(float2) * (size_t)pl->chirp_Q : 0));
  o = align256(o + (pl->use_chirp ? sizeof(float2) * ((size_t)1 << pl->chirp_logS) : 0));
  pl->tw_Q = (pow2 && (uint64_t)d->M >= kFftMinM) ? (d->M < kFftMaxQ ? d->M : kFftMaxQ) : 0;
  pl->off_tw = o;      o = align256(o + (pl->tw_Q ? sizeof(float2) * (size_t)(pl->tw_Q / 8 + 1) : 0));
  pl->off_FK = o;      o = align256(o + sizeof(float2) * (size_t)coef);
  pl->off_FV = o;      o = align256(o + sizeof(float2) * (size_t)coef);
  const size_t esz = d->kv_dtype == IWDFT_BF16 ? 2 : 4;
  const size_t n_sl = (size_t)d->n_layers * (size_t)slices_per_layer;
  pl->off_sinkK = o;   o = align256(o + esz * n_sl * (size_t)d->n_sink * kHeadDim);
  pl->off_sinkV = o;   o = align256(o + esz * n_sl * (size_t)d->n_sink * kHeadDim);
  pl->off_ringK = o;   o = align256(o + esz * n_sl * (size_t)d->n_recent * kHeadDim);
  pl->off_ringV = o;   o = align256(o + esz * n_sl * (size_t)d->n_recent * kHeadDim);
  pl->state_bytes = o;

  o = 0;
  pl->off_qc = o; o = align256(o + sizeof(float2) * (size_t)ws);
  pl->off_Pn = o; o = align256(o + sizeof(float2) * (size_t)ws);
  pl->off_pe = o; o = align256(o + sizeof(float) * n_sl * (size_t)pl->G * (size_t)(d->n_sink + d->n_recent));
  // Deferred write-back needs the FFT or chirp-z attention kernels, which weigh the pending tokens, and all query heads of a KV
  // head in one pass; otherwise every step writes back.  Contexts beyond kFftMaxBins bins have always written back at every step
  // (the kernels could weigh there too; not measured).  On chirp-z contexts deferral is taken where it is faster: not below 256
  // slots, and with more than two query heads per KV head from kDeferMinRows coefficient rows on, where a step reads 1 GB instead
  // of moving 2.  16 steps, every one written back / deferred, us a step, 4 heads: M = 1000, 250 bins, 94 slices 54 / 67, 219
  // slices 73 / 80, 512 slices 135 / 110; M = 4095, 1023 bins, 39 slices 84 / 84; M = 8132, 2033 bins, 12 slices 90 / 100, 64
  // slices 144 / 120; 8 heads, M = 1000: 94 slices 64 / 74, 258 slices 108 / 102; 2 heads: 16 slices 32 / 32, 94 slices 53 / 42.
  const bool weighs = (pl->use_fft && pl->max_nb <= kFftMaxBins) ||
                      (pl->use_chirp && (uint64_t)d->M >= kFftMinM && (pl->G <= 2 || coef / kHeadDim >= kDeferMinRows));
  pl->write_every = (d->write_every > 1 && weighs && heads_fit_one_pass(pl->G) && !(d->flags & IWDFT_FLAG_SHORTCUT))
                        ? (int)d->write_every
                        : 1;
  const size_t pend_rows = (d->n_recent || pl->write_every > 1) ? (size_t)pl->write_every : 0;
  pl->off_pendK = o; o = align256(o + esz * n_sl * pend_rows * kHeadDim);
  pl->off_pendV = o; o = align256(o + esz * n_sl * pend_rows * kHeadDim);
  pl->off_ps = o;    o = align256(o + (pl->write_every > 1 ? sizeof(float) * n_sl * (size_t)pl->G * kMaxPend : 0));
  pl->off_chirpW = o; o = align256(o + (pl->use_chirp ? sizeof(float2) * ((size_t)1 << pl->chirp_logN) : 0));
  pl->off_dec = o;   o = align256(o + (pl->use_any_prefill ? sizeof(float) * ((size_t)1 << pl->pf_logN) / 2 : 0));
  pl->off_taps = o;  o = align256(o + (pl->use_any_prefill ? sizeof(float) * tap_floats(pl->pf_Pb > 1 ? kSumTaps : kTaps) * ((size_t)pl->pf_period / 2 + 1) : 0));
  pl->off_direct = o;
  if (!pl->use_fft && !pl->use_chirp)
    o = align256(o + sizeof(float) * (size_t)d->n_layers * (size_t)slices_per_layer *
                         (size_t)pl->G * (size_t)d->M);
  // The grids of the prefill lie over everything above, which only lives between decode steps of the same context; their tables behind.
  if (pl->dec_logN) {
    const size_t n = ((size_t)1 << pl->dec_logN) / 4 + 1;
    o = std::max(o, align256((size_t)pl->dec_slices * 2 * kHeadDim * sizeof(double) << pl->dec_logN));
    pl->off_dec_w = o;    o = align256(o + sizeof(double) * kDecTaps * (size_t)(d->M >> pl->dec_logN));
    pl->off_dec_tw = o;   o = align256(o + sizeof(double2) * n);
    pl->off_dec_gain = o; o = align256(o + sizeof(double) * n);
  }
  if (pl->low_logN) {
    pl->off_low_gain = o; o = align256(o + sizeof(float) * (((size_t)1 << pl->low_logN) / 4 + 1));
    pl->off_low = o;
    o = align256(o + sizeof(float) * (pl->use_chirp ? 10 * ((size_t)d->M / 2 + 1) : (size_t)(d->M >> pl->low_logN) * kTaps));
    pl->off_grid = o;     o = align256(o + (pl->use_chirp ? 10 * sizeof(float) * (((size_t)1 << pl->low_logN) / 2 + 1) : 0));
  }
  if (pl->part_room > 1) {
    pl->off_parts = o; o = align256(o + sizeof(float2) * (size_t)ws * (size_t)pl->part_room);
    pl->off_stats = o; o = align256(o + stats_bytes(*pl, (int64_t)n_sl, pl->part_room));
  }
  pl->ws_bytes = o;
  return IWDFT_OK;
}

// The length-N transform (sign +) of h[n] = exp(-j pi n^2 / M), |n| < M, wrapped modulo N, divided by N, in double precision.
void make_chirp_transform(int64_t M, int logN, std::vector<float2>* H) {
  const double kPi = 3.14159265358979323846;
  const int64_t N = (int64_t)1 << logN;
  std::vector<std::complex<double>> h((size_t)N, 0.0), w((size_t)(N / 2));
  for (int64_t n = 0; n < M; ++n) {
    const double ph = kPi * (double)((n * n) % (2 * M)) / (double)M;
    const std::complex<double> v(std::cos(ph), -std::sin(ph));
    h[(size_t)n] = v;
    if (n) h[(size_t)(N - n)] = v;
  }
  for (int64_t j = 0; j < N / 2; ++j) w[(size_t)j] = std::polar(1.0, 2.0 * kPi * (double)j / (double)N);
  // iterative radix-2 transform, sign +
  for (int64_t i = 1, j = 0; i < N; ++i) {
    int64_t bit = N >> 1;
    for (; j & bit; bit >>= 1) j ^= bit;
    j ^= bit;
    if (i < j) std::swap(h[(size_t)i], h[(size_t)j]);
  }
  for (int64_t len = 2; len <= N; len <<= 1) {
    for (int64_t i = 0; i < N; i += len)
      for (int64_t j = 0; j < len / 2; ++j) {
        const std::complex<double> u = h[(size_t)(i + j)], z = h[(size_t)(i + j + len / 2)], t = w[(size_t)(j * (N / len))];
        const std::complex<double> v(z.real() * t.real() - z.imag() * t.imag(), z.real() * t.imag() + z.imag() * t.real());
        h[(size_t)(i + j)] = u + v;
        h[(size_t)(i + j + len / 2)] = u - v;
      }
  }
  H->resize((size_t)N);
  for (int64_t m = 0; m < N; ++m)
    (*H)[(size_t)m] = make_float2((float)(h[(size_t)m].real() / (double)N), (float)(h[(size_t)m].imag() / (double)N));
}
// Entry m of the transform sits at position digit_position(m) of the order that the in-LDS transforms of 2^logN points leave
// (fft_core.h, sample_at): the base-4 digits reversed, for odd logN behind the low bit, which moves to the top.
int64_t digit_position(int64_t m, int logN) {
  int64_t p = 0;
  const int odd = logN & 1, even = logN - odd;
  for (int t = 0; t < even / 2; ++t) p |= ((m >> (odd + 2 * t)) & 3) << (even - 2 * t - 2);
  return odd ? p | ((m & 1) << even) : p;
}

// The window of a grid of N = 2^logN points (tables.hip has its formulas).  beta after P. J. Beatty, D. G. Nishimura and
// J. M. Pauly, IEEE Trans. Med. Imaging 24 (2005).
Window grid_window(int logN, double reach, int taps) {
  Window w{(int64_t)1 << logN, reach, 0.0, 0.0, taps};
  const double a = taps * (1.0 - std::max(reach, 1.0) / (double)w.N);
  w.beta = 3.14159265358979323846 * std::sqrt(a * a - 0.8);
  w.W0 = std::sinh(w.beta) / w.beta;
  return w;
}

}  // namespace

struct iwdft_ctx {
  iwdft_desc desc;  // host pointers inside are cleared after create
  Plan plan;
  Params P;
  int device = 0;
  int64_t T = 0;
  char* state = nullptr;
  char* ws = nullptr;
  int pend = 0;  // tokens counted in T that only the pending rows hold (deferred write-back), < write_every
  // phase timing (iwdft_phase_timing): events of the calls since the last read-out
  bool timing = false;
  std::vector<iwdft::PhaseEvents> marks;  // pool, reused after every read-out
  size_t marks_used = 0;
};

namespace {

int check_ctx(const iwdft_ctx* c) {
  if (!c) return fail(IWDFT_ERR_ARG, "ctx is NULL");
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return fail(IWDFT_ERR_HIP, "hipGetDevice failed");
  if (dev != c->device)
    return fail(IWDFT_ERR_STATE, "context belongs to device %d but device %d is current", c->device,
                dev);
  return IWDFT_OK;
}

int launched(hipError_t e, const char* what) {
  if (e != hipSuccess) return fail(IWDFT_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
  return IWDFT_OK;
}

// Device address of this GPU's copy of `scratch`, looked up once per device with that device current.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

int static_scratch(int dev, char** out) {
  if (dev < 0 || dev >= kMaxDevices) return fail(IWDFT_ERR_UNSUPPORTED, "device index %d beyond %d", dev, kMaxDevices - 1);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fail(IWDFT_ERR_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
    g_scratch_ptr[dev] = p;
  }
  *out = (char*)g_scratch_ptr[dev];
  return IWDFT_OK;
}

// Next set of phase events of a timed call (created on demand), or null when timing is off.
int next_marks(iwdft_ctx* c, const PhaseEvents** out) {
  try {
    *out = nullptr;
    if (!c->timing) return IWDFT_OK;
    if (c->marks_used == c->marks.size()) {
      PhaseEvents m;
      for (int i = 0; i < 4; ++i) {
        hipError_t e = hipEventCreate(&m.ev[i]);
        if (e != hipSuccess) {
          for (int j = 0; j < i; ++j) (void)hipEventDestroy(m.ev[j]);
          return fail(IWDFT_ERR_HIP, "hipEventCreate: %s", hipGetErrorString(e));
        }
      }
      c->marks.push_back(m);
    }
    *out = &c->marks[c->marks_used++];
    return IWDFT_OK;

  } catch (...) {  // std::bad_alloc from the host-side containers: nothing may cross the C ABI
    return fail(IWDFT_ERR_ARG, "out of host memory");
  }
}

bool shortcut(const iwdft_ctx* c) { return (c->desc.flags & IWDFT_FLAG_SHORTCUT) != 0; }

// Readers of the coefficients: gain T / M with the Sec. 4.1 shortcut (the stored state is then M S_T, not T S_T).
void set_read_gain(iwdft_ctx* c) {
  c->P.gain = shortcut(c) ? (float)((double)c->T / (double)c->desc.M) : 1.0f;
}

uint32_t t_shift(const iwdft_ctx* c) {  // (T - M) mod M
  return (uint32_t)((c->T - c->desc.M) % c->desc.M);
}

// Writes the tokens that the fused decode step has deferred into the coefficients, oldest first, one
// streaming update each (the rare path: a call other than the fused step arrived in between).
int flush_pending(iwdft_ctx* c, hipStream_t st) {
  if (c->pend == 0) return IWDFT_OK;
  const Plan& pl = c->plan;
  const size_t esz = c->desc.kv_dtype == IWDFT_BF16 ? 2 : 4;
  for (int j = 0; j < c->pend; ++j) {
    const uint32_t tsh = (uint32_t)((c->T - c->pend + j - c->desc.M) % c->desc.M);
    hipError_t e = launch_absorb(c->P, c->ws + pl.off_pendK + (size_t)j * kHeadDim * esz,
                                 c->ws + pl.off_pendV + (size_t)j * kHeadDim * esz,
                                 (int64_t)pl.write_every * kHeadDim, tsh, st);
    if (e != hipSuccess) return fail(IWDFT_ERR_HIP, "write-back of deferred tokens: %s", hipGetErrorString(e));
  }
  c->pend = 0;
  return IWDFT_OK;
}

}  // namespace

extern "C" {

const char* iwdft_last_error(void) { return g_err; }

int iwdft_query_bytes(const iwdft_desc* desc, size_t* state_bytes, size_t* workspace_bytes) {
  try {
    if (!state_bytes || !workspace_bytes) return fail(IWDFT_ERR_ARG, "output pointer is NULL");
    Plan pl;
    int rc = make_plan(desc, &pl);
    if (rc != IWDFT_OK) return rc;
    *state_bytes = pl.state_bytes;
    *workspace_bytes = pl.ws_bytes < 256 ? 256 : pl.ws_bytes;
    return IWDFT_OK;

  } catch (...) {  // std::bad_alloc from the host-side containers: nothing may cross the C ABI
    return fail(IWDFT_ERR_ARG, "out of host memory");
  }
}

int iwdft_query_attn(const iwdft_desc* desc, int32_t pending, int32_t write_back, int32_t* workgroups) {
  try {
    if (!workgroups) return fail(IWDFT_ERR_ARG, "output pointer is NULL");
    if (pending < 0 || pending > kMaxPend) return fail(IWDFT_ERR_ARG, "pending = %d outside [0, %d]", pending, kMaxPend);
    Plan pl;
    int rc = make_plan(desc, &pl);
    if (rc != IWDFT_OK) return rc;
    Params P{};
    set_attn_shape(*desc, pl, &P);
    *workgroups = attn_slice_fits(P, pending, write_back != 0) ? 0 : pl.parts;
    return IWDFT_OK;
  } catch (...) {  // std::bad_alloc from the host-side containers: nothing may cross the C ABI
    return fail(IWDFT_ERR_ARG, "out of host memory");
  }
}

int iwdft_create(const iwdft_desc* desc, void* d_state, size_t state_bytes, void* d_workspace,
                 size_t workspace_bytes, iwdft_ctx** out) {
  try {
    if (!out) return fail(IWDFT_ERR_ARG, "out is NULL");
    *out = nullptr;
    std::unique_ptr<iwdft_ctx> c(new iwdft_ctx());  // freed on every early return and on exceptions
    int rc = make_plan(desc, &c->plan);
    if (rc != IWDFT_OK) return rc;
    const Plan& pl = c->plan;
    size_t need_ws = pl.ws_bytes < 256 ? 256 : pl.ws_bytes;
    if (!d_state || !d_workspace) { return fail(IWDFT_ERR_ARG, "d_state / d_workspace is NULL"); }
    if (((uintptr_t)d_state & 255) || ((uintptr_t)d_workspace & 255)) {
      return fail(IWDFT_ERR_ARG, "d_state and d_workspace must be 256-byte aligned");
    }
    if (state_bytes < pl.state_bytes) {
      return fail(IWDFT_ERR_SIZE, "state buffer has %zu bytes, %zu needed", state_bytes, pl.state_bytes);
    }
    if (workspace_bytes < need_ws) {
      return fail(IWDFT_ERR_SIZE, "workspace has %zu bytes, %zu needed", workspace_bytes, need_ws);
    }
    c->desc = *desc;
    c->state = (char*)d_state;
    c->ws = (char*)d_workspace;
    if (hipGetDevice(&c->device) != hipSuccess) { return fail(IWDFT_ERR_HIP, "hipGetDevice failed"); }
    {  // set-up of compressed_decode_attn_static: this device's scratch address (a failure is reported by that call)
      char* unused = nullptr;
      (void)static_scratch(c->device, &unused);
    }

    // Device copies of geometry, bins and weights live at the head of the state buffer.
    std::vector<float> w((size_t)pl.n_bins_total, 1.0f);
    if (desc->bin_weights) memcpy(w.data(), desc->bin_weights, sizeof(float) * w.size());
    hipError_t e = hipMemset(c->state, 0, pl.state_bytes);
    if (e == hipSuccess)
      e = hipMemcpy(c->state + pl.off_layers, pl.layers.data(), sizeof(LayerInfo) * pl.layers.size(),
                    hipMemcpyHostToDevice);
    if (e == hipSuccess)
      e = hipMemcpy(c->state + pl.off_bins, desc->bins, sizeof(int32_t) * (size_t)pl.n_bins_total,
                    hipMemcpyHostToDevice);
    if (e == hipSuccess)
      e = hipMemcpy(c->state + pl.off_weights, w.data(), sizeof(float) * w.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess)
      e = hipMemcpy(c->state + pl.off_fold, pl.fold.data(), sizeof(uint16_t) * pl.fold.size(),
                    hipMemcpyHostToDevice);
    if (e == hipSuccess && pl.use_chirp) {
      std::vector<float2> H, out;
      e = make_chirp((float2*)(c->state + pl.off_chirp), pl.chirp_Q);
      // In the workspace: a copy of the state buffer that is put back may be older than this order of the table.
      if (e == hipSuccess && !pl.low_logN) {
        make_chirp_transform(pl.chirp_Q, pl.chirp_logN, &H);
        out.resize(H.size());
        const int64_t T = (int64_t)H.size() / 16;
        for (int64_t m = 0; m < (int64_t)H.size(); ++m) {  // chirp.h: thread t owns the positions 16 t .. 16 t + 15, two per load
          const int64_t p = digit_position(m, pl.chirp_logN), t = p >> 4, j = (p & 15) >> 1;
          out[(size_t)((j * T + t) * 2 + (p & 1))] = H[(size_t)m];
        }
        e = hipMemcpy(c->ws + pl.off_chirpW, out.data(), sizeof(float2) * out.size(), hipMemcpyHostToDevice);
      }
      if (pl.use_any_prefill) {
        const Window gw = grid_window(pl.pf_logN, 0.5 * (double)pl.pf_A, pl.pf_Pb > 1 ? kSumTaps : kTaps);
        if (e == hipSuccess) e = make_samples((float*)(c->ws + pl.off_dec), pl.pf_A, pl.pf_logN, gw);
        if (e == hipSuccess) e = make_taps((float*)(c->ws + pl.off_taps), pl.pf_period, gw.N, 1.0, gw);
      }
    }
    if (e == hipSuccess && pl.tw_Q) {
      const double kTwoPi = 6.28318530717958647692;
      std::vector<float2> tw((size_t)(pl.tw_Q / 8 + 1));
      for (size_t m = 0; m < tw.size(); ++m) {
        const double ph = kTwoPi * (double)m / (double)pl.tw_Q;
        tw[m] = make_float2((float)std::cos(ph), (float)std::sin(ph));
      }
      e = hipMemcpy(c->state + pl.off_tw, tw.data(), sizeof(float2) * tw.size(), hipMemcpyHostToDevice);
    }
    if (e == hipSuccess && pl.dec_logN) {
      const Window gw = grid_window(pl.dec_logN, (double)pl.reach, kDecTaps);
      e = make_token_taps((double*)(c->ws + pl.off_dec_w), desc->M >> pl.dec_logN, gw);
      if (e == hipSuccess) e = make_low((double2*)(c->ws + pl.off_dec_tw), (double*)(c->ws + pl.off_dec_gain), gw);
    }
    if (e == hipSuccess && pl.low_logN) {
      const Window gw = grid_window(pl.low_logN, (double)pl.reach, kTaps);
      e = make_gain((float*)(c->ws + pl.off_low_gain), gw);
      if (e != hipSuccess) {
      } else if (!pl.use_chirp) {
        e = make_token_taps((float*)(c->ws + pl.off_low), desc->M >> pl.low_logN, gw);
      } else {
        e = make_taps((float*)(c->ws + pl.off_low), desc->M, gw.N, 1.0, gw);
        if (e == hipSuccess) e = make_taps((float*)(c->ws + pl.off_grid), gw.N, desc->M, (double)gw.N / (double)desc->M, gw);
      }
    }
    if (e == hipSuccess && (pl.use_chirp || pl.dec_logN || pl.low_logN)) e = hipStreamSynchronize(nullptr);  // the tables above
    const float2* tab = nullptr;
    if (e == hipSuccess) e = fft_table(&tab);
    if (e != hipSuccess) {
      return fail(IWDFT_ERR_HIP, "initialising the state buffer: %s", hipGetErrorString(e));
    }
    c->desc.bin_offsets = nullptr;
    c->desc.bins = nullptr;
    c->desc.bin_weights = nullptr;

    Params& P = c->P;
    P.n_layers = desc->n_layers;
    P.batch = desc->batch;
    P.n_kv = desc->n_kv_heads;
    set_attn_shape(*desc, pl, &P);
    P.kv_dtype = desc->kv_dtype;
    P.Mmask = ((desc->M & (desc->M - 1)) == 0) ? (uint32_t)(desc->M - 1) : 0u;
    if (desc->M == 1) P.Mmask = 0;  // M = 1: "mod 1" through the generic path
    P.max_nb = pl.max_nb;
    P.layers = (const LayerInfo*)(c->state + pl.off_layers);
    P.bins = (const int32_t*)(c->state + pl.off_bins);
    P.weights = (const float*)(c->state + pl.off_weights);
    P.fold = (const uint16_t*)(c->state + pl.off_fold);
    P.chirp = pl.use_chirp ? (const float2*)(c->state + pl.off_chirp) : nullptr;
    P.chirpW = pl.use_chirp && !pl.low_logN ? (const float4*)(c->ws + pl.off_chirpW) : nullptr;
    P.any_dec = pl.use_any_prefill ? (const float*)(c->ws + pl.off_dec) : nullptr;
    P.any_taps = pl.use_any_prefill ? (const float4*)(c->ws + pl.off_taps) : nullptr;
    P.any_logN = pl.chirp_logN;
    P.pf_logN = pl.pf_logN;
    P.pf_Pb = (uint32_t)pl.pf_Pb;
    P.pf_A = (uint32_t)pl.pf_A;
    P.pf_period = (uint32_t)pl.pf_period;
    P.pf_step = pl.pf_period ? (uint32_t)(pl.pf_Pb / (desc->M / pl.pf_period)) : 0u;
    P.dec_logN = pl.dec_logN;
    P.dec_slices = (int32_t)pl.dec_slices;
    P.dec_weights = pl.dec_logN ? (const double*)(c->ws + pl.off_dec_w) : nullptr;
    P.dec_tw = pl.dec_logN ? (const double2*)(c->ws + pl.off_dec_tw) : nullptr;
    P.dec_gain = pl.dec_logN ? (const double*)(c->ws + pl.off_dec_gain) : nullptr;
    P.dec_scratch = pl.dec_logN ? (double*)c->ws : nullptr;
    P.low_logN = pl.low_logN;
    P.low_gain = pl.low_logN ? (const float*)(c->ws + pl.off_low_gain) : nullptr;
    P.low_taps = pl.low_logN ? (const float*)(c->ws + pl.off_low) : nullptr;
    P.grid_taps = pl.low_logN && pl.use_chirp ? (const float4*)(c->ws + pl.off_grid) : nullptr;
    P.any_Q = (uint32_t)pl.chirp_Q;
    P.tab = tab;
    P.tw8 = pl.tw_Q ? (const float2*)(c->state + pl.off_tw) : nullptr;
    P.FK = (float2*)(c->state + pl.off_FK);
    P.FV = (float2*)(c->state + pl.off_FV);
    P.gain = 1.0f;
    P.x_scale = 1.0f;
    P.scale_pairs = pl.scale_pairs ? 1 : 0;
    P.sinkK = c->state + pl.off_sinkK;
    P.sinkV = c->state + pl.off_sinkV;
    P.ringK = c->state + pl.off_ringK;
    P.ringV = c->state + pl.off_ringV;
    c->T = 0;
    *out = c.release();
    return IWDFT_OK;

  } catch (...) {  // std::bad_alloc from the host-side containers: nothing may cross the C ABI
    return fail(IWDFT_ERR_ARG, "out of host memory");
  }
}

int iwdft_destroy(iwdft_ctx* ctx) {
  if (ctx)
    for (auto& m : ctx->marks)
      for (int i = 0; i < 4; ++i) (void)hipEventDestroy(m.ev[i]);
  delete ctx;
  return IWDFT_OK;
}

int iwdft_phase_timing(iwdft_ctx* ctx, int enable) {
  int rc = check_ctx(ctx);
  if (rc != IWDFT_OK) return rc;
  ctx->timing = enable != 0;
  return IWDFT_OK;
}

int iwdft_phase_times(iwdft_ctx* ctx, double* ms, int64_t* n_calls) {
  int rc = check_ctx(ctx);
  if (rc != IWDFT_OK) return rc;
  if (!ms || !n_calls) return fail(IWDFT_ERR_ARG, "ms / n_calls is NULL");
  ms[0] = ms[1] = ms[2] = 0.0;
  *n_calls = 0;
  for (size_t i = 0; i < ctx->marks_used; ++i) {
    const PhaseEvents& m = ctx->marks[i];
    hipError_t e = hipEventSynchronize(m.ev[3]);
    for (int p = 0; p < 3 && e == hipSuccess; ++p) {
      float t = 0.f;
      e = hipEventElapsedTime(&t, m.ev[p], m.ev[p + 1]);
      ms[p] += t;
    }
    if (e != hipSuccess) {
      ctx->marks_used = 0;
      return fail(IWDFT_ERR_HIP, "reading phase events: %s", hipGetErrorString(e));
    }
  }
  *n_calls = (int64_t)ctx->marks_used;
  ctx->marks_used = 0;
  return IWDFT_OK;
}

int64_t iwdft_num_tokens(const iwdft_ctx* ctx) { return ctx ? ctx->T : -1; }

int iwdft_prefill_kind(const iwdft_ctx* ctx) {
  return ctx ? (ctx->plan.use_fft_prefill ? 1 : (ctx->plan.use_any_prefill ? 2 : 0)) : -1;
}

int iwdft_attn_pipelined(const iwdft_ctx* ctx) { return ctx ? (attn_pipelines(ctx->P, ctx->plan.use_fft) ? 1 : 0) : -1; }

int iwdft_attn_kind(const iwdft_ctx* ctx) { return ctx ? (ctx->plan.use_fft ? 1 : (ctx->plan.use_chirp ? 2 : 0)) : -1; }

int iwdft_set_num_tokens(iwdft_ctx* ctx, int64_t T) {
  if (!ctx) return fail(IWDFT_ERR_ARG, "ctx is NULL");
  if (T < ctx->desc.M) return fail(IWDFT_ERR_ARG, "T = %lld is below M", (long long)T);
  ctx->T = T;
  ctx->pend = 0;  // the restored buffer is taken as complete
  return IWDFT_OK;
}

int iwdft_prefill(iwdft_ctx* ctx, const void* d_K, const void* d_V, void* hip_stream) {
  int rc = check_ctx(ctx);
  if (rc != IWDFT_OK) return rc;
  if (!d_K || !d_V) return fail(IWDFT_ERR_ARG, "d_K / d_V is NULL");
  {
    // the FFT prefill without sink / recent windows falls back to narrower loads; it still needs whole channel pairs
    const bool narrow_ok = ctx->plan.use_fft_prefill && ctx->desc.n_sink == 0 && ctx->desc.n_recent == 0;
    const uintptr_t mask = narrow_ok ? (ctx->desc.kv_dtype == IWDFT_BF16 ? 3u : 7u) : 15u;
    if ((((uintptr_t)d_K | (uintptr_t)d_V) & mask) != 0)
      return fail(IWDFT_ERR_ARG, "d_K / d_V must be %u-byte aligned for this prefill", (unsigned)mask + 1);
  }
  ctx->pend = 0;  // the prefill overwrites the whole state
  rc = launched(ctx->plan.use_fft_prefill ? launch_prefill_fft(ctx->P, d_K, d_V, (hipStream_t)hip_stream)
                : ctx->plan.use_any_prefill
                    ? launch_prefill_any(ctx->P, d_K, d_V, (hipStream_t)hip_stream)
                    : launch_prefill(ctx->P, d_K, d_V, (hipStream_t)hip_stream),
                "prefill launch");
  if (rc != IWDFT_OK) return rc;
  ctx->T = ctx->desc.M;
  return IWDFT_OK;
}

int iwdft_append(iwdft_ctx* ctx, const void* d_tok_k, const void* d_tok_v, void* hip_stream) {
  int rc = check_ctx(ctx);
  if (rc != IWDFT_OK) return rc;
  if (!d_tok_k || !d_tok_v) return fail(IWDFT_ERR_ARG, "d_tok_k / d_tok_v is NULL");
  if (misaligned16(d_tok_k) || misaligned16(d_tok_v)) return fail(IWDFT_ERR_ARG, kAlignMsg);
  if (ctx->T < ctx->desc.M) return fail(IWDFT_ERR_STATE, "iwdft_append before iwdft_prefill");
  if ((rc = flush_pending(ctx, (hipStream_t)hip_stream)) != IWDFT_OK) return rc;
  // The recent ring was filled oldest-first at prefill, so after T - M appends the oldest token
  // sits in slot (T - M) mod R.
  const uint32_t ring_pos = ctx->P.R ? (uint32_t)((ctx->T - ctx->desc.M) % ctx->P.R) : 0u;
  // Sec. 4.1 shortcut: S <- W (S + x / (T + 1)); on the stored M S_T that is the exact update of x M / (T + 1).
  ctx->P.x_scale = shortcut(ctx) ? (float)((double)ctx->desc.M / (double)(ctx->T + 1)) : 1.0f;
  rc = launched(launch_append(ctx->P, d_tok_k, d_tok_v, t_shift(ctx), ring_pos, (hipStream_t)hip_stream),
                "append launch");
  ctx->P.x_scale = 1.0f;
  if (rc != IWDFT_OK) return rc;
  ctx->T += 1;
  return IWDFT_OK;
}

int iwdft_export_coeffs(iwdft_ctx* ctx, int32_t layer, float* d_SK, float* d_SV, void* hip_stream) {
  int rc = check_ctx(ctx);
  if (rc != IWDFT_OK) return rc;
  if (layer < 0 || layer >= ctx->desc.n_layers) return fail(IWDFT_ERR_ARG, "layer %d out of range", layer);
  if (ctx->T < ctx->desc.M) return fail(IWDFT_ERR_STATE, "iwdft_export_coeffs before iwdft_prefill");
  if (!d_SK && !d_SV) return IWDFT_OK;
  if ((rc = flush_pending(ctx, (hipStream_t)hip_stream)) != IWDFT_OK) return rc;
  return launched(launch_export(ctx->P, layer, d_SK, d_SV, t_shift(ctx),
                                (float)(1.0 / (double)(shortcut(ctx) ? ctx->desc.M : ctx->T)),
                                (hipStream_t)hip_stream),
                  "export launch");
}

int iwdft_export_bins(iwdft_ctx* ctx, int32_t layer, int32_t* d_bins, void* hip_stream) {
  int rc = check_ctx(ctx);
  if (rc != IWDFT_OK) return rc;
  if (layer < 0 || layer >= ctx->desc.n_layers) return fail(IWDFT_ERR_ARG, "layer %d out of range", layer);
  if (!d_bins) return fail(IWDFT_ERR_ARG, "d_bins is NULL");
  const LayerInfo& L = ctx->plan.layers[layer];
  return launched(hipMemcpyAsync(d_bins, ctx->P.bins + L.bin_off, sizeof(int32_t) * (size_t)L.nb,
                                 hipMemcpyDeviceToDevice, (hipStream_t)hip_stream),
                  "export bins");
}

int iwdft_reconstruct_grid(iwdft_ctx* ctx, int32_t layer, int64_t a0, int64_t stride, int64_t n_slots, void* d_Kt,
                           void* d_Vt, void* hip_stream) {
  int rc = check_ctx(ctx);
  if (rc != IWDFT_OK) return rc;
  if (layer < 0 || layer >= ctx->desc.n_layers) return fail(IWDFT_ERR_ARG, "layer %d out of range", layer);
  if (stride < 1 || stride > ctx->desc.M) return fail(IWDFT_ERR_ARG, "stride %lld outside [1, M]", (long long)stride);
  if (a0 < 0 || n_slots < 0 || a0 > ctx->desc.M || (n_slots > 0 && a0 + (n_slots - 1) * stride >= ctx->desc.M))
    return fail(IWDFT_ERR_ARG, "slots %lld + %lld * [0, %lld) outside [0, M)", (long long)a0, (long long)stride,
                (long long)n_slots);
  if (ctx->T < ctx->desc.M) return fail(IWDFT_ERR_STATE, "iwdft_reconstruct before iwdft_prefill");
  if (n_slots == 0 || (!d_Kt && !d_Vt)) return IWDFT_OK;
  if ((rc = flush_pending(ctx, (hipStream_t)hip_stream)) != IWDFT_OK) return rc;
  set_read_gain(ctx);
  return launched(launch_reconstruct(ctx->P, layer, (uint32_t)a0, (uint32_t)stride, (uint32_t)n_slots, d_Kt, d_Vt,
                                     t_shift(ctx), ctx->plan.use_fft, (hipStream_t)hip_stream),
                  "reconstruct launch");
}

int iwdft_reconstruct(iwdft_ctx* ctx, int32_t layer, int64_t a0, int64_t n_slots, void* d_Kt, void* d_Vt,
                      void* hip_stream) {
  if (ctx && (a0 < 0 || n_slots < 0 || a0 + n_slots > ctx->desc.M))
    return fail(IWDFT_ERR_ARG, "slots [%lld, %lld) outside [0, M)", (long long)a0, (long long)(a0 + n_slots));
  return iwdft_reconstruct_grid(ctx, layer, a0, 1, n_slots, d_Kt, d_Vt, hip_stream);
}

int compressed_decode_attn(iwdft_ctx* ctx, const void* d_q, void* d_out, float scale, void* hip_stream) {
  int rc = check_ctx(ctx);
  if (rc != IWDFT_OK) return rc;
  if (!d_q || !d_out) return fail(IWDFT_ERR_ARG, "d_q / d_out is NULL");
  if (misaligned16(d_q) || misaligned16(d_out)) return fail(IWDFT_ERR_ARG, kAlignMsg);
  if (ctx->T < ctx->desc.M) return fail(IWDFT_ERR_STATE, "compressed_decode_attn before iwdft_prefill");
  if (!std::isfinite(scale)) return fail(IWDFT_ERR_ARG, "scale is not finite");
  if (scale <= 0.0f) scale = 1.0f / std::sqrt((float)ctx->desc.head_dim);
  if ((rc = flush_pending(ctx, (hipStream_t)hip_stream)) != IWDFT_OK) return rc;
  const Plan& pl = ctx->plan;
  const PhaseEvents* marks = nullptr;
  if ((rc = next_marks(ctx, &marks)) != IWDFT_OK) return rc;
  set_read_gain(ctx);
  return launched(launch_attn(ctx->P, d_q, d_out, scale, (float2*)(ctx->ws + pl.off_qc),
                              (float2*)(ctx->ws + pl.off_Pn), (float*)(ctx->ws + pl.off_pe),
                              (float*)(ctx->ws + pl.off_direct),
                              pl.use_fft, parts_at(pl, ctx->ws + pl.off_parts, ctx->ws + pl.off_stats), marks,
                              (hipStream_t)hip_stream),
                  "decode attention launch");
}

int compressed_decode_attn_static(iwdft_ctx* ctx, const void* d_q, void* d_out, float scale, void* hip_stream) {
  int rc = check_ctx(ctx);
  if (rc != IWDFT_OK) return rc;
  if (!d_q || !d_out) return fail(IWDFT_ERR_ARG, "d_q / d_out is NULL");
  if (misaligned16(d_q) || misaligned16(d_out)) return fail(IWDFT_ERR_ARG, kAlignMsg);
  if (ctx->T < ctx->desc.M) return fail(IWDFT_ERR_STATE, "compressed_decode_attn_static before iwdft_prefill");
  if (!std::isfinite(scale)) return fail(IWDFT_ERR_ARG, "scale is not finite");
  if (scale <= 0.0f) scale = 1.0f / std::sqrt((float)ctx->desc.head_dim);
  const Plan& pl = ctx->plan;
  // Same arrays as the workspace form, laid out inside the library's scratch: qc | Pn | pe | direct scores.
  const size_t n_heads = (size_t)ctx->P.n_slices * (size_t)pl.G;
  const size_t rows = align256(sizeof(float2) * (size_t)pl.ws_total);
  const size_t pe_bytes = align256(sizeof(float) * n_heads * (size_t)(ctx->P.S + ctx->P.R));
  const size_t direct_bytes = (pl.use_fft || pl.use_chirp) ? 0 : align256(sizeof(float) * n_heads * (size_t)ctx->desc.M);
  const size_t need = 2 * rows + pe_bytes + direct_bytes;
  if (need > kStaticScratchBytes)
    return fail(IWDFT_ERR_SIZE, "compressed_decode_attn_static needs %zu bytes of scratch, the library holds %zu", need,
                kStaticScratchBytes);
  // ... and as many parts of the softmax as there is room for (two of low frequencies do not pay, see softmax_parts); equal up to rounding whatever their number.
  Parts parts;
  const auto end_of = [&](int n) { return need + align256(rows * (size_t)n) + stats_bytes(pl, ctx->P.n_slices, n); };
  int n_parts = pl.parts;
  while (n_parts > 1 && end_of(n_parts) > kStaticScratchBytes) --n_parts;
  if (n_parts < (pl.use_fft && pl.low_logN ? 3 : 2)) n_parts = 1;
  char* sc = nullptr;
  if ((rc = static_scratch(ctx->device, &sc)) != IWDFT_OK) return rc;
  if ((rc = flush_pending(ctx, (hipStream_t)hip_stream)) != IWDFT_OK) return rc;
  set_read_gain(ctx);
  if (n_parts > 1) {
    parts = parts_at(pl, sc + need, sc + need + align256(rows * (size_t)n_parts));
    parts.n = n_parts;
  }
  // Every entry of the arrays is written by the kernels before it is read, so nothing needs clearing
  // although the scratch still holds the previous call's contents.
  return launched(launch_attn(ctx->P, d_q, d_out, scale, (float2*)sc, (float2*)(sc + rows), (float*)(sc + 2 * rows),
                              (float*)(sc + 2 * rows + pe_bytes), pl.use_fft, parts, nullptr, (hipStream_t)hip_stream),
                  "decode attention launch (static scratch)");
}

int iwdft_append_attn(iwdft_ctx* ctx, const void* d_tok_k, const void* d_tok_v, const void* d_q, void* d_out,
                      float scale, void* hip_stream) {
  int rc = check_ctx(ctx);
  if (rc != IWDFT_OK) return rc;
  if (!d_tok_k || !d_tok_v || !d_q || !d_out) return fail(IWDFT_ERR_ARG, "a token / query / output pointer is NULL");
  if (misaligned16(d_tok_k) || misaligned16(d_tok_v) || misaligned16(d_q) || misaligned16(d_out))
    return fail(IWDFT_ERR_ARG, kAlignMsg);
  if (ctx->T < ctx->desc.M) return fail(IWDFT_ERR_STATE, "iwdft_append_attn before iwdft_prefill");
  if (!std::isfinite(scale)) return fail(IWDFT_ERR_ARG, "scale is not finite");
  if (scale <= 0.0f) scale = 1.0f / std::sqrt((float)ctx->desc.head_dim);
  if (!step_can_fuse(ctx->P) || shortcut(ctx)) {  // more query heads per KV head than one pass holds, or the
                                                  // shortcut's per-token scale: plain sequence
    rc = iwdft_append(ctx, d_tok_k, d_tok_v, hip_stream);
    if (rc != IWDFT_OK) return rc;
    return compressed_decode_attn(ctx, d_q, d_out, scale, hip_stream);
  }
  const Plan& pl = ctx->plan;
  const uint32_t ring_pos = ctx->P.R ? (uint32_t)((ctx->T - ctx->desc.M) % ctx->P.R) : 0u;
  const PhaseEvents* marks = nullptr;
  if ((rc = next_marks(ctx, &marks)) != IWDFT_OK) return rc;
  const uint32_t tsh0 = (uint32_t)((ctx->T - ctx->pend - ctx->desc.M) % ctx->desc.M);  // oldest pending token
  rc = launched(launch_step(ctx->P, d_tok_k, d_tok_v, d_q, d_out, scale, (float2*)(ctx->ws + pl.off_qc),
                            (float2*)(ctx->ws + pl.off_Pn), (float*)(ctx->ws + pl.off_pe),
                            ctx->ws + pl.off_pendK, ctx->ws + pl.off_pendV, (float*)(ctx->ws + pl.off_ps),
                            (float*)(ctx->ws + pl.off_direct), pl.use_fft, tsh0, ring_pos, ctx->pend,
                            pl.write_every, parts_at(pl, ctx->ws + pl.off_parts, ctx->ws + pl.off_stats), marks,
                            (hipStream_t)hip_stream),
                "fused decode step launch");
  if (rc != IWDFT_OK) return rc;
  ctx->pend = (ctx->pend + 1) % pl.write_every;  // back to 0: this step wrote the coefficients
  ctx->T += 1;
  return IWDFT_OK;
}

int iwdft_flush(iwdft_ctx* ctx, void* hip_stream) {
  int rc = check_ctx(ctx);
  if (rc != IWDFT_OK) return rc;
  return flush_pending(ctx, (hipStream_t)hip_stream);
}

int iwdft_select_bins(const float* delta, int32_t n_layers, int32_t n_chunks, int64_t M, double r,
                      int64_t* bin_offsets, int32_t* bins, int64_t bins_capacity) {
  try {
    if (!delta || !bin_offsets) return fail(IWDFT_ERR_ARG, "delta / bin_offsets is NULL");
    if (n_layers <= 0 || n_chunks <= 0) return fail(IWDFT_ERR_ARG, "n_layers and n_chunks must be positive");
    if (M < 1 || M > ((int64_t)1 << 30)) return fail(IWDFT_ERR_ARG, "M = %lld outside [1, 2^30]", (long long)M);
    if (!(r >= 0.0) || !std::isfinite(r)) return fail(IWDFT_ERR_ARG, "retention ratio must be finite and >= 0");
    if (bins_capacity < 0 || (bins_capacity > 0 && !bins)) return fail(IWDFT_ERR_ARG, "bins is NULL");
    std::vector<int> keep;
    int64_t total = 0;
    bin_offsets[0] = 0;
    for (int l = 0; l < n_layers; ++l) {
      if (select_chunks(delta + (size_t)l * n_chunks, n_chunks, r, &keep) != 0)
        return fail(IWDFT_ERR_ARG, "delta of layer %d holds a NaN", l);
      for (int c : keep) {
        const int64_t a = chunk_edge(c, M, n_chunks), b = chunk_edge(c + 1, M, n_chunks);
        for (int64_t k = a; k < b; ++k, ++total)
          if (total < bins_capacity) bins[total] = (int32_t)k;
      }
      bin_offsets[l + 1] = total;
    }
    if (total > bins_capacity)
      return fail(IWDFT_ERR_SIZE, "bins holds %lld entries, %lld needed", (long long)bins_capacity, (long long)total);
    for (int l = 0; l < n_layers; ++l)
      if (bin_offsets[l + 1] == bin_offsets[l])
        return fail(IWDFT_ERR_BINS, "layer %d keeps no bin (M smaller than the number of chunks)", l);
    return IWDFT_OK;

  } catch (...) {  // std::bad_alloc from the host-side containers: nothing may cross the C ABI
    return fail(IWDFT_ERR_ARG, "out of host memory");
  }
}

int iwdft_ablate_chunk(const void* d_x, void* d_out, int64_t n_slices, int64_t M, int32_t head_dim,
                       int32_t kv_dtype, int32_t n_chunks, int32_t chunk, void* hip_stream) {
  if (!d_x || !d_out) return fail(IWDFT_ERR_ARG, "d_x / d_out is NULL");
  if (n_slices < 0 || n_slices > 0x3fffff) return fail(IWDFT_ERR_ARG, "n_slices = %lld out of range", (long long)n_slices);
  if (kv_dtype != IWDFT_F32 && kv_dtype != IWDFT_BF16) return fail(IWDFT_ERR_ARG, "bad kv_dtype %d", kv_dtype);
  if (n_chunks <= 0 || chunk < 0 || chunk >= n_chunks)
    return fail(IWDFT_ERR_ARG, "chunk %d outside [0, %d)", chunk, n_chunks);
  if (M < 1) return fail(IWDFT_ERR_ARG, "M must be positive");
  if (head_dim != kHeadDim) return fail(IWDFT_ERR_UNSUPPORTED, "head_dim %d: this build handles 128", head_dim);
  if ((M & (M - 1)) != 0 || M < (int64_t)kFftMinM || M > ((int64_t)1 << 24))
    return fail(IWDFT_ERR_UNSUPPORTED, "iwdft_ablate_chunk needs M = 2^m with 256 <= M <= 2^24 (got %lld)",
                (long long)M);
  const size_t esz = kv_dtype == IWDFT_BF16 ? 2 : 4;
  const size_t bytes = (size_t)n_slices * (size_t)M * kHeadDim * esz;
  const char *a = (const char*)d_x, *b = (const char*)d_out;
  if (a < b + bytes && b < a + bytes && bytes) return fail(IWDFT_ERR_ARG, "d_x and d_out overlap");
  if (n_slices == 0) return IWDFT_OK;
  return launched(launch_ablate(d_x, d_out, (int)n_slices, (uint32_t)M, kv_dtype,
                                (int)chunk_edge(chunk, M, n_chunks), (int)chunk_edge(chunk + 1, M, n_chunks),
                                (hipStream_t)hip_stream),
                  "ablation launch");
}

}  // extern "C"
