// Internal interface between the C-ABI host code and the gfx950 kernels.
#ifndef FABFT_KERNELS_H
#define FABFT_KERNELS_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fabft {

// Query rows per workgroup for head dimension d: 8 waves of 32 rows, or 4
// waves at d = 256 (one wave per SIMD, for the register file of 512).
constexpr int query_tile_for(int d) { return d == 256 ? 128 : 256; }

// Tile loads of the d = 256 forward. A workgroup loads 64-row K and V tiles in
// steps of 16 rows: the step's start goes into the scalar offset of a raw
// buffer load, the lane's row in the step and its column into the vector offset.
// The load's range check is vector offset >= size - scalar offset, which refuses
// a load only while the scalar offset is no larger than the size. Steps past
// the rows (of the ragged last tile, and of the two tiles past the last one,
// which every step of the loop issues) therefore start at the size itself,
// where the check refuses every lane: no memory past the rows is touched, and
// the rows of tiles that a causal workgroup does not use are not fetched.
constexpr uint32_t kWideRowBytes = 512, kWideStepBytes = 16 * kWideRowBytes;
// size: the rows of a head that the key tiles [0, t_end) hold
constexpr uint32_t wide_load_size(int Lk, int t_end) {
  return (uint32_t)(Lk < 64 * t_end ? Lk : 64 * t_end) * kWideRowBytes;
}
// scalar offset of 16-row step `step` of the head
constexpr uint32_t wide_load_start(uint32_t step, uint32_t size) {
  return step * kWideStepBytes < size ? step * kWideStepBytes : size;
}

// One injected single-bit fault (site numbers and fields as fabft_fault,
// with the head flattened to bh = b * H + h).
constexpr int kMaxFaults = 8;
struct FaultDesc {
  int site, bh, row, col, tile, bit;
};

struct FwdParams {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  uint16_t* o;
  float* resid;
  uint8_t* flags;
  float* pred;    // injection/debug kernels only; may be null
  float* actual;  // injection/debug kernels only; may be null
  float* pred_w;    // weighted check, debug kernels only; may be null
  float* actual_w;  // weighted check, debug kernels only; may be null
  // score check, debug kernels only; may be null: the row's sum of raw
  // scores over the key tiles without a mask (lhs), q_i . sum_k K_k over the
  // same keys (rhs) and |q_i| . sum_k |K_k| (the bound); 0 with the check off
  float* s_lhs;
  float* s_rhs;
  float* s_bound;
  int wcheck;     // 1: also run the weighted (alternating-sign) checksum
  // split over the keys (mode 3): workgroup (head, query tile, split) runs
  // key tiles [split*split_tiles, (split+1)*split_tiles) and writes the
  // partial state of each row to ws (see launch_merge)
  int nsplit;
  int split_tiles;
  float* ws;
  int dio;               // head dimension of q, k, v, o in memory (<= the
                         // kernel's width; the rest of the width is zero)
  // score check (modes 1, 2; null = off): per head, ntk + 1 rows of the
  // kernel's width D, the exclusive prefix over key tiles of the column sums
  // of K (kpre) and of |K| (kabs); tau_s its relative threshold
  const float* kpre;
  const float* kabs;
  int ntk;
  float tau_s;
  int Lq, Lk;
  int n_qt;       // query tiles per head
  int n_items;    // work items (head, query tile): B * H * n_qt
  int grid;       // workgroups: n_items (times nsplit in mode 3), or fewer
                  // with persist
  int persist;    // 1: each of the grid's workgroups runs a list of items
                  // (set by launch_fwd, modes 0 and 1 only)
  float sl2;      // scale * log2(e)
  float tau_rel, tau_abs;
  int nf;                          // faults in f (injection kernels only)
  FaultDesc f[kMaxFaults];
};

// mode 0: checksum off, 1: checksum on, 2: checksum on + debug/injection,
// 3: checksum on, one key split per workgroup (partial states to p.ws),
// 4: checksum on, two passes over the keys (Algorithm 1: the row max first),
// 5: mode 4 with injection/debug outputs.
// Modes 0 and 1 (without the score check) may run as many workgroups as fit
// on the device at once, each running a list of items, when there are more
// items than that (set_persistent: off, automatic, always).
int launch_fwd(const FwdParams& p, int d, bool causal, int mode, hipStream_t stream);
// Whether workgroups of half the waves (128 query rows) run a forward (modes 0
// and 1, d = 64, 96 or 128) faster than those of 256 rows on `cus` compute units. A
// wave alone on its SIMD takes about 0.7 of the time per key tile that two
// take together, and at d = 64 (96) three (two) half workgroups share a CU,
// none of them in step with the others, so that one's start-up and epilogue
// overlap another's products. Measured (us, full -> half workgroups, checksum
// on; H heads of L):
//  * every half workgroup has a CU of its own: d = 64, 32 of 512: 14.5 ->
//    11.0; d = 96, 32 of 256, causal: 10.4 -> 8.2; d = 128: 13.3 -> 10.1.
//    At d = 128 with at most 128 query rows there is nothing to spread and
//    the idle waves' share of the loads is missed (4,096 keys: 86 -> 96).
//  * no more full workgroups than CUs, causal: a light query tile shares the
//    CU of a heavy one (L = 2048, 32 heads: d = 64 42 -> 35, 96 49 -> 44,
//    128 59 -> 56; L = 1500: 32 -> 26, 37 -> 31, 44 -> 35), but not with
//    short rows (L = 1024, 64 heads: 23.8 -> 24.5, 28.0 -> 29.5, level) and not
//    where all query tiles see about the same keys (few queries over many),
//    which is as without a mask: two half workgroups do the work of one full one
//    in the same time. d = 64 gains there in short rows (without a mask 0.90 to
//    0.985 of the time up to 7 tiles, 1.00 to 1.07 from 8 to 128; with it up to 3:
//    192 heads of 130 8.2 -> 7.3) and, with the mask, while hardly a CU holds
//    two (66 heads of 512: 14.1 -> 11.6, 80: 14.5 -> 15.0; 88 heads of 384: 10.7 ->
//    10.0, 128: 10.9 -> 12.0).
//  * more than that, at d = 64 where all query tiles see about the same keys
//    (no mask, or few queries over many keys): rounds decide. Where half
//    workgroups save a half round of the CUs they win by 10 to 35% (17 heads
//    of 4,096: 156 -> 117; 300 heads of 256 x 2,048 causal: 82 -> 64), and over
//    many rounds or in short rows the overlap makes up for taking sumrow and the
//    loads of K and V twice (192 heads of 1,024 69.7 -> 68.0, 96 of 4,096 480 ->
//    477, 256 of 512 x 256 0.93). Without a mask long rows of two rounds (beyond 12
//    tiles) and of three (beyond 32) lose with the checksum or the score check:
//    by 3 to 5% over 4,096 keys (32 heads: 162 -> 167), 1 to 3% over 2,048 and
//    0 to 3% over 1,024; three rounds 0 to 2.5% (48 heads of 4,096: 242 -> 245);
//    without a check (157 -> 153) and with the weighted one (183 -> 181) they
//    gain or are level, as does one query tile per head (0.975 to 1.0). With the
//    mask the half order evens the rounds out (0.86 to 1.0) unless two rounds are full,
//    or nearly: 64 heads of 2,048 x 4,096 128 -> 138 (weighted 145 -> 152), of
//    2,048 x 8,192 279 -> 284 (weighted 323 -> 312, off 269 -> 262); with short
//    rows, whose full form is persistent, 256 heads of 512 x 1,024 42.4 -> 44.6
//    (weighted 47.2 -> 48.8, off 42.0 -> 41.0). (Ranges: several cards.)
//  * more than that otherwise: with the causal order long rows lose (d = 64,
//    32 heads of 4,096: 91 -> 109) and short ones gain (L = 700: 33 -> 21). At
//    d = 96 short rows gain (384 heads of 512: 59.9 -> 58.9, of 128: 23.3 ->
//    19.3); so do longer ones where half a round is saved (24 heads of 4,096
//    without a mask 190 -> 173), which this rule does not use. At d = 128 (one half
//    workgroup per CU: its LDS ring) whole query tiles lose (384 heads of 512
//    53 -> 70); mostly empty last tiles gain (414 heads of 330 x 272 without a
//    check 61 -> 55), not used either.
inline bool half_is_faster(int d, bool causal, bool check, bool weighted, int heads, int Lq, int Lk,
                           int cus) {
  const int rows = query_tile_for(d);
  const long long n_qt = ((long long)Lq + rows - 1) / rows;
  const long long full = heads * n_qt;
  const long long half = heads * (((long long)Lq + rows / 2 - 1) / (rows / 2));
  const int tiles = (Lk + 63) / 64;   // of the last query tile
  // query tiles of about the same work: no mask, or few queries over many keys
  const bool flat = !causal || 2LL * ((long long)Lk - Lq + rows) >= Lk;
  if (cus <= 0 || half > 0x7fffffff) return false;
  if (half <= cus) return d != 128 || half > full;
  if (full <= cus) {
    if (!flat) return tiles >= 20;
    if (d != 64) return false;
    return causal ? tiles <= 3 || (tiles <= 8 && 8 * half <= 9LL * cus) : tiles <= 7;
  }
  if (d == 128) return false;
  if (d == 64 && flat) {
    const long long rounds = (full + cus - 1) / cus;
    if ((half + cus - 1) / cus < 2 * rounds || rounds > 3) return true;
    const bool plain = check && !weighted;
    if (!causal) return !plain || n_qt == 1 || tiles <= (rounds == 2 ? 12 : 32);
    if (rounds == 3 || 16 * full < 30LL * cus) return true;
    if (n_qt >= 8 && (plain || Lk < 3LL * Lq)) return false;
    return !check || n_qt == 1 || tiles > 16;
  }
  return tiles <= (d == 64 ? 12 : 8);
}
enum { kPersistOff = 0, kPersistAuto = 1, kPersistAlways = 2 };
void set_persistent(int mode);
int get_persistent();
int key_tile(int d);
// Width the kernels compute with for a head dimension d (64, 96, 128 or
// 256): d itself, or 128 for d = 96 (columns 96..127 are zero on chip; the
// forward of modes 0 and 1 computes 96 columns itself, but the split records and
// the key prefix sums keep this width).
inline int compute_width(int d) { return d == 96 ? 128 : d; }
// Partial-state record of (head, row, split) in the split workspace, in
// floats: m (exp2 domain), l, c, c_w, then the d unnormalised outputs o.
inline int split_record_floats(int d) { return d + 4; }
// Merge the partial states of every row (mode 3 writes them) into O, resid
// and flags.
int launch_merge(const FwdParams& p, int d, int nheads, hipStream_t stream);
// Column sums of K per key tile and their exclusive prefix over the tiles
// (kpre) and the same for |K| (kabs): BH heads, (ceil(Lk/64) + 1) rows of
// compute_width(d) floats each.
int launch_kpre(const uint16_t* k, int BH, int Lk, int d, float* kpre, float* kabs,
                hipStream_t stream);
inline long long kpre_floats(long long BH, int Lk, int d) {
  return BH * ((Lk + 63) / 64 + 1) * (long long)compute_width(d);
}
// hflags_host: null, or pinned host memory (its device address) for a copy
int launch_head_flags(const uint8_t* flags, int BH, int Lq, uint8_t* hflags, uint8_t* hflags_host,
                      hipStream_t stream);
// Threads per head of the global check. Up to one workgroup per CU there is
// nothing else to keep loads in flight: 16 waves (B=1 H=32 L=2048 d=128: 256 threads
// 14, 1,024 9.2 us). With more heads the start of 16 waves per head costs
// more than the check (4,096 heads of 16 rows, d = 64: 64 threads 3.5, 256 6.2,
// 1,024 25.1; 2,048 of 256 rows: 256 threads 12.0, 1,024 20.6), except over long
// heads of many bytes in all (2,048 of 2,048 rows: 96.9, 90.4). A head of at most
// 512 chunks of 16 bytes takes one wave at any count (8,192 heads of 32 rows: 64
// threads 5.9, 256 11.0; 32 heads of 64 rows: 3.4 with each). (256: the chip's
// CUs; asking the runtime costs more than it could gain here.)
inline int global_threads(int BH, int Lq, int d) {
  const long long chunks = (long long)Lq * d / 8;
  if (chunks <= 512) return 64;
  return BH <= 256 || (chunks >= 8192 && BH * chunks >= (1 << 24)) ? 1024 : 256;
}
int launch_global(const uint16_t* o, const float* resid, int BH, int Lq, int d, float tau_rel,
                  float tau_abs, double* gsum, uint8_t* gflag, hipStream_t stream);

}  // namespace fabft

#endif
