// C ABI of the MI355X sparse-lexical LM head: host-side validation, workspace layout and kernel
// launches.  See include/lsr_head.h for the contract of every entry point.
#include "lsr_head.h"
#include "lsr_head_measure.h"

#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <mutex>

#include "bwd.hpp"
#include "fwd_few.hpp"
#include "fwd_mfma.hpp"
#include "fwd_misc.hpp"
#include "probes.hpp"

// Scratch of lsr_head_forward_static: device memory that lives in the library's code object, one copy
// per GPU, held until the process ends.  In host code this name is only a stand-in for the symbol; the
// device address comes from hipGetSymbolAddress (static_scratch below) and is what every launch uses.
static __device__ __align__(256) unsigned char scratch[LSR_STATIC_SCRATCH_BYTES];

namespace {

using namespace lsr;

constexpr size_t ALIGN = 256;
inline size_t align_up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }

struct Shape {
    int B, S, D, V;
    int dtype;
};

int check_desc(const lsr_head_desc* d, Shape* out) {
    if (!d) return LSR_ERR_NULL;
    if (d->hw_dtype != LSR_F32 && d->hw_dtype != LSR_BF16) return LSR_ERR_DTYPE;
    if (d->B < 1 || d->S < 1 || d->D < 1 || d->V < 1) return LSR_ERR_SHAPE;
    if (d->D % 8 != 0 || d->D > 8192 || d->S > 32768 || d->B > 65535) return LSR_ERR_SHAPE;
    if (d->V >= (int64_t(1) << 31) - 4096) return LSR_ERR_SHAPE;      // every factor is bounded before a product is formed
    if (d->B * d->S >= (int64_t(1) << 31) || d->B * d->V >= (int64_t(1) << 31)) return LSR_ERR_SHAPE;
    out->B = (int)d->B; out->S = (int)d->S; out->D = (int)d->D; out->V = (int)d->V;
    out->dtype = d->hw_dtype;
    return LSR_OK;
}

inline bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

// Chunks of the packed forward (see fwd_mfma.hpp).  The host does not know the lengths, so it sizes the
// grid and the workspace for the longest block list the shape allows (every sequence full:
// B * ceil(S/32) blocks, 8 per tile); chunks beyond the real list return at once.
// Chunks and launch mode.  A unit of work is (chunk of tiles, vocabulary tile).
// Deep problems launch one workgroup per unit, with chunks of four tiles: a workgroup that walks several
// tiles hides the start of each behind the one before, the hardware hands the next unit to whichever CU
// comes free (which keeps the CUs of an XCD on neighbouring units), and there are enough units that the
// last, partly filled round costs little.  Chunk lengths 1 / 2 / 4 / 8 measured (forward ms): B=16 S=256
// |V|=250002 0.966 / 0.944 / 0.958 / 1.007; B=64 S=512 D=1024 |V|=250002 8.91 / 8.92 / 8.78 / 8.95.
// Shallow problems (fewer than 24 units of one tile per CU; depth is estimated with sequences taken to
// fill 70 % of S) run one resident workgroup per CU over units of one tile each: no unit pays a workgroup
// launch, the next unit's row table and first slab are prefetched like the next tile's, and the last round
// is as full as the unit count allows (B=32 S=256 |V|=30522 and B=256 S=32: -1.5 to -3 %).  On deep problems
// resident workgroups drift apart and lose L2 locality (B=64 S=512 |V|=250002: L2 hit rate 0.82 -> 0.76,
// 16.1 -> 20.8 GB from the fabric, +1 % time), so they are not used there.
// Never more chunks than sequences: the per-chunk slots for cut sequences (8 bytes per vocabulary entry)
// then stay below the size of the outputs Y and I, whatever the sequence length.
// Rows per segment of the packed token list: the MFMA row block, or 8 for batches of short sequences
// (B=256, S=32, lengths 4..32: 8192 packed rows with 32-row segments, 5 400 with 8-row segments).
int fwd_seg(const Shape& s) { return s.S <= FWD_SEG_SHORT_MAX_S ? FWD_SEG_SHORT : FWD_BLK; }

// Kernel choice: the direct-to-LDS ring when H and W are each below 4 GiB (32-bit byte offsets per lane), else the
// register-staged loader (64-bit addresses).  Rows that are not a whole number of 128-byte K slabs take a variant of either
// that zero-fills the last slab.
bool fwd_direct(const Shape& s) {
    const size_t row = (size_t)s.D * (s.dtype == LSR_F32 ? 4 : 2);
    return (size_t)s.B * s.S * row < ((size_t)1 << 32) && (size_t)s.V * row < ((size_t)1 << 32);
}
bool fwd_whole_slabs(const Shape& s) { return (size_t)s.D * (s.dtype == LSR_F32 ? 4 : 2) % 128 == 0; }

// Calls of few tokens go through one launch of their own (fwd_few_kernel), where the hidden states fit the LDS.  Forward, us,
// packing and tile kernel -> one launch, all tokens valid (D=768 |V|=30522 bfloat16 where not said):
// The rule counts 256 CUs, as the others here do (a smaller partition of the device takes more rounds, with the same results).
//   one round of workgroups (|V| <= 32768), up to 16 sequences: B=1 S=32 22.1 -> 13.4, S=64 21.9 -> 17.3, D=2048 38.5 ->
//     28.1, B=8 S=8 24.6 -> 21.7, B=16 S=4 29.4 -> 25.3, B=1 S=16 D=384 14.1 -> 7.8, B=2 S=16 D=64 |V|=1000 11.3 -> 5.8; float32 B=1
//     S=32 38.6 -> 30.6, B=8 S=8 D=384 |V|=20000 39.4 -> 30.2, B=2 S=16 D=64 |V|=1000 13.9 -> 6.9
//   many rounds with long rows, which keep the loads of W going beside the sums: B=1 S=32 |V|=250002 97 -> 83, D=1024 115 -> 98,
//     |V|=160000 56 -> 44, B=1 S=16 D=512 |V|=250002 57.6 -> 47.4.  The sums grow with the sequences (and a little with the
//     tokens) and the loads with the columns, so what hides behind the loads is a number of sequences.
//     Odd numbers of rounds of 32768 entries, where the tile kernel's last round is at most half full: 4 (5 with up to 32 tokens),
//     from D=768 on 6 (8), from D=1024 on 8: B=4 S=16 D=512 |V|=270000 80 -> 70, B=6 S=10 D=768 |V|=425000 179 -> 167, B=8 S=4
//     D=1024 |V|=220000 126 -> 114; not B=8 S=8 D=512 |V|=147456 52 -> 56
//     Even numbers: one more than a row has whole batches of FEW_U k-steps, two more with up to 32 tokens from D=768 on, 8 from
//     D=1280 on: B=3 S=10 D=512 |V|=250002 62.7 -> 60.8, B=4 S=16 D=768 102 -> 92, B=5 S=6 D=1024 123 -> 115; not B=8 S=8 D=512
//     |V|=131072 40 -> 47.  Rows that end in a part of a batch: 2, and 3, 6, 7, 8 from D=768, 1024, 1280, 1600 on: B=2 S=16 D=640
//     |V|=250002 84 -> 77; not B=4 S=8 D=896 |V|=131072 49 -> 53.  Rows of 4 KiB, which share their memory channels: 2; not B=8 S=4
//     D=2048 |V|=301233 264 -> 288
//     Rows that are not whole slabs: 8 (B=8 S=8 D=568 |V|=702271 293 -> 263, B=2 S=16 D=712 |V|=250002 116 -> 88)
//   not: two or three rounds (B=4 S=16 |V|=40000 24.6 -> 27.6, B=1 S=32 |V|=60000 25.1 -> 26.1, |V|=119547 40.2 -> 40.2), many rounds of
//     short rows (B=1 S=64 D=384 |V|=119547 29.5 -> 33.5, B=8 S=8 D=128 |V|=250002 43 -> 58) or in float32 (B=1 S=16 D=512 |V|=250002
//     121 -> 134), more sequences (the lanes of a column take them one after the other: B=64 S=1 45.6 -> 51.1)
bool fwd_few(const Shape& s) {
    const long tokens = (long)s.B * s.S;
    if (tokens > FEW_MAX_TOKENS || few_lds((int)tokens, s.D * (s.dtype == LSR_F32 ? 4 : 2)) > FEW_LDS) return false;
    constexpr int round = 256 * FEW_COLS;                // vocabulary entries that 256 CUs take at a time
    if (s.V <= round) return s.B <= 16;
    if (s.dtype != LSR_BF16 || s.V < 4 * round || s.D < 512 || s.B > 8) return false;
    if (!fwd_direct(s) || !fwd_whole_slabs(s)) return true;
    const bool small = tokens <= 32;
    if ((s.V + round - 1) / round % 2 != 0) return s.B <= (s.D >= 1024 ? 8 : (s.D >= 768 ? (small ? 8 : 6) : (small ? 5 : 4)));
    constexpr int batch = 16 * FEW_U;                    // columns of a batch of loads
    if (s.D % 2048 == 0) return s.B <= 2;
    if (s.D % batch == 0) return s.B <= (s.D >= 1280 ? 8 : s.D / batch + 1 + (small && s.D >= 768 ? 1 : 0));
    return s.B <= (s.D >= 1600 ? 8 : s.D >= 1280 ? 7 : s.D >= 1024 ? 6 : s.D >= 768 ? 3 : 2);
}

// tpc: most tiles per chunk; window: float32 only, segments per window of a chunk (chunks are whole sequences, see
// fwd_f32_window); n_chunks: chunks the grid provides for
int fwd_f32_window(const Shape& s);
struct FwdChunks { int tpc, window, n_chunks; bool cut_possible, direct, tail, resident; };
FwdChunks fwd_chunks(const Shape& s) {
    const int seg = fwd_seg(s);
    const long segs_max = (long)s.B * ((s.S + seg - 1) / seg);
    const long tiles_max = (segs_max * seg + FWD_TM - 1) / FWD_TM;
    FwdChunks c;
    const double units1 = 0.7 * (double)tiles_max * (double)((s.V + 255) / 256) / 256.0;      // per workgroup at one tile per chunk
    const bool shallow = units1 < 24.0;
    c.tpc = shallow ? 1 : 4;
    const long per_seq = (tiles_max + s.B - 1) / s.B;
    if (c.tpc < per_seq) c.tpc = (int)per_seq;
    c.window = 0;
    c.n_chunks = (int)((tiles_max + c.tpc - 1) / c.tpc);
    if (s.dtype == LSR_F32) {
        c.window = fwd_f32_window(s);
        c.n_chunks = (int)((segs_max + c.window - 1) / c.window);
        const long longest = c.window - 1 + (s.S + seg - 1) / seg;        // segments of the sequences that begin in a window
        c.tpc = (int)(((longest < segs_max ? longest : segs_max) * seg + FWD_TM - 1) / FWD_TM);
    }
    // the register-staged loader has no prefetch across units to gain from residency, and rows with a partly filled last
    // slab were not tried
    c.direct = fwd_direct(s);
    c.tail = !fwd_whole_slabs(s);
    c.resident = shallow && c.direct && !c.tail;
    // a sequence of one segment can never lie across a chunk boundary: no pieces, no merge pass
    c.cut_possible = s.dtype == LSR_BF16 && s.S > seg && c.n_chunks > 1;
    return c;
}

// Float32 problems: segments per window of a chunk (FwdParams::tpc).  The float32 matrix rate makes a
// unit an order of magnitude longer than in bfloat16, so what matters is how full the last round of units
// is: the window of about half-tile granularity (short tiles cost what their live blocks cost) that gives the
// least rounds x rows, on 256 CUs, with sequences taken to fill 70 % of S; never less than the longest
// sequence, so that few windows come out empty.
int fwd_f32_window(const Shape& s) {
    const int seg = fwd_seg(s);
    const int per_seq = (s.S + seg - 1) / seg;
    const double segs = 0.7 * (double)s.B * per_seq;
    const double vtiles = (double)((s.V + fwd_tn(FWD_NWN) - 1) / fwd_tn(FWD_NWN));
    const int half = FWD_TM / seg / 2;
    int best = 0;
    double best_cost = 0.0;
    for (int k = 1; k <= 16; ++k) {
        const int L = k * half > per_seq ? k * half : per_seq;
        const double units = ceil(segs / L) * vtiles;
        const double cost = ceil(units / 256.0) * (L * seg + 32.0);
        if (!best || cost < best_cost) { best = L; best_cost = cost; }
    }
    // one workgroup of fwd_threads(FWD_NWN) threads per (window, vocabulary tile, in groups of FWD_GV_COLS columns), at most
    // 2^32 - 1 threads in a launch (a single window always fits)
    const long long max_units = (0xffffffffll / fwd_threads(FWD_NWN)) / 8 * 8;
    const long long groups = ((long long)s.V + FWD_GV_COLS - 1) / FWD_GV_COLS * (FWD_GV_COLS / fwd_tn(FWD_NWN));
    while (groups * (((long long)s.B * per_seq + best - 1) / best) > max_units) best *= 2;
    return best;
}

// ---- forward workspace: len[B] | pos[B*S] | seg0[B+1] | seg_meta[segs] | rows[segs*seg] |
//      part_m[chunks*V] | part_s[chunks*V]; segs = B * ceil(S/seg) being the most the packed layout can
//      need, the two part arrays only where a chunk boundary can fall inside a sequence ----
struct FwdWs { size_t len_off, pos_off, blk0_off, meta_off, rows_off, pm_off, ps_off, total; };
FwdWs fwd_ws(const Shape& s) {
    FwdWs w;
    const int seg = fwd_seg(s);
    const size_t blocks = (size_t)s.B * ((s.S + seg - 1) / seg);          // segments
    const FwdChunks c = fwd_chunks(s);
    const size_t part = c.cut_possible ? align_up(sizeof(float) * (size_t)c.n_chunks * s.V) : 0;
    w.len_off = 0;
    w.pos_off = w.len_off + align_up(sizeof(int) * (size_t)s.B);
    w.blk0_off = w.pos_off + align_up(sizeof(int) * (size_t)s.B * s.S);
    w.meta_off = w.blk0_off + align_up(sizeof(int) * ((size_t)s.B + 1));
    w.rows_off = w.meta_off + align_up(sizeof(int) * blocks);
    w.pm_off = w.rows_off + align_up(sizeof(int2) * blocks * seg);
    w.ps_off = w.pm_off + part;
    w.total = w.ps_off + part;
    return w;
}

// Column-sliced gathers (dH and dW), or whole rows by one workgroup each.  Slices gather what L2 holds, at the price of a pass
// over every list per slice and vocabulary chunk, whatever the list holds.  Where rows are a multiple of 64 columns that
// always paid; where they are not, pieces of rows straddle cache lines (reads and writes) and sparse gradients, which
// the host cannot see, ran up to 2.6 times slower in slices.  Backward, us, whole rows -> slices, for dense
// gradients; one in five; one in twenty (|V|=30522 where not said):
//   sliced: B=100 S=40 D=552 |V|=150000 6486 -> 2595; 1643 -> 921; 732 -> 577.  B=167 S=62 D=648 |V|=66407 5966 -> 2377; 1509 -> 858;
//     666 -> 555.  B=64 S=64 D=456 623 -> 347; 183 -> 144; 104 -> 106.  B=256 S=32 D=600 3861 -> 2026; 940 -> 621; 380 -> 278.
//     float32 B=32 S=64 D=712 840 -> 488; 220 -> 169; 101 -> 105.  Few waves: B=13 S=197 D=312 |V|=31091 172 -> 108; 84 -> 60;
//     71 -> 57.  B=16 S=100 D=456 |V|=60000 434 -> 240; 138 -> 108; 81 -> 86.  B=4 S=512 D=200 |V|=50000 141 -> 100; 75 -> 69; 62 -> 65
//     (dH alone loses where it has many waves: B=167 S=62 with one in twenty 195 -> 293)
//   whole rows: B=64 S=200 D=712 |V|=60000 1509 -> 1137; 373 -> 452; 172 -> 261.  B=45 S=110 D=680 |V|=70000 1270 -> 844; 331 -> 335;
//     156 -> 224.  B=16 S=250 D=904 |V|=200000 1385 -> 1586; 504 -> 806; 372 -> 547.  B=128 S=100 D=936 |V|=100000 7433 -> 4173;
//     1840 -> 1531; 771 -> 892.  B=64 S=64 D=776 |V|=60000 1473 -> 1077; 364 -> 376; 161 -> 251.  B=8 S=128 D=968 236 -> 145; 89 -> 90;
//     70 -> 76.  float32 B=64 S=24 D=904 |V|=30000 1610 -> 1028; 388 -> 358; 146 -> 163, B=16 S=128 D=328 |V|=20000 175 -> 187; 84 -> 79;
//     69 -> 62.  B=30 S=3000 D=312 |V|=60000 474 -> 584; 215 -> 271; 197 -> 236
bool sliced_gathers(const Shape& s) {
    if (s.D % DWS_COLS == 0) return true;
    const long long waves = (long long)s.B * s.S * n_slices(s.D);
    return s.D <= 720 && (s.S <= 64 || (s.dtype == LSR_BF16 && waves <= 16384));
}

// ---- backward workspace: perm[B*V + PERM_SLACK] (v, g) pairs | cnt[B*n_seg*S] | bstart[B*(S+1)] |
//      bounds[B*S*(n_vc+1)] (only when the dH gather is cut into n_vc > 1 vocabulary chunks; where D is not a
//      multiple of 64 they take the place of cnt, which nothing reads after the placement) ----
struct BwdWs { int n_seg, seg_len, key_bits, n_vc, vc_len; size_t perm_off, cnt_off, bs_off, cb_off, dh_stage_off, dw_stage_off, total; };

// Vocabulary chunks of the sliced dH gather.  A chunk is sized so that one 64-column slice of its
// rows of W is about 4 MB (what stays in L2 while every bucket gathers from it).  Each chunk after
// the first re-reads and re-writes dH once (8*B*S*D bytes), so the count is capped where that
// traffic would pass a quarter of the gather traffic itself (B*|V|*D elements): long sequences
// with few entries per bucket are gathered in one pass.
// Where row pieces straddle cache lines a window of half the rows takes the same lines.  Backward, us, whole -> half windows, for
// dense gradients; one in twenty: B=100 S=40 D=552 |V|=150000 3738 -> 2595; 520 -> 577, B=256 S=32 D=600 |V|=30522 2762 -> 2026;
// 289 -> 278, B=64 S=64 D=456 |V|=30522 405 -> 347; 89 -> 106, B=64 S=32 D=200 |V|=60000 430 -> 346; 107 -> 114; not for longer
// sequences (B=13 S=197 D=312 |V|=31091 108 -> 108; 57 -> 64) or few waves (B=2 S=64 D=328 |V|=30522 58 -> 66; 49 -> 57).
// n_seg: sort segments; where D is not a multiple of 64 the chunk bounds have to fit the count table.
void dh_chunks(const Shape& s, int n_seg, int* n_vc, int* vc_len) {
    const long esize = s.dtype == LSR_F32 ? 4 : 2;
    long rows_l2 = (4l << 20) / (DWS_COLS * esize);
    if (s.D * esize % 128 != 0 && s.S <= 64 && (long long)s.B * s.S * n_slices(s.D) > 4096) rows_l2 /= 2;
    long c = (s.V + rows_l2 - 1) / rows_l2;
    const long cap = (long)s.V * esize / (32l * s.S);
    if (c > cap) c = cap;
    if (c > 64) c = 64;
    if (s.D % DWS_COLS != 0 && c > n_seg - 1) c = n_seg - 1;
    if (c < 1 || !sliced_gathers(s)) c = 1;
    *n_vc = (int)c;
    *vc_len = (int)((s.V + c - 1) / c);
}
int dw_batch_chunk(const Shape& s);
int dw_stage_rows(const Shape& s);
int dw_tile_passes(const Shape& s);
// bf16_out: dH and dW are stored as bfloat16.  A result that several launches add up (dH over vocabulary
// chunks, dW over chunks of sequences) then keeps its float32 partial sums in a staging array of the
// workspace and is rounded once, by the last launch.
BwdWs bwd_ws(const Shape& s, bool bf16_out = false) {
    BwdWs w;
    // enough (b, segment) waves to fill the chip, segments of at least 512 entries, and a count
    // table no larger than B*V ints
    long n = 4096 / s.B;
    n = n < s.V / 512 ? n : s.V / 512;
    // short enough segments for the placement that sorts a segment in LDS, where it applies
    if (s.S <= PLACE_MAX_S) {
        const long fit = (s.V + PLACE_MAX_SEG - 129) / (PLACE_MAX_SEG - 128);
        n = n > fit ? n : fit;
    }
    n = n < s.V / s.S ? n : s.V / s.S;
    // one segment where a sequence fits it: the sort is then one launch (see bwd_place_staged_kernel)
    if (n < 1 || (s.S <= PLACE_MAX_S && s.V <= PLACE_MAX_SEG)) n = 1;
    w.n_seg = (int)n;
    w.seg_len = ((s.V + w.n_seg - 1) / w.n_seg + 63) / 64 * 64;
    w.n_seg = (s.V + w.seg_len - 1) / w.seg_len;
    w.key_bits = 0;
    while ((1 << w.key_bits) < s.S) ++w.key_bits;
    const size_t bv = (size_t)s.B * s.V;
    w.perm_off = 0;
    w.cnt_off = w.perm_off + align_up(sizeof(uint2) * (bv + PERM_SLACK));
    w.bs_off = w.cnt_off + align_up(sizeof(int) * (size_t)s.B * w.n_seg * s.S);
    w.cb_off = w.bs_off + align_up(sizeof(int) * (size_t)s.B * (s.S + 1));
    dh_chunks(s, w.n_seg, &w.n_vc, &w.vc_len);
    w.dh_stage_off = w.cb_off;
    if (s.D % DWS_COLS != 0) w.cb_off = w.cnt_off;
    else if (w.n_vc > 1) w.dh_stage_off += align_up(sizeof(int) * (size_t)s.B * s.S * (w.n_vc + 1));
    w.dw_stage_off = w.dh_stage_off + ((bf16_out && w.n_vc > 1) ? align_up(sizeof(float) * (size_t)s.B * s.S * s.D) : 0);
    // (the LDS-tile kernel takes one launch, and without dW nothing is staged)
    const bool dw_multi = dw_tile_passes(s) == 0 && dw_stage_rows(s) > 0 && dw_batch_chunk(s) < s.B;
    w.total = w.dw_stage_off + ((bf16_out && dw_multi) ? align_up(sizeof(float) * (size_t)s.V * s.D) : 0);
    return w;
}

// Buckets a wave of the sliced dH gather serves.  The lanes of a bucket load its entries in blocks of as many
// entries as the bucket has lanes (64 / k), two rounds of gathers per block.  Several buckets per wave pay
// off when a bucket holds too few entries per chunk to keep a wave busy for several blocks, and cost when
// their lists differ in length.  Lengths are not known on the host: sequences are taken to fill 70 % of S
// and every (b, v) pair to carry a gradient.  Measured (dH ms for k = 1 / 2 / 4 / 8; entries per bucket and
// chunk as estimated here, and as they really were): B=16 S=256 |V|=250002 (174; 217) 0.65 / 0.78 / 1.07 / -;
// B=64 S=512 |V|=250002, lengths 128..512 (87; 98) 2.93 / 2.32 / 2.41 / 3.5; B=256 S=512 |V|=30522, full
// lengths (85; 60) 0.91 / 0.75 / 0.79 / 0.90; B=256 S=512 |V|=250002, full lengths (87; 61) 9.3 / 8.0 / 7.7 /
// 8.6; B=128 S=8192 |V|=30522 (5; 4) 4.4 / 2.4 / 1.55 / 1.37.
int dh_buckets_per_wave(const Shape& s, int n_vc) {
    if (!sliced_gathers(s)) return 0;
    const double per_bucket = (double)s.V / ((0.7 * s.S > 1.0 ? 0.7 * s.S : 1.0) * n_vc);
    int bpw = per_bucket >= 128.0 ? 1 : (per_bucket >= 48.0 ? 2 : (per_bucket >= 12.0 ? 4 : 8));
    if (s.dtype == LSR_F32 && bpw > 4) bpw = 4;      // a float row piece takes 16 lanes
    return bpw;
}

// Waves that share a bucket of the sliced dH gather (then one bucket per workgroup, else four waves with buckets
// of their own).  One wave per long list leaves the launch waiting for its longest lists (a sequence of 4 tokens
// has |V| / 4 entries per bucket) and the chip half empty where buckets are few.  The price is paid where the lists turn
// out short, which the host cannot know: sparse gradients launch the same waves, and all but the first of a bucket of at
// most 64 entries leave at once (0.05 to 0.2 ns each).  The lines lie where one gradient in twenty costs about 3 % of a step.
// Forward and backward, us, one wave per bucket -> as chosen here, for dense gradients; one in five; one in twenty (D=768
// |V|=30522 where not said; in brackets the waves of a launch at one per bucket, x launches, and the estimated list):
//   4  B=64 S=32 (25k, 1363) 594 -> 462; 268 -> 259; 202 -> 200 (8 waves: 450; 272; 236).  float32 1576 -> 1216; 883 -> 848;
//      749 -> 736.  B=32 S=64 (25k, 681) 359 -> 297; 216 -> 208; 172 -> 170.  B=100 S=24 D=384 |V|=60000 (14k x 2, 1786) 916 ->
//      694; 412 -> 376; 303 -> 304.  B=24 S=50 D=512 |V|=120000 (10k x 4, 857) 793 -> 644; 398 -> 379; 317 -> 319.  B=128 S=24
//      D=512 (25k, 1817) 652 -> 534; 320 -> 302; 239 -> 247
//   2  B=32 S=128 D=1024 (66k, 341) 489 -> 446; 337 -> 343; 303 -> 313.  B=48 S=128 D=1024 (74k, 341) 517 -> 475; 366 -> 375;
//      340 -> 343.  B=16 S=128 (25k, 341) 234 -> 227; 183 -> 184; 174 -> 174.  B=128 S=40 (61k, 1090) 975 -> 863; 463 -> 439;
//      341 -> 348 (4 waves: 801; 447; 355).  B=60 S=40 |V|=200000 (29k x 7, 1020) 3448 -> 3062; 1470 -> 1412; 1085 -> 1093
//   1  (two waves instead) B=64 S=100 |V|=50000 (77k x 2, 357), backward 566 -> 550; -; 176 -> 197.  B=40 S=100 |V|=50000 (48k x 2, 357)
//      623 -> 590; 383 -> 381; 325 -> 333.  B=256 S=32 (98k, 1363), dH 904 -> 647; 187 -> 153; 61 -> 75 and the backward, where
//      it runs beside dW, 1677 -> 1753; -; 254 -> 257.  B=20 S=200 |V|=60000 (48k x 2, 214) 537 -> 510; 410 -> 414; 370 -> 377
// dH alone has no dW to hide the surplus behind: with one gradient in twenty B=10 S=60 |V|=200000 110 -> 128, B=32 S=128 D=1024 55 -> 62,
// B=60 S=40 |V|=200000 267 -> 271, B=24 S=50 D=512 |V|=120000 89 -> 86.
// List lengths as estimated above, in the time of bfloat16 entries (a float32 row piece takes twice the lanes).
int dh_waves_per_bucket(const Shape& s, int n_vc) {
    if (!sliced_gathers(s)) return 1;
    const double list = (double)s.V / ((0.7 * s.S > 1.0 ? 0.7 * s.S : 1.0) * n_vc) * (s.dtype == LSR_F32 ? 2.0 : 1.0);
    const long long waves = (long long)s.B * s.S * n_slices(s.D);      // per launch, at one per bucket
    if (waves <= 4096 && list >= 64.0) return 4;                       // latency alone (B=2 S=16 D=64 |V|=1000: 16 -> 6.4 us)
    if (list < 256.0) return 1;
    if (waves * n_vc > 80000) return list >= 512.0 && waves <= 80000 ? 2 : 1;
    return waves * n_vc <= 16384 || (waves <= 32768 && list >= 512.0) ? 4 : 2;
}

// Sequences per launch of the sliced dW gather.  The gather is L2-resident while the H slice of the
// sequences in flight (rows x 64 columns) is about 4 MB; larger batches are cut into chunks of
// consecutive sequences, each launch adding to dW (8*|V|*D bytes re-read and re-written per extra
// launch, capped at a quarter of the gather traffic and at 16 launches).  B=256, S=512, |V|=250002:
// dW 14.5 ms in one launch of 16-row tiles (16.8 MB slice).
int dw_batch_chunk(const Shape& s) {
    const long esize = s.dtype == LSR_F32 ? 4 : 2;
    const long per_seq = (long)s.S * DWS_COLS * esize;
    long bc = (4l << 20) / per_seq;
    bc = bc < 1 ? 1 : bc;
    long n = (s.B + bc - 1) / bc;
    const long cap = 1 + (long)s.B * esize / 32;
    n = n > cap ? cap : n;
    n = n > 16 ? 16 : n;
    if ((long)s.V < 16l * s.S) n = 1;      // a row of H is gathered about |V|/S times: too few for L2 to matter
    n = n < 1 ? 1 : n;
    return (int)((s.B + n - 1) / n);
}

// Vocabulary rows of the (g, I) staging tile of the sliced dW gather (at most 48 KiB of LDS for the sequences of
// one launch), or 0 when the whole-row kernel runs instead (see sliced_gathers, or too many sequences per launch for
// 16 rows).
int dw_stage_rows(const Shape& s) {
    const int nb = dw_batch_chunk(s);
    int VT = 64;
    while (VT > 1 && (size_t)nb * VT * 8 > 48 * 1024) VT /= 2;
    return VT >= 16 && sliced_gathers(s) ? VT : 0;
}

int check_device(int* n_cus) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return LSR_ERR_ARCH; }
    static int ok_dev[64] = {0};     // holds the CU count once a device has been checked
    if (dev >= 0 && dev < 64 && ok_dev[dev]) { *n_cus = ok_dev[dev]; return LSR_OK; }
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) { (void)hipGetLastError(); return LSR_ERR_ARCH; }
    if (strncmp(prop.gcnArchName, "gfx950", 6) != 0) return LSR_ERR_ARCH;
    if (prop.multiProcessorCount < 1) return LSR_ERR_ARCH;
    *n_cus = prop.multiProcessorCount;
    if (dev >= 0 && dev < 64) ok_dev[dev] = prop.multiProcessorCount;
    return LSR_OK;
}

// Device address of `scratch` on the current device, looked up once per device with that device
// current (every GPU holds its own copy at its own address).
int static_scratch(void** out) {
    static std::mutex mu;
    static void* ptr_of[64] = {nullptr};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) { (void)hipGetLastError(); return LSR_ERR_ARCH; }
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr_of[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) { (void)hipGetLastError(); return LSR_ERR_LAUNCH; }
        ptr_of[dev] = p;
    }
    *out = ptr_of[dev];
    return LSR_OK;
}

// Optional per-kernel event timing (the *_profiled entry points).
struct Prof {
    bool on = false;
    hipStream_t stream = nullptr;
    hipEvent_t ev[LSR_PROFILE_SLOTS][2];
    bool used[LSR_PROFILE_SLOTS] = {false};
    bool fail = false;
    void begin(int slot) {
        if (!on) return;
        if (hipEventCreate(&ev[slot][0]) != hipSuccess || hipEventCreate(&ev[slot][1]) != hipSuccess) { fail = true; return; }
        used[slot] = true;
        if (hipEventRecord(ev[slot][0], stream) != hipSuccess) fail = true;
    }
    void end(int slot) {
        if (!on || !used[slot]) return;
        if (hipEventRecord(ev[slot][1], stream) != hipSuccess) fail = true;
    }
    int finish(float* ms) {
        if (!on) return LSR_OK;
        if (hipStreamSynchronize(stream) != hipSuccess) fail = true;
        for (int i = 0; i < LSR_PROFILE_SLOTS; ++i) {
            ms[i] = 0.f;
            if (used[i]) {
                if (!fail && hipEventElapsedTime(&ms[i], ev[i][0], ev[i][1]) != hipSuccess) fail = true;
                (void)hipEventDestroy(ev[i][0]);
                (void)hipEventDestroy(ev[i][1]);
            }
        }
        return fail ? LSR_ERR_LAUNCH : LSR_OK;
    }
};

inline int launch_status() { return hipGetLastError() == hipSuccess ? LSR_OK : LSR_ERR_LAUNCH; }

// (see fwd_pack_kernel)
bool pack_in_one_launch(const Shape& s) {
    return (long)s.B * s.S <= PACK_MAX_TOKENS && s.B <= (s.S <= 64 ? PACK_MAX_B : 64);
}

template <typename T, bool DMA, int SEG, bool RES, bool TAIL = false>
void launch_fwd_cfg(FwdParams p, int V, bool arg, int n_cus, hipStream_t st) {
    constexpr int TN = fwd_tn(FWD_NWN);
    p.n_vtiles = (V + TN - 1) / TN;
    p.gv = FWD_GV_COLS / TN;
    // RES: one resident workgroup per CU (its LDS leaves room for no second one), a multiple of 8 so that
    // every XCD gets the same number.  Otherwise one workgroup per unit the longest possible token list
    // would need (workgroups beyond the real list return at once).
    const long long n_units = (long long)((p.n_vtiles + p.gv - 1) / p.gv) * p.gv * p.n_chunks;
    const int n_wg = RES ? (n_cus >= 8 ? n_cus / 8 * 8 : 8) : (int)((n_units + 7) / 8 * 8);
    const dim3 grid(n_wg), block(fwd_threads(FWD_NWN));
    if (arg) hipLaunchKernelGGL((fwd_mfma_kernel<T, true, DMA, SEG, RES, TAIL>), grid, block, 0, st, p);
    else     hipLaunchKernelGGL((fwd_mfma_kernel<T, false, DMA, SEG, RES, TAIL>), grid, block, 0, st, p);
}

template <typename T>
void launch_fwd(const FwdParams& p, int seg, bool direct, bool tail, bool resident, bool arg, int n_cus, hipStream_t st) {
    if (!direct) {
        if (seg == FWD_BLK) launch_fwd_cfg<T, false, FWD_BLK, false>(p, p.V, arg, n_cus, st);
        else launch_fwd_cfg<T, false, FWD_SEG_SHORT, false>(p, p.V, arg, n_cus, st);
    } else if (tail) {
        if (seg == FWD_BLK) launch_fwd_cfg<T, true, FWD_BLK, false, true>(p, p.V, arg, n_cus, st);
        else launch_fwd_cfg<T, true, FWD_SEG_SHORT, false, true>(p, p.V, arg, n_cus, st);
    } else if (seg == FWD_BLK) {
        if (resident) launch_fwd_cfg<T, true, FWD_BLK, true>(p, p.V, arg, n_cus, st);
        else launch_fwd_cfg<T, true, FWD_BLK, false>(p, p.V, arg, n_cus, st);
    } else {
        if (resident) launch_fwd_cfg<T, true, FWD_SEG_SHORT, true>(p, p.V, arg, n_cus, st);
        else launch_fwd_cfg<T, true, FWD_SEG_SHORT, false>(p, p.V, arg, n_cus, st);
    }
}

template <typename T>
void launch_few(const Shape& s, const void* H, const void* W, const float* bias, const uint8_t* mask, float* Y, int32_t* I, int n_cus,
                hipStream_t st) {
    const int row_bytes = s.D * (int)sizeof(T);
    const int n_tiles = (s.V + FEW_COLS - 1) / FEW_COLS;
    const dim3 grid(n_tiles < n_cus ? n_tiles : n_cus);
#define LSR_FEW(ARG) hipLaunchKernelGGL((fwd_few_kernel<T, ARG>), grid, dim3(FEW_THREADS), 0, st, static_cast<const T*>(H), \
                                        static_cast<const T*>(W), bias, mask, Y, I, s.B, s.S, s.D, s.V, few_stride(row_bytes), n_tiles)
    if (I) LSR_FEW(true);
    else LSR_FEW(false);
#undef LSR_FEW
}

int forward_impl(const lsr_head_desc* desc, const void* H, const void* W, const float* bias,
                 const uint8_t* mask, float* Y, int32_t* I, void* ws, size_t ws_bytes, hipStream_t st,
                 Prof& prof) {
    Shape s;
    int rc = check_desc(desc, &s);
    if (rc != LSR_OK) return rc;
    if (!H || !W || !bias || !mask || !Y) return LSR_ERR_NULL;
    if (misaligned(H) || misaligned(W) || misaligned(bias) || misaligned(Y) || (I && misaligned(I)) || misaligned(ws))
        return LSR_ERR_ALIGN;
    const FwdWs w = fwd_ws(s);
    if (!ws || ws_bytes < w.total) return LSR_ERR_WORKSPACE;
    int n_cus = 0;
    rc = check_device(&n_cus);
    if (rc != LSR_OK) return rc;

    prof.stream = st;
    if (fwd_few(s)) {
        prof.begin(1);
        if (s.dtype == LSR_F32) launch_few<float>(s, H, W, bias, mask, Y, I, n_cus, st);
        else launch_few<uint16_t>(s, H, W, bias, mask, Y, I, n_cus, st);
        prof.end(1);
        return launch_status();
    }
    int* len = reinterpret_cast<int*>(static_cast<char*>(ws) + w.len_off);
    int* pos = reinterpret_cast<int*>(static_cast<char*>(ws) + w.pos_off);

    prof.begin(0);
    // batches of few tokens are packed by one workgroup in one launch
    const bool one_launch = pack_in_one_launch(s);
    if (!one_launch) hipLaunchKernelGGL(fwd_prep_kernel, dim3(s.B), dim3(PREP_THREADS), 0, st, mask, len, pos, s.S);
    char* base = static_cast<char*>(ws);
    int* blk0 = reinterpret_cast<int*>(base + w.blk0_off);
    int* blk_meta = reinterpret_cast<int*>(base + w.meta_off);
    int2* rows = reinterpret_cast<int2*>(base + w.rows_off);
    float* part_m = reinterpret_cast<float*>(base + w.pm_off);
    int* part_s = reinterpret_cast<int*>(base + w.ps_off);
    const FwdChunks ck = fwd_chunks(s);
    const int seg = fwd_seg(s);
    if (one_launch) {
        hipLaunchKernelGGL(fwd_pack_kernel, dim3(1), dim3(PACK_THREADS), 0, st, mask, blk0, rows, blk_meta, s.B, s.S, seg);
    } else {
        hipLaunchKernelGGL(fwd_plan_kernel, dim3(1), dim3(PLAN_THREADS), 0, st, len, blk0, s.B, seg);
        hipLaunchKernelGGL(fwd_rows_kernel, dim3(s.B), dim3(FWD_ROWS_THREADS), 0, st, len, pos, blk0, rows, blk_meta, s.S, seg);
    }
    prof.end(0);
    if ((rc = launch_status()) != LSR_OK) return rc;

    prof.begin(1);
    FwdParams p;
    p.H = H; p.W = W;
    p.bias = bias; p.rows = rows; p.blk_meta = blk_meta; p.n_blocks = blk0 + s.B; p.Y = Y; p.I = I;
    p.part_m = part_m; p.part_s = part_s;
    p.B = s.B; p.S = s.S; p.D = s.D; p.V = s.V;
    p.n_chunks = ck.n_chunks; p.tpc = s.dtype == LSR_F32 ? ck.window : ck.tpc;
    if (s.dtype == LSR_F32) launch_fwd<float>(p, seg, ck.direct, ck.tail, ck.resident, I != nullptr, n_cus, st);
    else launch_fwd<uint16_t>(p, seg, ck.direct, ck.tail, ck.resident, I != nullptr, n_cus, st);
    prof.end(1);
    if (ck.cut_possible) {
        if ((rc = launch_status()) != LSR_OK) return rc;
        prof.begin(2);
        const int vgroups = (s.V + FWD_MERGE_THREADS - 1) / FWD_MERGE_THREADS;
        const dim3 grid(vgroups, fwd_merge_rows(vgroups, ck.n_chunks));
        if (I) hipLaunchKernelGGL((fwd_merge_kernel<true>), grid, dim3(FWD_MERGE_THREADS), 0, st, blk0, blk_meta, part_m, part_s,
                                  bias, Y, I, s.B, s.V, ck.tpc, FWD_TM / seg);
        else   hipLaunchKernelGGL((fwd_merge_kernel<false>), grid, dim3(FWD_MERGE_THREADS), 0, st, blk0, blk_meta, part_m, part_s,
                                  bias, Y, I, s.B, s.V, ck.tpc, FWD_TM / seg);
        prof.end(2);
    }
    return launch_status();
}

template <typename T, typename OT>
void launch_dh(int cpt, dim3 grid, hipStream_t st, const T* W, const int* bstart, const uint2* pm,
               OT* dH, int S, int D, int V, int accumulate) {
    switch (cpt) {
        case 1: hipLaunchKernelGGL((bwd_dh_kernel<T, 1, OT>), grid, dim3(ROW_THREADS), 0, st, W, bstart, pm, dH, S, D, V, accumulate); break;
        case 2: hipLaunchKernelGGL((bwd_dh_kernel<T, 2, OT>), grid, dim3(ROW_THREADS), 0, st, W, bstart, pm, dH, S, D, V, accumulate); break;
        case 4: hipLaunchKernelGGL((bwd_dh_kernel<T, 4, OT>), grid, dim3(ROW_THREADS), 0, st, W, bstart, pm, dH, S, D, V, accumulate); break;
        case 8: hipLaunchKernelGGL((bwd_dh_kernel<T, 8, OT>), grid, dim3(ROW_THREADS), 0, st, W, bstart, pm, dH, S, D, V, accumulate); break;
        default: hipLaunchKernelGGL((bwd_dh_kernel<T, 16, OT>), grid, dim3(ROW_THREADS), 0, st, W, bstart, pm, dH, S, D, V, accumulate); break;
    }
}

template <typename T, typename OT>
void launch_dw(int cpt, dim3 grid, size_t lds, hipStream_t st, const T* H, const float* dY, const float* Y, const int* I,
               OT* dW, float* db, int B, int S, int D, int V, int VT, int accumulate) {
    switch (cpt) {
        case 1: hipLaunchKernelGGL((bwd_dw_kernel<T, 1, OT>), grid, dim3(ROW_THREADS), lds, st, H, dY, Y, I, dW, db, B, S, D, V, VT, accumulate); break;
        case 2: hipLaunchKernelGGL((bwd_dw_kernel<T, 2, OT>), grid, dim3(ROW_THREADS), lds, st, H, dY, Y, I, dW, db, B, S, D, V, VT, accumulate); break;
        case 4: hipLaunchKernelGGL((bwd_dw_kernel<T, 4, OT>), grid, dim3(ROW_THREADS), lds, st, H, dY, Y, I, dW, db, B, S, D, V, VT, accumulate); break;
        case 8: hipLaunchKernelGGL((bwd_dw_kernel<T, 8, OT>), grid, dim3(ROW_THREADS), lds, st, H, dY, Y, I, dW, db, B, S, D, V, VT, accumulate); break;
        default: hipLaunchKernelGGL((bwd_dw_kernel<T, 16, OT>), grid, dim3(ROW_THREADS), lds, st, H, dY, Y, I, dW, db, B, S, D, V, VT, accumulate); break;
    }
}

// 32-bit byte offsets into W (one multiplication of 24-bit factors per entry) where W allows them.
bool off32_w(const Shape& s) {
    const size_t row = (size_t)s.D * (s.dtype == LSR_F32 ? 4 : 2);
    return (size_t)s.V * row <= 0xffffffffull && s.V <= (1 << 24) && row < (1u << 24);
}
// One launch of the sliced dH gather (vocabulary chunk vc) / of the sliced dW gather (sequences b0 .. b0+nb-1).
template <typename T, typename OT>
void launch_dh_sliced(int bpw, int wpb, dim3 grid, hipStream_t st, const T* W, const int* bounds, const uint2* perm, const float* prev,
                      OT* dst, int add_dst, int write_all, const Shape& s, int n_groups, int n_vc, int vc, bool xcd_own) {
    const bool off32 = off32_w(s);
#define LSR_DH2(BPW, WPB, O32) hipLaunchKernelGGL((bwd_dh_sliced_kernel<T, BPW, WPB, OT, O32>), grid, dim3(dh_threads(WPB)), 0, st, W, bounds, \
                                                  perm, prev, dst, add_dst, write_all, s.B, s.S, s.D, s.V, n_groups, n_vc, vc, xcd_own ? 1 : 0)
#define LSR_DH(BPW, WPB) do { if (off32) LSR_DH2(BPW, WPB, true); else LSR_DH2(BPW, WPB, false); } while (0)
    if (wpb == 4) LSR_DH(1, 4);
    else if (wpb == 2) LSR_DH(1, 2);
    else if (bpw == 1) LSR_DH(1, 1);
    else if (bpw == 2) LSR_DH(2, 1);
    else if (bpw == 4 || sizeof(T) == 4) LSR_DH(4, 1);   // a float row piece takes 16 lanes: at most four buckets per wave
    else if constexpr (sizeof(T) == 2) LSR_DH(8, 1);
#undef LSR_DH
#undef LSR_DH2
}
template <typename T, typename OT>
void launch_dh_dw(int bpw, int wpb, unsigned grid, size_t lds, hipStream_t st, const DhDwArgs& a) {
#define LSR_DH_DW(BPW, WPB) hipLaunchKernelGGL((bwd_dh_dw_kernel<T, BPW, WPB, OT>), dim3(grid), dim3(dh_threads(WPB)), lds, st, a)
    if (wpb == 4) LSR_DH_DW(1, 4);
    else if (bpw == 1) LSR_DH_DW(1, 1);
    else if (bpw == 2) LSR_DH_DW(2, 1);
    else if (bpw == 4 || sizeof(T) == 4) LSR_DH_DW(4, 1);
    else if constexpr (sizeof(T) == 2) LSR_DH_DW(8, 1);
#undef LSR_DH_DW
}
template <typename T, typename OT>
void launch_dw_sliced(dim3 grid, dim3 block, size_t lds, hipStream_t st, const T* H, const float* dY, const float* Y,
                      const int* I, const float* prev, OT* dst, int add_dst, float* db, int add_db, int b0, int nb, const Shape& s,
                      int VT, int NDC) {
    if (VT < 32)
        hipLaunchKernelGGL((bwd_dw_sliced_kernel<T, true, OT>), grid, block, lds, st, H, dY, Y, I, prev, dst, add_dst, db, add_db, b0, nb,
                           s.S, s.D, s.V, VT, NDC);
    else
        hipLaunchKernelGGL((bwd_dw_sliced_kernel<T, false, OT>), grid, block, lds, st, H, dY, Y, I, prev, dst, add_dst, db, add_db, b0, nb,
                           s.S, s.D, s.V, VT, NDC);
}

// The dW/db gather does not depend on the bucket sort that feeds dH, so the plain (not profiled)
// backward can run it on an auxiliary stream beside the dH chain: fork after the caller's prior
// work, join before returning control of the caller's stream.  The fork and the join cost the host about 30 us
// (two event records, two waits), and two gathers at a time help while they leave each other's windows in L2:
//   - up to AUX_MIN_GATHER_BYTES of worst-case gather traffic (2 * B * |V| rows of D elements) the host's time is
//     the longer one (forward and backward, us, without -> with: B=2 S=16 D=64 |V|=1000 float32 42.6 -> 52.1; backward alone B=4 S=64
//     D=512 |V|=20000, 0.16 GB, 55 -> 59, B=8 S=32 |V|=8000, 0.2 GB, 70 -> 71, B=2 S=128 |V|=30522, 0.19 GB, 64 -> 68), and up to 0.9 GB
//     dW shares a launch of the chain where it can (share_dw);
//   - up to AUX_MAX_GATHER_BYTES it pays nearly everywhere (backward, dense; one gradient in twenty: B=30 S=80 D=256 |V|=25000
//     101 -> 87; 62 -> 61, B=64 S=100 D=768 |V|=50000 646 -> 579; 195 -> 176, B=24 S=400 |V|=100000 674 -> 626; 411 -> 363,
//     B=16 S=256 |V|=250002 1026 -> 988; 581 -> 566; but B=256 S=512 D=384 |V|=30522 955 -> 985; 463 -> 371);
//   - beyond, where dW gathers from L2 and a 64-column slice of H is at most 1.375 MiB (at 0.75 MiB, B=256 S=24 |V|=60000, 3958 ->
//     3656; 510 -> 448, at 1, B=128 S=64 |V|=60000, 1374 -> 1316; 300 -> 270, at 1.25, B=256 S=40, 1843 -> 1670; 296 -> 264, at 1.5,
//     B=256 S=48, 1818 -> 1750; 305 -> 271, at 1.56, B=200 S=64 |V|=40000, 1479 -> 1511; 344 -> 317, at 2.5, B=200 S=100, 1845 -> 2049),
//     or from LDS and dH has one window
//     (B=256 S=512 6757 -> 6409 with the forward, B=128 S=512 D=1024 1075 -> 994; 737 -> 637, B=200 S=256 1124 -> 1008; 752 -> 618,
//     B=256 S=128 D=1024 1530 -> 1517; 780 -> 746).  With several windows a dW that gathers from LDS gains or loses beside dH
//     (B=60 S=128 D=1024 |V|=80000 1069 -> 1109; 575 -> 596, B=40 S=200 D=1024 |V|=130000 1356 -> 1361; 705 -> 712, B=16 S=512 D=1024
//     |V|=250002 1507 -> 1567; 834 -> 829, B=128 S=512 |V|=50000 1461 -> 1361; 1003 -> 933, B=64 S=512 D=1024 |V|=250002 13.29 ->
//     13.37 ms with the forward), so it runs behind (D=768 |V|=30522 where not said).
constexpr double AUX_MIN_GATHER_BYTES = 100e6;
constexpr double AUX_MAX_GATHER_BYTES = 16e9;
constexpr size_t AUX_SMALL_SLICE_BYTES = 11u << 17;      // 1.375 MiB
//
// The lane (one stream, one fork and one join event per device, default priority, non-blocking with
// respect to the null stream) is created by the first backward on that device and kept until the
// process ends.  It is shared by every caller on the device, so a call holds the lane's mutex from the
// record of the fork event to the wait on the join event: the three enqueue steps that name the
// shared events (record fork on the caller's stream, wait for it on the lane, ... record join on the
// lane, wait for it on the caller's stream) can then not interleave with another host thread's, and
// a wait always refers to the record made by the same call (a stream wait binds to the event's most
// recent record at the time of the wait call).  Only enqueueing is serialised; the device work of
// two callers still overlaps as their streams allow, except that their dW gathers share one lane.
struct AuxLane {
    std::mutex mu;
    hipStream_t stream = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
    bool ready = false;
};
AuxLane* aux_lane_of_current_device() {
    static AuxLane lanes[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) { (void)hipGetLastError(); return nullptr; }
    return &lanes[dev];
}
// Holds the lane from fork to join.  forked() is false when the lane could not be used; the caller
// then runs everything on its own stream.
class AuxFork {
public:
    AuxFork(AuxLane* lane, hipStream_t main) : main_(main) {
        if (!lane) return;
        lock_ = std::unique_lock<std::mutex>(lane->mu);
        if (!lane->ready) {
            if (hipStreamCreateWithFlags(&lane->stream, hipStreamNonBlocking) != hipSuccess ||
                hipEventCreateWithFlags(&lane->fork, hipEventDisableTiming) != hipSuccess ||
                hipEventCreateWithFlags(&lane->join, hipEventDisableTiming) != hipSuccess) {
                (void)hipGetLastError();
                lock_.unlock();
                return;
            }
            lane->ready = true;
        }
        if (hipEventRecord(lane->fork, main) != hipSuccess || hipStreamWaitEvent(lane->stream, lane->fork, 0) != hipSuccess) {
            (void)hipGetLastError();
            lock_.unlock();
            return;
        }
        lane_ = lane;
    }
    bool forked() const { return lane_ != nullptr; }
    hipStream_t side() const { return lane_ ? lane_->stream : main_; }
    // Joins the lane back into the caller's stream; called on every path once forked, errors included,
    // so that the caller's stream (possibly one that is being captured) is never left with an open fork.
    int join() {
        if (!lane_) return LSR_OK;
        const bool ok = hipEventRecord(lane_->join, lane_->stream) == hipSuccess &&
                        hipStreamWaitEvent(main_, lane_->join, 0) == hipSuccess;
        if (!ok) (void)hipGetLastError();
        lane_ = nullptr;
        lock_.unlock();
        return ok ? LSR_OK : LSR_ERR_LAUNCH;
    }
    ~AuxFork() { (void)join(); }
private:
    hipStream_t main_;
    AuxLane* lane_ = nullptr;
    std::unique_lock<std::mutex> lock_;
};

enum class DwShare { none, placement, dh };
// Everything the backward launches is decided here, from the shape alone, before anything is enqueued.
struct BwdLaunch {
    int cpt;                 // 16-byte chunks per thread of the whole-row kernels
    bool staged_place;       // the bucket sort places through LDS
    bool one_sort;           // ... and is one launch, because a sequence is one segment (but see backward_impl)
    bool dh_sliced;          // column-sliced dH gather, else whole rows
    int bpw, wpb, dh_groups; // buckets per wave, waves per bucket and workgroups per slice of the sliced dH gather
    int dw_vt;               // rows of the dW staging tile: sliced gather if dw_sliced, else whole-row kernel
    bool dw_sliced;
    int dw_bc, dw_ndc, dw_slice_groups, dw_vtiles;
    bool dh_xcd_own;         // sliced dH gather: column slices owned by XCDs
    int dw_tile_passes;      // LDS-tile dW kernel: copy passes per tile (ceil(S / 128)), or 0 when it does not apply
    int dw_tile_vtiles;
    DwShare share;           // whose launch the sliced dW gather may share
};
// The sliced dH gather with its column slices owned by XCDs (xcd_slice_unit).  In the slice-major order every
// XCD fetches the slice's window of W for itself and sees one eighth of its reuse, which is B / 8 gathers
// per row and vocabulary chunk; owned slices pay off while that is small.  Measured (dH, slice-major ->
// owned): B=8 S=512 |V|=30522 0.062 -> 0.047 ms; B=16 S=256 |V|=250002 0.88 -> 0.73; B=32 S=256 |V|=250002
// 1.06 -> 1.01; from B=32 at D=1024 on it loses (B=32 1.45 -> 1.67, B=64 S=512 2.65 -> 3.1: fewer L2 misses
// but a slower kernel; the slice-major order happens to keep every sequence's bucket lists on one XCD).
bool dh_slices_owned(const Shape& s) { return sliced_gathers(s) && s.B <= 16; }
// The LDS-tile dW kernel (bwd_dw_tile_kernel): bfloat16, D a multiple of 64, S within the tile, and at least
// one workgroup per CU of a 256-CU device.  Measured against the sliced gather (dW): B=64 S=512 D=1024
// |V|=250002 1.98 -> 1.72 ms; B=256 S=512 D=768 |V|=250002 7.84 -> 5.43; B=16 S=256 |V|=250002 0.407 ->
// 0.363; B=256 S=512 |V|=30522 1.02 -> 0.94; B=8 S=512 |V|=30522 0.0445 -> 0.0463; 60 workgroups (D=128,
// |V|=30522) 0.030 -> 0.052.
int dw_tile_passes(const Shape& s) {
    if (s.dtype != LSR_BF16 || s.D % DWS_COLS != 0 || s.S < DWT_MIN_S || s.S > DWT_MAX_S) return 0;
    if (s.V > (1 << 28)) return 0;                       // the kernel keeps byte offsets within a row of dY / Y / I in 32 bits
    const long long units = (long long)((s.V + DWT_ROWS - 1) / DWT_ROWS) * (s.D / DWS_COLS);
    if (units < 256 || units > 0x7fffffffll) return 0;
    return (s.S + 127) / 128;
}
double worst_gather_bytes(const Shape& s) { return 2.0 * s.B * s.V * s.D * (s.dtype == LSR_F32 ? 4 : 2); }
// Whose launch the sliced dW gather shares where all of dW/db is one launch, in tiles of 32 rows or more.
//   The dH gather's (bwd_dh_dw_kernel) where that gathers slices with 32-bit offsets in workgroups of four waves, a dW tile is at most an eighth of
//   a CU's LDS, and bfloat16 gradients need no staging: up to 0.9 GB of worst-case gathers, 0.6 GB with several vocabulary windows (dW then overlaps the
//   first window alone).  Backward; forward and backward; the same through autograd, us, auxiliary stream (below 0.1 GB: one after the other) -> here:
//     0.02 GB  B=1 S=21 D=312 |V|=18974 37 -> 29; 45 -> 36; 136 -> 133          0.07  B=6 S=11 D=312 |V|=9013 37 -> 26; 57 -> 45; 138 -> 135
//     0.15  B=7 S=52 D=312 |V|=17108 56 -> 35; 77 -> 59; 201 -> 148             0.43  B=25 S=63 D=512 |V|=8494 95 -> 85; 123 -> 113; 204 -> 140
//     0.47  B=10 S=32 D=312 |V|=18822 float32 76 -> 80; 132 -> 137; 194 -> 143  0.50  B=16 S=78 D=600 |V|=13048, one in twenty, 57 -> 43; 94 -> 84; 192 -> 145
//     0.71  B=10 S=21 D=256 |V|=34715 float32 103 -> 100; 166 -> 163; 203 -> 163  0.86  B=14 S=38 D=512 |V|=29935, one in twenty, 50 -> 43; 80 -> 73; 198 -> 138
//     not  1.02  B=17 S=41 D=200 |V|=37401 float32 129 -> 137, 1.27  B=32 S=32 D=200 |V|=24838 float32 131 -> 157, and with windows
//     0.64  B=2 S=15 D=512 |V|=77818 float32, one in twenty, 71 -> 84, 1.06  B=4 S=151 D=512 |V|=65002 float32, one in twenty, 73 -> 99
//     not where two waves share a bucket: the dW workgroups of such a launch have two waves too, which walk their tile in twice the rounds
//     (backward; forward and backward; autograd, us, auxiliary stream -> two-wave launch: 0.89  B=15 S=52 D=1536 |V|=4855 float32 221 -> 367; 466 -> 614; 466 -> 615,
//     0.85  B=18 S=76 D=832 |V|=14269 117 -> 187; 172 -> 243; 202 -> 243, 0.86  B=13 S=109 D=768 |V|=21410 95 -> 129; 147 -> 183; 205 -> 189, 0.83  B=15
//     S=150 D=512 |V|=26974, one in twenty, 57 -> 65; 106 -> 121; 195 -> 138), and sum db in another order than four
//     (the tile is what is counted: four waves that share a bucket keep 1 KiB of their own beside it, so at 39 and 40 sequences seven of eight
//     workgroups fit, which still is the better side of the auxiliary stream: 0.77  B=39 S=6 D=256 |V|=9611 float32 111 -> 98; 162 -> 148; 163 -> 148,
//     0.62  B=40 S=86 D=128 |V|=30092 63 -> 60; 116 -> 113; 196 -> 136; 0.52  B=40 S=56 D=256 |V|=6376 float32, one in twenty, 53 -> 36; 136 -> 127)
//   Neither, from 0.1 GB on, for up to three sequences with several windows and a dW of more than SHARE_MAX_DW elements: dW is then bound by its own output and outlasts
//   the window (or the placement) that it overlaps, and the others follow it (backward; forward and backward, us, auxiliary stream -> the launch of
//   dH: B=1 S=69 D=1024 |V|=46510 91 -> 107; 108 -> 99, B=1 S=130 D=768 |V|=86259 float32, one in twenty, 98 -> 117; 256 -> 274, B=1 S=71 D=1536 |V|=71646
//   217 -> 231; 272 -> 307; into the placement's B=1 S=11 D=832 |V|=28884 float32 82 -> 99; 109 -> 126).  Of 210 shapes with several windows none with
//   more sequences lost (0.55 to 0.97; 0.8 to 1.01), and with up to three 73 below the line 0.58 to 1.06; 0.79 to 1.02 and 98 above it
//   0.83 to 1.19; 0.85 to 1.13.
//   Else the placement's (bwd_place_dw_kernel): below 0.1 GB, and there always where a sequence is one segment, because the sort then is that launch
//   alone (placement against dH: B=5 S=163 D=64 |V|=1936 15 and 17, B=17 S=49 D=128 |V|=3023 float32 28 and 35); up to 0.3 GB otherwise
//     0.25  B=3 S=870 D=200 |V|=105469 72 -> 69; 191 -> 187; 220 -> 187         0.30  B=3 S=11 D=512 |V|=49397, one in twenty, 66 -> 54; 78 -> 75; 192 -> 145
//     not  0.62  B=91 S=155 D=128 |V|=13260 91 -> 115; 163 -> 184, 0.82  B=8 S=26 D=768 |V|=17108 float32 93 -> 108
constexpr double SHARE_MAX_DW = 17.5e6;      // 70 MB in float32
DwShare share_dw(const Shape& s, const BwdWs& w, bool bf16_out) {
    const int vt = dw_stage_rows(s);
    if (dw_tile_passes(s) > 0 || vt < 32 || dw_batch_chunk(s) < s.B) return DwShare::none;
    const double bytes = worst_gather_bytes(s);
    const bool staged_place = s.S <= PLACE_MAX_S && w.seg_len <= PLACE_MAX_SEG;
    if (bytes < AUX_MIN_GATHER_BYTES && staged_place && w.n_seg == 1) return DwShare::placement;
    if (bytes >= AUX_MIN_GATHER_BYTES && w.n_vc > 1 && s.B <= 3 && (double)s.V * s.D > SHARE_MAX_DW) return DwShare::none;
    // (a tile of 32 rows means sliced gathers.  Eight workgroups of four waves are the eight waves per SIMD of the dH gather.)
    if (dh_waves_per_bucket(s, w.n_vc) != 2 && off32_w(s) && (w.n_vc == 1 || !bf16_out) && (size_t)s.B * vt * 8 * 8 <= 160 * 1024 &&
        bytes < (w.n_vc == 1 ? 0.9e9 : 0.6e9))
        return DwShare::dh;
    return staged_place && bytes < 0.3e9 ? DwShare::placement : DwShare::none;
}
// Whether dW/db run on the auxiliary stream beside dH (see AUX_MAX_GATHER_BYTES).
bool dw_beside_dh(const Shape& s, const BwdWs& w, bool want_dw, bool bf16_out) {
    const double gather_bytes = worst_gather_bytes(s);
    const size_t h_slice = (size_t)s.B * s.S * DWS_COLS * (s.dtype == LSR_F32 ? 4 : 2);
    const bool tile = dw_tile_passes(s) > 0 && want_dw;      // dW gathers from LDS
    const bool apart = gather_bytes <= AUX_MAX_GATHER_BYTES || (tile ? w.n_vc == 1 : sliced_gathers(s) && h_slice <= AUX_SMALL_SLICE_BYTES);
    return gather_bytes >= AUX_MIN_GATHER_BYTES && apart && share_dw(s, w, bf16_out) == DwShare::none;
}
int plan_backward(const Shape& s, const BwdWs& w, bool bf16_out, BwdLaunch* L) {
    const int chunk_elems = s.dtype == LSR_F32 ? 4 : 8;
    const int n_chunks = s.D / chunk_elems;
    L->cpt = 1;
    while (L->cpt * ROW_THREADS < n_chunks) L->cpt *= 2;
    L->staged_place = s.S <= PLACE_MAX_S && w.seg_len <= PLACE_MAX_SEG;      // plan[3] of lsr_head_plan
    L->one_sort = L->staged_place && w.n_seg == 1;
    L->dh_sliced = sliced_gathers(s);
    L->bpw = dh_buckets_per_wave(s, w.n_vc);
    L->wpb = dh_waves_per_bucket(s, w.n_vc);
    L->dh_groups = !L->dh_sliced ? 0 : (L->wpb > 1 ? s.B * s.S : s.B * ((s.S + 4 * L->bpw - 1) / (4 * L->bpw)));
    if ((long long)L->dh_groups * n_slices(s.D) > 0x7fffffffll) return LSR_ERR_SHAPE;
    L->dh_xcd_own = dh_slices_owned(s);
    if (L->dh_xcd_own && xcd_slice_grid(n_slices(s.D), L->dh_groups, 1) > 0x7fffffffll) return LSR_ERR_SHAPE;
    L->dw_tile_passes = dw_tile_passes(s);
    L->dw_tile_vtiles = (s.V + DWT_ROWS - 1) / DWT_ROWS;
    // column-sliced dW gathers (L2-resident slices of H) need a (g, I) staging tile (at most 48 KiB) at least
    // 16 vocabulary rows wide, i.e. at most 384 sequences per launch.  Larger batches take the whole-row
    // kernel, which also skips zero gradients.
    L->dw_bc = dw_batch_chunk(s);
    L->dw_vt = dw_stage_rows(s);
    L->dw_sliced = L->dw_vt > 0;
    if (L->dw_sliced) {
        // slices per group: a workgroup walks the slices of its group with one staging of (g, I), and
        // the groups run one after the other.  Up to 9 MiB of H rows per group measured best (C5: two
        // 4 MiB slices, dW 2.21 -> 2.02 ms; C3 0.22 -> 0.175; 3 per group at C5 2.11, all 16: 2.48):
        // fewer stagings against a wider window of H in flight.
        const int n_dc = n_slices(s.D);
        const size_t slice_bytes = (size_t)L->dw_bc * s.S * DWS_COLS * (s.dtype == LSR_F32 ? 4 : 2);
        int ndc = (int)((size_t)(9u << 20) / slice_bytes);
        L->dw_ndc = ndc < 1 ? 1 : (ndc > n_dc ? n_dc : ndc);
        L->dw_slice_groups = (n_dc + L->dw_ndc - 1) / L->dw_ndc;
        L->dw_vtiles = (s.V + L->dw_vt - 1) / L->dw_vt;
        if ((long long)L->dw_vtiles * L->dw_slice_groups > 0x7fffffffll) return LSR_ERR_SHAPE;
    } else {
        // whole-row gathers; rows of the (g, I) staging tile: as wide as 48 KiB of LDS allows, at most 32
        int VT = 32;
        while (VT > 1 && (size_t)s.B * VT * 8 > 48 * 1024) VT /= 2;
        L->dw_vt = VT;
        L->dw_ndc = L->dw_slice_groups = 0;
        L->dw_vtiles = (s.V + VT - 1) / VT;
    }
    L->share = share_dw(s, w, bf16_out);
    if (L->share == DwShare::dh) {
        // one grid dimension for all workgroups, of 256 threads each
        const long long n_dh = L->dh_xcd_own ? xcd_slice_grid(n_slices(s.D), L->dh_groups, 1) : (long long)L->dh_groups * n_slices(s.D);
        if (n_dh + (long long)L->dw_vtiles * L->dw_slice_groups + 8 > 0xffffffffll / 256) L->share = DwShare::none;
    }
    return LSR_OK;
}

// The whole backward for element types T (H, W) and OT (dH, dW), after every check.
template <typename T, typename OT>
int backward_launches(const Shape& s, const BwdWs& w, const BwdLaunch& L, const T* H, const T* W, const float* dY, const float* Y,
                      const int32_t* I, OT* dH, OT* dW, float* db, int accumulate, char* base, hipStream_t st, hipStream_t st_dw,
                      Prof& prof);

int backward_impl(const lsr_head_desc* desc, const void* H, const void* W, const float* dY, const float* Y,
                  const int32_t* I, void* dH, void* dW, float* db, const lsr_backward_opts* opts, void* ws, size_t ws_bytes,
                  hipStream_t st, Prof& prof) {
    Shape s;
    int rc = check_desc(desc, &s);
    if (rc != LSR_OK) return rc;
    const int grad_dtype = opts ? opts->grad_dtype : LSR_F32;
    const int accumulate = (opts && opts->accumulate) ? 1 : 0;
    if (grad_dtype != LSR_F32 && grad_dtype != LSR_BF16) return LSR_ERR_DTYPE;
    if (grad_dtype == LSR_BF16 && s.dtype != LSR_BF16) return LSR_ERR_DTYPE;      // bfloat16 gradients belong to bfloat16 parameters
    const bool bf16_out = grad_dtype == LSR_BF16;
    if (!H || !W || !dY || !Y || !I) return LSR_ERR_NULL;
    if (misaligned(H) || misaligned(W) || misaligned(dY) || misaligned(Y) || misaligned(I) || misaligned(ws) ||
        (dH && misaligned(dH)) || (dW && misaligned(dW)) || (db && misaligned(db)))
        return LSR_ERR_ALIGN;
    if (s.S > 8192 || s.B > 6144) return LSR_ERR_SHAPE;      // LDS tables of the bucket sort / dW staging
    const BwdWs w = bwd_ws(s, bf16_out);
    if (!ws || ws_bytes < w.total) return LSR_ERR_WORKSPACE;
    BwdLaunch L;
    if ((rc = plan_backward(s, w, bf16_out, &L)) != LSR_OK) return rc;
    int n_cus = 0;
    rc = check_device(&n_cus);
    if (rc != LSR_OK) return rc;
    // ---- nothing has been enqueued up to here; every check is behind us ----

    prof.stream = st;
    char* base = static_cast<char*>(ws);

    // fork: dW/db on the auxiliary stream, the dH chain on the caller's
    const bool overlap = !prof.on && dH && (dW || db) && dw_beside_dh(s, w, dW != nullptr, bf16_out);
    // A sort of one launch ends before a dW of more than 384 sequences (whole rows, or several launches) has begun, and the two then gather from
    // the first workgroup on side by side; behind a count and a scan dH comes when dW has the chip.  Backward, us, one launch -> three (the same segments):
    // B=2887 S=29 D=384 |V|=1430 2422 -> 1308, B=781 S=7 D=1024 |V|=3128 853 -> 660, B=2995 S=6 D=256 |V|=1324 float32, one in twenty, 250 -> 161; not
    // B=2292 S=50 D=256 |V|=3692 2351 -> 2898, B=1782 S=38 D=768 |V|=740 828 -> 973; 70 shapes 0.97 in the mean, and with up to 384
    // sequences 1.03 (one in twenty B=255 S=44 D=256 |V|=815 float32 44 -> 53).
    if (overlap && s.B > 384) L.one_sort = false;
    AuxFork lane(overlap ? aux_lane_of_current_device() : nullptr, st);
    const hipStream_t st_dw = lane.side();

    // A failed launch ends the sequence; the join below still runs.
    if (s.dtype == LSR_F32)
        rc = backward_launches<float, float>(s, w, L, static_cast<const float*>(H), static_cast<const float*>(W), dY, Y, I,
                                             static_cast<float*>(dH), static_cast<float*>(dW), db, accumulate, base, st, st_dw, prof);
    else if (!bf16_out)
        rc = backward_launches<uint16_t, float>(s, w, L, static_cast<const uint16_t*>(H), static_cast<const uint16_t*>(W), dY, Y, I,
                                                static_cast<float*>(dH), static_cast<float*>(dW), db, accumulate, base, st, st_dw, prof);
    else
        rc = backward_launches<uint16_t, uint16_t>(s, w, L, static_cast<const uint16_t*>(H), static_cast<const uint16_t*>(W), dY, Y, I,
                                                   static_cast<uint16_t*>(dH), static_cast<uint16_t*>(dW), db, accumulate, base, st,
                                                   st_dw, prof);
    const int rj = lane.join();
    return rc != LSR_OK ? rc : rj;
}

template <typename T, typename OT>
int backward_launches(const Shape& s, const BwdWs& w, const BwdLaunch& L, const T* H, const T* W, const float* dY, const float* Y,
                      const int32_t* I, OT* dH, OT* dW, float* db, int accumulate, char* base, hipStream_t st, hipStream_t st_dw,
                      Prof& prof) {
    constexpr bool OUT_F32 = sizeof(OT) == 4;
    uint2* perm = reinterpret_cast<uint2*>(base + w.perm_off);
    int* cnt = reinterpret_cast<int*>(base + w.cnt_off);
    int* bstart = reinterpret_cast<int*>(base + w.bs_off);
    // Positions in use per sequence, for the LDS-tile dW kernel where it runs behind dH on the same stream: left by the launch
    // that cuts the lists into windows, in place of the counts, which nothing reads after the placement.
    int* tops = dH && dW && w.n_vc > 1 && L.dw_tile_passes > 0 && st_dw == st ? cnt : nullptr;
    // launches that dW shares (what is profiled runs apart)
    const bool shared = dH && (dW || db) && !prof.on;
    const bool place_dw = shared && L.share == DwShare::placement, dh_dw = shared && L.share == DwShare::dh;
    int r;
    if (dH) {
        const dim3 seg_grid(w.n_seg, s.B);
        if (!L.one_sort) {
            prof.begin(0);
            // few segments (long sequences, small problems): more threads per workgroup instead
            const int count_threads = (long long)s.B * w.n_seg < 512 ? SORT_MAX_THREADS : 256;
            hipLaunchKernelGGL(bwd_count_kernel, seg_grid, dim3(count_threads), sizeof(int) * s.S, st, dY, Y, I, cnt, s.S, s.V, w.n_seg, w.seg_len);
            prof.end(0);
            if ((r = launch_status()) != LSR_OK) return r;
            prof.begin(1);
            if (s.S > 256) hipLaunchKernelGGL(bwd_scan_kernel<1024>, dim3(s.B), dim3(1024), 0, st, cnt, bstart, s.S, w.n_seg);
            else hipLaunchKernelGGL(bwd_scan_kernel<256>, dim3(s.B), dim3(256), 0, st, cnt, bstart, s.S, w.n_seg);
            prof.end(1);
            if ((r = launch_status()) != LSR_OK) return r;
        }
        prof.begin(2);
        const dim3 place_block(64 * PLACE_WAVES);
        auto place_lds = [&](int waves) { return sizeof(int) * (waves / 2) * s.S + sizeof(uint2) * w.seg_len; };
        if (place_dw) {
            const size_t lds = place_lds(PLACE_WAVES), lds_dw = (size_t)s.B * L.dw_vt * 8;
#define LSR_PLACE_DW2(STEPS, ONE) hipLaunchKernelGGL((bwd_place_dw_kernel<T, OT, STEPS, ONE>), dim3(s.B * w.n_seg + L.dw_vtiles * L.dw_slice_groups), \
                                                     place_block, lds > lds_dw ? lds : lds_dw, st, H, dY, Y, I, cnt, bstart, perm, dW, db, \
                                                     accumulate, s.B, s.S, s.D, s.V, w.n_seg, w.seg_len, w.key_bits, L.dw_vt, L.dw_ndc, L.dw_vtiles)
#define LSR_PLACE_DW(STEPS) do { if (L.one_sort) LSR_PLACE_DW2(STEPS, true); else LSR_PLACE_DW2(STEPS, false); } while (0)
            if (w.seg_len <= 4 * 64 * PLACE_WAVES) LSR_PLACE_DW(4);
            else if (w.seg_len <= 8 * 64 * PLACE_WAVES) LSR_PLACE_DW(8);
            else LSR_PLACE_DW(16);
#undef LSR_PLACE_DW
#undef LSR_PLACE_DW2
        } else if (L.staged_place) {
#define LSR_PLACE2(STEPS, NW, ONE) hipLaunchKernelGGL((bwd_place_staged_kernel<STEPS, NW, ONE>), seg_grid, dim3(64 * NW), place_lds(NW), st, dY, Y, I, cnt, \
                                                      bstart, perm, s.S, s.V, w.n_seg, w.seg_len, w.key_bits)
#define LSR_PLACE(STEPS) do { if (L.one_sort) LSR_PLACE2(STEPS / 2, PLACE_ONE_WAVES, true); \
                              else if (w.n_seg == 1) LSR_PLACE2(STEPS / 2, PLACE_ONE_WAVES, false); \
                              else LSR_PLACE2(STEPS, PLACE_WAVES, false); } while (0)
            static_assert(PLACE_ONE_WAVES == 2 * PLACE_WAVES, "half the steps");
            if (w.seg_len <= 4 * 64 * PLACE_WAVES) LSR_PLACE(4);
            else if (w.seg_len <= 8 * 64 * PLACE_WAVES) LSR_PLACE(8);
            else LSR_PLACE(16);
#undef LSR_PLACE
#undef LSR_PLACE2
        } else {
            hipLaunchKernelGGL(bwd_place_kernel, seg_grid, place_block, sizeof(int) * PLACE_WAVES * s.S, st, dY, Y, I, cnt, bstart, perm,
                               s.S, s.V, w.n_seg, w.seg_len, w.key_bits);
        }
        prof.end(2);
        if ((r = launch_status()) != LSR_OK) return r;
        prof.begin(3);
        if (!L.dh_sliced) {
            launch_dh<T, OT>(L.cpt, dim3(s.B, s.S), st, W, bstart, perm, dH, s.S, s.D, s.V, accumulate);
        } else {
            // column-sliced gathers, one launch per vocabulary chunk: the rows of W in use stay in L2
            const int* bounds = bstart;
            if (w.n_vc > 1) {
                int* cb = reinterpret_cast<int*>(base + w.cb_off);
                const long long n = (long long)s.B * s.S * (w.n_vc + 1);
                hipLaunchKernelGGL(bwd_chunk_bounds_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, bstart, perm, cb, tops,
                                   s.B * s.S, s.S, s.V, w.n_vc, w.vc_len);
                bounds = cb;
            }
            const dim3 grid = L.dh_xcd_own ? dim3((unsigned)xcd_slice_grid(n_slices(s.D), L.dh_groups, 1))
                                           : dim3((unsigned)s.B, (unsigned)(L.dh_groups / s.B), (unsigned)n_slices(s.D));
            float* stage = reinterpret_cast<float*>(base + w.dh_stage_off);
            for (int vc = 0; vc < w.n_vc; ++vc) {
                if (vc == 0 && dh_dw) {
                    DhDwArgs a;
                    a.H = H; a.W = W; a.dY = dY; a.Y = Y; a.I = I; a.bounds = bounds; a.perm = perm; a.dH = dH; a.dW = dW; a.db = db;
                    a.accumulate = accumulate;
                    a.B = s.B; a.S = s.S; a.D = s.D; a.V = s.V;
                    a.n_groups = L.dh_groups; a.n_vc = w.n_vc; a.xcd_own = L.dh_xcd_own ? 1 : 0;
                    a.VT = L.dw_vt; a.NDC = L.dw_ndc; a.n_vtiles = L.dw_vtiles;
                    a.n_dw = L.dw_vtiles * L.dw_slice_groups; a.n_dw_pad = (a.n_dw + 7) / 8 * 8;
                    const long long n_dh = L.dh_xcd_own ? xcd_slice_grid(n_slices(s.D), L.dh_groups, 1) : (long long)L.dh_groups * n_slices(s.D);
                    launch_dh_dw<T, OT>(L.bpw, L.wpb, (unsigned)(a.n_dw_pad + n_dh), (size_t)s.B * L.dw_vt * 8, st, a);
                    continue;
                }
                const bool last = vc + 1 == w.n_vc;
                if (OUT_F32) {
                    // partial sums live in dH itself; the first chunk of a fresh result writes every bucket
                    float* d = reinterpret_cast<float*>(dH);
                    const bool fresh = vc == 0 && !accumulate;
                    launch_dh_sliced<T, float>(L.bpw, L.wpb, grid, st, W, bounds, perm, fresh ? nullptr : d, d, 0, fresh ? 1 : 0, s, L.dh_groups,
                                               w.n_vc, vc, L.dh_xcd_own);
                } else if (w.n_vc == 1) {
                    launch_dh_sliced<T, OT>(L.bpw, L.wpb, grid, st, W, bounds, perm, nullptr, dH, accumulate, accumulate ? 0 : 1, s, L.dh_groups,
                                            w.n_vc, vc, L.dh_xcd_own);
                } else if (!last) {
                    launch_dh_sliced<T, float>(L.bpw, L.wpb, grid, st, W, bounds, perm, vc > 0 ? stage : nullptr, stage, 0, vc == 0 ? 1 : 0, s,
                                               L.dh_groups, w.n_vc, vc, L.dh_xcd_own);
                } else {
                    launch_dh_sliced<T, OT>(L.bpw, L.wpb, grid, st, W, bounds, perm, stage, dH, accumulate, 1, s, L.dh_groups, w.n_vc, vc, L.dh_xcd_own);
                }
            }
        }
        prof.end(3);
        if ((r = launch_status()) != LSR_OK) return r;
    }
    if ((dW || db) && !place_dw && !dh_dw) {
        prof.begin(4);
        const int VT = L.dw_vt;
        if (L.dw_tile_passes > 0 && dW) {
            // one launch for all sequences; the sums start from zero, so bfloat16 results need no staging
            if constexpr (sizeof(T) == 2) {
                const dim3 grid((unsigned)L.dw_tile_vtiles * (unsigned)(s.D / DWS_COLS));
#define LSR_DWT2(NP, ALONE) hipLaunchKernelGGL((bwd_dw_tile_kernel<OT, NP, ALONE>), grid, dim3(DWT_ROWS), 0, st_dw, H, dY, Y, I, dW, accumulate, db, \
                                       accumulate, tops, s.B, s.S, s.D, s.V, L.dw_tile_vtiles)
                const bool alone = w.n_vc == 1 && grid.x % 256 != 0;
#define LSR_DWT(NP) do { if (alone) LSR_DWT2(NP, true); else LSR_DWT2(NP, false); } while (0)
                switch (L.dw_tile_passes) {
                    case 1: LSR_DWT(1); break;
                    case 2: LSR_DWT(2); break;
                    case 3: LSR_DWT(3); break;
                    default: LSR_DWT(4); break;
                }
#undef LSR_DWT
#undef LSR_DWT2
            }
        } else if (L.dw_sliced) {
            // four waves also where the tile has fewer row groups than that (16 rows of bf16: two): the
            // others still share the staging and the compaction (C3: dW 0.264 -> 0.222 ms)
            const int waves = 4;
            const int bc = L.dw_bc;                            // sequences per launch
            const size_t lds = (size_t)bc * VT * 8;
            const dim3 grid((unsigned)L.dw_vtiles, (unsigned)L.dw_slice_groups), block(64 * waves);
            float* stage = reinterpret_cast<float*>(base + w.dw_stage_off);
            for (int b0 = 0; b0 < s.B; b0 += bc) {
                const int nb = s.B - b0 < bc ? s.B - b0 : bc;
                const bool first = b0 == 0, last = b0 + bc >= s.B;
                const int add_db = (!first || accumulate) ? 1 : 0;
                if (OUT_F32) {
                    float* d = reinterpret_cast<float*>(dW);
                    launch_dw_sliced<T, float>(grid, block, lds, st_dw, H, dY, Y, I, (!first || accumulate) ? d : nullptr, d, 0, db,
                                               add_db, b0, nb, s, VT, L.dw_ndc);
                } else if (first && last) {
                    launch_dw_sliced<T, OT>(grid, block, lds, st_dw, H, dY, Y, I, nullptr, dW, accumulate, db, add_db, b0, nb, s, VT,
                                            L.dw_ndc);
                } else if (!last) {
                    launch_dw_sliced<T, float>(grid, block, lds, st_dw, H, dY, Y, I, first ? nullptr : stage, dW ? stage : nullptr, 0,
                                               db, add_db, b0, nb, s, VT, L.dw_ndc);
                } else {
                    launch_dw_sliced<T, OT>(grid, block, lds, st_dw, H, dY, Y, I, stage, dW, accumulate, db, add_db, b0, nb, s, VT,
                                            L.dw_ndc);
                }
            }
        } else {
            const size_t lds = (size_t)s.B * VT * 8;
            launch_dw<T, OT>(L.cpt, dim3(L.dw_vtiles), lds, st_dw, H, dY, Y, I, dW, db, s.B, s.S, s.D, s.V, VT, accumulate);
        }
        prof.end(4);
        if ((r = launch_status()) != LSR_OK) return r;
    }
    return LSR_OK;
}

// Runs `launch` `launches` times on st and returns the duration of the last one in ms (< 0 on error).
template <typename F>
float time_last_launch(int launches, hipStream_t st, F&& launch) {
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) { (void)hipGetLastError(); return -1.f; }
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipGetLastError(); (void)hipEventDestroy(e0); return -1.f; }
    bool ok = true;
    for (int l = 0; l < launches && ok; ++l) {
        const bool timed = l + 1 == launches;
        if (timed) ok = hipEventRecord(e0, st) == hipSuccess;
        launch();
        ok = ok && hipGetLastError() == hipSuccess;
        if (timed) ok = ok && hipEventRecord(e1, st) == hipSuccess;
    }
    float ms = -1.f;
    ok = ok && hipEventSynchronize(e1) == hipSuccess && hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (!ok) { (void)hipGetLastError(); return -1.f; }
    return ms;
}

}  // namespace

extern "C" {

size_t lsr_head_workspace_bytes(const lsr_head_desc* desc, int for_backward) {
    Shape s;
    if (check_desc(desc, &s) != LSR_OK) return 0;
    return for_backward ? bwd_ws(s).total : fwd_ws(s).total;
}

int lsr_head_forward(const lsr_head_desc* desc, const void* H, const void* W, const float* bias, const uint8_t* mask,
                     float* Y, int32_t* I, void* workspace, size_t workspace_bytes, lsr_stream_t stream) {
    Prof prof;
    return forward_impl(desc, H, W, bias, mask, Y, I, workspace, workspace_bytes, stream, prof);
}

int lsr_head_forward_static(const lsr_head_desc* desc, const void* H, const void* W, const float* bias,
                            const uint8_t* mask, float* Y, int32_t* I, lsr_stream_t stream) {
    Shape s;
    const int rc = check_desc(desc, &s);
    if (rc != LSR_OK) return rc;
    if (fwd_ws(s).total > (size_t)LSR_STATIC_SCRATCH_BYTES) return LSR_ERR_STATIC_SCRATCH;
    int n_cus = 0;
    const int rd = check_device(&n_cus);      // a usable gfx950 device is current before its symbol is looked up
    if (rd != LSR_OK) return rd;
    void* ws = nullptr;
    const int rs = static_scratch(&ws);
    if (rs != LSR_OK) return rs;
    // Every word of the scratch that a kernel reads has been written earlier in the same call (lengths,
    // position lists, block tables), so nothing has to be cleared between calls.
    Prof prof;
    return forward_impl(desc, H, W, bias, mask, Y, I, ws, (size_t)LSR_STATIC_SCRATCH_BYTES, stream, prof);
}

int lsr_head_backward(const lsr_head_desc* desc, const void* H, const void* W, const float* dY, const float* Y,
                      const int32_t* I, float* dH, float* dW, float* db, void* workspace, size_t workspace_bytes,
                      lsr_stream_t stream) {
    Prof prof;
    return backward_impl(desc, H, W, dY, Y, I, dH, dW, db, nullptr, workspace, workspace_bytes, stream, prof);
}

size_t lsr_head_backward_ex_workspace_bytes(const lsr_head_desc* desc, const lsr_backward_opts* opts) {
    Shape s;
    if (check_desc(desc, &s) != LSR_OK) return 0;
    const int grad_dtype = opts ? opts->grad_dtype : LSR_F32;
    if (grad_dtype != LSR_F32 && !(grad_dtype == LSR_BF16 && s.dtype == LSR_BF16)) return 0;
    return bwd_ws(s, grad_dtype == LSR_BF16).total;
}

int lsr_head_backward_ex(const lsr_head_desc* desc, const void* H, const void* W, const float* dY, const float* Y,
                         const int32_t* I, void* dH, void* dW, float* db, const lsr_backward_opts* opts, void* workspace,
                         size_t workspace_bytes, lsr_stream_t stream) {
    Prof prof;
    return backward_impl(desc, H, W, dY, Y, I, dH, dW, db, opts, workspace, workspace_bytes, stream, prof);
}

int lsr_head_forward_profiled(const lsr_head_desc* desc, const void* H, const void* W, const float* bias,
                              const uint8_t* mask, float* Y, int32_t* I, void* workspace, size_t workspace_bytes,
                              lsr_stream_t stream, float* kernel_ms) {
    if (!kernel_ms) return LSR_ERR_NULL;
    Prof prof;
    prof.on = true;
    const int rc = forward_impl(desc, H, W, bias, mask, Y, I, workspace, workspace_bytes, stream, prof);
    const int rc2 = prof.finish(kernel_ms);
    return rc != LSR_OK ? rc : rc2;
}

int lsr_head_backward_profiled(const lsr_head_desc* desc, const void* H, const void* W, const float* dY,
                               const float* Y, const int32_t* I, float* dH, float* dW, float* db, void* workspace,
                               size_t workspace_bytes, lsr_stream_t stream, float* kernel_ms) {
    if (!kernel_ms) return LSR_ERR_NULL;
    Prof prof;
    prof.on = true;
    const int rc = backward_impl(desc, H, W, dY, Y, I, dH, dW, db, nullptr, workspace, workspace_bytes, stream, prof);
    const int rc2 = prof.finish(kernel_ms);
    return rc != LSR_OK ? rc : rc2;
}

int lsr_mfma_peak_probe(int64_t iters, int launches, void* sink, double* tflops, lsr_stream_t stream) {
    if (!sink || !tflops) return LSR_ERR_NULL;
    if (iters < 1 || iters > (1 << 24) || launches < 1 || launches > 64) return LSR_ERR_SHAPE;
    int n_cus = 0;
    int rc = check_device(&n_cus);
    if (rc != LSR_OK) return rc;
    hipStream_t st = stream;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) { (void)hipGetLastError(); return LSR_ERR_LAUNCH; }
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipGetLastError(); (void)hipEventDestroy(e0); return LSR_ERR_LAUNCH; }
    // two workgroups of four waves per CU: two waves on every SIMD, each with four independent MFMA chains
    const dim3 grid(2 * n_cus);
    float ms = 0.f;
    bool ok = true;
    for (int l = 0; l < launches && ok; ++l) {        // the last launch is the one that is timed
        const bool timed = l + 1 == launches;
        if (timed) ok = hipEventRecord(e0, st) == hipSuccess;
        hipLaunchKernelGGL(mfma_probe_kernel, grid, dim3(PROBE_THREADS), 0, st, (int)iters, static_cast<float*>(sink));
        ok = ok && hipGetLastError() == hipSuccess;
        if (timed) ok = ok && hipEventRecord(e1, st) == hipSuccess;
    }
    ok = ok && hipEventSynchronize(e1) == hipSuccess && hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (!ok || ms <= 0.f) { (void)hipGetLastError(); return LSR_ERR_LAUNCH; }
    const double flops = 2.0 * 32 * 32 * 16 * PROBE_MFMA_PER_ITER * (double)iters * (PROBE_THREADS / 64) * grid.x;
    *tflops = flops / (ms * 1e-3) / 1e12;
    return LSR_OK;
}

int lsr_copy_probe(void* dst, const void* src, size_t bytes, int launches, double* gbytes_per_s, lsr_stream_t stream) {
    if (!dst || !src || !gbytes_per_s) return LSR_ERR_NULL;
    if (misaligned(dst) || misaligned(src)) return LSR_ERR_ALIGN;
    if (bytes < 16 || bytes % 16 != 0 || launches < 1 || launches > 64) return LSR_ERR_SHAPE;
    int n_cus = 0;
    const int rc = check_device(&n_cus);
    if (rc != LSR_OK) return rc;
    const size_t n16 = bytes / 16;
    size_t blocks = (n16 + COPY_THREADS - 1) / COPY_THREADS;
    const size_t cap = (size_t)n_cus * 32;            // grid-stride loop over a grid that fills the chip a few times
    if (blocks > cap) blocks = cap;
    const float ms = time_last_launch(launches, stream, [&] {
        hipLaunchKernelGGL(copy_probe_kernel, dim3((unsigned)blocks), dim3(COPY_THREADS), 0, stream, static_cast<uint4*>(dst),
                           static_cast<const uint4*>(src), n16);
    });
    if (ms <= 0.f) return LSR_ERR_LAUNCH;
    *gbytes_per_s = 2.0 * (double)bytes / (ms * 1e-3) / 1e9;      // bytes read + bytes written
    return LSR_OK;
}

int lsr_gather_probe(const void* table, size_t window_bytes, int steps, int launches, void* out, size_t out_bytes,
                     double* gbytes_per_s, lsr_stream_t stream) {
    if (!table || !out || !gbytes_per_s) return LSR_ERR_NULL;
    if (misaligned(table) || misaligned(out)) return LSR_ERR_ALIGN;
    if (window_bytes < 128 || window_bytes % 128 != 0 || window_bytes > ((size_t)1 << 38) || steps < 1 || steps > (1 << 20) ||
        launches < 1 || launches > 64)
        return LSR_ERR_SHAPE;
    int n_cus = 0;
    const int rc = check_device(&n_cus);
    if (rc != LSR_OK) return rc;
    const unsigned blocks = (unsigned)n_cus * 16;                // eight waves resident per SIMD's worth of work in flight
    const size_t groups = (size_t)blocks * GATHER_THREADS / 8;
    if (out_bytes < groups * 8 * 8 * sizeof(float)) return LSR_ERR_WORKSPACE;
    const uint32_t rows = (uint32_t)(window_bytes / 128);
    const float ms = time_last_launch(launches, stream, [&] {
        hipLaunchKernelGGL(gather_probe_kernel, dim3(blocks), dim3(GATHER_THREADS), 0, stream, static_cast<const uint16_t*>(table),
                           rows, steps, static_cast<float*>(out));
    });
    if (ms <= 0.f) return LSR_ERR_LAUNCH;
    *gbytes_per_s = (double)groups * steps * GATHER_NLD * 128.0 / (ms * 1e-3) / 1e9;
    return LSR_OK;
}

int lsr_head_plan_ex(const lsr_head_desc* desc, int32_t* plan, int slots) {
    Shape s;
    const int rc = check_desc(desc, &s);
    if (rc != LSR_OK) return rc;
    if (!plan) return LSR_ERR_NULL;
    if (slots < 1) return LSR_ERR_SHAPE;
    const FwdChunks f = fwd_chunks(s);
    const BwdWs w = bwd_ws(s);
    const int32_t all[LSR_PLAN_EX_SLOTS] = {
        f.tpc, w.n_seg, w.seg_len, (s.S <= PLACE_MAX_S && w.seg_len <= PLACE_MAX_SEG) ? 1 : 0,
        w.n_vc, w.vc_len, dh_buckets_per_wave(s, w.n_vc), dw_stage_rows(s),
        dw_batch_chunk(s), f.n_chunks, fwd_seg(s), f.resident ? 1 : 0,
        dh_slices_owned(s) ? 1 : 0, dw_tile_passes(s), dh_waves_per_bucket(s, w.n_vc), f.window,
        dw_beside_dh(s, w, true, false) ? 1 : 0, fwd_few(s) ? 1 : 0};
    for (int i = 0; i < slots && i < LSR_PLAN_EX_SLOTS; ++i) plan[i] = all[i];
    return LSR_OK;
}

int lsr_head_dw_route(const lsr_head_desc* desc, const lsr_backward_opts* opts, int32_t* route) {
    Shape s;
    int rc = check_desc(desc, &s);
    if (rc != LSR_OK) return rc;
    const int grad_dtype = opts ? opts->grad_dtype : LSR_F32;
    if (grad_dtype != LSR_F32 && (grad_dtype != LSR_BF16 || s.dtype != LSR_BF16)) return LSR_ERR_DTYPE;
    if (!route) return LSR_ERR_NULL;
    if (s.S > 8192 || s.B > 6144) return LSR_ERR_SHAPE;
    const bool bf16_out = grad_dtype == LSR_BF16;
    const BwdWs w = bwd_ws(s, bf16_out);
    BwdLaunch L;
    if ((rc = plan_backward(s, w, bf16_out, &L)) != LSR_OK) return rc;
    *route = L.share == DwShare::dh ? LSR_DW_IN_DH_LAUNCH
             : L.share == DwShare::placement ? LSR_DW_IN_PLACEMENT_LAUNCH
             : dw_beside_dh(s, w, true, bf16_out) ? LSR_DW_ON_AUX_STREAM : LSR_DW_BEHIND_DH;
    return LSR_OK;
}

int lsr_head_plan(const lsr_head_desc* desc, int32_t* plan) { return lsr_head_plan_ex(desc, plan, LSR_PLAN_SLOTS); }

const char* lsr_status_string(int status) {
    switch (status) {
        case LSR_OK: return "ok";
        case LSR_ERR_NULL: return "a required pointer is NULL";
        case LSR_ERR_SHAPE: return "shape outside the supported range";
        case LSR_ERR_DTYPE: return "unknown hw_dtype";
        case LSR_ERR_ALIGN: return "pointer not 16-byte aligned";
        case LSR_ERR_WORKSPACE: return "workspace missing or too small";
        case LSR_ERR_ARCH: return "no gfx950 device";
        case LSR_ERR_LAUNCH: return "HIP launch or event error";
        case LSR_ERR_STATIC_SCRATCH: return "shape needs more scratch than the static array of lsr_head_forward_static holds";
        default: return "unknown status";
    }
}

}  // extern "C"
