// Launch-shape heuristics of the forward path.
#include "../../include/lbscan.h"
#include "lbscan_internal.h"

#include <limits.h>

namespace lbscan {
namespace {

struct Shape { int nseg, seg_tiles; };

// Up to this many segments the full forward pass folds the carry chain itself.
// (Measured, up to 16 / up to 4, us, fp32: 4 x 384 x 576 17.7 / 19.0, 16 x 384 x 576 34.6 / 37.7,
// 8 x 384 x 1500 48.2 / 48.7.)
constexpr int kFoldChainSegments = 16;

// Cuts the rows into want_seg segments of whole forward tiles, at least 64 tokens each
// (force_nseg: as many as asked for).
Shape cut_rows(const FwdParams& p, long want_seg)
{
    const int ntiles = (p.seqlen + kFwdTileTokens - 1) / kFwdTileTokens;
    Shape s{1, ntiles};
    if (p.force_nseg >= 1) want_seg = p.force_nseg;
    if (want_seg > 1) {
        int st = (int)((ntiles + want_seg - 1) / want_seg);
        if (p.force_nseg < 1 && st < 2) st = 2;
        if (st < 1) st = 1;
        s.seg_tiles = st;
        s.nseg = (ntiles + st - 1) / st;
    }
    return s;
}

size_t carry_floats(const FwdParams& p, int nseg)
{
    return (size_t)nseg * p.batch * p.dim * (size_t)p.dstate;
}

// Scratch of rows cut into nseg segments: the states and the sums of time steps.
size_t summary_bytes(const FwdParams& p, int nseg)
{
    return nseg <= 1 ? 0 : (carry_floats(p, nseg) + (size_t)nseg * p.batch * p.dim) * sizeof(float);
}

// Rows that the kernels gather token by token (a scan order without copies).  The summary launch
// gathers x, delta and Bm a second time, which costs the more the less of the rows the caches
// hold.  Measured on MI355X (us, uncut / cut; rows x tokens, MB of x):
//   blocks  fp32                                     bf16
//   96      2305, 28 MB  650 / 509                   4097, 25 MB  1139 / 789
//   120     1601, 25 MB  508 / 430                   4097, 31 MB  1365 / 1140
//   120     2305, 35 MB  754 / 767                   5185, 40 MB  1661 / 1956
//   144     1025, 19 MB  377 / 337                   2305, 21 MB  700 / 658
//   144     4097, 76 MB  1534 / 1954                 4097, 38 MB  1537 / 1875
//   192     1025, 25 MB  472 / 516                   1601, 20 MB  556 / 526
//   192     4097, 101 MB 1903 / 2567                 2305, 28 MB  882 / 1007
//   240     577, 18 MB   201 / 206                   1601, 25 MB  651 / 762
//   336     401, 17 MB   150 / 157                   1025, 22 MB  513 / 572
//   288     145          26 / 28                     145          23 / 25
//   288     257          61 / 53                     401          72 / 62
// (square grids; few rows or few columns keep more of the lines: 360 blocks of 4 x 256 tokens in bf16
// 238 / 191 with kernels whose loads waited for one another.  On the wrong side: bf16 at 384 blocks of 401
// tokens, 90 / 87.)
bool gather_cut_pays(const FwdParams& p, long nrb)
{
    if (p.seqlen <= 160) return nrb < 208;
    const double bytes = (double)p.batch * p.dim * p.seqlen * (p.dtype == 0 ? 4 : 2);
    const int side = p.order.H < p.order.W ? p.order.H : p.order.W;
    return nrb < 120 || (nrb < 384 && (side < 16 || nrb * bytes < 4.4e9));
}

// The forward kernels run one block per (32 rows, segment), five to seven of them on a CU.  Rows that
// cannot fill the chip are cut into segments scanned in parallel: a summary launch, the
// carry chain, then the full pass started from the carried-in states.  That costs a second
// read of x, delta, Bm and ~60% more arithmetic, so only when rows are scarce.  Number of blocks
// aimed at (us, 1 x 256 x 65536): 1024: 146, 1536: 142, 2048: 139, 2560: 150; 1 x 512 x 16384:
// 768: 80, 1024: 77, 1536: 82, 2048: 79.  Up to 256 row blocks a CU has one block of uncut rows at most, and
// all rows that one block cannot take whole (in_block_shape) are cut; beyond, the longer the rows
// the more a cut can pay for its launches.  cut_pays says which calls take scratch for a cut: its lines
// are those of the kernels before the ways of loading had kernels of their own, and callers
// size their scratch by them.  whole_is_faster leaves rows whole within them where that is
// faster now.  Measured on MI355X (us, uncut / cut; fp32 with window 4, bf16 with window 8):
//   tokens  blocks  fp32          bf16             tokens  blocks  fp32          bf16
//   197     300     21.6 / 25.5   22.3 / 25.8      700     300     65.2 / 63.1   66.5 / 61.0
//   197     348     21.9 / 29.4   22.6 / 29.2      700     324     65.8 / 68.4   66.5 / 64.5
//   256     324     25.3 / 27.4   26.0 / 28.4      700     348     66.2 / 75.2   66.6 / 68.2
//   300     192     24.8 / 23.6   24.9 / 22.6      1100    300     101 / 98.4    102 / 92.7
//   300     216     25.0 / 26.6   25.1 / 25.8      1100    324     102 / 106     103 / 94.7
//   300     252     25.3 / 27.5   25.2 / 26.9      1100    372     103 / 116     105 / 107
//   300     348     31.0 / 36.2   32.1 / 34.9      1600    324     140 / 138     149 / 131
//   400     252     31.6 / 33.8   32.0 / 33.1      1600    348     139 / 144     150 / 143
//   400     276     38.7 / 37.8   40.0 / 37.1      1600    372     140 / 153     151 / 153
//   400     300     38.7 / 40.3   40.1 / 40.0      3001    300     273 / 264     278 / 244
//   400     324     39.0 / 42.9   40.8 / 42.5      3001    348     279 / 297     281 / 271
//   512     300     46.7 / 44.0   48.7 / 44.0      3001    372     270 / 310     281 / 283
// With eight states 300 tokens cross at 300 blocks (24.2 / 24.6, 24.6 / 23.6) and not below 257 (240:
// 21.6 / 21.1), and long bf16 rows beyond cut_pays' lines (64 x 168 x 3555, 384 blocks, 250 / 230); reversed
// rows and windows 1 and 16 cross at the same lines within 3%.
bool cut_pays(const FwdParams& p, long nrb)
{
    const int L = p.seqlen;
    if (p.order.kind != 0) return gather_cut_pays(p, nrb);
    if (L <= 192) return nrb < 257;
    if (L <= 256) return nrb < 348;
    if (p.dtype == 0 || L <= 320) return nrb < (L <= 1024 ? 360 : 384);
    return nrb < (L <= 1024 ? 390 : 410);
}

bool whole_is_faster(const FwdParams& p)
{
    const long nrb = (long)((p.dim + 31) / 32) * p.batch;
    const int L = p.seqlen;
    if (p.order.kind != 0) return false;
    if (L <= 256) return nrb > 256;
    if (L <= 320) return p.dstate > 8 ? nrb > 207 : nrb > 311;
    if (p.dtype == 0) return nrb > (L <= 448 ? 287 : 317);
    if (p.dstate <= 8 && L > 448) return false;
    return nrb > (L <= 448 ? 311 : L <= 1024 ? 341 : 365);
}

// Segments aimed at where rows are cut.  With at most eight states a lane has half the work for the
// same launches, and long rows of few channels notice how the blocks fill the chip: whole rounds of
// 1536 blocks, and no chain of more segments than one block of the chain kernel takes (256).
// Measured on MI355X (us, fp32, N = 8, window 2; 2048 blocks / this):
//   4 blocks x 30000    40.4 / 35.7      12 blocks x 30000   81.3 / 78.6
//   6 blocks x 20000    38.2 / 33.6      12 blocks x 65536   150 / 148
//   8 blocks x 30000    59.3 / 56.4      16 blocks x 41432   146 / 140
//   8 blocks x 65536    101 / 104        24 blocks x 30000   145 / 143
// (Shorter rows, 16 x 14000 51.4 / 53.1 us at 1536 blocks, and 16 states gain at some lengths and lose at others.)
long segments_wanted(const FwdParams& p, long nrb)
{
    if (p.dstate > 8 || nrb > 32 || p.seqlen < 20000) return (2048 + nrb - 1) / nrb;
    const long want = (nrb <= 8 ? 1536 : 3072) / nrb;
    return want < 256 ? want : 256;
}

// The summaries alone take 5.4 MB at most.  Beside a first pass's result they may not fit what
// lbscan_fwd_static holds: the rows are then cut into as many segments as do, but into no fewer
// than 768 blocks of 64 rows need (uncut from 256 such row blocks on).
Shape pick_shape(const FwdParams& p)
{
    const long nrb = (long)((p.dim + 31) / 32) * p.batch;
    const Shape s = cut_rows(p, cut_pays(p, nrb) ? segments_wanted(p, nrb) : 1);
    if (p.beside + summary_bytes(p, s.nseg) <= LBSCAN_STATIC_SCRATCH_BYTES || p.beside > LBSCAN_STATIC_SCRATCH_BYTES) return s;
    const long nrb64 = (long)((p.dim + 63) / 64) * p.batch;
    const long coarse = nrb64 < 256 ? (768 + nrb64 - 1) / nrb64 : 1;
    const long fitting = (long)((LBSCAN_STATIC_SCRATCH_BYTES - p.beside) / (summary_bytes(p, 2) / 2));
    const Shape t = cut_rows(p, fitting > coarse ? fitting : coarse);
    return p.beside + summary_bytes(p, t.nseg) <= LBSCAN_STATIC_SCRATCH_BYTES ? t : s;
}

// Few short rows: the segments of a row as waves of one block of 8 rows, one launch instead of two;
// nseg 0 where it is not taken.  Every block stages all of Bm and Cm for its 8 rows, so it
// wins only while the chip is not full.  Measured on MI355X (us, fp32 with window 4 / bf16 with window 8, separate launches
// or uncut rows -> one launch):
//   64 rows, 256 tokens    16.2 / 16.3 -> 11.2 / 11.2    1920 rows, 401 tokens   17.7 / 18.1 -> 13.3 / 14.0
//   3072 rows, 197 tokens  15.7 / 16.3 -> 11.1 / 11.2    2304 rows, 401 tokens   17.6 / 17.6 -> 19.7 / 20.0
//   6144 rows, 197 tokens  20.0 / 20.1 -> 15.1 / 15.8    3072 rows, 401 tokens   20.7 / 20.7 -> 20.1 / 20.4
//   8064 rows, 197 tokens  21.4 / 22.1 -> 18.7 / 19.8    6144 rows, 401 tokens   28.8 / 29.4 -> 30.1 / 30.5
//   8448 rows, 197 tokens  21.6 / 22.3 -> 21.8 / 23.6    384 rows, 576 tokens    16.3 / 16.0 -> 17.2 / 17.9
//   12288 rows, 197 tokens 22.0 / 22.9 -> 28.0 / 30.8    1536 rows, 576 tokens   17.7 / 17.4 -> 17.8 / 18.3
//   9216 rows, 100 tokens  12.5 / 12.5 -> 15.9 / 16.0    64 rows, 50 tokens      11.1 / 11.4 -> 11.1 / 11.2
// (On the wrong side: 2304 and 3072 rows of 290 tokens, 15.9 / 15.8 -> 13.9 / 14.1 and 16.8 / 17.1 -> 14.5 / 14.2.)
// Gathered rows pay more for the eightfold Bm and Cm (fp32 / bf16, 145 tokens: 6144 rows 21.3 / 19.4 -> 15.4 / 15.3,
// 7680 rows 22.9 / 19.0 -> 24.5 / 23.1; 197 tokens, 7680 rows: 30.6 / 26.0 -> 24.1 / 23.2, and 9216 rows, beyond the
// line, 38.4 / 30.6 -> 28.8 / 28.0).
Shape in_block_shape(const FwdParams& p)
{
    const int ntiles = (p.seqlen + kFwdTileTokens - 1) / kFwdTileTokens;
    const long blocks = (long)((p.dim + 7) / 8) * p.batch;
    if (p.force_nseg >= 1 || ntiles < 3) return {0, 0};
    const long most = p.order.kind != 0 && ntiles <= 5 ? 832 : 1024;
    if (blocks > (ntiles <= kInBlockSegments ? most : ntiles <= 2 * kInBlockSegments ? 256 : 0)) return {0, 0};
    const int st = (ntiles + kInBlockSegments - 1) / kInBlockSegments;
    return {(ntiles + st - 1) / st, st};
}

// The backward kernel runs one block per (64 rows, segment), two on a CU.  Where rows are
// cut: three rounds of 512 blocks, so that a block's end leaves little idle, but not more than 64
// segments unless one round needs them (long chains, more summaries to read).  Backward call on
// MI355X, us, at 512 / 1536 blocks:
//   8 x 768 x 4096 bf16    575 / 539      4 x 768 x 2048 bf16    167 / 157
//   16 x 768 x 2048 bf16   671 / 551      2 x 768 x 4096 bf16    167 / 159
//   16 x 768 x 1024 fp32   332 / 298      8 x 768 x 1100 fp32    183 / 192
//   4 x 768 x 4096 bf16    297 / 287      6 x 768 x 2048 fp32    229 / 231
//   1 x 256 x 65536 fp32   373 / 401      1 x 512 x 16384 fp32   192 / 207
// (On the wrong side: rows that three rounds cut into segments of two or three tiles, as 8 x 768 x
// 1100 above; 32 x 384 x 197 95.8 us in four segments, 85.2 in two; 4 x 768 x 1100 107.5 and 102.2.  The next
// lengths go the other way, 8 x 768 x 1300 215 / 213.)
Shape pick_bwd_shape(const FwdParams& p)
{
    const long nrb = (long)((p.dim + 63) / 64) * p.batch;
    if (nrb >= 256) return cut_rows(p, 1);
    const long fill = 512 / nrb, rounds = 1536 / nrb < 64 ? 1536 / nrb : 64;
    return cut_rows(p, fill > rounds ? fill : rounds);
}

// The chunk-per-lane kernel (one wave per row, 1024-token chunks, one launch; 768 blocks of four rows
// in flight, so 3072 rows are a full round) against the wave-tile kernels (rows cut where that is
// faster), measured on MI355X (us, wave tiles / chunk; fp32 with window 4, bf16 with window 8;
// 16 states).  Whole chunks:
//   rows x tokens      fp32           bf16           rows x tokens      fp32           bf16
//   192 x 1024         17.9 / 14.3    18.2 / 14.2    1536 x 4096        57.1 / 65.3    59.3 / 62.1
//   3072 x 1024        36.4 / 25.1    36.5 / 22.9    3072 x 4096        103 / 86.1     102 / 79.4
//   12288 x 1024       91.0 / 85.6    95.3 / 73.2    6144 x 4096        192 / 164      188 / 152
//   24576 x 1024       128 / 160      128 / 141      12288 x 4096       351 / 331      343 / 286
//   1536 x 2048        35.6 / 34.2    35.7 / 32.5    16128 x 2048       179 / 210      192 / 188
// A chunk that the row does not fill takes its loads element by element, in every state,
//   192 x 900          17.3 / 21.4    17.4 / 23.3    6144 x 1700        93.9 / 106     86.4 / 100
//   1920 x 1020        30.3 / 29.8    30.5 / 33.5    6144 x 5000        254 / 234      235 / 227
//   2688 x 900         32.0 / 34.4    31.7 / 36.9    9216 x 2000        144 / 168      141 / 175
//   3072 x 960         34.6 / 35.5    35.1 / 37.9    12288 x 1700       154 / 206      160 / 219
//   3456 x 960         36.7 / 56.3    38.7 / 61.4    12288 x 4000       341 / 372      342 / 368
//   6144 x 1000        57.9 / 69.9    56.0 / 72.1    16128 x 2000       183 / 300      191 / 316
//   3072 x 2000        58.0 / 55.2    57.2 / 55.4    1536 x 3000        49.0 / 58.7    47.9 / 61.7
// and less so with fewer states, while a wave tile has lanes for 8 or 16 of them (rows x tokens x N):
//   192 x 1000 x 12    17.6 / 18.3    17.5 / 19.5    14592 x 1700 x 8   118 / 172      122 / 172
//   6144 x 1000 x 12   56.7 / 60.0    55.0 / 60.4    14592 x 1000 x 8   71.8 / 129     72.6 / 129
//   192 x 1000 x 5     16.4 / 12.4    15.5 / 12.7    768 x 1000 x 8     15.2 / 16.9    15.5 / 16.8
// It needs chunks that are mostly full, and rows enough for a wave each unless a row is one whole
// chunk.  Ragged chunks of 15 and 16 states pay where the rows about fill one round of blocks, or two
// with three chunks and more; of fewer states from two thirds of a round on (with two and three chunks not a little
// over one), up to two rounds with two chunks or four with more; rows of one ragged chunk where they fill a round or
// are few.  Where the wave tile's lanes are half idle (5, 6, 9, 10 states, and up to 4) fewer rows are
// enough.  Whole chunks pay up to 13312 rows in fp32 (four rows share a staged Bm / Cm chunk, so those reads
// are twice the row reads) and 20480 in bf16, and further with fewer states.  On 420 calls drawn over
// 600 to 49000 rows, 820 to 12000 tokens, 5 to 16 states, both types and directions and windows 1 to
// 16 the rule takes 1.6% more time than the faster side of each (the lines before the present kernels 3.8%; single
// sizes of theirs up to 77%, 14592 x 1000 x 8).
// (On the wrong side: rows of 2 to 8 states and two chunks or more below the lines, where the chunk
// kernel would be up to a third faster; whole chunks of 13000 fp32 rows of 8 states, of a little over a
// round.)
// It leaves no checkpoints for a backward call.
bool use_chunk_mapping(const FwdParams& p, const float* saved)
{
    if (p.force_mapping == 1) return false;
    FwdParams q = p;
    q.ckpt = nullptr; q.summary_only = 0;
    if (!fwd_chunk_supported(q)) return false;
    if (saved) return false;
    if (p.force_mapping == 2) return true;
    if (p.force_nseg >= 1) return false;                              // (it takes its rows whole)
    const long rows = (long)p.batch * p.dim;
    const long chunk = 1024, nchunks = (p.seqlen + chunk - 1) / chunk;
    const long taken = (p.dim + 31) / 32 * 32L * p.batch;             // rows that wave tiles work on
    const int N = p.dstate;
    if (p.seqlen * 5 < nchunks * chunk * 4) return false;             // chunks less than 80% full
    if (p.seqlen % chunk == 0) {
        if (p.dtype == 0)
            return rows <= (N > 8 ? 13312 : N > 4 ? 14336 : 16384) && (nchunks == 1 || rows >= (nchunks == 2 ? 1536 : 3072));
        if (N > 8 && rows > 20480) return false;
        return nchunks == 1 || (N <= 8 || nchunks < 4 ? rows >= 1536 : taken >= (nchunks < 8 ? 1920 : 2048));
    }
    if (N <= 4) {
        if (nchunks == 1) return rows <= 8192 || (p.dtype != 0 && N <= 2);
        return p.dtype != 0 ? rows >= 1536 : rows <= 16384 && rows >= (nchunks == 2 ? 1536 : 3072);
    }
    const bool one_round = taken > 2720 && rows <= 3072;
    const bool light = N <= 6 || (N > 8 && N <= 10);                  // few of the lanes that a wave tile has for states
    if (nchunks == 1) {
        if (light) return rows <= 6144;
        return N <= 8 ? rows <= 768 || one_round : one_round && (N <= 14 || p.seqlen >= 1000);
    }
    if (N > 14) {
        if (nchunks < 5) return one_round || (nchunks >= 3 && rows > 5632 && rows <= 6144);
        return one_round || (rows > 4900 && rows <= 9216);
    }
    if (rows > (nchunks == 2 || (N > 12 && p.dtype == 0) ? 6144 : N > 6 && nchunks < 4 ? 12288 : 14336)) return false;
    if (p.dtype == 0 && nchunks > 2 && rows < 2817) return false;
    return light && (p.dtype != 0 || nchunks == 2) ? rows >= 1536 : taken >= 1920 && (N <= 6 || nchunks > 3 || rows <= 3072 || rows > 4096);
}

hipError_t launch_fwd_wave(const FwdParams& p, hipStream_t stream)
{
    // (the second pass of the any-window path starts segments anywhere and tells them apart itself)
    switch (p.generic_window ? Rows::aligned : rows_of(p.order, p.dtype, p.pitch, p.seqlen, p.reverse)) {
        case Rows::gathered: return p.dtype == 0 ? launch_fwd_gather_f32(p, stream) : launch_fwd_gather_bf16(p, stream);
        case Rows::odd: return launch_fwd_odd_bf16(p, stream);
        case Rows::aligned: break;
    }
    return p.dtype == 0 ? launch_fwd_wave_f32(p, stream) : launch_fwd_wave_bf16(p, stream);
}

hipError_t launch_bwd_wave(const BwdParams& p, hipStream_t stream)
{
    switch (rows_of(p.order, p.dtype, p.pitch, p.seqlen, p.reverse)) {
        case Rows::gathered: return p.dtype == 0 ? launch_bwd_gather_f32(p, stream) : launch_bwd_gather_bf16(p, stream);
        case Rows::odd: return launch_bwd_odd_bf16(p, stream);
        case Rows::aligned: break;
    }
    return p.dtype == 0 ? launch_bwd_wave_f32(p, stream) : launch_bwd_wave_bf16(p, stream);
}

}  // namespace

size_t fwd_workspace_bytes(const FwdParams& p)
{
    if (p.batch == 0 || p.dim == 0 || p.seqlen == 0) return 0;
    return in_block_shape(p).nseg ? 0 : summary_bytes(p, pick_shape(p).nseg);
}

size_t saved_state_bytes(const FwdParams& p)
{
    if (p.batch == 0 || p.dim == 0 || p.seqlen == 0) return 0;
    if (pick_bwd_shape(p).nseg > 1) return 0;
    const size_t ntiles16 = (p.seqlen + kTileTokens - 1) / kTileTokens;
    return ntiles16 * p.batch * p.dim * (size_t)p.dstate * sizeof(float);
}

hipError_t launch_fwd(FwdParams p, void* workspace, float* saved, hipStream_t stream)
{
    if (p.batch == 0 || p.dim == 0 || p.seqlen == 0) return hipSuccess;
    // (a pass that leaves checkpoints takes its rows whole: its callers have rows enough)
    const bool whole = saved || (p.force_nseg < 1 && whole_is_faster(p));
    const Shape s = whole ? Shape{1, (p.seqlen + kFwdTileTokens - 1) / kFwdTileTokens} : pick_shape(p);
    if (use_chunk_mapping(p, saved)) return launch_fwd_chunk(p, stream);
    p.ckpt = saved;
    p.cum = nullptr;
    auto launch = [&](const FwdParams& q) { return launch_fwd_wave(q, stream); };
    p.nseg = s.nseg;
    p.seg_tiles = s.seg_tiles;
    p.in_block = 0;
    p.summary_only = 0;
    // (uncut rows read the entering state from h0)
    p.carry = nullptr;
    p.dsum = nullptr;
    p.fold_chain = 0;
    const Shape rows = saved ? Shape{0, 0} : in_block_shape(p);
    if (rows.nseg) {
        p.nseg = rows.nseg;
        p.seg_tiles = rows.seg_tiles;
        p.in_block = 1;
        return launch(p);
    }
    if (s.nseg > 1) {
        if (!workspace) return hipErrorInvalidValue;
        p.carry = static_cast<float*>(workspace);
        p.dsum = p.carry + carry_floats(p, s.nseg);
        FwdParams q = p;
        q.summary_only = 1;
        hipError_t e = launch(q);
        if (e != hipSuccess) return e;
        // few segments: the full pass folds the chain itself (one launch less);
        // many: the chain kernel, which shares them out to the waves of a block
        p.fold_chain = s.nseg <= kFoldChainSegments;
        if (!p.fold_chain) {
            e = launch_carry_chain(p, stream);
            if (e != hipSuccess) return e;
        }
    }
    return launch(p);
}

// ---- window lengths without a compiled kernel ---------------------------------
//
// Eq. 8 splits into the plain forward scan (sum_n Cm f + Dskip x: the kernel
// compiled for window 1, entering and leaving states included) and the local
// backward part sum_n Cm g, which never crosses a window end.  Pass 1 leaves the
// first in fp32 (in y itself when y is fp32, else at the start of the
// workspace); pass 2 adds the second for any window length, gates and writes y.

static size_t generic_partial_bytes(const FwdParams& p)
{
    return p.dtype == 0 ? 0 : (size_t)p.batch * p.dim * p.seqlen * sizeof(float);
}

size_t fwd_generic_workspace_bytes(const FwdParams& p)
{
    if (p.batch == 0 || p.dim == 0 || p.seqlen == 0) return 0;
    FwdParams p1 = p;
    p1.window = 1;
    p1.beside = generic_partial_bytes(p);
    return p1.beside + fwd_workspace_bytes(p1);
}

hipError_t launch_fwd_generic(FwdParams p, void* workspace, hipStream_t stream)
{
    if (p.batch == 0 || p.dim == 0 || p.seqlen == 0) return hipSuccess;
    float* partial = static_cast<float*>(p.y);
    char* scratch = static_cast<char*>(workspace);
    if (p.dtype != 0) {
        if (!workspace) return hipErrorInvalidValue;
        partial = static_cast<float*>(workspace);
        scratch += generic_partial_bytes(p);
    }
    FwdParams p1 = p;
    p1.beside = generic_partial_bytes(p);
    p1.window = 1; p1.z = nullptr; p1.y = partial; p1.y_is_f32 = 1;
    hipError_t e = launch_fwd(p1, scratch, nullptr, stream);
    if (e != hipSuccess) return e;

    FwdParams p2 = p;
    p2.generic_window = 1; p2.Dskip = nullptr; p2.yprev = partial;
    p2.h0 = nullptr; p2.hT = nullptr; p2.carry = nullptr; p2.dsum = nullptr;
    p2.ckpt = nullptr; p2.cum = nullptr; p2.summary_only = 0; p2.seg_tiles = 0;
    // segments of whole windows, at least 64 steps each, enough of them to fill the chip
    const long nrb = (long)((p.dim + 31) / 32) * p.batch;
    const long M = p.window, L = p.seqlen;
    const long nw = (L + M - 1) / M;
    long want_seg = nrb < 1536 ? (1536 + nrb - 1) / nrb : 1;
    if (p.force_nseg >= 1) want_seg = p.force_nseg;
    long wps = (nw + want_seg - 1) / want_seg;
    if (p.force_nseg < 1 && wps * M < 64) wps = (64 + M - 1) / M;
    if (wps < 1) wps = 1;
    p2.seg_tokens = (int)(wps * M);
    p2.nseg = (int)((L + p2.seg_tokens - 1) / p2.seg_tokens);
    return launch_fwd_wave(p2, stream);
}

// ---- backward ----------------------------------------------------------------

namespace {

// A window that straddles the start of a 16-token tile needs the part of the adjoint
// of the local backward state that enters the tile from the left (BwdParams::gck).
bool needs_gamma_checkpoints(const FwdParams& f)
{
    return f.seqlen > kTileTokens && kTileTokens % f.window != 0;
}

struct BwdLayout {
    Shape shape;            // segments in forward tiles (32 tokens)
    size_t ntiles16;        // backward tiles (16 tokens) per row
    size_t ckpt, cum, gck, carry, dsum, psi, part;   // float offsets into the workspace
    size_t total;           // floats
};

BwdLayout bwd_layout(const FwdParams& f)
{
    BwdLayout l;
    l.shape = pick_bwd_shape(f);
    const bool gamma = needs_gamma_checkpoints(f);
    if (gamma && l.shape.nseg > 1) {
        // segments must start at window starts: whole windows per segment
        long g = f.window, r = kFwdTileTokens;
        while (r) { const long t = g % r; g = r; r = t; }          // gcd(window, 32)
        const long unit = f.window / g;                            // forward tiles per window period
        const long ntiles = (f.seqlen + kFwdTileTokens - 1) / kFwdTileTokens;
        long st = ((l.shape.seg_tiles + unit - 1) / unit) * unit;
        if (st >= ntiles) st = ntiles;
        l.shape.seg_tiles = (int)st;
        l.shape.nseg = (int)((ntiles + st - 1) / st);
    }
    const size_t rows = (size_t)f.batch * f.dim, N = f.dstate;
    l.ntiles16 = (f.seqlen + kTileTokens - 1) / kTileTokens;
    size_t o = 0;
    l.ckpt = o; o += l.ntiles16 * rows * N;
    l.cum = o;  o += l.ntiles16 * rows;
    l.gck = o;  if (gamma) o += l.ntiles16 * rows * N;
    const size_t ns = l.shape.nseg > 1 ? l.shape.nseg : 0;
    l.carry = o; o += ns * rows * N;
    l.dsum = o;  o += ns * rows;
    l.psi = o;   o += ns * rows * N;
    l.part = o;                                // per block of 64 channels: fp32 dBm, dCm
    o += 2 * (size_t)((f.dim + 63) / 64) * f.batch * N * f.seqlen;
    l.total = o;
    return l;
}

}  // namespace

size_t bwd_workspace_bytes(const FwdParams& f)
{
    if (f.batch == 0 || f.dim == 0 || f.seqlen == 0) return 0;
    return bwd_layout(f).total * sizeof(float);
}

hipError_t launch_bwd(const FwdParams& f, BwdParams p, void* dBm, void* dCm, void* workspace,
                      const float* saved, const float* dhT, hipStream_t stream)
{
    if (f.batch == 0 || f.dim == 0 || f.seqlen == 0) return hipSuccess;
    if (!workspace) return hipErrorInvalidValue;
    const BwdLayout l = bwd_layout(f);
    const Shape& s = l.shape;
    const bool gamma = needs_gamma_checkpoints(f);
    float* ws = static_cast<float*>(workspace);
    const long bnl = (long)f.batch * f.dstate * f.seqlen;
    p.dBpart = ws + l.part;
    p.ckpt = ws + l.ckpt;
    p.cum = ws + l.cum;
    p.gck = gamma ? ws + l.gck : nullptr;
    p.nseg = s.nseg;
    p.seg_tiles = s.seg_tiles * (kFwdTileTokens / kTileTokens);
    // uncut rows: the entering state and the gradient arriving at the leaving state
    // take the places of the chained values
    p.carry = s.nseg > 1 ? ws + l.carry : f.h0;
    p.psi_in = s.nseg > 1 ? ws + l.psi : dhT;

    hipError_t e;
    const ZeroMany z{{p.dA, p.dDskip, p.dbias, nullptr, nullptr},
                     {(long)f.dim * f.dstate, f.dim, f.dim, 0, 0}};
    if ((e = launch_zero_many(z, stream)) != hipSuccess) return e;

    // after the backward kernel: dBm, dCm from the per-block partial sums
    auto finish = [&]() -> hipError_t {
        const int nbx = (f.dim + 63) / 64;
        return f.dtype == 0 ? launch_reduce_f32(p.dBpart, dBm, dCm, bnl, nbx, stream)
                            : launch_reduce_bf16(p.dBpart, dBm, dCm, bnl, nbx, stream);
    };

    if (saved && s.nseg == 1 && !gamma) {
        // the forward call left the checkpoints (entering state included): no summary pass
        p.ckpt = saved;
        p.cum = nullptr;
        p.carry = nullptr;
        e = launch_bwd_wave(p, stream);
        return e != hipSuccess ? e : finish();
    }

    // summary pass (the forward kernel in summary mode): checkpoints of f for every
    // 16-token tile and, when the rows are cut, the per-segment summaries of the
    // forward and of the right-to-left recurrence; for windows that straddle tile
    // starts also the checkpoints of the adjoint of the local backward state
    FwdParams q = f;
    q.nseg = s.nseg;
    q.seg_tiles = s.seg_tiles;
    q.summary_only = 1;
    q.ckpt = ws + l.ckpt;
    q.cum = ws + l.cum;
    q.gck = gamma ? ws + l.gck : nullptr;
    q.carry = q.nseg > 1 ? ws + l.carry : nullptr;
    q.dsum = q.nseg > 1 ? ws + l.dsum : nullptr;
    q.psi = q.nseg > 1 ? ws + l.psi : nullptr;
    q.dout = p.dout;
    e = launch_fwd_wave(q, stream);
    if (e != hipSuccess) return e;
    if (q.nseg > 1) {
        if ((e = launch_carry_chains(q, q.psi, dhT, stream)) != hipSuccess) return e;
    }

    e = launch_bwd_wave(p, stream);
    return e != hipSuccess ? e : finish();
}

// ---- a scan order through reordered copies --------------------------------------
//
// The wave-tile kernels can gather the tokens of a scan order themselves, which
// needs no scratch; given scratch, the row tensors are copied into scanned order
// first, the stored-order path runs on the copies, and its results are copied back.
// The forward pass leaves z where it is: the scan returns the ungated sum in fp32 and
// the copy back applies the gate.
//
// What a gather costs depends on how far apart the tokens of a tile lie and on how much
// of the rows the caches hold between tiles: rows of few bytes, grids of few rows or few
// columns and small calls gather well.  Measured on MI355X (us, gather / copies):
//   rows x tokens (grid)            forward fp32   forward bf16   backward fp32  backward bf16
//   128 x 384, 50 (7 x 7)           21 / 39        21 / 39        92 / 110       88 / 105
//   1042 x 384, 50 (7 x 7)          138 / 219      133 / 198      616 / 686      554 / 610
//   88 x 384, 65 (8 x 8)            25 / 42        25 / 42        108 / 120      110 / 119
//   127 x 384, 82 (9 x 9)           38 / 55        31 / 53        162 / 152      133 / 141
//   103 x 384, 101 (10 x 10)        44 / 54        34 / 52        207 / 164      158 / 157
//   72 x 384, 145 (12 x 12)         62 / 54        38 / 52        237 / 154      161 / 141
//   90 x 384, 145 (12 x 12)         78 / 64        45 / 58        341 / 208      235 / 198
//   29 x 384, 197 (14 x 14)         47 / 42        35 / 42        206 / 119      151 / 115
//   106 x 384, 197 (14 x 14)        151 / 90       78 / 74        632 / 296      388 / 259
//   132 x 384, 197 (14 x 14)        199 / 109      104 / 94       811 / 370      482 / 318
//   128 x 768, 197 (14 x 14)        351 / 188      177 / 149      1408 / 604     833 / 525
//   30 x 384, 257 (16 x 16)         70 / 53        44 / 51        302 / 146      190 / 128
//   35 x 384, 257 (16 x 16)         80 / 56        45 / 53        370 / 157      234 / 145
//   32 x 384, 325 (18 x 18)         118 / 60       60 / 64        417 / 167      231 / 151
//   4 x 768, 1025 (32 x 32)         130 / 67       89 / 66        259 / 140      185 / 132
//   1 x 768, 4096 (64 x 64)         100 / 78       99 / 78        223 / 152      209 / 151
//   119 x 384, 197 (2 x 98)         90 / 97        72 / 86        334 / 312      302 / 274
//   119 x 384, 197 (65 x 3)         117 / 98       75 / 86        388 / 311      296 / 275
//   8 x 384, 1025 (4 x 256)         44 / 67        41 / 66        136 / 139      116 / 132
//   30 x 384, 1025 (4 x 256)        220 / 165      167 / 156      624 / 415      553 / 388
//   6 x 384, 1025 (8 x 128)         44 / 58        41 / 59        182 / 121      153 / 119
//   8 x 384, 1025 (8 x 128)         52 / 67        47 / 66        170 / 139      140 / 132
//   11 x 384, 1025 (8 x 128)        87 / 78        70 / 76        356 / 189      336 / 179
//   3 x 384, 2049 (8 x 256)         44 / 63        42 / 64        198 / 131      177 / 132
//   4 x 384, 2049 (8 x 256)         50 / 71        46 / 70        159 / 151      129 / 150
//   8 x 768, 4096 (64 x 64)         1850 / 347     1883 / 375     4507 / 870     4075 / 839
// (The lines stand where the kernels before the wave tiles put them, and callers size their scratch
// by them.  On the wrong side are now, forward, where calls copy: fp32 at 8 x 128 and 8 x 256 below 4 million
// elements, bf16 at 35 x 384 x 257, 32 x 384 x 325 and 11 x 384 x 1025; where they gather: fp32 at
// 72 x 384 x 145, bf16 at 106 x 384 x 197.  Backward, where they copy: bf16 at 65 and 82 tokens, by 6 and 8%, and
// at 4 x 256 and 4 x 384 x 2049, by 14 and 16%; where they gather: fp32 at 2 x 98, by 7%.)
// The copies ask for an fp32 result, which the chunk-per-lane kernel gives for bf16 only
// with window 1: bf16 images of 4096 tokens run the wave-tile kernels here.
namespace {

// Elements of a (B,D,L) tensor from which the forward pass copies.  Never below 2^21:
// it pays for two more launches.
long reorder_fwd_elements(const FwdParams& p)
{
    const int L = p.seqlen, side = p.order.H < p.order.W ? p.order.H : p.order.W;
    const long never = LONG_MAX;
    if (side <= 2) return never;
    long line;
    if (p.dtype == 0) line = L >= 160 ? 1L << 21 : (L >= 112 ? 4500000L : never);
    else line = L >= 320 ? 1L << 21 : (L >= 208 ? 3250000L : (L >= 160 ? 9500000L : never));
    if (side <= 4) return line < 8000000L ? 8000000L : line;
    return p.dtype != 0 && side <= 8 && L >= 1000 ? 4000000L : line;
}

// The backward call makes several launches anyway; it moves more per token, so copies
// win from shorter rows on, and also where the call is too small to fill the chip.
bool reorder_bwd(const FwdParams& p)
{
    const int side = p.order.H < p.order.W ? p.order.H : p.order.W;
    if ((long)p.batch * p.dim * p.seqlen < 400000L) return true;
    return p.dtype == 0 ? p.seqlen >= 80 && side > 2 : p.seqlen >= 60;
}

constexpr size_t kCopyAlign = 256;
size_t aligned_bytes(size_t n) { return (n + kCopyAlign - 1) / kCopyAlign * kCopyAlign; }

bool reorder_applies(const FwdParams& p)
{
    return p.order.kind != 0 && p.seqlen <= kReorderMaxTokens && p.batch > 0 && p.dim > 0 && p.seqlen > 0;
}

// stored index -> scanned index: the same map with the grid's sides exchanged
TokenOrder inverse_order(const TokenOrder& o)
{
    TokenOrder r = o;
    r.H = o.W;
    r.W = o.H;
    r.rH = 1.0f / (float)r.H;
    return r;
}

TokenOrder stored_order()
{
    TokenOrder r{};
    r.H = r.W = r.HW = 1;
    r.rH = 1.0f;
    return r;
}

// The rows of the copies start at multiples of 32 elements: a tile is then whole lines of
// memory, where rows of 197 tokens straddle them (the scan of such rows takes 10% longer).
int copy_pitch(const FwdParams& p) { return (p.seqlen + 31) / 32 * 32; }

struct CopySizes {
    size_t row, mat;      // bytes of a (B,D,L) and of a (B,N,L) copy in the storage type, rounded up
    size_t row32;         // of a (B,D,L) copy in fp32
};
CopySizes copy_sizes(const FwdParams& p)
{
    const size_t e = p.dtype == 0 ? 4 : 2;
    const size_t bdl = (size_t)p.batch * p.dim * copy_pitch(p), bnl = (size_t)p.batch * p.dstate * copy_pitch(p);
    return {aligned_bytes(bdl * e), aligned_bytes(bnl * e), aligned_bytes(bdl * 4)};
}

FwdParams in_stored_order(FwdParams p)
{
    p.order = stored_order();
    p.pitch = copy_pitch(p);
    return p;
}

// Copies of one tensor list, filled in the order of the calls.
struct Copies {
    ReorderMany m{};
    int n = 0;
    void add(const void* src, int src_pitch, void* dst, long rows)
    {
        if (!src) return;
        m.src[n] = src; m.src_pitch[n] = src_pitch; m.dst[n] = dst; m.rows[n] = rows;
        ++n;
    }
};

}  // namespace

size_t fwd_reordered_workspace_bytes(const FwdParams& p)
{
    if (!reorder_applies(p) || (long)p.batch * p.dim * p.seqlen < reorder_fwd_elements(p)) return 0;
    const CopySizes c = copy_sizes(p);
    return aligned_bytes(fwd_workspace_bytes(in_stored_order(p))) + 2 * c.row + 2 * c.mat + c.row32;
}

hipError_t launch_fwd_reordered(FwdParams p, void* workspace, float* saved, hipStream_t stream)
{
    const CopySizes c = copy_sizes(p);
    FwdParams q = in_stored_order(p);
    const long rows = (long)p.batch * p.dim, mats = (long)p.batch * p.dstate;
    char* at = static_cast<char*>(workspace) + aligned_bytes(fwd_workspace_bytes(q));
    auto take = [&](size_t n) { char* r = at; at += n; return r; };
    Copies in;
    const int L = p.seqlen;
    in.m.dst_pitch = q.pitch;
    q.x = take(c.row);     in.add(p.x, L, const_cast<void*>(q.x), rows);
    q.delta = take(c.row); in.add(p.delta, L, const_cast<void*>(q.delta), rows);
    q.Bm = take(c.mat);    in.add(p.Bm, L, const_cast<void*>(q.Bm), mats);
    q.Cm = take(c.mat);    in.add(p.Cm, L, const_cast<void*>(q.Cm), mats);
    hipError_t e = launch_reorder(in.m, p.dtype, p.seqlen, p.order, stream);
    if (e != hipSuccess) return e;
    q.z = nullptr;
    q.y = take(c.row32);
    q.y_is_f32 = 1;
    e = launch_fwd(q, workspace, saved, stream);
    if (e != hipSuccess) return e;
    Copies out;
    out.add(q.y, q.pitch, p.y, rows);
    out.m.dst_pitch = L;
    out.m.gate = p.z;
    return launch_reorder_gate(out.m, p.dtype, p.seqlen, inverse_order(p.order), stream);
}

size_t bwd_reordered_workspace_bytes(const FwdParams& f)
{
    if (!reorder_applies(f) || !reorder_bwd(f)) return 0;
    const CopySizes c = copy_sizes(f);
    return aligned_bytes(bwd_workspace_bytes(in_stored_order(f))) + (5 + (f.z ? 2 : 0)) * c.row + 4 * c.mat;
}

hipError_t launch_bwd_reordered(FwdParams f, BwdParams p, void* dBm, void* dCm, void* workspace,
                                const float* saved, const float* dhT, hipStream_t stream)
{
    const CopySizes c = copy_sizes(f);
    FwdParams q = in_stored_order(f);
    BwdParams r = p;
    r.order = q.order;
    r.pitch = q.pitch;
    const long rows = (long)f.batch * f.dim, mats = (long)f.batch * f.dstate;
    char* at = static_cast<char*>(workspace) + aligned_bytes(bwd_workspace_bytes(q));
    auto take = [&](size_t n) { char* t = at; at += n; return t; };
    Copies in, out;
    auto copy_in = [&](const void* src, size_t bytes, long n) -> const void* {
        if (!src) return nullptr;
        void* d = take(bytes);
        in.add(src, f.seqlen, d, n);
        return d;
    };
    auto copy_out = [&](void* dst, size_t bytes, long n, int pitch) -> void* {
        if (!dst) return nullptr;
        void* t = take(bytes);
        out.add(t, pitch, dst, n);
        return t;
    };
    in.m.dst_pitch = q.pitch;
    out.m.dst_pitch = f.seqlen;
    q.x = r.x = copy_in(f.x, c.row, rows);
    q.delta = r.delta = copy_in(f.delta, c.row, rows);
    q.z = r.z = copy_in(f.z, c.row, rows);
    r.dout = copy_in(p.dout, c.row, rows);
    q.Bm = r.Bm = copy_in(f.Bm, c.mat, mats);
    q.Cm = r.Cm = copy_in(f.Cm, c.mat, mats);
    r.dx = copy_out(p.dx, c.row, rows, q.pitch);
    r.ddelta = copy_out(p.ddelta, c.row, rows, q.pitch);
    r.dz = copy_out(p.dz, c.row, rows, q.pitch);
    void* dB = copy_out(dBm, c.mat, mats, f.seqlen);      // (the sums over channels are dense)
    void* dC = copy_out(dCm, c.mat, mats, f.seqlen);
    hipError_t e = launch_reorder(in.m, f.dtype, f.seqlen, f.order, stream);
    if (e != hipSuccess) return e;
    e = launch_bwd(q, r, dB, dC, workspace, saved, dhT, stream);
    if (e != hipSuccess) return e;
    return launch_reorder(out.m, f.dtype, f.seqlen, inverse_order(f.order), stream);
}

}  // namespace lbscan
