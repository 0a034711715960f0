// Internal helpers shared by the HIP translation units of libsagnn (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "sagnn.h"

#define SAGNN_EXPORT extern "C" __attribute__((visibility("default")))

namespace sagnn {

constexpr int kWave = 64;  // CDNA wavefront width

void set_hip_error(hipError_t e);

inline int hip_fail(hipError_t e) {
  set_hip_error(e);
  return SAGNN_EHIP;
}

#define SAGNN_HIP(expr)                                   \
  do {                                                    \
    hipError_t _e = (expr);                               \
    if (_e != hipSuccess) return ::sagnn::hip_fail(_e);   \
  } while (0)

// launch check: catches configuration errors without synchronising
#define SAGNN_LAUNCH_CHECK() SAGNN_HIP(hipGetLastError())

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// --- SpMM workspace geometry (host and device agree through these) -----------------------
// Chunks of the nonzero-splitting schedule: about T entries each, T a multiple of 16.  Long enough that what a
// chunk costs besides its entries does not count, short enough that small matrices fill the chip: 8192 wavefronts
// (32 per CU) of 64 / lanes-per-entry chunks.  Serial sums stay below T + 32 <= 160 terms.
constexpr int kSpmmChunkMax = 128;
inline int64_t spmm_chunk_groups(int32_t f) { return f <= 16 ? 16 : (f <= 32 ? 8 : (f <= 64 ? 4 : (f <= 128 ? 2 : 1))); }
inline int64_t spmm_chunk_entries(int64_t nnz, int32_t f) {
  const int64_t t = (nnz / (8192 * spmm_chunk_groups(f)) + 15) / 16 * 16;
  return t < 16 ? 16 : (t > kSpmmChunkMax ? kSpmmChunkMax : t);
}
constexpr uint32_t kSpmmMagic = 0x53A66E02u;

// Slab-sweep schedule (long rows): a wavefront owns kSweepSlots row pieces.
constexpr int kSweepSlots = 16;
// longest run of entries summed into one register before it is folded into the piece's slot
constexpr int kSweepRunMax = 128;
constexpr int kSweepMaxSlabs = 384;
constexpr int kSweepColBits = 27;           // column id bits in an encoded entry
constexpr int kSweepMinLong = 16;           // smallest degree a "long" row can be given
// The sweep is cut into intervals of `sync_slabs` slabs; between two intervals the workgroups of
// an XCD that run at the same time wait for each other (bounded), so that they stay in the same
// part of B.  A wavefront's stream is padded to a whole batch at every interval boundary.
constexpr int kSweepMaxIntervals = 64;
constexpr int kSweepBarrierSlots = 65536;   // arrival counters (cohort x XCD x interval)
constexpr int kSweepMaxWindows = 2048;      // dealing windows of a matrix (11 bits of a sort key)

// Longest piece of a swept row where the caller does not say: about what a stream holds on average when 8192
// wavefronts share the entries (a longer piece makes one stream the whole product waits for: 2.4 M entries at f = 128
// took 433 us with pieces of 4096 and 167 with 1024), a power of two up to 4096.
inline int64_t sweep_piece_streams(int32_t f) { return 8192 * (f > 128 ? 1 : (f > 64 ? 2 : 4)); }
inline int32_t sweep_piece_default(int64_t nnz, int32_t f) {
  const int64_t streams = sweep_piece_streams(f);
  int32_t p = 256;
  while (p < 4096 && 2 * (int64_t)p * streams <= nnz) p *= 2;
  return p;
}
inline int32_t sweep_piece_floor(int64_t nnz, int32_t f) {   // no piece is cut shorter
  const int32_t p = sweep_piece_default(nnz, f);
  return p < 1024 ? p : 1024;
}

// Columns one launch of the sweep covers when `rest` are left: slabs of 256, 128 and 64 (the exact kernels; max_slab
// 128: none wider), a width that is no multiple of 64 in one launch as soon as at most max_slab are left.
inline int32_t sweep_slab(int32_t rest, int32_t max_slab) {
  if (rest >= max_slab) return max_slab;
  if ((rest & 63) == 0 && rest > 128) return 128;
  return rest;
}
inline int32_t sweep_widest_launch(int32_t f, int32_t max_slab) {
  int32_t widest = 0;
  for (int32_t c = 0; c < f;) {
    const int32_t fw = sweep_slab(f - c, max_slab);
    widest = fw > widest ? fw : widest;
    c += fw;
  }
  return widest;
}

// Cache lines of 128 bytes a row of f floats touches on average when rows lie ldb floats apart (the first row aligned)
inline double spmm_row_lines(int32_t f, int64_t ldb) {
  int lines = 0;
  for (int i = 0; i < 32; ++i) lines += (int)(((ldb * 4 * i) % 128 + (int64_t)f * 4 + 127) / 128);
  return lines / 32.0;
}
inline int32_t spmm_padded_width(int32_t f) { return f <= 16 ? 16 : (f + 31) / 32 * 32; }
// Whether k rows of B are copied to rows that begin on a cache line (on half of one where f <= 16) before nnz of them
// are gathered.  Time of the saved lines and of the copy at the rates both run at (7.5 TB/s of lines that miss the L2,
// copies 4.8 TB/s); hits save a quarter of that, hence the margin: 400 k vertices, 8 M entries lose 10 us of 143 at f = 24
// (3.6 times the copy), 1 M vertices, 50 M entries gain 95 of 680 (9 times), 300 of 1323 at f = 60 (6 times) and 310 of
// 2212 at f = 124 (3 times).  Small operands stay in the L2s and are not copied.
inline bool spmm_pad_pays(int64_t k, int64_t nnz, int32_t f, int64_t ldb) {
  const int32_t fp = spmm_padded_width(f);
  if (f > 128 || k * (int64_t)f * 4 < (8 << 20)) return false;
  const double saved = spmm_row_lines(f, ldb) - spmm_row_lines(f, fp);
  return (double)nnz * saved * 128 / 7.5 > (f <= 64 ? 4 : 2) * ((double)k * (f + fp) * 4 / 4.8);
}

struct SpmmWsHeader {       // first 256 bytes of the SpMM workspace (device copy)
  uint32_t magic;
  int32_t has_empty_rows;   // some row of the matrix has no entries
  int64_t m, nnz;
  int32_t f;
  int32_t mode;             // 0: nonzero splitting over the caller's CSR; 1: slab sweep
  uint64_t generation;      // matches the host descriptor of the same prepare call
  // chunk part (the caller's CSR in mode 0, the short-row CSR in mode 1)
  int64_t c_rows, c_nnz, c_nchunks;
  // sweep part
  int64_t n_waves, n_long_entries, n_multi_rows, n_multi_pieces;
  int32_t n_slabs, slab_width;
  int32_t groups;           // lane groups per wavefront in the sweep streams (1, 2 or 4)
  int32_t n_intervals;      // >= 1; interval boundaries are barrier points when sync_slabs > 0
  int32_t sync_slabs;       // slabs per interval (0: no barriers, one interval)
  int32_t wg_per_cohort;    // workgroups that are resident together (a multiple of 8)
  int32_t sync_timeout_ticks;  // bounded wait at a barrier, in 100 MHz ticks
  int32_t sync_test_extra;  // test hook: added to the expected arrivals (forces the give-up path)
  int32_t slots;            // accumulator rows (pieces) per wavefront actually used, <= kSweepSlots
  int32_t barriers;         // 1: barriers at interval boundaries
  int32_t pace_ps_per_step; // pacing asked for at prepare time (0: none)
  int32_t max_slab;         // widest column slab of B per launch (256 or 128)
  int32_t col_slab;         // columns per launch where the width is a multiple of it (0: as max_slab says)
  int32_t launch_waves;     // wavefronts per launch (0: all in one)
  int32_t fused_waves;      // the same with the layer's dense transform behind the sweep
};
static_assert(sizeof(SpmmWsHeader) <= 256, "header must fit its slot");

// Fixed layout (a function of m, k, nnz, f only; every array has its worst-case size):
struct SpmmWsLayout {
  size_t header, chunks, fix_list, flags, rowptr_s, rowmap_s, code, vals, piece_info, piece_target,
      wave_base, wave_steps, sync_off, barrier, sched, multi_row, multi_first, partial, carry, plan, wpack, padded, total;
  size_t need;           // enough for every call; with `total` there is room for the padded copy
  int64_t max_chunks, max_pieces, max_waves, max_multi_rows, max_multi_pieces, stream_cap;
  int64_t padded_rows;   // rows of B the padded copy has room for
};

inline int64_t spmm_nchunks(int64_t nnz, int64_t T) { return ceil_div(nnz, T); }

// A workspace that is enough for a matrix is enough for every smaller one: fewer rows, entries or columns of B.  Chunks
// and pieces get longer with the number of entries and with the width, so what they need is the most that any smaller
// count, and any narrower operand, comes to.
// Chunks of any count up to nnz at width f (the short rows of a sweep are such a part of the entries)
inline int64_t spmm_most_chunks(int64_t nnz, int32_t f) {
  const int64_t T = spmm_chunk_entries(nnz, f);
  int64_t most = spmm_nchunks(nnz, T) + 1;
  for (int64_t t = 16; t < T; t += 16) {
    const int64_t upto = (t + 1) * 8192 * spmm_chunk_groups(f);   // the most entries that get chunks of t
    const int64_t chunks = (upto < nnz ? upto : nnz) / t + 2;
    most = chunks > most ? chunks : most;
  }
  return most;
}
// Times that rows of any count up to nnz are cut at width f (a piece has at least sweep_piece_floor entries)
inline int64_t sweep_most_cuts(int64_t nnz, int32_t f) {
  int64_t most = nnz / sweep_piece_floor(nnz, f);
  for (int64_t p = 256; p < sweep_piece_floor(nnz, f); p *= 2) {
    const int64_t cuts = (2 * p * sweep_piece_streams(f) - 1) / p;   // at the most entries that get pieces of p
    most = cuts > most ? cuts : most;
  }
  return most;
}

inline SpmmWsLayout spmm_ws_layout(int64_t m, int64_t nnz, int32_t f) {
  SpmmWsLayout L{};
  int64_t cuts = 0, carry_floats = 0, partial_floats = 0;
  for (int32_t top = 16;; top *= 2) {   // widths up to 16, 32, 64, 128 and beyond differ
    const int32_t w = top > 128 || f < top ? f : top;
    const int64_t chunks = spmm_most_chunks(nnz, w), c = sweep_most_cuts(nnz, w);
    L.max_chunks = chunks > L.max_chunks ? chunks : L.max_chunks;
    cuts = c > cuts ? c : cuts;
    carry_floats = chunks * w > carry_floats ? chunks * w : carry_floats;
    partial_floats = (2 * c + 2) * w > partial_floats ? (2 * c + 2) * w : partial_floats;
    if (w == f) break;
  }
  // every long row has >= kSweepMinLong entries; splitting adds at most `cuts` pieces; every
  // short row may become a piece of its own (whole-row wavefronts behind those of the long rows)
  const int64_t long_pieces = nnz / kSweepMinLong + cuts + kSweepSlots;
  const int64_t long_waves = ceil_div(long_pieces, kSweepSlots) + 1;
  const int64_t short_waves = ceil_div(m, kSweepSlots) + 4;
  L.max_pieces = long_pieces + m;
  L.max_waves = long_waves + short_waves;
  L.max_multi_rows = cuts + 1;
  L.max_multi_pieces = partial_floats / f;   // (at least twice the cuts at width f, and 2)
  // sweep streams + gap + short CSR entries + padding.  A wavefront's stream is padded to the
  // batch of 8 steps at every interval boundary; with lane groups (2 to 16 zipped streams per
  // wavefront) also to the longest of its group streams inside every interval.  If a pattern
  // needs more than this, the planner lays the streams out as one interval.  A whole-row
  // wavefront has one interval, and short rows of like length: with up to 4 group streams at most
  // 8 steps of padding for each, 32 words; 8 and 16 streams (up to 128 words) sweep short rows whole
  // only where the rest of the room takes that, and if the long rows' padding has filled it the
  // planner starts over with the short rows beside the sweep.  What fits neither way is not swept.
  L.stream_cap = nnz + nnz / 4 + 256 * long_waves + 32 * short_waves + 1024;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += round_up(bytes, 256); return o; };
  L.header = take(256);
  L.chunks = take(4 * sizeof(int32_t) * (size_t)L.max_chunks);
  L.fix_list = take(2 * sizeof(int32_t) * (size_t)L.max_chunks);
  L.flags = take(sizeof(uint32_t) * (size_t)(nnz / 32 + 4));
  L.rowptr_s = take(sizeof(int32_t) * (size_t)(m + 1));
  L.rowmap_s = take(sizeof(int32_t) * (size_t)(m + 1));
  L.code = take(sizeof(uint32_t) * (size_t)L.stream_cap);
  L.vals = take(sizeof(float) * (size_t)L.stream_cap);
  L.piece_info = take(sizeof(int32_t) * 2 * (size_t)(L.max_waves * kSweepSlots));
  L.piece_target = take(sizeof(int32_t) * (size_t)(L.max_waves * kSweepSlots));
  L.wave_base = take(sizeof(int32_t) * (size_t)(L.max_waves + 1));
  L.wave_steps = take(sizeof(int32_t) * (size_t)(L.max_waves + 1));
  L.sync_off = take(sizeof(int32_t) * (size_t)L.max_waves * (kSweepMaxIntervals + 1));
  L.barrier = take(sizeof(uint32_t) * (size_t)(kSweepBarrierSlots + 64));
  L.sched = take(sizeof(float) * (size_t)(kSweepMaxIntervals + 2));
  L.multi_row = take(sizeof(int32_t) * (size_t)L.max_multi_rows);
  L.multi_first = take(sizeof(int32_t) * (size_t)(L.max_multi_rows + 1));
  L.partial = take(sizeof(float) * (size_t)partial_floats);
  L.carry = take(sizeof(float) * (size_t)carry_floats);
  // planner: totals, per-window arrays, tile sums of the five row scans (2048 rows per tile)
  L.plan = take(256 + (size_t)kSweepMaxWindows * 8 + 3 * 4 * (size_t)(kSweepMaxWindows + 64) +
                5 * sizeof(int32_t) * (size_t)(ceil_div(m, 2048) + 2));
  // W of a fused layer call packed for the bfloat16 matrix instructions (at most 256 x 256, up to
  // three terms per element)
  L.wpack = take(3 * 256 * 256 * 2);
  L.need = off;
  // the layout does not know how many rows B has: as many as A where a copy pays then
  L.padded_rows = spmm_pad_pays(m, nnz, f, f) ? m : 0;
  L.padded = take(sizeof(float) * (size_t)L.padded_rows * (size_t)spmm_padded_width(f));
  L.total = off;
  return L;
}
inline size_t spmm_ws_bytes(int64_t m, int64_t nnz, int32_t f) { return spmm_ws_layout(m, nnz, f).total; }

// Host descriptor of a prepared workspace (what the launcher needs without reading the device)
struct SpmmHostDesc {
  uint64_t generation;
  int64_t m, nnz;
  int32_t f, mode;
  int64_t c_rows, c_nnz, c_nchunks;
  int64_t n_fix, n_fix_big; // rows whose shares the carry fix-up adds: with few, with many chunks
  int64_t n_waves, n_multi_rows, sweep_stream_len;
  int32_t has_empty_rows;
  int32_t groups;
  int64_t k;                // rows of B the schedule was prepared for (stream columns are < k)
  int32_t n_intervals, sync_slabs, wg_per_cohort, sync_timeout_ticks, sync_test_extra;
  int32_t slots;
  int32_t barriers, pace_ps_per_step;
  int32_t max_slab;         // widest column slab of B per launch (256, or 128 for the lane-group kernels at wider f)
  int32_t n_slabs;          // slabs of B that a stream passes over
  int32_t col_slab;         // columns per launch where the width is a multiple of it (0: as max_slab says)
  int32_t launch_waves;     // wavefronts per launch (0: all in one)
  int32_t fused_waves;      // the same with the layer's dense transform behind the sweep
  int32_t apart;            // a small matrix without hubs: the layer's dense transform is not the sweep's epilogue.  Its wavefronts
                            // may hold fewer than 16 rows, which the epilogue multiplies all the same: 60 k vertices of 20 in
                            // communities, f = 128 to 128 173 us, 256 to 256 455; product and transform apart 109, 253
  float reuse;              // uses of a row of B among the rows of A that an XCD holds (see sweep_prepare)
  bool turns, layer_turns;  // wavefronts take turns in the product, in the layer with lane groups (see there)
  int32_t long_waves;       // wavefronts of a sweep before those of whole short rows
  int32_t run_blocks;       // workgroups that are resident at once where the order of the rows carries locality, else 0
  float run_rows;           // rows of a generation from which the XCDs take runs of workgroups (see sweep_prepare)
  int32_t narrow_sums;      // sums of eight lane groups: 0 plain, 1 two, 2 two and folded (see there)
  float mean_steps;         // average stream steps per wavefront (the end of the pacing schedule)
  float max_steps;          // steps of the longest stream
  // dense-tile schedule (tiles.hip): when tiles != 0 everything above describes the rest CSR
  // stored in the tile region behind the plain workspace, nnz included; full_nnz is the caller's
  int32_t tiles;
  int64_t full_nnz, tile_count, tile_items, tile_entries, tile_rows;
  uint64_t tile_generation;
};

// Workgroups of `lds` bytes of LDS each that a CU really holds at once.  Measured on MI355X:
// 5 x 32000 bytes fit, 5 x 32768 do not (the runtime's occupancy query says 5 for both), 2 x 65536
// fit, 3 x 53248 were not tried.  Modelled as 160 KB minus 2 KB, allocations rounded up to 1280
// bytes; an estimate on the low side is harmless wherever this is used.
inline int lds_resident_workgroups(size_t lds) {
  const size_t unit = round_up(lds > 0 ? lds : 1, 1280);
  size_t n = (160u * 1024u - 2048u) / unit;
  if (n > 8) n = 8;   // 32 wavefronts per CU, four per workgroup
  return (int)n;
}
void spmm_desc_put(const void* ws, const SpmmHostDesc& d);
bool spmm_desc_get(const void* ws, SpmmHostDesc* d);
void spmm_desc_erase(const void* ws);

// --- entry points implemented per translation unit (called by the layer functions) --------
int launch_spmm(const int32_t* rowptr, const int32_t* colidx, const float* val, int64_t m,
                int64_t k, int64_t nnz, const float* B, int64_t ldb, int32_t f, float* C,
                int64_t ldc, int32_t accumulate, void* ws, size_t ws_bytes, hipStream_t s);

// rows of H into `out`, and of a second list into `out2` in the same launch (N2 = 0: none)
int launch_pack(const float* H, int64_t n, int64_t ldh, int32_t f, const int32_t* rows, int64_t N, float* out,
                const int32_t* rows2, int64_t N2, float* out2, int64_t ldo, hipStream_t s);

// nonzero-splitting part (spmm_flat.hip)
struct FlatArgs {
  int64_t rows, nnz, nchunks;          // of the CSR being walked
  const int32_t* colidx; const float* val; const float* B; int64_t ldb; uint32_t kmax;
  float* C; int64_t ldc; int32_t accumulate;
  const SpmmWsHeader* hdr; uint64_t generation;
  const int4* chunks; const uint32_t* flags; float* carry; int64_t carry_ld; const int32_t* rowmap;
  bool hubs;                           // rows that many chunks share (the back fix-up list)
};
// d_stat (4 ints of device memory): [0] 1 if some row is empty, [1] / [2] rows on the front / back fix-up list
int flat_build_tables(const int32_t* d_rowptr, int64_t rows, int64_t nnz, int64_t T, char* ws, const SpmmWsLayout& L,
                      int32_t* d_stat, hipStream_t s);
int flat_launch(const FlatArgs& a, int32_t col0, int32_t fw, hipStream_t s);   // columns [col0, col0 + fw), fw <= 256
int flat_fixup(const FlatArgs& a, const int2* list, int64_t list_cap, int64_t n_small, int64_t n_big, int32_t f_total,
               hipStream_t s);

// slab-sweep part (spmm_sweep.hip)
struct SweepPlanResult {
  bool use_sweep;
  float reuse;       // see SpmmHostDesc
  bool turns, layer_turns;
  int32_t narrow_sums, run_blocks, long_waves;
  float run_rows;
  float mean_steps;  // average stream steps per wavefront
  float max_steps;   // steps of the longest stream
  SpmmWsHeader hdr;  // filled in for mode 1 (sweep part + short CSR sizes)
};
// Sizes at which every matrix is looked at for the sweep (see sweep_prepare); below them those without hubs are
inline bool sweep_size(int64_t k, int64_t nnz, int32_t f) { return nnz >= (3 << 20) && k * (int64_t)f * 4 > (8ll << 20); }
// no_hubs: no row is known to hold many times the others' entries
int sweep_prepare(const int32_t* d_rowptr, const int32_t* d_colidx, const float* d_val, int64_t m,
                  int64_t k, int64_t nnz, int32_t f, char* ws, const SpmmWsLayout& L,
                  const sagnn_spmm_options& opt, bool no_hubs, hipStream_t s, SweepPlanResult* out);
// device side of the planner (sweep_plan.hip); the scratch arrays live in the stream arrays of the
// workspace, which are written last
struct SweepRowTotals {
  int64_t pieces, short_rows, short_entries, multi_rows, multi_pieces;
  int32_t min_long;
  int32_t locality;   // permille: how far the columns of neighbouring rows differ from those of all rows
  int32_t span;       // permille of the columns that neighbouring rows choose from
  int32_t slide;      // permille: how often they change a little from one run of rows to the next
  bool has_empty, bad;
};
bool sweep_plan_fits(const SpmmWsLayout& L);
// what the rows look like: the threshold of long rows, locality, span (d_colidx may be null: no locality then).  With `out`
// the host waits for it: bad, min_long, locality, span, slide, and short_entries where the threshold is the lowest (0 otherwise)
int sweep_plan_sample(const int32_t* d_rowptr, const int32_t* d_colidx, int64_t m, int64_t k, int64_t nnz, int32_t opt_min_long,
                      char* ws, const SpmmWsLayout& L, hipStream_t s, SweepRowTotals* out);
// behind sweep_plan_sample: classify rows, build the short-row CSR, the list of split rows and the piece records; one
// stream synchronisation (a 128-byte copy)
// (short_pieces: the short rows also get piece records, one whole row each, behind those of the long rows)
int sweep_plan_rows(const int32_t* d_rowptr, int64_t m, int32_t piece_max, char* ws, const SpmmWsLayout& L, hipStream_t s,
                    SweepRowTotals* out, bool short_pieces = false);
// entries of the pieces of every window (only needed with several windows; synchronises)
int sweep_plan_window_entries(char* ws, const SpmmWsLayout& L, int64_t P, int64_t window, int32_t nwin,
                              hipStream_t s, std::vector<int64_t>* entries);
// sort the pieces and deal them to the streams: fills piece_info / piece_target; synchronises
// (it looks at a flag every few batches to see whether pieces are left); flags[2] of the carry
// area stays 1 if pieces were left over (whole: all of a window's streams get a piece in a batch, else half of them)
int sweep_plan_deal(char* ws, const SpmmWsLayout& L, int64_t P, int64_t window, const int32_t* h_win_unit0,
                    int32_t nwin, int64_t n_waves4, int32_t R, int32_t SL, int32_t piece_max, bool snake, bool whole, hipStream_t s);
// the short rows' pieces (records P_long .. P_long + n_short), longest first, 16 consecutive ones
// per wavefront from wavefront first_wave on (n_waves4 of sweep_plan_deal must cover them); no
// synchronisation
int sweep_plan_deal_short(char* ws, const SpmmWsLayout& L, int64_t P_long, int64_t n_short, int64_t first_wave,
                          hipStream_t s);
// the sweep with the dense transform of a GCN layer as its epilogue (spmm_sweep.hip)
struct SweepFusedArgs {
  const float* W;        // f_in x f_out, row-major
  const void* Wp;        // bfloat16 products: W packed for the matrix cores (set by the launcher)
  float *Z, *Hout, *T;   // m x f_out, m x f_out, m x f_in; each may be NULL (not both Z and Hout)
  int32_t f_out, act;
};
int sweep_launch_fused(const SpmmHostDesc& d, const SpmmWsLayout& L, char* ws, const float* B, int64_t ldb,
                       int32_t f_in, uint32_t kmax, const SweepFusedArgs& fa, int32_t mode, hipStream_t s);
// the layer through that kernel plus a small kernel for the rows it leaves out (spmm.hip);
// returns 1 if the workspace / shapes do not allow it (the caller then uses another form)
bool fused_sweep_layer_applicable(const void* ws, int32_t f_in, int32_t f_out);
int launch_fused_sweep_layer(const int32_t* rowptr, const int32_t* colidx, const float* val, int64_t m,
                             int64_t k, int64_t nnz, const float* H, int64_t ldh, int32_t f_in,
                             const float* W, int32_t f_out, int32_t act, int32_t prec, float* T, float* Z,
                             float* Hout, void* ws, size_t ws_bytes, hipStream_t s);
// `fused` / `fuse` (lane-group schedules only): the layer form, see SweepFusedArgs
int sweep_launch(const SpmmHostDesc& d, const SpmmWsLayout& L, char* ws, const float* B,
                 int64_t ldb, int32_t col0, int32_t fw, uint32_t kmax, float* C, int64_t ldc,
                 int32_t accumulate, int32_t f_total, hipStream_t s,
                 const SweepFusedArgs* fused = nullptr, int32_t fuse = 0);

// Dense-tile schedule (tiles.hip): the tiles of A that are dense enough to re-use staged rows of
// the dense operand are multiplied out of LDS, the rest of A goes through the other schedules.
constexpr int64_t kTileMaxRows = 131072;   // ranked rows / columns that can form tiles
constexpr int64_t kTileMaxCols = 65536;
constexpr int64_t kTileItemEntries = 32768;   // entries of a work item (several tiles of one row group)
struct TileGeom { int fpl, rpw, rg, tc; };    // floats per lane, rows per wavefront, rows per group, columns per tile
bool tile_geom(int32_t f, TileGeom* g);       // false: no tile kernel for this width
struct TileWsLayout {   // the tile region (a function of m, k, nnz, f; worst-case sizes)
  size_t header, rowrank, colrank, hubrow, hubcol, tilecnt, tileslot, ts_chunk, ts_item, item_g, item_ts0,
      item_nch, group_item0, cnt16, roff16, wstart, ent, partial, rest_rowptr, rest_col, rest_val, keys, colcnt,
      err, radix, total;
  int64_t kr, kc, ng, nc, max_ts, max_items;
};
TileWsLayout tile_ws_layout(int64_t m, int64_t k, int64_t nnz, int32_t f);
struct TilePlan { int64_t n_ts, n_items, entries, rest_nnz, rows; };
int tile_prepare(const int32_t* d_rowptr, const int32_t* d_colidx, const float* d_val, int64_t m, int64_t k,
                 int64_t nnz, int32_t f, char* base, const TileWsLayout& L, int32_t reuse_x10, uint64_t generation,
                 hipStream_t s, TilePlan* out);
// C += (kept tiles of A) * B
int tile_launch(const TilePlan& p, uint64_t generation, char* base, const TileWsLayout& L, const float* B,
                int64_t ldb, uint32_t kmax, int32_t f, int64_t m, float* C, int64_t ldc, hipStream_t s);

// Stable least-significant-digit radix sort of (key, payload) pairs on the device (radix.hip),
// over key bits [0, bits).  With pay_in == NULL the payload is the index of the
// pair.  The sorted pairs end up in w.keys[*result], w.pay[*result].  A workspace carved for n
// pairs serves any smaller count.  With limit > 0, err[0] (device, cleared by the caller) is set to 1 if
// some key is >= limit.
struct RadixWs {
  uint32_t *keys[2], *pay[2];
  int32_t* counts;     // [digits][tiles]
  int32_t* totals;     // [digits], then a word for radix_order's flag
  int64_t cap;         // pairs the workspace was carved for
  size_t bytes;
};
RadixWs carve_radix(void* base, int64_t n);   // base == NULL: sizes only
// Stable order of keys of up to 8 bits: order[place] = index, inverse[index] = place.  w.totals = pairs of every key, behind 256 of
// them the flag of a key >= limit (cleared by the caller).
int radix_order(const uint32_t* keys, int64_t n, int bits, const RadixWs& w, int32_t* order, int32_t* inverse, hipStream_t s,
                int64_t limit);
int radix_sort_pairs(const uint32_t* keys_in, const uint32_t* pay_in, int64_t n, int bits, const RadixWs& w,
                     hipStream_t s, int* result, int64_t limit = 0, int32_t* err = nullptr);
// rowptr[c] = number of the cnt sorted keys below c, c in [0, n]
int launch_sorted_rowptr(const uint32_t* keys, int64_t cnt, int64_t n, int32_t* rowptr, hipStream_t s);
// the transpose without its argument checks and error read-back; ws: transpose_ws_bytes(nnz)
size_t transpose_ws_bytes(int64_t nnz);
int launch_transpose(const int32_t* rowptr, const int32_t* colidx, const float* val, int64_t m, int64_t n, int64_t nnz,
                     int32_t* rowptr_t, int32_t* colidx_t, float* val_t, void* ws, int32_t* d_err, hipStream_t s);

int launch_gemm(const float* X, int64_t ldx, const float* W, int64_t ldw, int32_t transW,
                int64_t m, int32_t kdim, int32_t nout, int32_t prec, int32_t act,
                const float* mask, int64_t ldmask, float* Z, int64_t ldz, float* A, int64_t lda,
                hipStream_t s);

// fused layer forward (fused.hip): T = A H stays on the chip; T may be NULL
bool fused_layer_supported(int32_t f_in, int32_t f_out, int32_t prec);
int launch_fused_layer(const int32_t* rowptr, const int32_t* colidx, const float* val, int64_t m,
                       int64_t k, int64_t nnz, const float* H, int64_t ldh, int32_t f_in,
                       const float* W, int32_t f_out, int32_t act, int32_t prec, float* T, float* Z,
                       float* Hout, hipStream_t s);

int launch_gemm_tn(const float* X, int64_t ldx, const float* S, int64_t lds_, int64_t m,
                   int32_t fi, int32_t fo, int32_t prec, float* Y, void* yws, size_t yws_bytes,
                   hipStream_t s);
size_t gemm_tn_ws_bytes(int64_t m, int32_t fi, int32_t fo);

}  // namespace sagnn
