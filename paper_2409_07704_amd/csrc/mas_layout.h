// Workspace and bit layout shared by the libmas kernels and host code.
//
// Rows of an item are processed by 64-lane waves.  Lane 0 of wave g carries
// the row above the wave (row 63g-1, a copy handed down by the previous
// wave; for g = 0 the virtual -inf row above row 0) and lanes 1..63 own
// rows 63g .. 63g+62, one text row per lane.  Two such waves (126 rows)
// share a workgroup with the waves that feed them.  Speech columns are
// processed in chunks of 32, and every lane packs its row's 32 forward
// decisions of a chunk into one 32-bit word.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace mas {

constexpr int kWave = 64;                    // lanes per wavefront (CDNA)
constexpr int kRowsPerWave = kWave - 1;      // text rows a wave owns (lanes 1..63)
constexpr int kWavesPerBlock = 2;            // sweep waves of a workgroup
constexpr int kChunk = 32;                   // speech columns per decision word
constexpr size_t kAlign = 256;
constexpr int kMaxRows = 8192;               // largest T (the walker keeps row_start in LDS)

// Decision bit of text row i at speech column j (j >= 1): 1 when the forward
// max took the diagonal predecessor Q[i-1][j-1] (the backtrack then moves to
// row i-1), 0 when it kept Q[i][j-1].  A sweep wave packs a row's decisions
// of one chunk into one 32-bit word, the chunk's first column in bit 31.
// Those words never leave the CU: they are turned into step masks.
//
// Step mask of row i in chunk c: the set of positions p (column 32c + 31 - p)
// at which the backtrack, entering the chunk in row i at its last column,
// moves up one row while walking back to the chunk's first column; row i - k
// begins at the column of the k-th lowest position.  Per chunk, pm[b][c] holds
// EP = kEntPerWave * NW entries:
//   32g + q (q < 32):  mid entry q of wave g: the mask of the wave's last row
//                      entered at position q (column 32c + 31 - q), positions
//                      >= q, which completes a path of the next wave that
//                      climbs out of it, at q = p + 1 (below);
//   ent_row0 + i:      the mask of text row i, for the path while it stays in
//                      the rows of i's wave; a path that climbs into the row
//                      above the wave ends there, with that step as its
//                      highest position p.
// Rows lie in a row whatever waves they belong to, so that the walk reads 64
// rows' entries with one subtraction per lane.  A path climbs at most 32 rows
// per chunk, so it crosses at most one wave boundary in a chunk.
constexpr int kEntPerWave = 96;
// Descent bytes pd[b][c], the walk's own copy of the step masks at a quarter of
// their size, entry by entry:
//   row i:        the number of rows the path climbs in the chunk while it
//                 stays in the wave's rows (the mask's popcount), or 64 + p
//                 when it climbs into the row above the wave at position p
//                 (the highest position of the mask);
//   mid entry q:  the popcount of mid entry q's mask.
constexpr uint32_t kEscape = 64;
__host__ __device__ constexpr int ent_row0(int NW) { return kChunk * NW; }

// Boundary hand-off between consecutive workgroups of an item: the last wave
// g of a workgroup publishes Q[63g+62][j] (its last row) for every column j it
// computes as one 64-bit word {low: fp32 bits, high: tag} (waves of one
// workgroup hand on through LDS).  The tag identifies the call (see
// WsHeader), so stale words from earlier calls are never mistaken for fresh
// ones.
// Dense path of large batches: written in tiles of kPathTileRows rows of one
// item, taken in the order the items' row_start tables are published, by at
// most kPathWorkgroups path-writer workgroups: enough to keep up; with more the
// sweeps still running lose what the path gains.  With 96, 112, 128, 160 and
// 192 (us): 64 x 1024 x 4096 mixed lengths, eight draws 170.8, 166.0, 162.6,
// 161.7, 162.4, ragged 211, 204, 199, 199, 203, full 312, 303, 298, 295, 295; 32
// x 2048 x 8192 518, 512, 513, 518, 522; 300 x 200 x 1200 122, 117, 117, 115, 124.
constexpr int kPathTileRows = 32;
constexpr int kPathWorkgroups = 128;
constexpr uint64_t kShapeSlack = 192;  // (shapes are accepted up to this much below 2^31 boundary regions)

// Batches of at most this many cells (B T S) get their path from the sweep
// workgroups themselves, zeros first (KParams::early): their launches wait on
// chains of dependent steps, not on HBM, so that the zeros cost little before
// the sweeps and only the ones are left after the walks.  Larger ones also
// start their items by length (KParams::stagger).  Measured, path writers /
// early (us): 200 x 128 x 1500 65 / 45, 32 x 512 x 2048 60 / 58, 48 x 400 x 2400
// 64 / 62, 64 x 500 x 2000 64 / 65, 16 x 1024 x 4000 125 / 131, 64 x 252 x 4096
// 104 / 113 (the last three just below the limit); above it 300 x 200 x 1200 115
// / 83, 600 x 128 x 1000 200 / 175, 64 x 300 x 4096 113 / 114, 64 x 500 x 3000
// 107 / 112, 24 x 1024 x 4096 132 / 138, 64 x 1024 x 4096 162 / 218.  So cells
// alone draw the line coarsely: items of many cells would have it a fifth lower,
// batches of many small ones above 128 M.
constexpr uint64_t kEarlyMaxCells = (uint64_t)64 << 20;

// Generations run from 0 to kGenEnd - 1 and start over: a call's tags, 2 gen + 1
// and 2 gen + 2, are never 0, which is what a clear workspace and a load that
// was dropped hold.
constexpr uint32_t kGenEnd = 0x7fffffffu;
struct WsHeader {
  uint32_t gen;         // call generation; tag of a call = 2 * gen + 1 (and the even number after it, see slot_region)
  uint32_t exit_count;  // workgroups that finished the current call
  uint32_t error;       // sticky: non-zero once a device-side wait timed out
  uint32_t walk_count;  // row_start tables published in the current call
  uint32_t tile_next;   // path tiles taken in the current call
  uint32_t magic;       // kWsMagic once the workspace has been initialised
  uint32_t path_fail;   // tag of the last call in which a path writer gave up a wait
  uint32_t pad[57];
};
constexpr uint32_t kWsMagic = 0x3153414du;  // "MAS1"
constexpr int kWsMagicPiece = 1;            // the header's 16-byte piece holding magic (bytes 16..31)
static_assert(sizeof(WsHeader) == kAlign, "header is one alignment unit");

__host__ __device__ inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct Layout {
  int32_t B, T, S;
  int32_t NW;      // waves per item = ceil(T / 63)
  int32_t NB;      // workgroups per item = ceil(NW / 2)
  int32_t NS;      // boundary word regions per item = ceil(NW / 4), shared by two workgroups each
  int32_t NC;      // chunks per item = ceil(S / 32)
  int32_t EP;      // step-mask entries per chunk of an item = kEntPerWave * NW
  size_t off_done;   // uint32 [B][NW] sweep-finished flags (tag values)
  size_t off_tmo;    // uint32 [B] per-item timeout flags (tag values)
  size_t off_order;  // uint64 [B] items in the order their row_start tables were published: tag << 32 | item
  size_t off_slots;  // uint64 [B][NS][NC*32] boundary hand-off words of each workgroup's last wave
  size_t off_pm;     // uint32 [B][NC][EP] step masks
  size_t off_rs;     // int32  [B][T+1] row_start table (mas_forward_ex)
  size_t off_pd;     // uint8  [B][NC][EP] descent bytes
  size_t bytes;
};

// Returns false when the shape is invalid or its byte counts overflow.
__host__ inline bool make_layout(int32_t B, int32_t T, int32_t S, Layout* L) {
  if (B < 1 || T < 1 || S < 1 || T > kMaxRows) return false;
  L->B = B;
  L->T = T;
  L->S = S;
  L->NW = (T + kRowsPerWave - 1) / kRowsPerWave;
  L->NB = (L->NW + kWavesPerBlock - 1) / kWavesPerBlock;
  L->NS = (L->NW + 3) / 4;
  L->NC = (S + kChunk - 1) / kChunk;
  L->EP = kEntPerWave * L->NW;
  // Overflow guard: every product below stays far under 2^62 when these hold.
  if ((uint64_t)B * (uint64_t)L->NS + kShapeSlack > 0x7fffffffull) return false;
  if ((uint64_t)B * (uint64_t)T * (uint64_t)S > (1ull << 46)) return false;
  // One item's value slab is addressed with signed 32-bit byte offsets.
  if ((uint64_t)T * (uint64_t)S * 4u >= (1ull << 31)) return false;
  size_t off = sizeof(WsHeader);
  L->off_done = off;
  off = round_up(off + (size_t)B * L->NW * sizeof(uint32_t), kAlign);
  L->off_tmo = off;
  off = round_up(off + (size_t)B * sizeof(uint32_t), kAlign);
  L->off_order = off;
  off = round_up(off + (size_t)B * sizeof(uint64_t), kAlign);
  L->off_slots = off;
  off = round_up(off + (size_t)B * L->NS * (size_t)L->NC * kChunk * sizeof(uint64_t), kAlign);
  L->off_pm = off;
  off = round_up(off + (size_t)B * L->NC * (size_t)L->EP * sizeof(uint32_t), kAlign);
  L->off_rs = off;
  off = round_up(off + (size_t)B * ((size_t)T + 1) * sizeof(int32_t), kAlign);
  L->off_pd = off;
  off = round_up(off + (size_t)B * L->NC * (size_t)L->EP, kAlign);
  L->bytes = off;
  return true;
}

// Per-item status codes (same values as MAS_ITEM_* in the public header).
enum ItemStatus : int32_t {
  kItemOk = 0,
  kItemEmpty = 1,
  kItemInfeasible = 2,
  kItemOutOfRange = 3,
  kItemSyncTimeout = 4,
  kItemBadWorkspace = 5
};

__host__ __device__ inline int32_t item_status(int32_t tx, int32_t ty, int32_t T, int32_t S) {
  if (tx < 0 || ty < 0 || tx > T || ty > S) return kItemOutOfRange;
  if (tx == 0 || ty == 0) return kItemEmpty;
  if (ty < tx) return kItemInfeasible;
  return kItemOk;
}

}  // namespace mas
