// Internal layout shared by the host side and the HIP kernels of libepm.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace epm {

// ---------------------------------------------------------------- angle keys
// A pencil angle phi in [0, pi) is stored as the u32 key round(phi / pi * 2^32):
// 2^32 key units are pi, so a difference of keys taken mod 2^32 is the
// circular difference of undirected line angles and the wrap-around at 0/pi
// (Sec. 4.4) needs no splitting.
constexpr double kKeyPerRad = 4294967296.0 / 3.14159265358979323846;
// Key units added to every half-width on top of outward rounding.
constexpr uint32_t kGuard = 4;
// A half-width of 2^31 key units (pi/2) covers every angle: the "full"
// interval of a circle that contains the epipole (Sec. 4.4).
constexpr uint32_t kFullHalf = 0x80000000u;

// Keys of a pair are angles minus the pair's cut, the middle of the gap that
// the lines through the epipole leave beside image 2 (a far epipole sees the
// image under a small angle); differences of keys do not notice.  The
// position code of a key has kCentreBits bits: the arc of the lines that meet
// image 2 takes all of them but kSideCodes on either side, for the rest of the
// circle, since keypoints may lie outside their image.  Half of those resolve
// what borders on the arc, up to twice its length away.  (With the keys beyond
// the arc all at its ends' codes, a pair of 60000 whose keypoints reach twice
// as far as the stated image took 3450 us fused, now 167; twenty times as far
// 187, and 269 with seven in eight beside the arc.  The three pieces add 5 us
// to 65 for four million keys.)  The code never decreases
// with the key, so windows of keys are windows of codes, whatever the arc is.
//
// Records are sorted by (width class, position code of the centre).  Class c
// holds half-widths H with 2^(c-1) <= H < 2^c, so a query at key P only has
// to scan class-c centres in [P - 2^c + 1, P + 2^c - 1]; class 31 holds every
// half-width >= 2^30 and is scanned whole.
constexpr int kClassBits = 5;
constexpr int kNumClasses = 32;
constexpr int kCentreBits = 17;
constexpr uint32_t kSideCodes = 1u << (kCentreBits - 4);
constexpr uint32_t kNearCodes = kSideCodes / 2;
constexpr int kRadixBits = 11;  // bits per pass of the sort
constexpr int kSortBits = kClassBits + kCentreBits;  // two passes
constexpr int kWideClass = 31;
static_assert(kSortBits == 2 * kRadixBits, "the records take two passes");

// Query flags.
constexpr uint32_t kQueryNormal = 0;
constexpr uint32_t kQueryEmpty = 1;  // a = b = 0: no distance is defined
constexpr uint32_t kQueryBrute = 2;  // scan every record of the pair

// Relative miss of a query line from the epipole that the record intervals
// absorb; queries beyond it scan the whole pair (exact either way).
constexpr double kKappaBuild = 1.0 / (1 << 24);
// Tolerance inflation used when building intervals (pixels): relative and
// absolute slack that dominates every FP64 rounding in the key pipeline.
constexpr double kEpsRelSlack = 1.0 / (1 << 30);
constexpr double kEpsAbsSlackPx = 1e-7;

// ------------------------------------------------------------ pair records
// Position codes of a pair's keys: codes per key, times 2^32, of the arc (for
// keys shifted up by arc_shift), near it and beyond; keys minus `cut` have the
// arc in their middle (arc_len 0: no arc).
struct KeyArc {
  uint32_t arc_mul, arc_shift, near_mul, far_mul, cut, arc_len;
};

struct PairDev {
  double F[9];          // row-major, pixel space, exactly as given
  double u[3], v[3], e[3];  // orthonormal pencil basis in normalised line space
  double s, cx, cy;     // image-2 normalisation p^ = s (p - c)
  double G11, G12, G22; // Gram matrix of (u_12, v_12)
  double e12;           // |e_12|
  double kappa;         // miss bound absorbed by the record intervals
  KeyArc arc;
  int64_t q_begin, m, k_begin, n;
};

// Angle key of a pencil line at phi: phi reduced to [0, pi), in key units.
__host__ __device__ inline uint32_t angle_key(double phi) {
  if (phi < 0.0) phi += M_PI;
  if (phi >= M_PI) phi -= M_PI;
  return (uint32_t)(uint64_t)(int64_t)nearbyint(phi * kKeyPerRad);
}

// Keys below an arc of len keys in the middle of the circle (one more may lie
// above it), and how far the finer codes beside it reach.
__host__ __device__ inline uint32_t arc_side(uint32_t len) { return (0u - len) >> 1; }
__host__ __device__ inline uint32_t arc_near(uint32_t len) {
  const uint32_t side = arc_side(len);
  return len < side / 4u ? 2u * len : side / 2u;
}

// The pair's arc of keys: those of the pencil lines that meet image 2, a
// little wider on both sides; the whole circle when the epipole lies in the
// image or close to it, or the pair has no pencil.  (Only the resolution of
// the position codes depends on it.)
__host__ __device__ inline void set_key_arc(PairDev& pd) {
  KeyArc& arc = pd.arc;
  arc.cut = arc.arc_len = arc.arc_mul = arc.arc_shift = arc.near_mul = arc.far_mul = 0u;
  if (pd.kappa < 0.0) return;
  // d = e_w p - (e_x, e_y) is the direction from the epipole to the point p
  // (normalised coordinates, centre 0; up to a common sign).  While the four
  // corners lie ahead of the epipole as it looks at the centre, the lines
  // through them are ordered by cross(d0, p) / dot(d0, d), also for an
  // epipole at infinity.
  const double dx0 = -pd.e[0], dy0 = -pd.e[1];
  const double hx = pd.s * pd.cx, hy = pd.s * pd.cy;
  const uint32_t kc = angle_key(atan2(pd.u[2], -pd.v[2]));  // the line through the centre
  double tmin = 0.0, tmax = 0.0;
  uint32_t kmin = kc, kmax = kc;
  for (int k = 0; k < 4; ++k) {
    const double x = k & 1 ? hx : -hx, y = k & 2 ? hy : -hy;
    const double ahead = dx0 * (pd.e[2] * x + dx0) + dy0 * (pd.e[2] * y + dy0);
    if (!(ahead > 1e-3 * (dx0 * dx0 + dy0 * dy0))) return;
    const double t = (dx0 * y - dy0 * x) / ahead;
    const uint32_t key = angle_key(atan2(pd.u[0] * x + pd.u[1] * y + pd.u[2],
                                         -(pd.v[0] * x + pd.v[1] * y + pd.v[2])));
    if (t < tmin) {
      tmin = t;
      kmin = key;
    }
    if (t > tmax) {
      tmax = t;
      kmax = key;
    }
  }
  // from one extreme corner to the other, through the centre
  uint32_t lo = kmin, len = kmax - kmin;
  if (kc - kmin > len) {
    lo = kmax;
    len = kmin - kmax;
  }
  const uint64_t margin = (uint64_t)(len >> 5) + 65536u;
  const uint64_t wide = (uint64_t)len + 2u * margin;
  if (wide >= 0xF0000000ull) return;
  lo -= (uint32_t)margin;
  arc.arc_len = (uint32_t)wide;
  const uint32_t off = arc_side(arc.arc_len), near = arc_near(arc.arc_len);
  arc.cut = lo - off;
  while (!((arc.arc_len << arc.arc_shift) & 0x80000000u)) ++arc.arc_shift;
  // (a key beyond the arc is at most `off` keys away, which is at least 2^27;
  // all rounded down, whatever the divisions' last bits)
  arc.arc_mul = (uint32_t)(((1u << kCentreBits) - 2u * kSideCodes) * 0x1p32 /
                          (arc.arc_len << arc.arc_shift)) - 1u;
  arc.near_mul = (uint32_t)(kNearCodes * 0x1p32 / near) - 1u;
  arc.far_mul = (uint32_t)((kSideCodes - kNearCodes) * 0x1p32 / (off - near + 2u)) - 1u;
}

// Position code of a key (an angle minus the pair's cut); never decreases
// with the key.
__host__ __device__ inline uint32_t position_code(const KeyArc& arc, uint32_t key) {
  const uint32_t off = arc_side(arc.arc_len), near = arc_near(arc.arc_len);
  const uint32_t y = key - off;  // (past the arc's end below the arc)
  const bool below = key < off, inside = !below && y < arc.arc_len;
  const uint32_t d = below ? off - 1u - key : y - arc.arc_len;  // keys to the arc
  const bool far = d >= near;
  const uint32_t mul = inside ? arc.arc_mul : far ? arc.far_mul : arc.near_mul;
  const uint32_t x = inside ? y << arc.arc_shift : far ? d - near : d;
  const uint32_t c = (uint32_t)(((uint64_t)x * mul) >> 32), s = far ? kNearCodes + c : c;
  const uint32_t code = inside  ? kSideCodes + c
                        : below ? kSideCodes - 1u - s
                                : (1u << kCentreBits) - kSideCodes + s;
  return arc.arc_len == 0u ? key >> (32 - kCentreBits) : code;
}

struct SortTile {
  int64_t begin;  // global element index
  int32_t count;
  int32_t seg;
};

// A segment of the sort and its tiles.  Segments of several tiles have a row
// of digit counts per tile from hist_begin on; one tile counts for itself.
struct SortSeg {
  int64_t begin;
  int64_t count;
  int32_t tile_begin, tile_count;
  int32_t hist_begin;
  int32_t tile;  // the queries' segments: queries per stabbing tile
};

constexpr int kSortThreads = 1024;
constexpr int kSortTileMin = 1024, kSortTileMax = 32768;  // elements per sort tile
constexpr int kRadix = 1 << kRadixBits;
constexpr int kHistWords = kRadix / 2;  // a row of counts: two 16-bit counts per word

constexpr int kClassSlots = kNumClasses + 1;  // class_begin entries per pair

// Longest row sorted in LDS by the fill kernel; longer rows are rebuilt in
// ascending j order by a direct scan of the pair.
constexpr int kRowSortMax = 2048;

// Stabbing tiles: up to kTileQ consecutive angle-sorted queries of one pair share
// one window search per width class; the window's records are staged in LDS
// a round at a time (256, 512 or 1024 records, a tile shape chosen per index;
// kChunk by default).  Rows of up to kStage candidates are parked in a staging
// buffer by the tile kernel and sorted by the copy pass; longer rows are
// rebuilt by the fill kernel.
constexpr int kTileQ = 64;
constexpr int kStage = 128;
constexpr int kChunk = 512;

// Queries with equal upper kRadixBits bits of their codes form a group of the
// one-pass query sort.  What the window pass does with a segment's groups:
// sort around the boundaries of neighbouring tiles, where groups are small;
// sort its workgroups' queries, where groups exceed a tile or tiles hold fewer
// than kTileQ of them; and bring groups of more than two tiles into the order
// of their keys.
constexpr uint32_t kGroupsSmall = 0, kGroupsLocal = 1, kGroupsLarge = 2;
static_assert(kCentreBits >= kRadixBits, "a group's queries differ in the bits below");

// Per-tile record windows found by the window pass: up to two ranges of
// sorted positions per width class (the second one when the window wraps
// through angle 0), as start positions and a running prefix of lengths.
constexpr int kSlots = 2 * kNumClasses;
struct TileWindow {
  uint32_t slot_b[kSlots];
  uint32_t slot_pref[kSlots + 1];
};

// per-tile counters of the tile pass: records scanned, angle hits,
// brute-force queries, empty queries; BF16 fused selection: rows ranked on
// bounds, rows left uncertified, exact distances evaluated; one spare
constexpr int kTileCounts = 8;

struct StabTile {
  int64_t begin;  // first angle-sorted query position of the tile
  int32_t count;  // queries in the tile (<= kTileQ; 0: not needed)
  int32_t pair;
};

// One query of a stabbing tile as the window pass leaves it for the tile
// pass: the epipolar line (a, b, c), the query's index, flag and key (slots
// past the tile's count: empty, index 0).
struct TileQuery {
  double a, b, c;
  uint32_t i, flag, key, pad;
};

// The fewest queries per tile of a pair with m queries and n records, which
// say how many tiles it gets; how many queries they take is decided when the
// pair is queried (launch_tile_split).  A tile's window holds the records
// between its first and last query, n / m per query, beside those within the
// tolerance, and windows of more than 1024 records are left to slower passes;
// so a pair with many records per query may take fewer queries per tile, such
// that they hold up to 512.
__host__ __device__ inline int tile_queries(int64_t m, int64_t n) {
  return n <= 8 * m ? kTileQ : n <= 16 * m ? kTileQ / 2 : n <= 32 * m ? kTileQ / 4 : kTileQ / 8;
}

}  // namespace epm
