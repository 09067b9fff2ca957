// The C ABI of libbitrev: argument validation (before any HIP call), the
// plan (which path, tile width, grid), the tuning table, and the launches.
#include <errno.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "bitrev.h"
#include "bitrev_device.hpp"
#include "bitrev_launch.hpp"

namespace {

using namespace bitrev;

thread_local int g_last_hip_error = 0;

bitrev_status_t hip_fail(hipError_t e) {
  g_last_hip_error = (int)e;
  return BITREV_ERROR_HIP;
}

// ---------------------------------------------------------------------------
// Device properties (cached per device).
// ---------------------------------------------------------------------------
struct DeviceInfo {
  int cus = 256;                 // compute units
  size_t lds_per_block = 163840; // LDS bytes a workgroup may use
  int xcds = 8;                  // XCDs the dispatcher deals workgroups over
  char arch[32] = "gfx950";      // gcnArchName without its feature suffix
};

constexpr int kMaxDevices = 64;
std::mutex g_dev_mu;
bool g_dev_known[kMaxDevices];
DeviceInfo g_dev[kMaxDevices];

// The current device's properties; MI355X figures when `allow_default` and
// no device is present (plan queries on a host without a GPU).
bitrev_status_t device_info(DeviceInfo* out, bool allow_default, bool* present = nullptr) {
  int dev = 0;
  if (present) *present = false;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    if (allow_default) {
      (void)hipGetLastError();
      *out = DeviceInfo();
      return BITREV_SUCCESS;
    }
    return hip_fail(e != hipSuccess ? e : hipErrorInvalidDevice);
  }
  std::lock_guard<std::mutex> lock(g_dev_mu);
  if (!g_dev_known[dev]) {
    hipDeviceProp_t p;
    e = hipGetDeviceProperties(&p, dev);
    if (e != hipSuccess) return hip_fail(e);
    DeviceInfo d;
    d.cus = p.multiProcessorCount > 0 ? p.multiProcessorCount : 1;
    snprintf(d.arch, sizeof d.arch, "%.*s", (int)strcspn(p.gcnArchName, ":"), p.gcnArchName);
    d.lds_per_block = p.sharedMemPerBlock;
    // gfx950 has 32 compute units per XCD; a partitioned device shows fewer.
    int x = (d.cus + 16) / 32;
    if (strncmp(p.gcnArchName, "gfx942", 6) == 0) x = (d.cus + 19) / 38;
    if (x < 1) x = 1;
    if (const char* env = getenv("BITREV_XCDS")) {
      const int v = atoi(env);
      if (v >= 1 && v <= 64) x = v;
    }
    d.xcds = x;
    g_dev[dev] = d;
    g_dev_known[dev] = true;
  }
  *out = g_dev[dev];
  if (present) *present = true;
  return BITREV_SUCCESS;
}

// ---------------------------------------------------------------------------
// Tuning table: (mode, elem_size, log2n or -1) -> tile bits, workgroups per
// CU, order.  Loaded from a text file; the built-in defaults apply otherwise.
// ---------------------------------------------------------------------------
struct TuneEntry {
  int tile_bits = 0;
  int wg_per_cu = 0;
  int order = 0;
  int variant = 0;
  int xcd_remap = 0;
  int cache_hints = 0;
};

std::mutex g_tune_mu;
std::map<std::tuple<int, int, int>, TuneEntry> g_tune;
std::once_flag g_tune_env_once;

const char kTuningFormat[] =
    "libbitrev tuning v3: one entry per line, '#' starts a comment.  Plan rows: arch(* = any, "
    "else a gcnArchName such as gfx950) cus(0 = any) kind(inplace|outofplace|batched|batched_oop|"
    "dit_inplace|dit_outofplace|digit_inplace|digit_outofplace) elem_size(0 = any) "
    "digit_bits(0 = any) tile_match(tile width in use, 0 = any) class_min class_max(footprint "
    "class floor(log2 bytes), -1 = open) tile_bits wg_per_cu order variant xcd_remap cache_hints "
    "(0 = not set here; codes as in bitrev_config_t), consulted before the built-in table; per "
    "field the first matching row that sets it wins.  Exact entries (v2): mode"
    "(inplace|outofplace|batched) elem_size log2n(-1 = any) tile_bits wg_per_cu order variant "
    "xcd_remap [cache_hints], which override the table for that size";

int mode_from_name(const char* s) {
  if (strcmp(s, "inplace") == 0) return 0;
  if (strcmp(s, "outofplace") == 0) return 1;
  if (strcmp(s, "batched") == 0) return 2;
  return -1;
}

bool valid_elem_size(size_t s) { return s == 1 || s == 2 || s == 4 || s == 8 || s == 16; }

// ---------------------------------------------------------------------------
// Plan table: the tile width, kernel variant, work order, XCD mapping, cache
// hints and workgroups per CU of each kind of launch, by device
// (gcnArchName and compute units), element size, digit width, tile width in
// use and footprint class.  The built-in rows are data (plans_gfx950.inc,
// regenerated by the autotuner); rows of the same form in a tuning file are
// consulted before them.
// ---------------------------------------------------------------------------
enum PlanKind {
  kKindInplace = 0,
  kKindOutofplace,
  kKindBatched,
  kKindBatchedOop,
  kKindDitInplace,
  kKindDitOutofplace,
  kKindDigitInplace,
  kKindDigitOutofplace,
  kKindCount
};
const char* const kKindNames[kKindCount] = {"inplace",        "outofplace",  "batched",
                                            "batched_oop",    "dit_inplace", "dit_outofplace",
                                            "digit_inplace",  "digit_outofplace"};
// The kind whose rows fill the fields a kind's own rows leave unset.
const int kKindParent[kKindCount] = {-1, -1, -1, kKindBatched, kKindInplace, kKindOutofplace,
                                     kKindInplace, kKindOutofplace};

struct PlanFields {
  int b = 0, wg = 0, order = 0, variant = 0, xcd = 0, hints = 0;
};

struct PlanRow {
  char arch[32];  // "*" or a gcnArchName without its feature suffix
  int cus;        // compute units, 0 = any
  int kind;
  int s, d, bm;   // element size, digit bits, tile width in use; 0 = any
  int cmin, cmax; // footprint class range, -1 = open
  PlanFields f;
};

const char kBuiltinPlans[] =
#include "plans_gfx950.inc"
    ;

// floor(log2(bytes)): the footprint class of a launch.
int footprint_class(uint64_t bytes) {
  int c = -1;
  while (bytes) {
    bytes >>= 1;
    ++c;
  }
  return c;
}

int kind_from_name(const char* s) {
  for (int k = 0; k < kKindCount; ++k)
    if (strcmp(s, kKindNames[k]) == 0) return k;
  return -1;
}

// One table row from a line: 0 = parsed, 1 = not a table row, -1 = malformed.
int parse_plan_row(const char* line, PlanRow* r) {
  char arch[32], kind[32], extra[8];
  int v[12];
  const int got = sscanf(line, "%31s %d %31s %d %d %d %d %d %d %d %d %d %d %d %7s", arch, &v[0],
                         kind, &v[1], &v[2], &v[3], &v[4], &v[5], &v[6], &v[7], &v[8], &v[9],
                         &v[10], &v[11], extra);
  if (got <= 0) return 1;
  if (!(strcmp(arch, "*") == 0 || strncmp(arch, "gfx", 3) == 0)) return 1;
  if (got != 14) return -1;
  const int kd = kind_from_name(kind);
  const int s = v[1];
  if (kd < 0 || v[0] < 0 || v[0] > 4096 || !(s == 0 || valid_elem_size((size_t)s)) || v[2] < 0 ||
      v[2] > 3 || v[3] < 0 || v[3] > kMaxTileBits || v[4] < -1 || v[4] > 62 || v[5] < -1 ||
      v[5] > 62 || v[6] < 0 || v[6] > kMaxTileBits || v[7] < 0 || v[7] > 1024 || v[8] < 0 ||
      v[8] > 3 || v[9] < 0 || v[9] > 3 || v[10] < 0 || v[10] > 2 || v[11] < 0 || v[11] > 4)
    return -1;
  snprintf(r->arch, sizeof r->arch, "%s", arch);
  r->cus = v[0];
  r->kind = kd;
  r->s = s;
  r->d = v[2];
  r->bm = v[3];
  r->cmin = v[4];
  r->cmax = v[5];
  r->f.b = v[6];
  r->f.wg = v[7];
  r->f.order = v[8];
  r->f.variant = v[9];
  r->f.xcd = v[10];
  r->f.hints = v[11];
  return 0;
}

std::vector<PlanRow> g_builtin_rows[kKindCount];
std::vector<PlanRow> g_user_rows;  // guarded by g_tune_mu
std::once_flag g_builtin_once;

// The built-in rows of one kind: a call looks at these and its parents' only
// (the whole table in every call cost 0.1 us of a small array's 3.6).
const std::vector<PlanRow>& builtin_rows(int kind) {
  std::call_once(g_builtin_once, [] {
    const char* p = kBuiltinPlans;
    char line[512];
    while (*p) {
      size_t n = strcspn(p, "\n");
      const size_t len = n < sizeof line - 1 ? n : sizeof line - 1;
      memcpy(line, p, len);
      line[len] = '\0';
      char* hash = strchr(line, '#');
      if (hash) *hash = '\0';
      PlanRow r;
      if (parse_plan_row(line, &r) == 0) g_builtin_rows[r.kind].push_back(r);
      p += n + (p[n] == '\n');
    }
  });
  return g_builtin_rows[kind];
}

bool arch_matches(const char* row, const char* dev) {
  if (strcmp(row, "*") == 0) return true;
  const size_t n = strlen(row);
  return strncmp(row, dev, n) == 0 && (dev[n] == '\0' || dev[n] == ':');
}

void merge_rows(const std::vector<PlanRow>& rows, int kind, int s, int d, int bm, int c,
                const DeviceInfo& dev, PlanFields* f) {
  for (const PlanRow& r : rows) {
    if (r.kind != kind || (r.s && r.s != s) || (r.d && r.d != d) || (r.bm && r.bm != bm) ||
        (r.cmin >= 0 && c < r.cmin) || (r.cmax >= 0 && c > r.cmax) ||
        (r.cus && r.cus != dev.cus) || !arch_matches(r.arch, dev.arch))
      continue;
    if (!f->b) f->b = r.f.b;
    if (!f->wg) f->wg = r.f.wg;
    if (!f->order) f->order = r.f.order;
    if (!f->variant) f->variant = r.f.variant;
    if (!f->xcd) f->xcd = r.f.xcd;
    if (!f->hints) f->hints = r.f.hints;
  }
}


void load_env_tuning();

// Whether a tuning file's plan rows, the kind's own or those it falls back to,
// decide anything for this launch.
bool user_rows_apply(int kind, int s, uint64_t footprint, const DeviceInfo& dev) {
  load_env_tuning();
  std::lock_guard<std::mutex> lock(g_tune_mu);
  if (g_user_rows.empty()) return false;
  const int c = footprint_class(footprint);
  for (int k = kind; k >= 0; k = kKindParent[k])
    for (const PlanRow& r : g_user_rows)  // whatever digit or tile width a row is for
      if (r.kind == k && (!r.s || r.s == s) && (r.cmin < 0 || c >= r.cmin) &&
          (r.cmax < 0 || c <= r.cmax) && (!r.cus || r.cus == dev.cus) &&
          arch_matches(r.arch, dev.arch))
        return true;
  return false;
}

bitrev_status_t load_tuning_file(const char* path) {
  if (path == NULL) {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    g_tune.clear();
    g_user_rows.clear();
    return BITREV_SUCCESS;
  }
  FILE* f = fopen(path, "r");
  if (!f) return BITREV_ERROR_INVALID_VALUE;
  std::map<std::tuple<int, int, int>, TuneEntry> table;
  std::vector<PlanRow> rows;
  char line[512];
  bool ok = true;
  while (fgets(line, sizeof line, f)) {
    char* hash = strchr(line, '#');
    if (hash) *hash = '\0';
    PlanRow row;
    const int pr = parse_plan_row(line, &row);
    if (pr == 0) {
      rows.push_back(row);
      continue;
    }
    if (pr < 0) {
      ok = false;
      break;
    }
    char mode[32];
    int s, k, b, wg, order, variant, xcd, hints = 0;
    char extra[8];
    const int got = sscanf(line, "%31s %d %d %d %d %d %d %d %d %7s", mode, &s, &k, &b, &wg,
                           &order, &variant, &xcd, &hints, extra);
    if (got <= 0) continue;  // blank or comment-only line
    const int md = got >= 8 ? mode_from_name(mode) : -1;
    if ((got != 8 && got != 9) || md < 0 || !valid_elem_size((size_t)s) || k < -1 ||
        k > BITREV_MAX_LOG2N || b < 0 || b > kMaxTileBits || wg < 0 || wg > 1024 || order < 0 ||
        order > 3 || variant < 0 || variant > 3 || xcd < 0 || xcd > 2 || hints < 0 || hints > 4) {
      ok = false;
      break;
    }
    TuneEntry t;
    t.tile_bits = b;
    t.wg_per_cu = wg;
    t.order = order;
    t.variant = variant;
    t.xcd_remap = xcd;
    t.cache_hints = hints;
    table[std::make_tuple(md, s, k)] = t;
  }
  fclose(f);
  if (!ok) return BITREV_ERROR_INVALID_VALUE;
  std::lock_guard<std::mutex> lock(g_tune_mu);
  g_tune.swap(table);
  g_user_rows.swap(rows);
  return BITREV_SUCCESS;
}

void load_env_tuning() {
  std::call_once(g_tune_env_once, [] {
    const char* p = getenv("BITREV_TUNING_FILE");
    if (p && *p) (void)load_tuning_file(p);
  });
}

TuneEntry tune_lookup(int mode, int s, int k) {
  load_env_tuning();
  std::lock_guard<std::mutex> lock(g_tune_mu);
  auto it = g_tune.find(std::make_tuple(mode, s, k));
  if (it == g_tune.end()) it = g_tune.find(std::make_tuple(mode, s, -1));
  return it == g_tune.end() ? TuneEntry() : it->second;
}

// The table's plan for a launch of `kind` covering `footprint` bytes; bm is
// the tile width in use (0 while it is being chosen), d the digit width.
// Fields no row sets stay 0.  `f` starts with what is already decided; *file,
// where given, gets the width, count, order and XCD mapping that a tuning file's
// rows set.
PlanFields table_plan(int kind, int s, int d, int bm, uint64_t footprint, const DeviceInfo& dev,
                      PlanFields f = PlanFields(), PlanFields* file = nullptr) {
  load_env_tuning();
  const int c = footprint_class(footprint);
  std::lock_guard<std::mutex> lock(g_tune_mu);
  for (int k = kind; k >= 0; k = kKindParent[k]) {
    const PlanFields before = f;
    merge_rows(g_user_rows, k, s, d, bm, c, dev, &f);
    if (file) {
      if (!before.b) file->b = f.b;
      if (!before.wg) file->wg = f.wg;
      if (!before.xcd) file->xcd = f.xcd;
      if (!before.order) file->order = f.order;
    }
    merge_rows(builtin_rows(k), k, s, d, bm, c, dev, &f);
  }
  return f;
}

// What the bytes and rows of a launch on MI355X decide before the table, whose
// rows know only powers of two and were measured on single arrays (its choices
// stay wherever nothing is set here).  Kernel us, three states in turn, before
// -> now.
//  - Several rows, in dispatch order, which walks the rows one after the
//    other where contiguous XCD ranges keep eight distant rows in flight:
//    complex128 rows of 1 to 8 MiB from 64 MiB on (68 MiB of 2^17 22.8 ->
//    21.8, 124 MiB 46.2 -> 41.4; level at 204 MiB of 2^18, 67.5), float32
//    rows of 256 KiB to 4 MiB from 256 MiB on at b = 7 (330 MiB of 2^17 128.6
//    -> 117.2, 488 MiB of 2^16 179.4 -> 172.7), fused levels up to five on
//    complex128 rows of 1 to 8 MiB from 128 MiB on (152 MiB of 2^17 57.0 ->
//    51.7, 216 MiB of 2^19 82.6 -> 75.0).  For complex64 the same gained 7%
//    or lost 6% with the buffers' places, and is left.
//  - Several rows of 40 to 64 MiB out of place by the one-item kernels: their
//    write-through stores, where the table's pipelined kernels at 32 MiB keep
//    plain ones (44 MiB of 2^16: complex64 16.8 -> 15.9, float32 17.1 -> 16.0,
//    uint8 17.8 -> 16.5).  In place the wide pipelined tiles stay where a single
//    array takes narrower ones, which lose there (float32 40 MiB of 2^17 13.2,
//    narrower 13.7; complex64 31 MiB 10.6, 10.7; complex128 19.5 MiB of 2^14
//    7.8, 8.4, 56 MiB 18.1, 18.5).
//  - Off the 16-byte grid, and rows at a padded pitch, keep the wide pipelined
//    tiles to 64 MiB (out of place to 32), and the table beyond: single
//    elements want them (int16 2^14 at n + 1, 6.7 MiB 5.0, narrower 6.0), and
//    the narrower ones gain most where a pitch of a power of two maps rows to
//    the same channels (complex128 2^16 at n + 4, 6 MiB 4.1, narrower 4.9).
//  - Fused levels from 12 to 16 MiB on rectangular tiles at b = 6, smaller
//    workgroups (complex64 16 MiB, five levels 8.0 -> 6.5; complex128 2^20,
//    four 8.3 -> 6.9), complex64 with two levels and more to 18 MiB and with
//    five from 6 MiB (10 MiB of 2^14 6.2 -> 5.4).  Outside those lines they
//    lose (17 MiB of complex128 2^14 7.5 -> 8.4, 4 MiB 3.5 -> 4.2; one
//    complex64 level at 8 MiB 4.1 -> 4.4).
//  - Six complex64 levels at 24 to 40 MiB with plain accesses, whose stores the
//    L2s still hold there (2^22 15.0 -> 12.4, from cold caches 18.3 -> 18.2).
//    Fewer gain 1 to 8% so and lose up to 14% from cold caches (one level 15.5
//    -> 18.0): left to the table.
//  - Up to four complex128 levels in place at 4 to 64 MiB, where the table's
//    in-place rows give two tiles at b = 4: the register-staged pair at b = 5
//    stays for rows of 2^10 and 2^11, where b = 5 is one tile or two a row
//    (2^10 15 MiB, four levels 6.8 -> 5.6, 2^11 12 MiB 6.0 -> 5.0), for two
//    levels (2^12 15 MiB 6.3 -> 5.7, 2^19 4.7 -> 4.4; against it 2^13 23 MiB
//    8.2 -> 9.7, 2^20 7.0 -> 7.6), and for rows of 2^14 from 16 MiB (30 MiB,
//    four levels 11.2 -> 10.5).  Elsewhere it loses (one level: 2^13 23 MiB
//    8.2 -> 10.2, 2^16 15 MiB 5.8 -> 7.3, one array of 2^21 12.1 -> 13.8) or
//    is level from cold caches (2^12 15 MiB, four levels 6.7 -> 6.1, 10.2).
// `width`: the tile width that the caller or an exact tuning entry sets, if any.
// The rule's fields were measured together: at another width than its own the
// table decides.
PlanFields bytes_rule(int kind, int s, int k, uint64_t rows, uint64_t footprint, int stages,
                      bool linear, int width, const DeviceInfo& dev) {
  PlanFields f;
  if (dev.cus != 256 || !arch_matches("gfx950", dev.arch)) return f;
  auto set = [&f](int b, int variant, int order, int xcd, int hints) {
    f.b = b;
    f.variant = variant;
    f.order = order;
    f.xcd = xcd;
    f.hints = hints;
  };
  const uint64_t mib = 1ull << 20, row = (uint64_t)s << k;
  const bool many = rows >= 2 && row >= mib / 4 && row <= 8 * mib;
  const int c = footprint_class(footprint);
  if (kind == kKindDitInplace) {
    if (s == 16 && stages <= 4 && c >= 22 && c <= 25 && k >= 10 &&
        (k <= 11 || stages == 2 || (k == 14 && c >= 24)))
      set(5, 3, 2, 2, 4);
  } else if (stages == 0 && !linear) {
    if (kind == kKindInplace && c <= 25 && s != 1) set(s == 2 ? 7 : s == 4 ? 6 : 5, 2, 1, 2, 1);
    if (kind == kKindOutofplace && s == 2 && c <= 24) set(7, 2, 2, 2, 1);
    if (kind == kKindOutofplace && s == 16 && c <= 24) set(5, 2, 2, 2, 1);
  } else if (kind == kKindInplace) {
    if (rows >= 2 && ((s == 4 && c == 25) || (s == 8 && c == 24) ||
                      (s == 16 && footprint > 18 * mib && c <= 25)))
      set(s == 4 ? 6 : 5, 2, 1, 2, 1);
  } else if (kind == kKindOutofplace) {
    if (rows >= 2 && footprint >= 40 * mib && footprint < 64 * mib) {
      if (s <= 4) set(s == 1 ? 7 : 6, 1, 1, 1, 4);
      if (s >= 8) set(5, 1, 2, 2, 4);
    }
    if (many && s == 16 && row >= mib && footprint >= 64 * mib) set(5, 1, 3, 2, 4);
    if (many && s == 4 && row <= 4 * mib && footprint >= 256 * mib) set(7, 1, 1, 2, 4);
  } else if (many && s == 16 && row >= mib && stages <= 5 && footprint >= 128 * mib) {
    set(5, 1, 3, 2, 4);
  } else if (footprint <= 18 * mib) {
    const bool large = footprint >= 12 * mib, one = stages == 1;
    if (s == 8 && (k >= 12 || (k == 11 && large)) &&
        (stages == 5 || (large && k >= 12 && (!one || footprint <= 16 * mib))) &&
        footprint >= 6 * mib)
      set(6, 2, 3, 2, 4);
    if (s == 16 && k >= 12 && large && footprint <= 16 * mib) set(6, 2, 1, 1, 4);
  } else if (footprint >= 24 * mib && footprint <= 40 * mib && s == 8 && stages == 6) {
    set(6, 2, 1, rows >= 2 ? 2 : 1, 1);
  }
  if (!f.b || (width && width != f.b) || user_rows_apply(kind, s, footprint, dev))
    return PlanFields();
  return f;
}

// ---------------------------------------------------------------------------
// Plans.
// ---------------------------------------------------------------------------
enum { kModeInplace = 0, kModeOutofplace = 1, kModeBatched = 2 };

int occupancy_of(int s, int b, bool vec, bool inplace, bool pipelined) {
  switch (s) {
    case 1: return tile_occupancy_s1(b, vec, inplace, pipelined);
    case 2: return tile_occupancy_s2(b, vec, inplace, pipelined);
    case 4: return tile_occupancy_s4(b, vec, inplace, pipelined);
    case 8: return tile_occupancy_s8(b, vec, inplace, pipelined);
    default: return tile_occupancy_s16(b, vec, inplace, pipelined);
  }
}

int rs_threads_of(int s, int b, bool vec) {
  switch (s) {
    case 1: return tile_rs_threads_s1(b, vec);
    case 2: return tile_rs_threads_s2(b, vec);
    case 4: return tile_rs_threads_s4(b, vec);
    case 8: return tile_rs_threads_s8(b, vec);
    default: return tile_rs_threads_s16(b, vec);
  }
}

int threads_of(int s, int b, bool vec) {
  switch (s) {
    case 1: return tile_threads_s1(b, vec);
    case 2: return tile_threads_s2(b, vec);
    case 4: return tile_threads_s4(b, vec);
    case 8: return tile_threads_s8(b, vec);
    default: return tile_threads_s16(b, vec);
  }
}

#ifndef BITREV_GROUP_J
#define BITREV_GROUP_J 3
#endif

// The kernels' order code (bit 0 balanced, bits 1.. group width) for a
// plan's order: 1 natural, 2 balanced, 3 grouped.
int order_code(int order) {
  // grouped: groups in pair_at's natural order (measured 1% ahead of the
  // balanced group order for complex64 2^24-2^26); the kernels clamp j
  if (order == 3) return BITREV_GROUP_J << 1;
  return order == 2 ? 1 : 0;
}

bool valid_config(const bitrev_config_t* c) {
  if (!c) return true;
  return c->tile_bits >= 0 && c->tile_bits <= kMaxTileBits && c->grid_blocks >= 0 &&
         c->order >= 0 && c->order <= 3 && c->variant >= 0 && c->variant <= 3 &&
         c->xcd_remap >= 0 && c->xcd_remap <= 2 && c->cache_hints >= 0 && c->cache_hints <= 4;
}

bool config_set(const bitrev_config_t* c) {
  return c && (c->tile_bits || c->grid_blocks || c->order || c->variant || c->xcd_remap ||
               c->cache_hints);
}

uint32_t round_up(uint64_t v, uint32_t to) {
  const uint64_t r = (v + to - 1) / to * to;
  return (uint32_t)(r > 0xFFFFFFFFull ? 0xFFFFFFFFull / to * to : r);
}

// Grid for `items` work items: one workgroup per item up to 2^20
// workgroups (then a grid-stride loop), a multiple of the XCD count.
uint32_t default_grid(uint64_t items, const DeviceInfo& d) {
  const uint64_t cap = 1ull << 20;
  return round_up(items < cap ? items : cap, (uint32_t)d.xcds);
}

int resident_per_cu(int threads, size_t lds);

struct Plan {
  int path = BITREV_PATH_NONE;
  int b = 0;
  int m = 0;
  int threads = 0;
  uint32_t grid = 0;
  int order = 2;
  int variant = 1;
  int xcd_remap = 1;
  int hints = kHintPlain;  // CacheHint of the one-item 16-byte tile kernels
  bool vec = true;
  uint64_t items_per_seg = 0;
  uint64_t total = 0;
  size_t lds = 0;
  bool persistent = false; // batched: the caller or a tuning file set the grid
  bool forced_width = false;  // batched: ... set the tile width
  bool forced_xcd = false;    // batched: ... set the XCD mapping
  bool forced_order = false;  // batched: ... set the order
  int chunk_log2 = 0;      // whole-row path: bytes per workgroup
  bool gather = false;
};

// The whole-row path (bitrev_rows.hpp) for `rows` >= 2 arrays of 2^k elements
// whose accesses stay 4-byte aligned: true and *p filled where it is taken,
// unless the tile plan is one linear tile per row (which plan_plain asks).  The
// lines, each with both sides measured (kernel time, three matrices in turn):
//  - rows of at most 16 KiB, from 8 KiB on only bytes or 64 MiB (complex64
//    2^11 128 MiB 43.1 -> 41.4, 36 MiB 12.2 against 12.6; rows of 32 KiB lose
//    1-8%); off the 16-byte grid, where the tile kernels move single elements,
//    rows of up to 64 KiB (float32 2^14 at a pitch of n + 2, 32 MiB: 15.6 ->
//    11.4 us);
//  - where the tile plan has one tile per row (k = 2b), its accesses are
//    linear too: it stays from 2 KiB rows (complex64 2^8 33 MiB out of place:
//    10.8 against 11.4, int16 2^10 12 MiB 5.8 against 6.2), of bytes from 1 KiB
//    rows and, at 64 MiB and more, from 1 KiB rows of b >= 4 (float32 2^8: 64
//    MiB 20.9 -> 19.8, but 96 MiB 31.2 against 32.9; 12.2 -> 10.5 at 32 MiB);
//  - the gathers of rows of 16 bytes and more from 512 KiB on, of shorter
//    ones from 32 KiB: their four vectors per thread are a serial chain that
//    costs 1 us from cold caches (uint8 2^6 0.3 MiB 6.1 against 7.1, at 2.5
//    MiB 8.6 -> 7.8; 2^3 0.3 MiB 9.5 -> 7.2).
// Write-through stores with streaming loads from 64 MiB (complex64 2^10 64
// MiB 20.1 -> 19.6 us, 128 MiB 47.5 -> 42.4; at 32 MiB out of place 10.5
// against 10.8) and for the gathers of 1- and 2-byte elements from 32 MiB
// (int16 2^4 in place 12.2 -> 10.8); plain stores where rows end inside a
// 64-byte line, which two workgroups then write (float64 2^9 at n + 2, 256
// MiB: 95 against 107 us).
bool plan_rows(int k, int s, uint64_t rows, size_t align, bool contiguous, bool whole_lines,
               uint64_t footprint, Plan* p) {
  const uint64_t rb = (uint64_t)s << k;
  const int c = s == 16 ? 0 : s == 8 ? 1 : s == 4 ? 2 : s == 2 ? 3 : 4;
  if (rows < 2 || k > 16 || align < 4 || (rb < 16 && !contiguous)) return false;
  const bool aligned = align == 16;
  if (rb > 65536u) return false;
  if (aligned && rb >= 8192 && (rb > 16384 || (s > 1 && footprint < (64ull << 20)))) return false;
  const bool gather = k < 2 * c;
  if (gather && footprint < ((rb >= 16 ? 512u : 32u) << 10)) return false;
  int lb;
  if (gather) {
    lb = s > 1 ? 14 : 12;
  } else {
    lb = s == 16 ? 13 : 14;
    while ((1ull << lb) < rb) ++lb;
  }
  const uint64_t runs = rb < 16 ? (rows * rb) / 16 : rows;
  const uint64_t per = rb < 16 ? (1u << lb) / 16 : (1ull << lb) / rb;
  const uint64_t chunks = runs ? (runs + per - 1) / per : 1;
  const int hints = (align == 16 && whole_lines &&
                     footprint >= ((gather && s <= 2 ? 32ull : 64ull) << 20))
                        ? kHintStreamWriteThrough
                        : kHintPlain;
  *p = Plan();
  p->path = BITREV_PATH_ROWS;
  p->order = 1;
  p->xcd_remap = 2;
  p->variant = 0;
  p->threads = rows_block_threads(s, lb, gather);
  p->total = chunks;
  p->grid = (uint32_t)(chunks < (1u << 20) ? chunks : (1u << 20));
  p->hints = hints;
  p->lds = (size_t)1 << lb;
  p->chunk_log2 = lb;
  p->gather = gather;
  return true;
}

// Plan for a plain call (mode 0 or 1) on `rows` arrays of 2^k elements by the
// tile and wavefront kernels.
// align: the largest power of two (<= 16) dividing both data pointers.
bitrev_status_t plan_tiles(int mode, int k, int s, int64_t rows, const bitrev_config_t* cfg,
                           size_t align, bool contiguous, const DeviceInfo& d, bool have_device,
                           Plan* p) {
  *p = Plan();
  if (rows == 0 || (mode == kModeInplace && k <= 1)) return BITREV_SUCCESS;
  const int forced_b = cfg ? cfg->tile_bits : 0;
  const TuneEntry te = tune_lookup(mode, s, k);
  // the size class is the launch's whole footprint: 256 rows of 2^16 float32
  // (64 MiB) run 15% faster on the 64 MiB plan than on the plan of one
  // 256 KiB row
  const uint64_t row_bytes = ((uint64_t)s) << k;
  const uint64_t rows_u = rows > 0 ? (uint64_t)rows : 1u;
  const uint64_t footprint = row_bytes > UINT64_MAX / rows_u ? UINT64_MAX : row_bytes * rows_u;
  const int kind = mode == kModeInplace ? kKindInplace : kKindOutofplace;
  const PlanFields tp = table_plan(kind, s, 0, 0, footprint, d,
                                   bytes_rule(kind, s, k, rows_u, footprint, 0,
                                              contiguous && align == 16,
                                              forced_b ? forced_b : te.tile_bits, d));
  p->order = (cfg && cfg->order) ? cfg->order : (te.order ? te.order : (tp.order ? tp.order : 2));
  p->xcd_remap = (cfg && cfg->xcd_remap) ? cfg->xcd_remap
                                         : (te.xcd_remap ? te.xcd_remap : (tp.xcd ? tp.xcd : 1));
  if (forced_b == 0 && k <= 6) {
    p->path = BITREV_PATH_WAVE;
    p->threads = 256;
    const uint64_t wg = ((uint64_t)rows + 3) / 4;
    p->grid = (uint32_t)(wg < 65536 ? wg : 65536);
    if (cfg && cfg->grid_blocks > 0) p->grid = (uint32_t)cfg->grid_blocks;
    p->total = (uint64_t)rows;
    return BITREV_SUCCESS;
  }
  p->variant = (cfg && cfg->variant) ? cfg->variant
                                     : (te.variant ? te.variant : (tp.variant ? tp.variant : 1));
  if (p->variant == 3 && mode != kModeInplace) p->variant = 1;  // register staging is in place only
  // LDS tiles per workgroup: a pair in place (one when register-staged)
  const int inplace_tiles = (mode == kModeInplace && p->variant != 3) ? 2 : 1;
  int b;
  if (forced_b > 0) {
    b = forced_b;
    if (2 * b > k || b > max_tile_bits(s) ||
        tile_lds_bytes_for(s, b, inplace_tiles) > d.lds_per_block)
      return BITREV_ERROR_NOT_SUPPORTED;
  } else {
    b = te.tile_bits ? te.tile_bits : (tp.b ? tp.b : max_tile_bits(s));
    if (b > max_tile_bits(s)) b = max_tile_bits(s);
    if (2 * b > k) b = k / 2;
    while (b > 0 && tile_lds_bytes_for(s, b, inplace_tiles) > d.lds_per_block) --b;
  }
  const int m = k - 2 * b;
  if (m > 32) return BITREV_ERROR_NOT_SUPPORTED;
  const size_t vb = ((size_t)s << b) < 16 ? ((size_t)s << b) : 16;
  p->vec = (align % vb) == 0;
  p->path = BITREV_PATH_TILE;
  p->b = b;
  p->m = m;
  p->items_per_seg = (mode == kModeInplace) ? pair_count(m) : (1ull << m);
  if ((uint64_t)rows > (1ull << 62) / p->items_per_seg) return BITREV_ERROR_NOT_SUPPORTED;
  p->total = p->items_per_seg * (uint64_t)rows;
  p->threads = p->variant == 3 ? rs_threads_of(s, b, p->vec) : threads_of(s, b, p->vec);
  p->lds = tile_lds_bytes_for(s, b, inplace_tiles);
  p->hints = (cfg && cfg->cache_hints)
                 ? cfg->cache_hints - 1
                 : (te.cache_hints ? te.cache_hints - 1 : (tp.hints ? tp.hints - 1 : kHintPlain));
  if (cfg && cfg->grid_blocks > 0) {
    p->grid = round_up((uint64_t)cfg->grid_blocks, (uint32_t)d.xcds);
  } else if (te.wg_per_cu > 0) {
    p->grid = round_up((uint64_t)te.wg_per_cu * d.cus, (uint32_t)d.xcds);
  } else if (p->variant == 2) {
    // persistent: the workgroups that are resident at once
    int occ = have_device ? occupancy_of(s, b, p->vec, mode == kModeInplace, true) : 0;
    if (occ <= 0) occ = resident_per_cu(p->threads, p->lds);
    const uint64_t g = (uint64_t)occ * d.cus;
    p->grid = round_up(g < p->total ? g : p->total, (uint32_t)d.xcds);
  } else {
    p->grid = default_grid(p->total, d);
  }
  return BITREV_SUCCESS;
}

// Plan for a plain call: whole rows where that path is the better one and
// neither the caller's configuration nor a tuning file decides.  The pitches
// are in elements between consecutive arrays.
bitrev_status_t plan_plain(int mode, int k, int s, int64_t rows, uint64_t src_pitch,
                           uint64_t dst_pitch, const bitrev_config_t* cfg, size_t align,
                           const DeviceInfo& d, bool have_device, Plan* p) {
  const uint64_t n = 1ull << k;
  const bool contiguous = rows < 2 || (src_pitch == n && dst_pitch == n);
  const auto tiles = [&] {
    return plan_tiles(mode, k, s, rows, cfg, align, contiguous, d, have_device, p);
  };
  if (rows < 2 || k > 16 || (mode == kModeInplace && k <= 1) || config_set(cfg) ||
      (uint64_t)rows > (1ull << 62) >> k)
    return tiles();
  // arithmetic before the tuning tables' locks and lookups, which a call that
  // stays with the tiles makes once more
  const uint64_t footprint = (n * (uint64_t)s) * (uint64_t)rows;
  const bool whole_lines = contiguous || ((src_pitch * s) % 64 == 0 && (dst_pitch * s) % 64 == 0);
  Plan whole;
  if (!plan_rows(k, s, (uint64_t)rows, align, contiguous, whole_lines, footprint, &whole))
    return tiles();
  // the tile plan is made only where it may be one linear tile per row
  const uint64_t rb = n * (uint64_t)s;
  if (align == 16 && k >= 8 && k % 2 == 0 &&
      (rb >= 2048 || (rb == 1024 && (s == 1 || footprint >= (64ull << 20))))) {
    const bitrev_status_t st = tiles();
    if (st != BITREV_SUCCESS || (p->path == BITREV_PATH_TILE && p->m == 0 && p->vec && p->b >= 4))
      return st;
  }
  const TuneEntry te = tune_lookup(mode, s, k);
  if (te.tile_bits || te.wg_per_cu || te.order || te.variant || te.xcd_remap || te.cache_hints ||
      user_rows_apply(mode == kModeInplace ? kKindInplace : kKindOutofplace, s, footprint, d))
    return tiles();
  *p = whole;
  return BITREV_SUCCESS;
}

// Workgroups of the batched kernel that fit on one CU at once: limited by
// LDS (160 KiB per CU) and by 32 wavefronts per CU.
int resident_per_cu(int threads, size_t lds) {
  const int by_waves = 32 / ((threads + 63) / 64);
  const int by_lds = lds ? (int)(163840 / lds) : by_waves;
  const int r = by_waves < by_lds ? by_waves : by_lds;
  return r < 1 ? 1 : r;
}

int batched_occupancy_of(int s, int b, bool oop) {
  switch (s) {
    case 1: return batched_occupancy_s1(b, oop);
    case 2: return batched_occupancy_s2(b, oop);
    case 4: return batched_occupancy_s4(b, oop);
    case 8: return batched_occupancy_s8(b, oop);
    default: return batched_occupancy_s16(b, oop);
  }
}

bitrev_status_t plan_batched(int s, const bitrev_config_t* cfg, const DeviceInfo& d,
                             bool have_device, bool oop, Plan* p) {
  *p = Plan();
  const TuneEntry te = tune_lookup(kModeBatched, s, -1);
  const int kind = oop ? kKindBatchedOop : kKindBatched;
  PlanFields file;
  const PlanFields t1 = table_plan(kind, s, 0, 0, 0, d, PlanFields(), &file);
  p->forced_width = (cfg && cfg->tile_bits) || te.tile_bits || file.b;
  int b = (cfg && cfg->tile_bits) ? cfg->tile_bits
                                  : (te.tile_bits ? te.tile_bits : (t1.b ? t1.b : max_tile_bits(s)));
  if (!(cfg && cfg->tile_bits) && b > max_tile_bits(s)) b = max_tile_bits(s);
  p->lds = tile_lds_bytes_for(s, b, oop ? 1 : 2);
  if (b < kMinBatchedTileBits || b > max_tile_bits(s) || p->lds > d.lds_per_block)
    return BITREV_ERROR_NOT_SUPPORTED;
  p->path = BITREV_PATH_BATCHED;
  p->b = b;
  // order, XCD mapping and workgroups per CU for the width in use (the
  // table's per-CU counts belong to the widths they were measured at)
  const PlanFields tp = table_plan(kind, s, 0, b, 0, d, PlanFields(), &file);
  p->order = (cfg && cfg->order) ? cfg->order : (te.order ? te.order : (tp.order ? tp.order : 2));
  p->xcd_remap = (cfg && cfg->xcd_remap) ? cfg->xcd_remap
                                         : (te.xcd_remap ? te.xcd_remap : (tp.xcd ? tp.xcd : 1));
  // (a file that leaves the count open leaves the library its own grid: one
  // tile per workgroup, which the tuner timed such a row with)
  p->persistent = (cfg && cfg->grid_blocks > 0) || te.wg_per_cu > 0 || file.wg > 0;
  p->forced_xcd = (cfg && cfg->xcd_remap) || te.xcd_remap || file.xcd;
  p->forced_order = (cfg && cfg->order) || te.order || file.order;
  p->threads = threads_of(s, b, true);
  int per_cu = te.wg_per_cu > 0 ? te.wg_per_cu : tp.wg;
  if (per_cu <= 0) {
    // resident at once: LDS and threads, and the registers the kernel needs
    per_cu = resident_per_cu(p->threads, p->lds);
    const int occ = have_device ? batched_occupancy_of(s, b, oop) : 0;
    if (occ > 0 && occ < per_cu) per_cu = occ;
  }
  if (cfg && cfg->grid_blocks > 0) {
    p->grid = round_up((uint64_t)cfg->grid_blocks, (uint32_t)d.xcds);
  } else {
    p->grid = round_up((uint64_t)per_cu * d.cus, (uint32_t)d.xcds);
  }
  return BITREV_SUCCESS;
}

// ---------------------------------------------------------------------------
// Launches.
// ---------------------------------------------------------------------------
hipError_t launch_tile(bool inplace, int s, const Plan& p, const void* src, void* dst,
                       uint64_t src_stride, uint64_t dst_stride, const DeviceInfo& d,
                       hipStream_t st, void* ev_start = nullptr, void* ev_stop = nullptr) {
  TileLaunch a;
  a.ev_start = ev_start;
  a.ev_stop = ev_stop;
  a.src = src;
  a.dst = dst;
  a.m = p.m;
  a.items_per_seg = p.items_per_seg;
  a.total_items = p.total;
  a.seg_elems = src_stride;
  a.dst_seg_elems = dst_stride;
  a.balanced = order_code(p.order);
  a.xcds = p.xcd_remap == 2 ? 1 : d.xcds;
  a.grid = p.grid;
  a.pipelined = p.variant == 2 ? 1 : (p.variant == 3 ? 2 : 0);
  a.hints = p.hints;
  switch (s) {
    case 1: return inplace ? launch_tile_inplace_s1(p.b, p.vec, a, st) : launch_tile_outofplace_s1(p.b, p.vec, a, st);
    case 2: return inplace ? launch_tile_inplace_s2(p.b, p.vec, a, st) : launch_tile_outofplace_s2(p.b, p.vec, a, st);
    case 4: return inplace ? launch_tile_inplace_s4(p.b, p.vec, a, st) : launch_tile_outofplace_s4(p.b, p.vec, a, st);
    case 8: return inplace ? launch_tile_inplace_s8(p.b, p.vec, a, st) : launch_tile_outofplace_s8(p.b, p.vec, a, st);
    default: return inplace ? launch_tile_inplace_s16(p.b, p.vec, a, st) : launch_tile_outofplace_s16(p.b, p.vec, a, st);
  }
}

hipError_t launch_wave(int s, const Plan& p, const void* src, void* dst, int k, int64_t rows,
                       uint64_t src_stride, uint64_t dst_stride, hipStream_t st) {
  WaveLaunch a;
  a.src = src;
  a.dst = dst;
  a.k = k;
  a.nseg = (uint64_t)rows;
  a.grid = p.grid;
  a.src_stride = src_stride;
  a.dst_stride = dst_stride;
  switch (s) {
    case 1: return launch_wave_s1(a, st);
    case 2: return launch_wave_s2(a, st);
    case 4: return launch_wave_s4(a, st);
    case 8: return launch_wave_s8(a, st);
    default: return launch_wave_s16(a, st);
  }
}

hipError_t launch_row_chunks(int s, const Plan& p, const void* src, void* dst, int k,
                             int64_t rows, uint64_t src_stride, uint64_t dst_stride,
                             hipStream_t st) {
  const uint64_t rb = (uint64_t)s << k;
  RowsLaunch a;
  a.src = src;
  a.dst = dst;
  a.k = k;
  if (rb < 16) {  // contiguous: one run of vectors, then what is left
    a.runs = (uint64_t)rows * rb / 16;
    a.run_log2 = 0;
    a.tail = (uint32_t)((uint64_t)rows * rb % 16 / s);
    a.src_pitch = a.dst_pitch = 16;
  } else {
    a.runs = (uint64_t)rows;
    a.run_log2 = footprint_class(rb / 16);
    a.tail = 0;
    a.src_pitch = src_stride * s;
    a.dst_pitch = dst_stride * s;
  }
  a.chunk_log2 = p.chunk_log2;
  a.gather = p.gather;
  a.hints = p.hints;
  a.grid = p.grid;
  return launch_rows(s, a, st);
}

size_t pointer_align(const void* a, const void* b) {
  const uintptr_t v = reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b);
  size_t al = 16;
  while (al > 1 && (v & (al - 1))) al >>= 1;
  return al;
}

bool overlap(const void* a, const void* b, size_t bytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + bytes && y < x + bytes;
}

// Common body of bitrev_inplace/outofplace/rows (+ _ex).
// Largest power of two <= 16 dividing v (16 for v = 0).
size_t align_of(uint64_t v) {
  size_t al = 16;
  while (al > 1 && (v & (al - 1))) al >>= 1;
  return al;
}

// Bytes spanned by `rows` arrays of n elements placed `stride` elements apart.
uint64_t footprint(uint64_t n, int64_t rows, uint64_t stride, size_t s) {
  return rows <= 0 ? 0 : ((uint64_t)(rows - 1) * stride + n) * s;
}

bool ranges_overlap(const void* a, uint64_t abytes, const void* b, uint64_t bbytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + bbytes && y < x + abytes;
}

// Common body of the plain, rows and strided entry points.  Strides are in
// elements between consecutive arrays; 0 means 2^k (contiguous rows).
// ev_start / ev_stop: optional hipEvent_t recorded as the path's one kernel
// starts and ends (around the launch where the path is not a tile kernel).
bitrev_status_t run_plain(const void* src, void* dst, int k, int64_t rows, size_t s,
                          const bitrev_config_t* cfg, void* stream, uint64_t src_stride = 0,
                          uint64_t dst_stride = 0, void* ev_start = nullptr,
                          void* ev_stop = nullptr) {
  // ---- validation: no HIP call before this block completes ----
  if (src == NULL || dst == NULL) return BITREV_ERROR_INVALID_VALUE;
  if (k < 0 || k > BITREV_MAX_LOG2N || !valid_elem_size(s) || rows < 0 || !valid_config(cfg))
    return BITREV_ERROR_INVALID_VALUE;
  if ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) % s)
    return BITREV_ERROR_INVALID_VALUE;
  const uint64_t n = 1ull << k;
  if (src_stride == 0) src_stride = n;
  if (dst_stride == 0) dst_stride = n;
  if (src_stride < n || dst_stride < n || src_stride > (1ull << 50) || dst_stride > (1ull << 50))
    return BITREV_ERROR_INVALID_VALUE;
  if (rows > 0 && ((uint64_t)rows > (1ull << 62) / (src_stride * s) ||
                   (uint64_t)rows > (1ull << 62) / (dst_stride * s)))
    return BITREV_ERROR_INVALID_VALUE;
  const bool inplace = (src == dst);
  if (inplace && src_stride != dst_stride) return BITREV_ERROR_INVALID_VALUE;
  if (!inplace && ranges_overlap(src, footprint(n, rows, src_stride, s), dst,
                                 footprint(n, rows, dst_stride, s)))
    return BITREV_ERROR_ALIAS;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const bool timed = ev_start != nullptr && ev_stop != nullptr;
  if (rows == 0 || (inplace && k <= 1)) {
    if (!timed) return BITREV_SUCCESS;  // nothing to run: the events bracket nothing
    hipError_t e = hipEventRecord(static_cast<hipEvent_t>(ev_start), hs);
    if (e == hipSuccess) e = hipEventRecord(static_cast<hipEvent_t>(ev_stop), hs);
    return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
  }
  // ---- plan and launch ----
  DeviceInfo d;
  bitrev_status_t st = device_info(&d, false);
  if (st != BITREV_SUCCESS) return st;
  Plan p;
  size_t align = pointer_align(src, dst);
  // (contiguous rows shorter than a vector are one run of bytes: 2^1 uint8, 40
  // MiB, 899 us by single elements)
  if (rows > 1 && !(src_stride == n && dst_stride == n && n * s < 16)) {
    const size_t sa = align_of(src_stride * s), da = align_of(dst_stride * s);
    if (sa < align) align = sa;
    if (da < align) align = da;
  }
  st = plan_plain(inplace ? kModeInplace : kModeOutofplace, k, (int)s, rows, src_stride,
                  dst_stride, cfg, align, d, true, &p);
  if (st != BITREV_SUCCESS) return st;
  hipError_t e = hipSuccess;
  if (p.path == BITREV_PATH_WAVE || p.path == BITREV_PATH_ROWS) {
    if (timed) e = hipEventRecord(static_cast<hipEvent_t>(ev_start), hs);
    if (e == hipSuccess)
      e = p.path == BITREV_PATH_ROWS
              ? launch_row_chunks((int)s, p, src, dst, k, rows, src_stride, dst_stride, hs)
              : launch_wave((int)s, p, src, dst, k, rows, src_stride, dst_stride, hs);
    if (timed && e == hipSuccess) e = hipEventRecord(static_cast<hipEvent_t>(ev_stop), hs);
  } else if (p.path == BITREV_PATH_TILE) {
    e = launch_tile(inplace, (int)s, p, src, dst, src_stride, dst_stride, d, hs,
                    timed ? ev_start : nullptr, timed ? ev_stop : nullptr);
  }
  return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
}

hipError_t launch_transpose(int s, int b, bool vec, const TransposeLaunch& a, hipStream_t st) {
  switch (s) {
    case 1: return launch_transpose_s1(b, vec, a, st);
    case 2: return launch_transpose_s2(b, vec, a, st);
    case 4: return launch_transpose_s4(b, vec, a, st);
    case 8: return launch_transpose_s8(b, vec, a, st);
    default: return launch_transpose_s16(b, vec, a, st);
  }
}

// In-place transpose of the 2^h x 2^h matrix at data (validated by callers).
bitrev_status_t run_transpose(void* data, int h, size_t s, hipStream_t st) {
  if (h == 0) return BITREV_SUCCESS;
  DeviceInfo d;
  bitrev_status_t status = device_info(&d, false);
  if (status != BITREV_SUCCESS) return status;
  const PlanFields tp = table_plan(kKindInplace, (int)s, 0, 0, ((uint64_t)s) << (2 * h), d);
  int b = tp.b ? tp.b : max_tile_bits((int)s);
  if (b > h) b = h;
  if (b > max_tile_bits((int)s)) b = max_tile_bits((int)s);
  while (b > 0 && tile_lds_bytes_for((int)s, b, 2) > d.lds_per_block) --b;
  const size_t vb = (s << b) < 16 ? (s << b) : 16;
  TransposeLaunch a;
  a.data = data;
  a.h = h;
  const uint64_t nt = 1ull << (h - b);
  a.total_items = nt * (nt + 1) / 2;
  a.xcds = tp.xcd == 2 ? 1 : d.xcds;
  a.grid = default_grid(a.total_items, d);
  const hipError_t e = launch_transpose((int)s, b, pointer_align(data, data) % vb == 0, a, st);
  return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
}

hipError_t launch_digit(int s, int d, int b, bool vec, const TileLaunch& a, hipStream_t st) {
  switch (s) {
    case 1: return launch_digit_s1(d, b, vec, a, st);
    case 2: return launch_digit_s2(d, b, vec, a, st);
    case 4: return launch_digit_s4(d, b, vec, a, st);
    case 8: return launch_digit_s8(d, b, vec, a, st);
    default: return launch_digit_s16(d, b, vec, a, st);
  }
}

hipError_t launch_wave_digit(int s, const WaveLaunch& a, int d, hipStream_t st) {
  switch (s) {
    case 1: return launch_wave_digit_s1(a, d, st);
    case 2: return launch_wave_digit_s2(a, d, st);
    case 4: return launch_wave_digit_s4(a, d, st);
    case 8: return launch_wave_digit_s8(a, d, st);
    default: return launch_wave_digit_s16(a, d, st);
  }
}

// Digit-reversed permutation (d-bit digits) of one array; src == dst in place.
// cfg (may be NULL): tile_bits (a whole number of digits), grid_blocks,
// order (out of place: the source tile order; in place the grouped digit
// order is fixed), xcd_remap and cache_hints as for the plain calls.
bitrev_status_t run_digit(const void* src, void* dst, int k, int d, size_t s,
                          const bitrev_config_t* cfg, void* stream) {
  // ---- validation: no HIP call before this block completes ----
  if (src == NULL || dst == NULL || k < 0 || k > BITREV_MAX_LOG2N || !valid_elem_size(s) ||
      d < 1 || d > 3 || k % d || !valid_config(cfg))
    return BITREV_ERROR_INVALID_VALUE;
  if ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) % s)
    return BITREV_ERROR_INVALID_VALUE;
  const uint64_t n = 1ull << k;
  const bool inplace = (src == dst);
  if (!inplace && overlap(src, dst, (size_t)(n * s))) return BITREV_ERROR_ALIAS;
  if (d == 1) return run_plain(src, dst, k, 1, s, cfg, stream);
  if (inplace && k <= d) return BITREV_SUCCESS;  // one digit: the identity
  // ---- plan and launch ----
  DeviceInfo dev;
  bitrev_status_t st = device_info(&dev, false);
  if (st != BITREV_SUCCESS) return st;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  hipError_t e;
  if (k <= 6) {
    WaveLaunch w;
    w.src = src;
    w.dst = dst;
    w.k = k;
    w.nseg = 1;
    w.grid = 1;
    e = launch_wave_digit((int)s, w, d, hs);
    return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
  }
  const int kind = inplace ? kKindDigitInplace : kKindDigitOutofplace;
  const PlanFields t1 = table_plan(kind, (int)s, d, 0, n * s, dev);
  int b = t1.b ? t1.b : max_tile_bits((int)s);
  const int tiles = inplace ? 2 : 1;  // staged by a workgroup
  if (cfg && cfg->tile_bits) {
    b = cfg->tile_bits;  // forced: whole digits, within the array, compiled, fits
    if (b % d || 2 * b > k || b > max_tile_bits((int)s) ||
        tile_lds_bytes_for((int)s, b, tiles) > dev.lds_per_block)
      return BITREV_ERROR_NOT_SUPPORTED;
  } else {
    // b must be a multiple of d: round up where the element size and the
    // array allow (radix 8 out of place, complex64 2^24: b = 3 moved 2.2 TB/s)
    const int bu = (b + d - 1) / d * d;
    if (bu <= max_tile_bits((int)s) && 2 * bu <= k) b = bu;
    if (b > max_tile_bits((int)s)) b = max_tile_bits((int)s);
    if (2 * b > k) b = k / 2;
    b -= b % d;
    while (b >= d && tile_lds_bytes_for((int)s, b, tiles) > dev.lds_per_block) b -= d;
  }
  if (b < d) return BITREV_ERROR_NOT_SUPPORTED;
  const int m = k - 2 * b;
  if (m > 32) return BITREV_ERROR_NOT_SUPPORTED;
  TileLaunch a;
  a.src = src;
  a.dst = dst;
  a.m = m;
  a.total_items = inplace ? dpair_count(m, d) : (1ull << m);
  a.items_per_seg = a.total_items;
  a.seg_elems = n;
  const PlanFields tp = table_plan(kind, (int)s, d, b, n * s, dev);
  a.balanced = order_code((cfg && cfg->order) ? cfg->order : (tp.order ? tp.order : 1));
  const int xr = (cfg && cfg->xcd_remap) ? cfg->xcd_remap : (tp.xcd ? tp.xcd : 1);
  a.xcds = xr == 2 ? 1 : dev.xcds;
  a.grid = (cfg && cfg->grid_blocks > 0) ? round_up((uint64_t)cfg->grid_blocks, (uint32_t)dev.xcds)
                                         : default_grid(a.total_items, dev);
  a.hints = (cfg && cfg->cache_hints) ? cfg->cache_hints - 1
                                      : (tp.hints ? tp.hints - 1 : kHintPlain);
  a.pipelined = 0;
  const size_t vb = (s << b) < 16 ? (s << b) : 16;
  e = launch_digit((int)s, d, b, pointer_align(src, dst) % vb == 0, a, hs);
  return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
}

}  // namespace

extern "C" {

bitrev_status_t bitrev_digitrev_inplace(void* data, int log2n, int digit_bits, size_t elem_size,
                                        void* stream) {
  return run_digit(data, data, log2n, digit_bits, elem_size, NULL, stream);
}

bitrev_status_t bitrev_digitrev_outofplace(const void* src, void* dst, int log2n, int digit_bits,
                                           size_t elem_size, void* stream) {
  if (src != NULL && src == dst) return BITREV_ERROR_ALIAS;
  return run_digit(src, dst, log2n, digit_bits, elem_size, NULL, stream);
}

bitrev_status_t bitrev_digitrev_inplace_ex(void* data, int log2n, int digit_bits,
                                           size_t elem_size, const bitrev_config_t* cfg,
                                           void* stream) {
  return run_digit(data, data, log2n, digit_bits, elem_size, cfg, stream);
}

bitrev_status_t bitrev_digitrev_outofplace_ex(const void* src, void* dst, int log2n,
                                              int digit_bits, size_t elem_size,
                                              const bitrev_config_t* cfg, void* stream) {
  if (src != NULL && src == dst) return BITREV_ERROR_ALIAS;
  return run_digit(src, dst, log2n, digit_bits, elem_size, cfg, stream);
}

uint32_t bitrev_debug_digit_rev(uint32_t v, int j, int d) {
  return (j < 0 || j > 32 || d < 1 || d > 3) ? 0u : drev_bits(v, j, d);
}

uint64_t bitrev_debug_digit_pair_count(int m, int d) {
  return (m < 0 || m > 32 || d < 1 || d > 3 || m % d) ? 0 : dpair_count(m, d);
}

uint32_t bitrev_debug_digit_pair_at(int m, uint64_t w, int d) {
  if (m < 0 || m > 32 || d < 1 || d > 3 || m % d || w >= dpair_count(m, d)) return 0xFFFFFFFFu;
  return dpair_at(m, w, d);
}

uint32_t bitrev_debug_digit_inplace_pair_at(int m, uint64_t w, int d) {
  if (m < 0 || m > 32 || d < 1 || d > 3 || m % d || w >= dpair_count(m, d)) return 0xFFFFFFFFu;
  return dinplace_pair_at(m, w, d);
}

bitrev_status_t bitrev_transpose_inplace(void* data, int log2side, size_t elem_size, void* stream) {
  if (data == NULL || log2side < 0 || 2 * log2side > BITREV_MAX_LOG2N || !valid_elem_size(elem_size) ||
      reinterpret_cast<uintptr_t>(data) % elem_size)
    return BITREV_ERROR_INVALID_VALUE;
  if (log2side > 32) return BITREV_ERROR_NOT_SUPPORTED;
  return run_transpose(data, log2side, elem_size, static_cast<hipStream_t>(stream));
}

// Whether several short rows with fused levels take k_rows_dit: 4 <= k < 8,
// whose tiles are at most 2^3 elements wide (three levels at most).  From k = 8
// on the tiles read whole lines and are level or ahead (complex64 2^8, three
// levels, 73 MiB 24.5 us against 26.0; complex128 2^10 12 MiB 5.3 against 5.8).
static bool rows_dit_applies(int k, uint64_t rows, const bitrev_config_t* cfg) {
  return rows >= 2 && !config_set(cfg) && k >= 4 && k < 8;
}

// How a call with fused levels runs: whole rows in LDS, or tiles of width b.
// The pointers and the direction are the caller's to fill in.
struct DitPlan {
  bool whole_rows = false;
  RowsDitLaunch r = {};
  DitLaunch a = {};
  int b = 0;
  bool vec = true;
  int order = 0, xcd_remap = 0;
};

static bitrev_status_t plan_dit(bool inplace, int log2n, int64_t rows, int stages, size_t s,
                                const bitrev_config_t* cfg, size_t align, const DeviceInfo& d,
                                DitPlan* p) {
  const uint64_t n = 1ull << log2n;
  const int kind = inplace ? kKindDitInplace : kKindDitOutofplace;
  const uint64_t footprint = n * s * (uint64_t)rows;
  if (rows_dit_applies(log2n, (uint64_t)rows, cfg) &&
      !user_rows_apply(kind, (int)s, footprint, d)) {
    RowsDitLaunch& r = p->r;
    p->whole_rows = true;
    r.k = log2n;
    r.rows = (uint64_t)rows;
    r.stages = stages;
    r.hints = footprint >= (64ull << 20) && align == 16 ? kHintStreamWriteThrough : kHintPlain;
    const uint64_t per = (1ull << kRowsDitLog2) / (n * s);
    const uint64_t chunks = ((uint64_t)rows + per - 1) / per;
    r.grid = (uint32_t)(chunks < (1u << 20) ? chunks : (1u << 20));
    return BITREV_SUCCESS;
  }
  const PlanFields rule = bytes_rule(kind, (int)s, log2n, (uint64_t)rows, footprint, stages,
                                     true, cfg ? cfg->tile_bits : 0, d);
  const PlanFields t1 = table_plan(kind, (int)s, 0, 0, footprint, d, rule);
  int b;
  if (cfg && cfg->tile_bits) {
    b = cfg->tile_bits;  // forced: must hold the levels and fit (a
                         // rectangular tile needs only b + (b - 1) or
                         // b + (b - 2) bits, checked below)
    const bool rect = cfg->variant >= 2;
    if ((2 * b > log2n && !rect) || b > max_tile_bits((int)s)) return BITREV_ERROR_NOT_SUPPORTED;
  } else {
    b = t1.b ? t1.b : max_tile_bits((int)s);
    if (b < stages) b = stages;
    if (b > max_tile_bits((int)s)) b = max_tile_bits((int)s);
    if (2 * b > log2n) b = log2n / 2;
  }
  const size_t lds = tile_lds_bytes_for((int)s, b, 2) + ((size_t)1 << b) * (s / 2);
  if (b < stages || lds > d.lds_per_block) return BITREV_ERROR_NOT_SUPPORTED;
  // square tiles (a forced rectangular plan with 2b > log2n gets its own
  // geometry below or is rejected there)
  const int m = 2 * b <= log2n ? log2n - 2 * b : 0;
  if (m > 32) return BITREV_ERROR_NOT_SUPPORTED;
  DitLaunch& a = p->a;
  a.t.m = m;
  a.t.items_per_seg = inplace ? pair_count(m) : (1ull << m);
  a.t.total_items = a.t.items_per_seg * (uint64_t)rows;
  a.t.seg_elems = n;
  const PlanFields tp = table_plan(kind, (int)s, 0, b, footprint, d, rule);
  // rectangular tiles out of place (variant 2: source rows of 2^(b-1)
  // elements, 3: of 2^(b-2); b = 5 or 6, 16-byte aligned arrays)
  const int dvar = (cfg && cfg->variant) ? cfg->variant : (tp.variant ? tp.variant : 1);
  if (inplace && dvar == 3 && 2 * b <= log2n) {
    // in place: the pair in registers, each tile staged in turn through one
    // LDS tile
    a.rs = 1;
  } else if (dvar >= 2) {
    const int bz = b - (dvar - 1);
    const bool fits = !inplace && (b == 5 || b == 6) && align % 16 == 0 &&
                      log2n >= b + bz && log2n - b - bz <= 32;
    if (fits) {
      a.rect_bz = bz;
      a.t.m = log2n - b - bz;
      a.t.items_per_seg = 1ull << a.t.m;
      a.t.total_items = a.t.items_per_seg * (uint64_t)rows;
    } else if (cfg && cfg->variant) {
      return BITREV_ERROR_NOT_SUPPORTED;
    }
  }
  p->order = (cfg && cfg->order) ? cfg->order : (tp.order ? tp.order : 2);
  a.t.balanced = order_code(p->order);
  p->xcd_remap = (cfg && cfg->xcd_remap) ? cfg->xcd_remap : (tp.xcd ? tp.xcd : 1);
  a.t.xcds = p->xcd_remap == 2 ? 1 : d.xcds;
  a.t.grid = (cfg && cfg->grid_blocks > 0) ? round_up((uint64_t)cfg->grid_blocks, (uint32_t)d.xcds)
                                           : default_grid(a.t.total_items, d);
  a.t.pipelined = 0;
  a.t.hints = (cfg && cfg->cache_hints) ? cfg->cache_hints - 1
                                        : (tp.hints ? tp.hints - 1 : kHintPlain);
  a.stages = stages;
  const size_t vb = (s << b) < 16 ? (s << b) : 16;
  p->b = b;
  p->vec = align % vb == 0;
  return BITREV_SUCCESS;
}

bitrev_status_t bitrev_dit_stages_ex(const void* src, void* dst, int log2n, int64_t rows,
                                     int stages, int inverse, int dtype,
                                     const bitrev_config_t* cfg, void* stream) {
  // ---- validation: no HIP call before this block completes ----
  if (src == NULL || dst == NULL || log2n < 0 || log2n > BITREV_MAX_LOG2N || rows < 0 ||
      stages < 0 || stages > 7 || (inverse != 0 && inverse != 1) || (dtype != 0 && dtype != 1) ||
      !valid_config(cfg))
    return BITREV_ERROR_INVALID_VALUE;
  const size_t s = dtype == 0 ? 8 : 16;
  if ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) % s)
    return BITREV_ERROR_INVALID_VALUE;
  const uint64_t n = 1ull << log2n;
  if (rows > 0 && (uint64_t)rows > (1ull << 62) / (n * s)) return BITREV_ERROR_INVALID_VALUE;
  const bool inplace = (src == dst);
  if (!inplace && overlap(src, dst, (size_t)(n * s * (uint64_t)rows))) return BITREV_ERROR_ALIAS;
  if (2 * stages > log2n || stages > max_tile_bits((int)s)) return BITREV_ERROR_NOT_SUPPORTED;
  if (stages == 0) {
    // the plain permutation: the config's variant names DIT tile shapes, not
    // the plain kernels' variants, and a width only rectangular tiles could
    // take is left to the plan
    bitrev_config_t plain_cfg;
    if (cfg) {
      plain_cfg = *cfg;
      plain_cfg.variant = 0;
      if (2 * plain_cfg.tile_bits > log2n) plain_cfg.tile_bits = 0;
    }
    return run_plain(src, dst, log2n, rows, s, cfg ? &plain_cfg : NULL, stream);
  }
  if (rows == 0) return BITREV_SUCCESS;
  // ---- plan and launch ----
  DeviceInfo d;
  bitrev_status_t st = device_info(&d, false);
  if (st != BITREV_SUCCESS) return st;
  DitPlan p;
  st = plan_dit(inplace, log2n, rows, stages, s, cfg, pointer_align(src, dst), d, &p);
  if (st != BITREV_SUCCESS) return st;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  hipError_t e;
  if (p.whole_rows) {
    p.r.src = src;
    p.r.dst = dst;
    p.r.inverse = inverse;
    e = launch_rows_dit((int)s, p.r, hs);
  } else {
    p.a.t.src = src;
    p.a.t.dst = dst;
    p.a.inverse = inverse;
    e = s == 8 ? launch_dit_s8(p.b, p.vec, p.a, hs) : launch_dit_s16(p.b, p.vec, p.a, hs);
  }
  return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
}

bitrev_status_t bitrev_dit_stages(const void* src, void* dst, int log2n, int64_t rows, int stages,
                                  int inverse, int dtype, void* stream) {
  return bitrev_dit_stages_ex(src, dst, log2n, rows, stages, inverse, dtype, NULL, stream);
}

// The block-local reversals with the second recursion level in LDS: 2^h
// contiguous blocks of 2^h elements each.
static bitrev_status_t run_block_recursive(void* data, int h, size_t s, hipStream_t st) {
  DeviceInfo d;
  bitrev_status_t status = device_info(&d, false);
  if (status != BITREV_SUCCESS) return status;
  const uint64_t nblocks = 1ull << h;
  // two 64 KiB blocks fit a compute unit's LDS at once
  const uint64_t cap = (uint64_t)d.cus * 8;
  const uint32_t grid = (uint32_t)(nblocks < cap ? nblocks : cap);
  const bool vec = reinterpret_cast<uintptr_t>(data) % 16 == 0 && (s << h) % 16 == 0;
  hipError_t e;
  switch (s) {
    case 1: e = launch_block_recursive_s1(data, h, nblocks, vec, grid, st); break;
    case 2: e = launch_block_recursive_s2(data, h, nblocks, vec, grid, st); break;
    case 4: e = launch_block_recursive_s4(data, h, nblocks, vec, grid, st); break;
    case 8: e = launch_block_recursive_s8(data, h, nblocks, vec, grid, st); break;
    default: e = launch_block_recursive_s16(data, h, nblocks, vec, grid, st); break;
  }
  return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
}

// Largest block the LDS stage of the second recursion level holds.
constexpr size_t kRecursiveBlockBytes = 65536;

bitrev_status_t bitrev_inplace_recursive_ex(void* data, int log2n, size_t elem_size, int levels,
                                            void* stream) {
  if (data == NULL || log2n < 0 || log2n > BITREV_MAX_LOG2N || !valid_elem_size(elem_size) ||
      reinterpret_cast<uintptr_t>(data) % elem_size || levels < 0 || levels > 2)
    return BITREV_ERROR_INVALID_VALUE;
  if (log2n % 2) return BITREV_ERROR_NOT_SUPPORTED;
  const int h = log2n / 2;
  const bool two_fit = h % 2 == 0 && (elem_size << h) <= kRecursiveBlockBytes;
  if (levels == 2 && !two_fit) return BITREV_ERROR_NOT_SUPPORTED;
  if (log2n <= 1) return BITREV_SUCCESS;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const int64_t rows = (int64_t)1 << h;
  const bool two = levels == 2 || (levels == 0 && two_fit);
  bitrev_status_t st = two ? run_block_recursive(data, h, elem_size, hs)
                           : run_plain(data, data, h, rows, elem_size, NULL, stream);
  if (st == BITREV_SUCCESS) st = run_transpose(data, h, elem_size, hs);
  if (st == BITREV_SUCCESS)
    st = two ? run_block_recursive(data, h, elem_size, hs)
             : run_plain(data, data, h, rows, elem_size, NULL, stream);
  return st;
}

bitrev_status_t bitrev_inplace_recursive(void* data, int log2n, size_t elem_size, void* stream) {
  return bitrev_inplace_recursive_ex(data, log2n, elem_size, 0, stream);
}

bitrev_status_t bitrev_inplace(void* data, int log2n, size_t elem_size, void* stream) {
  return run_plain(data, data, log2n, 1, elem_size, NULL, stream);
}

bitrev_status_t bitrev_inplace_ex(void* data, int log2n, size_t elem_size,
                                  const bitrev_config_t* cfg, void* stream) {
  return run_plain(data, data, log2n, 1, elem_size, cfg, stream);
}

bitrev_status_t bitrev_inplace_timed(void* data, int log2n, size_t elem_size,
                                     const bitrev_config_t* cfg, void* start_event,
                                     void* stop_event, void* stream) {
  if (start_event == NULL || stop_event == NULL) return BITREV_ERROR_INVALID_VALUE;
  return run_plain(data, data, log2n, 1, elem_size, cfg, stream, 0, 0, start_event, stop_event);
}

bitrev_status_t bitrev_outofplace_timed(const void* src, void* dst, int log2n, size_t elem_size,
                                        const bitrev_config_t* cfg, void* start_event,
                                        void* stop_event, void* stream) {
  if (start_event == NULL || stop_event == NULL) return BITREV_ERROR_INVALID_VALUE;
  return run_plain(src, dst, log2n, 1, elem_size, cfg, stream, 0, 0, start_event, stop_event);
}

bitrev_status_t bitrev_timing_event_create(void** event) {
  if (event == NULL) return BITREV_ERROR_INVALID_VALUE;
  *event = NULL;
  hipEvent_t ev = NULL;
  // no system-scope fence when the event is reached: the stop timestamp is
  // then not delayed by the writeback of the L2 that such a fence performs
  const hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableSystemFence);
  if (e != hipSuccess) return hip_fail(e);
  *event = (void*)ev;
  return BITREV_SUCCESS;
}

bitrev_status_t bitrev_timing_event_destroy(void* event) {
  if (event == NULL) return BITREV_SUCCESS;
  const hipError_t e = hipEventDestroy((hipEvent_t)event);
  return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
}

bitrev_status_t bitrev_timing_elapsed_ms(void* start_event, void* stop_event, float* ms) {
  if (start_event == NULL || stop_event == NULL || ms == NULL) return BITREV_ERROR_INVALID_VALUE;
  hipError_t e = hipEventSynchronize((hipEvent_t)stop_event);
  if (e == hipSuccess) e = hipEventElapsedTime(ms, (hipEvent_t)start_event, (hipEvent_t)stop_event);
  return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
}

bitrev_status_t bitrev_outofplace(const void* src, void* dst, int log2n, size_t elem_size,
                                  void* stream) {
  if (src != NULL && src == dst) return BITREV_ERROR_ALIAS;
  return run_plain(src, dst, log2n, 1, elem_size, NULL, stream);
}

bitrev_status_t bitrev_outofplace_ex(const void* src, void* dst, int log2n, size_t elem_size,
                                     const bitrev_config_t* cfg, void* stream) {
  if (src != NULL && src == dst) return BITREV_ERROR_ALIAS;
  return run_plain(src, dst, log2n, 1, elem_size, cfg, stream);
}

bitrev_status_t bitrev_rows(const void* src, void* dst, int log2n, int64_t rows,
                            size_t elem_size, void* stream) {
  return run_plain(src, dst, log2n, rows, elem_size, NULL, stream);
}

bitrev_status_t bitrev_rows_ex(const void* src, void* dst, int log2n, int64_t rows,
                               size_t elem_size, const bitrev_config_t* cfg, void* stream) {
  return run_plain(src, dst, log2n, rows, elem_size, cfg, stream);
}

bitrev_status_t bitrev_rows_strided(const void* src, void* dst, int log2n, int64_t rows,
                                    int64_t src_stride, int64_t dst_stride, size_t elem_size,
                                    void* stream) {
  if (src_stride <= 0 || dst_stride <= 0) return BITREV_ERROR_INVALID_VALUE;
  return run_plain(src, dst, log2n, rows, elem_size, NULL, stream, (uint64_t)src_stride,
                   (uint64_t)dst_stride);
}

bitrev_status_t bitrev_evenodd(const void* src, void* dst, int log2n, int64_t rows,
                               size_t elem_size, void* stream) {
  if (src == NULL || dst == NULL || log2n < 1 || log2n > BITREV_MAX_LOG2N || rows < 0 ||
      !valid_elem_size(elem_size) ||
      (reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) % elem_size)
    return BITREV_ERROR_INVALID_VALUE;
  const uint64_t n = 1ull << log2n;
  if (rows > 0 && (uint64_t)rows > (1ull << 62) / (n * elem_size)) return BITREV_ERROR_INVALID_VALUE;
  const uint64_t bytes = n * elem_size * (uint64_t)rows;
  if (ranges_overlap(src, bytes, dst, bytes)) return BITREV_ERROR_ALIAS;
  if (rows == 0) return BITREV_SUCCESS;
  DeviceInfo d;
  bitrev_status_t st = device_info(&d, false);
  if (st != BITREV_SUCCESS) return st;
  const uint64_t pairs = (n / 2) * (uint64_t)rows;
  const uint64_t want = (pairs + 255) / 256;
  const uint32_t grid = (uint32_t)(want < (uint64_t)d.cus * 16 ? (want ? want : 1) : (uint64_t)d.cus * 16);
  hipStream_t hs = static_cast<hipStream_t>(stream);
  hipError_t e;
  switch (elem_size) {
    case 1: e = launch_evenodd_s1(src, dst, log2n, (uint64_t)rows, grid, hs); break;
    case 2: e = launch_evenodd_s2(src, dst, log2n, (uint64_t)rows, grid, hs); break;
    case 4: e = launch_evenodd_s4(src, dst, log2n, (uint64_t)rows, grid, hs); break;
    case 8: e = launch_evenodd_s8(src, dst, log2n, (uint64_t)rows, grid, hs); break;
    default: e = launch_evenodd_s16(src, dst, log2n, (uint64_t)rows, grid, hs); break;
  }
  return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
}

size_t bitrev_batched_workspace_size(int64_t num_arrays) {
  if (num_arrays < 0 || num_arrays > (1ll << 40)) return 0;
  const size_t raw = ((size_t)num_arrays + 3) * 8;
  return (raw + 255) / 256 * 256;
}

// Common body of the batched entry points; src != NULL means out of place
// (src -> data, the same packed layout).
// Host-side checks of a batched call's arguments other than the workspace
// (no HIP call is made).  *nothing_to_do is set for num_arrays == 0.
static bitrev_status_t check_batched_args(const void* src, void* data, int64_t data_elems,
                                          const int64_t* offsets, const int32_t* log2n,
                                          int64_t num_arrays, size_t elem_size,
                                          const bitrev_config_t* cfg, bool* nothing_to_do) {
  *nothing_to_do = false;
  if (num_arrays < 0 || num_arrays > (1ll << 40) || data_elems < 0 || !valid_elem_size(elem_size) ||
      !valid_config(cfg))
    return BITREV_ERROR_INVALID_VALUE;
  if (num_arrays == 0) {
    *nothing_to_do = true;
    return BITREV_SUCCESS;
  }
  if (data == NULL || offsets == NULL || log2n == NULL) return BITREV_ERROR_INVALID_VALUE;
  if (reinterpret_cast<uintptr_t>(data) % elem_size || reinterpret_cast<uintptr_t>(offsets) % 8 ||
      reinterpret_cast<uintptr_t>(log2n) % 4)
    return BITREV_ERROR_INVALID_VALUE;
  if (src != NULL) {
    if (reinterpret_cast<uintptr_t>(src) % elem_size) return BITREV_ERROR_INVALID_VALUE;
    if ((uint64_t)data_elems > (1ull << 62) / elem_size) return BITREV_ERROR_INVALID_VALUE;
    const uint64_t bytes = (uint64_t)data_elems * elem_size;
    if (src == data || ranges_overlap(src, bytes, data, bytes)) return BITREV_ERROR_ALIAS;
  }
  return BITREV_SUCCESS;
}

// What a batched launch takes from the plan and from the batch: a->src, a->num
// and a->data_elems are set, the geometry is filled in.
static void batched_geometry(const Plan& p, size_t elem_size, const DeviceInfo& d,
                             BatchedLaunch* a) {
  a->b = p.b;
  // Arrays that move whole through LDS: those too short for a tile and, where
  // neither the caller nor a tuning file sets the width (a tuned width is timed
  // as a forced one), all up to 16 KiB (5000 complex128 arrays of 2^10 35.8 ->
  // 28.8 us), in batches of short arrays (under 16 KiB on average) up to 32 KiB
  // (20000 complex64 arrays of 2^0-2^12: 69 -> 51 us; 1500 complex128 arrays
  // of 2^8-2^14, 75 KiB on average, would lose 47 -> 52)
  a->whole = 2 * p.b - 1;
  const bool shorts = (uint64_t)a->data_elems / (uint64_t)a->num < 16384 / elem_size;
  if (!p.forced_width)
    while ((elem_size << (a->whole + 1)) <= (shorts ? 32768u : 16384u)) ++a->whole;
  a->hints =
      (uint64_t)a->data_elems >= (64ull << 20) / elem_size ? kHintStreamWriteThrough : kHintPlain;
  // Long complex128 arrays in place in the grouped order (8 arrays of 32 MiB
  // 107.5 -> 97.1 us, from cold caches 101.1 -> 84.0, where one item per
  // workgroup in the balanced order had lost to the persistent grid's 92.9; 2 of
  // 256 MiB 231 -> 221 and 184 -> 178; 64 of 2^0-2^20 52.6 -> 50.4; one of 256
  // MiB 118 -> 109, but 87 -> 94).  Below 1 MiB on average it is level or loses
  // 1 to 3% (5000 of 2^3-2^13 51.6 -> 52.7, 700 of 2^10-2^16 70.7 -> 71.3).
  const bool grouped = elem_size == 16 && !p.forced_order && a->src == nullptr &&
                       (uint64_t)a->data_elems / (uint64_t)a->num >= (1ull << 20) / 16;
  a->order = grouped ? 3 : p.order;
  a->balanced = order_code(a->order);
  // one item per workgroup runs in dispatch order unless the caller or a tuning
  // file asks otherwise: contiguous XCD ranges walk eight distant regions at
  // once (4096 complex64 arrays: +10%)
  const bool ranges = p.xcd_remap != 2 && (p.persistent || p.forced_xcd);
  a->xcds = ranges ? d.xcds : 1;
  a->grid = p.grid;
  if (!p.persistent) {
    // no more workgroups than the data hold tiles: those without an item
    // cost 1 us per thousand (in short batches few arrays have tiles)
    uint64_t most = ((uint64_t)a->data_elems >> (2 * p.b)) + 1;
    if (shorts) most = most / 2 > 2u * (uint32_t)d.cus ? most / 2 : 2u * (uint32_t)d.cus;
    if (most < a->grid) a->grid = round_up(most, (uint32_t)d.xcds);
  }
}

static bitrev_status_t run_batched(const void* src, void* data, int64_t data_elems,
                                   const int64_t* offsets, const int32_t* log2n,
                                   int64_t num_arrays, size_t elem_size, void* workspace,
                                   size_t workspace_bytes, const bitrev_config_t* cfg,
                                   void* stream) {
  // ---- validation: no HIP call before this block completes ----
  bool nothing = false;
  const bitrev_status_t chk = check_batched_args(src, data, data_elems, offsets, log2n, num_arrays,
                                                 elem_size, cfg, &nothing);
  if (chk != BITREV_SUCCESS || nothing) return chk;
  if (workspace == NULL || reinterpret_cast<uintptr_t>(workspace) % 8 ||
      workspace_bytes < bitrev_batched_workspace_size(num_arrays))
    return BITREV_ERROR_WORKSPACE;
  // ---- plan and launch ----
  DeviceInfo d;
  bitrev_status_t st = device_info(&d, false);
  if (st != BITREV_SUCCESS) return st;
  Plan p;
  st = plan_batched((int)elem_size, cfg, d, true, src != NULL, &p);
  if (st != BITREV_SUCCESS) return st;
  BatchedLaunch a;
  a.src = src;
  a.data = data;
  a.offsets = offsets;
  a.log2n = log2n;
  a.num = num_arrays;
  a.data_elems = data_elems;
  a.ws = static_cast<int64_t*>(workspace);
  batched_geometry(p, elem_size, d, &a);
  hipStream_t hs = static_cast<hipStream_t>(stream);
  hipError_t e = launch_batched_front((int)elem_size, a, hs);
  if (e != hipSuccess) return hip_fail(e);
  switch (elem_size) {
    case 1: e = launch_batched_s1(a, hs); break;
    case 2: e = launch_batched_s2(a, hs); break;
    case 4: e = launch_batched_s4(a, hs); break;
    case 8: e = launch_batched_s8(a, hs); break;
    default: e = launch_batched_s16(a, hs); break;
  }
  return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
}

bitrev_status_t bitrev_batched_ex(void* data, int64_t data_elems, const int64_t* offsets,
                                  const int32_t* log2n, int64_t num_arrays, size_t elem_size,
                                  void* workspace, size_t workspace_bytes,
                                  const bitrev_config_t* cfg, void* stream) {
  return run_batched(NULL, data, data_elems, offsets, log2n, num_arrays, elem_size, workspace,
                     workspace_bytes, cfg, stream);
}

bitrev_status_t bitrev_batched_outofplace(const void* src, void* dst, int64_t data_elems,
                                          const int64_t* offsets, const int32_t* log2n,
                                          int64_t num_arrays, size_t elem_size, void* workspace,
                                          size_t workspace_bytes, void* stream) {
  if (src == NULL) return BITREV_ERROR_INVALID_VALUE;
  return run_batched(src, dst, data_elems, offsets, log2n, num_arrays, elem_size, workspace,
                     workspace_bytes, NULL, stream);
}

bitrev_status_t bitrev_batched(void* data, int64_t data_elems, const int64_t* offsets,
                               const int32_t* log2n, int64_t num_arrays, size_t elem_size,
                               void* workspace, size_t workspace_bytes, void* stream) {
  return bitrev_batched_ex(data, data_elems, offsets, log2n, num_arrays, elem_size, workspace,
                           workspace_bytes, NULL, stream);
}

// ---------------------------------------------------------------------------
// Allocation-free batched call: the workspace lives in a file-scope device
// array.  Host code never uses the array's name as an address (on the host it
// is only a stand-in for the symbol); it asks the runtime for the array's
// device address once per device and passes that to the kernels.
// ---------------------------------------------------------------------------
}  // extern "C"

// bitrev_batched_workspace_size(BITREV_NOALLOC_MAX_ARRAYS) bytes: the
// header and scan words, rounded up to 256 bytes
static __device__ __align__(256) int64_t scratch[(BITREV_NOALLOC_MAX_ARRAYS + 3 + 31) / 32 * 32];
static_assert(sizeof(scratch) == ((size_t)(BITREV_NOALLOC_MAX_ARRAYS + 3) * 8 + 255) / 256 * 256,
              "scratch must hold the workspace of the largest allowed batch");

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];  // device address of `scratch`, per device

// The current device's address of `scratch`, looked up on the first call on
// each device with that device current.
bitrev_status_t scratch_address(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e);
  if (dev < 0 || dev >= kMaxDevices) return hip_fail(hipErrorInvalidDevice);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr) return hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol);
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return BITREV_SUCCESS;
}
}  // namespace

extern "C" {

bitrev_status_t bitrev_batched_noalloc(void* data, int64_t data_elems, const int64_t* offsets,
                                       const int32_t* log2n, int64_t num_arrays, size_t elem_size,
                                       void* stream) {
  // every argument, and the size limit, is checked before any HIP call
  bool nothing = false;
  const bitrev_status_t chk = check_batched_args(NULL, data, data_elems, offsets, log2n,
                                                 num_arrays, elem_size, NULL, &nothing);
  if (chk != BITREV_SUCCESS || nothing) return chk;
  if (num_arrays > BITREV_NOALLOC_MAX_ARRAYS) return BITREV_ERROR_WORKSPACE;
  void* ws = nullptr;
  const bitrev_status_t st = scratch_address(&ws);
  if (st != BITREV_SUCCESS) return st;
  // the first kernel writes every workspace word the second one reads
  // (header and scan), so the previous call's contents need no clearing
  return run_batched(NULL, data, data_elems, offsets, log2n, num_arrays, elem_size, ws,
                     sizeof(scratch), NULL, stream);
}

bitrev_status_t bitrev_batched_errors(const void* workspace, int64_t* num_rejected,
                                      int64_t* first_rejected, void* stream) {
  if (workspace == NULL || reinterpret_cast<uintptr_t>(workspace) % 8) return BITREV_ERROR_WORKSPACE;
  hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(e);
  int64_t hdr[2] = {0, -1};
  e = hipMemcpy(hdr, workspace, sizeof hdr, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return hip_fail(e);
  if (num_rejected) *num_rejected = hdr[0];
  if (first_rejected) *first_rejected = hdr[1];
  return BITREV_SUCCESS;
}

bitrev_status_t bitrev_plan_query(int log2n, size_t elem_size, int64_t rows, int mode,
                                  const bitrev_config_t* cfg, bitrev_plan_t* plan) {
  if (plan == NULL || mode < 0 || mode > 2 || !valid_elem_size(elem_size) || !valid_config(cfg) ||
      rows < 0 || (mode != 2 && (log2n < 0 || log2n > BITREV_MAX_LOG2N)))
    return BITREV_ERROR_INVALID_VALUE;
  DeviceInfo d;
  bool have_device = false;
  bitrev_status_t st = device_info(&d, true, &have_device);
  if (st != BITREV_SUCCESS) return st;
  Plan p;
  st = (mode == 2) ? plan_batched((int)elem_size, cfg, d, have_device, false, &p)
                   : plan_plain(mode, log2n, (int)elem_size, rows, 1ull << log2n, 1ull << log2n,
                                cfg, 16, d, have_device, &p);
  if (st != BITREV_SUCCESS) return st;
  memset(plan, 0, sizeof *plan);
  plan->path = p.path;
  plan->tile_bits = p.b;
  plan->mid_bits = p.m;
  plan->block_threads = p.threads;
  plan->grid_blocks = (int)p.grid;
  plan->order = p.order;
  plan->vector_access = p.vec ? 1 : 0;
  plan->variant = p.path == BITREV_PATH_TILE ? p.variant : 0;
  plan->xcd_remap = (p.path == BITREV_PATH_TILE || p.path == BITREV_PATH_BATCHED) ? p.xcd_remap : 0;
  plan->cache_hints =
      (p.path == BITREV_PATH_TILE || p.path == BITREV_PATH_ROWS) ? p.hints + 1 : 0;
  plan->work_items = p.total;
  plan->lds_bytes = p.lds;
  return BITREV_SUCCESS;
}

bitrev_status_t bitrev_debug_batched_plan(int64_t data_elems, int64_t num_arrays,
                                          size_t elem_size, int outofplace,
                                          const bitrev_config_t* cfg, bitrev_plan_t* plan,
                                          int* whole_bits) {
  if (plan == NULL || whole_bits == NULL || data_elems < 0 || num_arrays < 1 ||
      num_arrays > (1ll << 40) || !valid_elem_size(elem_size) || !valid_config(cfg))
    return BITREV_ERROR_INVALID_VALUE;
  DeviceInfo d;
  bool have_device = false;
  bitrev_status_t st = device_info(&d, true, &have_device);
  if (st != BITREV_SUCCESS) return st;
  Plan p;
  st = plan_batched((int)elem_size, cfg, d, have_device, outofplace != 0, &p);
  if (st != BITREV_SUCCESS) return st;
  BatchedLaunch a = {};
  a.src = outofplace ? plan : nullptr;  // (only whether there is one counts)
  a.num = num_arrays;
  a.data_elems = data_elems;
  batched_geometry(p, elem_size, d, &a);
  memset(plan, 0, sizeof *plan);
  plan->path = p.path;
  plan->tile_bits = a.b;
  plan->block_threads = p.threads;
  plan->grid_blocks = (int)a.grid;
  plan->order = a.order;
  plan->vector_access = 1;
  plan->xcd_remap = a.xcds > 1 ? 1 : 2;
  plan->cache_hints = a.hints + 1;
  plan->lds_bytes = p.lds;
  *whole_bits = a.whole;
  return BITREV_SUCCESS;
}

bitrev_status_t bitrev_debug_dit_plan(int log2n, int64_t rows, int stages, int outofplace,
                                      int dtype, size_t align, const bitrev_config_t* cfg,
                                      bitrev_plan_t* plan) {
  if (plan == NULL || log2n < 0 || log2n > 40 || rows < 1 || rows > (1ll << (50 - log2n)) ||
      stages < 1 || 2 * stages > log2n || (dtype != 0 && dtype != 1) ||
      stages > max_tile_bits(dtype == 0 ? 8 : 16) || !(align == 16 || (align == 8 && dtype == 0)) ||
      !valid_config(cfg))
    return BITREV_ERROR_INVALID_VALUE;
  DeviceInfo d;
  bitrev_status_t st = device_info(&d, true);
  if (st != BITREV_SUCCESS) return st;
  DitPlan p;
  st = plan_dit(outofplace == 0, log2n, rows, stages, dtype == 0 ? 8 : 16, cfg, align, d, &p);
  if (st != BITREV_SUCCESS) return st;
  memset(plan, 0, sizeof *plan);
  plan->vector_access = p.vec ? 1 : 0;
  if (p.whole_rows) {
    plan->path = BITREV_PATH_ROWS;
    plan->grid_blocks = (int)p.r.grid;
    plan->cache_hints = p.r.hints + 1;
    return BITREV_SUCCESS;
  }
  plan->path = BITREV_PATH_TILE;
  plan->tile_bits = p.b;
  plan->mid_bits = p.a.t.m;
  plan->grid_blocks = (int)p.a.t.grid;
  plan->order = p.order;
  plan->variant = p.a.rs ? 3 : p.a.rect_bz ? 1 + p.b - p.a.rect_bz : 1;
  plan->xcd_remap = p.xcd_remap;
  plan->cache_hints = p.a.t.hints + 1;
  plan->work_items = p.a.t.total_items;
  return BITREV_SUCCESS;
}

bitrev_status_t bitrev_load_tuning(const char* path) {
  load_env_tuning();  // an explicit load always wins over the environment
  return load_tuning_file(path);
}

const char* bitrev_tuning_format(void) { return kTuningFormat; }

bitrev_status_t bitrev_copy_ex(const void* src, void* dst, size_t bytes, int cache_hints,
                               void* stream) {
  if (src == NULL || dst == NULL || cache_hints < 0 || cache_hints > 4)
    return BITREV_ERROR_INVALID_VALUE;
  if (bytes == 0) return BITREV_SUCCESS;
  if (overlap(src, dst, bytes)) return BITREV_ERROR_ALIAS;
  DeviceInfo d;
  bitrev_status_t st = device_info(&d, false);
  if (st != BITREV_SUCCESS) return st;
  // streaming loads with write-through stores: the fastest form measured at
  // 128 MiB and at 4 GiB (plain and streaming-load copies trail by 1-4%)
  const int h = cache_hints ? cache_hints - 1 : kHintStreamWriteThrough;
  const hipError_t e = launch_copy(src, dst, bytes, (uint32_t)(d.cus * 4), h,
                                   static_cast<hipStream_t>(stream));
  return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
}

bitrev_status_t bitrev_copy(const void* src, void* dst, size_t bytes, void* stream) {
  return bitrev_copy_ex(src, dst, bytes, 0, stream);
}

bitrev_status_t bitrev_copy_tiled(const void* src, void* dst, int log2n, size_t elem_size,
                                  const bitrev_config_t* cfg, void* stream) {
  // ---- validation: no HIP call before this block completes ----
  if (src == NULL || dst == NULL || log2n < 0 || log2n > BITREV_MAX_LOG2N ||
      !valid_elem_size(elem_size) || !valid_config(cfg) ||
      (reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) % elem_size)
    return BITREV_ERROR_INVALID_VALUE;
  const uint64_t bytes = (uint64_t)elem_size << log2n;
  if (overlap(src, dst, (size_t)bytes)) return BITREV_ERROR_ALIAS;
  // ---- plan and launch ----
  DeviceInfo d;
  bitrev_status_t st = device_info(&d, false);
  if (st != BITREV_SUCCESS) return st;
  Plan p;
  st = plan_tiles(kModeOutofplace, log2n, (int)elem_size, 1, cfg, pointer_align(src, dst), true, d,
                  true, &p);
  if (st != BITREV_SUCCESS) return st;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  if (p.path != BITREV_PATH_TILE) {
    // arrays of at most 64 elements have no tiles: a plain copy
    const hipError_t e = launch_copy(src, dst, (size_t)bytes, 1, kHintPlain, hs);
    return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
  }
  if (!p.vec) return BITREV_ERROR_NOT_SUPPORTED;
  TileLaunch a;
  a.src = src;
  a.dst = dst;
  a.m = p.m;
  a.items_per_seg = a.total_items = 1ull << p.m;
  a.seg_elems = a.dst_seg_elems = 1ull << log2n;
  a.balanced = order_code(p.order);
  a.xcds = p.xcd_remap == 2 ? 1 : d.xcds;
  a.grid = (cfg && cfg->grid_blocks > 0) ? p.grid : default_grid(a.total_items, d);
  a.pipelined = 0;
  a.hints = p.hints;
  hipError_t e;
  switch (elem_size) {
    case 1: e = launch_tile_copy_s1(p.b, a, hs); break;
    case 2: e = launch_tile_copy_s2(p.b, a, hs); break;
    case 4: e = launch_tile_copy_s4(p.b, a, hs); break;
    case 8: e = launch_tile_copy_s8(p.b, a, hs); break;
    default: e = launch_tile_copy_s16(p.b, a, hs); break;
  }
  return e == hipSuccess ? BITREV_SUCCESS : hip_fail(e);
}

const char* bitrev_status_string(bitrev_status_t status) {
  switch (status) {
    case BITREV_SUCCESS: return "success";
    case BITREV_ERROR_INVALID_VALUE: return "invalid value";
    case BITREV_ERROR_ALIAS: return "source and destination overlap";
    case BITREV_ERROR_WORKSPACE: return "workspace missing, misaligned or too small";
    case BITREV_ERROR_HIP: return "HIP runtime error";
    case BITREV_ERROR_NOT_SUPPORTED: return "not supported by this build or device";
  }
  return "unknown status";
}

int bitrev_last_hip_error(void) { return g_last_hip_error; }

int bitrev_abi_version(void) { return BITREV_ABI_VERSION; }

uint32_t bitrev_debug_rev(uint32_t v, int j) {
  return (j < 0 || j > 32) ? 0u : rev_bits(v, j);
}

uint64_t bitrev_debug_pair_count(int m) { return (m < 0 || m > 32) ? 0 : pair_count(m); }

uint32_t bitrev_debug_pair_at(int m, uint64_t w, int balanced) {
  if (m < 0 || m > 32 || w >= pair_count(m)) return 0xFFFFFFFFu;
  return pair_at(m, w, balanced != 0);
}

uint32_t bitrev_debug_oop_tile_at(int m, uint32_t w, int order) {
  if (m < 0 || m > 32 || (m < 32 && w >= (1u << m)) || order < 1 || order > 3) return 0xFFFFFFFFu;
  return oop_tile_at(m, w, order_code(order));
}

uint32_t bitrev_debug_inplace_pair_at(int m, uint64_t w, int order) {
  if (m < 0 || m > 32 || w >= pair_count(m) || order < 1 || order > 3) return 0xFFFFFFFFu;
  return inplace_pair_at(m, w, order_code(order));
}

void bitrev_debug_tri_pair(uint64_t w, uint32_t* r, uint32_t* c) {
  uint32_t rr = 0, cc = 0;
  tri_pair(w, &rr, &cc);
  if (r) *r = rr;
  if (c) *c = cc;
}

uint32_t bitrev_debug_spread(uint32_t w, int width) {
  return (width < 0 || width > 32) ? 0u : spread_bits(w, width);
}

}  // extern "C"
