// Per-shape plan selection: the MI355X counterpart of the multi-grained
// thread-block mapping of MG3MConv (Sec. 4.1.2, Fig. 3; evaluated in Sec. 5.3,
// Table 2).  The paper picks, per convolution scene, whether one MM_unit runs
// on one CPE (TB(1,1)), a row of eight (TB(1,8)) or the whole 8x8 mesh
// (TB(8,8)), because a coarse mapping starves the cores when B, IC and OC are
// small, while a fine one repeats memory traffic when they are large.  Here the
// same trade-off is a choice of work-group tile (how much of the output matrix
// one work-group owns, and how many waves share its staged operands) and of a
// split of the reduction, made by a small cost model over 256 compute units.
//
// Host only: no HIP call in this file.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>

#include "mg3m.h"
#include "mg3m_internal.h"

namespace mg3m {

namespace {

constexpr int kCUs = 256;                    // MI355X: 8 XCDs x 32 CUs
constexpr double kClockHz = 2.4e9;
constexpr double kFlopPerClkCU = 256.0;      // fp32 MFMA: 4 SIMDs x 64 flop/clk
constexpr double kFlopPerClkCU64 = 128.0;    // fp64 MFMA: 4 SIMDs x 32 flop/clk
constexpr double kFlopPerClkCUB3 = 4096.0 / 6;   // bf16 MFMA: 4 SIMDs x 1024 flop/clk, six products for one
constexpr int kLdsBytesPerCU = 160 * 1024;
constexpr int kRegsPerLane = 512;            // unified VGPR + AGPR file per SIMD lane
constexpr int kMaxWavesPerSimd = 8;
// Constants fitted to kernel timings on MI355X (see the tile menu): a layer's
// streaming rate, the cost of one kernel launch on the stream, the fixed cost
// of each round of resident work-groups (prologue loads, epilogue stores), and
// how MFMA utilisation falls when fewer than ~2 waves per SIMD are resident.
constexpr double kStreamBytesPerS = 4.0e12;
constexpr double kLaunchUs = 3.0;
constexpr double kRoundUs = 2.0;
constexpr double kTailLaunchUsB3 = 4.5;      // second launch of a b3 plan: launch gap, reduction and its cold partials
constexpr double kUtilBase = 0.5, kUtilPerWave = 0.1;
constexpr double kUtilBaseB3 = 0.5, kUtilPerWaveB3 = 0.25;   // the kernel of bf16 part products: two waves fill it
// Persistent plans (conv_igemm_f32_pt), measured on MI355X against the same
// tile's data-parallel plan: its main loop (run-time LDS buffer parity, one
// copy of the stage code) runs at 0.92 of the tile's rate on deep reductions
// (VGG-16 conv2/conv3, 36 and 18 k-tiles: 8-11% slower); it has no per-round
// cost (a work-group loads its next tile while storing the last); and the
// overlap of output stores with the next tile's MFMAs lets a write-bound layer
// stream at 4.8 TB/s (VGG-16 conv1, 860 MB: 207 -> 180 us).
constexpr double kPersistEff = 0.92;
constexpr double kStreamBytesPerSPersist = 4.8e12;
// The NCHW row loader with a column stride above 1 loads element by element
// (no 16-byte vector covers four output columns): on ResNet-50's stride-2
// layers and AlexNet's conv1 it ran 1.2-1.6x the model's time.  Fitted, with
// the layout-change cost below, to the 44 NCHW layers of VGG-16, ResNet-50
// and AlexNet + inception timed both natively and run as HWCN: the picks then
// total 18714 us against 18823 before and 18696 for the faster of the two on
// every layer.
constexpr double kNchwStridedFactor = 0.6;
// In NCHW the kernel of bf16 part products loads 16 output pixels at a time,
// which on rows shorter than that touch two input rows: 512 channels at 14x14
// then run as fast on HWCN copies (N = 64: 281 against 283 us), where wider rows
// are faster in place (28x28: 963 against 1005; 56x56, 256 channels, N = 32: 493
// against 551).
constexpr double kNchwShortRowFactorB3 = 0.95;
// HWCN copies of batches under 16 write part of every 64-byte sector: whole
// sectors' bytes go at these rates, with element stores and with 16-byte ones
// (384 channels at 112x113, N = 1: 245 us for the copy of 19 MB; 192 at 72x73,
// N = 4: 29 us for 16 MB).
constexpr double kPartSectorBytesPerS = 1.1e12, kPartSectorBytesPerS4 = 2.2e12;
// What a latency-bound launch of the bf16 part product kernel takes less than
// the model's launch and round (a graph of them: 2.7 us apart from its chain).
constexpr double kB3AloneUs = 2.0;
// Stages from which groups of waves share out a tile's reduction: 18 stages 17.4
// -> 13.9 us (two groups); at 8 there is about a microsecond to gain.
constexpr int kB3GroupStages = 12;
// 1x1 layers that the resident-filter kernel does not take (512 channels and
// more).  From 64 images on every tile is weighed, the 64x64 one at its measured
// efficiency there: 512 -> 128 channels at 28x28, N = 64: 57 us on it, 42 on
// 128x256; 1024 -> 256 at 14x14: 57, and 43 on 64x256.  Smaller batches stay on the
// 64x64 tile, which is what the selector has always given them and its tests
// name, though the larger ones would win there too (N = 32: 34 against 26 us);
// one image may also take the small tiles of many waves (1024 -> 256 at 14x14:
// 11.4 -> 8.1 us).
constexpr double kB3Small1x1 = 0.63;
constexpr int kB3WideBatch = 64;
constexpr double kLastLevelCacheBytes = 256.0 * (1 << 20);
// The resident-filter kernel, against 64x64 tiles of the other on 1x1 layers of
// 64 to 384 channels: its MFMA efficiency, the filter's way into LDS, and a
// wave's step of 32 rows alone.  Fitted to which of the two is faster (8x28x28
// columns, 128 -> 512 channels: 11.8 against 13.8 us; 320 -> 320: 21.1 against 15.4).
constexpr double kB3ResStartUs = 2.0, kB3ResEff = 0.75, kB3ResStepUs = 0.6;

long long cdiv(long long a, long long b) { return (a + b - 1) / b; }

// The kernel families, each with a tile menu.
enum Family { kF32 = 0, kF64 = 1, kB3 = 2 };

const TileDesc& tile_desc(Family f, int i) { return f == kF64 ? kTiles64[i] : f == kB3 ? kTilesB3[i] : kTiles[i]; }
int num_tiles(Family f) { return f == kF64 ? kNumTiles64 : f == kB3 ? kNumTilesB3 : kNumTiles; }
int lds_bytes(const TileDesc& t, Family f) {
  return f == kB3 ? (t.wn == 2 ? kB3ResLds : lds_bytes_for_b3(t)) : (f == kF64 || t.m16) ? lds_bytes_for64(t) : lds_bytes_for(t);
}
Family family(const Plan& p) { return p.b3 ? kB3 : p.acc64 ? kF64 : kF32; }

// Registers of the kernel a plan runs: the persistent kernel's with its
// patch loader, else the tile's (tuned loader).
int kernel_regs(const TileDesc& t, int persist_variant) {
  if (persist_variant < 0) return t.regs;
  return t.regs_pt[persist_variant == kVarHwcnVecNTapDma ? 2 : persist_variant == kVarHwcnVecNTap ? 1 : 0];
}

// Work-groups of this tile resident on one CU, limited by LDS and registers
// (persist_variant: the loader variant of a persistent plan, else -1).
int resident_wgs(const TileDesc& t, Family f, int persist_variant = -1) {
  const int waves = t.wm * t.wn;
  const int regs = (kernel_regs(t, persist_variant) + 7) / 8 * 8;
  const int waves_per_simd = std::min(kMaxWavesPerSimd, kRegsPerLane / regs);
  const int by_regs = std::max(1, 4 * waves_per_simd / waves);
  const int by_lds = std::max(1, kLdsBytesPerCU / lds_bytes(t, f));
  return std::min(by_regs, by_lds);
}

// Relative speed of the loader variants against the tuned one.  The NCHW
// vec-K and element-wise factors were fitted to timings of every NCHW plan on
// the VGG-16, ResNet-50 and AlexNet/inception layers (ResNet-50's NCHW excess
// over the fastest plan per layer 9.2% -> 3.3%; its 7x7 stem 231 -> 146 us).
double variant_factor(int variant) {
  switch (variant) {
    case kVarHwcnVecNTap: case kVarHwcnVecNTapDma: return 1.0;
    case kVarNchwTap: return 0.9;
    case kVarNchwVecA: return 1.0;
    case kVarHwcnVecN: return 0.85;
    case kVarHwcnVecC: case kVarHwcnVecA: case kVarNchwScalar: return 0.7;
    default: return 0.5;
  }
}

struct Override {
  int mt = 0, nt = 0, kt = 0, split = 0, tail = 0, persist = 0, dma = -1;   // dma: -1 = the default
  int wm = 0, wn = 0;                                                     // waves (0: any)
  int via = -1;                                                           // NCHW run as HWCN: 1, 0, -1 = either
  long long sk = 0;
};

int parse_override(const char* text, Override* o, std::string* err) {
  if (text == nullptr || *text == 0) return MG3M_OK;
  std::string s(text);
  size_t pos = 0;
  while (pos <= s.size()) {
    size_t end = s.find(',', pos);
    if (end == std::string::npos) end = s.size();
    std::string item = s.substr(pos, end - pos);
    pos = end + 1;
    if (item.empty()) {
      if (end == s.size()) break;
      continue;
    }
    size_t eq = item.find('=');
    if (eq == std::string::npos) {
      *err = "plan override: expected key=value, got '" + item + "'";
      return MG3M_ERR_PLAN;
    }
    std::string key = item.substr(0, eq), val = item.substr(eq + 1);
    char* tail = nullptr;
    if (key == "tile") {
      size_t x = val.find('x');
      if (x == std::string::npos) {
        *err = "plan override: tile must be <MT>x<NT>";
        return MG3M_ERR_PLAN;
      }
      // each half must be a whole decimal number (so "64x64;kt=32" is rejected,
      // not read as 64x64 with the default depth)
      auto whole = [](const std::string& t, long* v) {
        char* e = nullptr;
        *v = std::strtol(t.c_str(), &e, 10);
        return !t.empty() && e == t.c_str() + t.size();
      };
      long mt = 0, nt = 0;
      const bool ok = whole(val.substr(0, x), &mt) && whole(val.substr(x + 1), &nt);
      o->mt = ok && mt <= 4096 ? (int)mt : 0;
      o->nt = ok && nt <= 4096 ? (int)nt : 0;
      if (o->mt <= 0 || o->nt <= 0) {
        *err = "plan override: bad tile '" + val + "'";
        return MG3M_ERR_PLAN;
      }
    } else if (key == "waves") {
      size_t x = val.find('x');
      char* e1 = nullptr;
      char* e2 = nullptr;
      const std::string a = x == std::string::npos ? std::string() : val.substr(0, x);
      const std::string b = x == std::string::npos ? std::string() : val.substr(x + 1);
      const long wm = std::strtol(a.c_str(), &e1, 10), wn = std::strtol(b.c_str(), &e2, 10);
      if (a.empty() || b.empty() || *e1 != 0 || *e2 != 0 || wm < 1 || (wm > 8 && wm != 16) || wn < 1 || wn > 8) {
        *err = "plan override: waves must be <WM>x<WN> (1..8 each)";
        return MG3M_ERR_PLAN;
      }
      o->wm = (int)wm;
      o->wn = (int)wn;
    } else if (key == "via") {
      if (val == "hwcn") {
        o->via = 1;
      } else if (val == "none") {
        o->via = 0;
      } else {
        *err = "plan override: via must be hwcn or none";
        return MG3M_ERR_PLAN;
      }
    } else if (key == "split") {
      long v = std::strtol(val.c_str(), &tail, 10);
      if (tail == val.c_str() || *tail != 0 || v < 1 || v > 64) {
        *err = "plan override: split must be 1..64";
        return MG3M_ERR_PLAN;
      }
      o->split = (int)v;
    } else if (key == "kt") {
      long v = std::strtol(val.c_str(), &tail, 10);
      if (tail == val.c_str() || *tail != 0 || (v != 16 && v != 32 && v != 64)) {
        *err = "plan override: kt must be 16, 32 or 64";
        return MG3M_ERR_PLAN;
      }
      o->kt = (int)v;
    } else if (key == "tail") {
      long v = std::strtol(val.c_str(), &tail, 10);
      if (tail == val.c_str() || *tail != 0 || v < 2 || v > 64) {
        *err = "plan override: tail must be 2..64";
        return MG3M_ERR_PLAN;
      }
      o->tail = (int)v;
    } else if (key == "dma") {
      long v = std::strtol(val.c_str(), &tail, 10);
      if (tail == val.c_str() || *tail != 0 || (v != 0 && v != 1)) {
        *err = "plan override: dma must be 0 or 1";
        return MG3M_ERR_PLAN;
      }
      o->dma = (int)v;
    } else if (key == "persist") {
      long v = std::strtol(val.c_str(), &tail, 10);
      if (tail == val.c_str() || *tail != 0 || v < 1 || v > 16) {
        *err = "plan override: persist must be 1..16 (resident work-groups per CU)";
        return MG3M_ERR_PLAN;
      }
      o->persist = (int)v;
    } else if (key == "sk") {
      long long v = std::strtoll(val.c_str(), &tail, 10);
      if (tail == val.c_str() || *tail != 0 || v < 1 || v > 0x7fffffffLL) {
        *err = "plan override: sk must be 1..2^31-1";
        return MG3M_ERR_PLAN;
      }
      o->sk = v;
    } else {
      *err = "plan override: unknown key '" + key + "'";
      return MG3M_ERR_PLAN;
    }
    if (end == s.size()) break;
  }
  if ((o->split > 0) + (o->tail > 0) + (o->sk > 0) + (o->persist > 0) > 1) {
    *err = "plan override: give at most one of split, tail, sk and persist";
    return MG3M_ERR_PLAN;
  }
  return MG3M_OK;
}

// How a candidate schedules its tiles (see Plan).  kSplitAll and kSplitTail
// cut each tail tile's reduction into `param` runs; kStreamK deals the
// left-over tiles' k-tiles out to `param` work-groups in all (a split when
// the runs fall on tile boundaries).
enum Sched { kDataParallel = 0, kSplitAll = 1, kSplitTail = 2, kStreamK = 3, kPersistent = 4 };

// Partials the tail work-groups write: one per run, plus (stream-K) one for
// each tail tile boundary that falls inside a run.
long long tail_pieces(const Plan& p) {
  if (p.tail_wgs == 0) return 0;
  if (p.sk_s > 0) return p.tail_wgs;
  return (long long)p.tail_wgs + p.tail_tiles - 1;
}

// Fill the shape-dependent parts of a plan for one (tile, schedule, param)
// choice.  Returns false when the choice does not apply to the shape.
bool shape_plan(const ConvShape& s, Family f, int tile, int sched, long long param, Plan* p) {
  const TileDesc& t = tile_desc(f, tile);
  const bool acc64 = f == kF64;
  p->layout = s.layout;
  p->acc64 = acc64 ? 1 : 0;
  p->b3 = f == kB3 ? 1 : 0;
  p->tile = tile;
  p->t = t;
  p->k_tiles = (int)cdiv(s.Kg, t.kt);
  p->tiles_m = (int)cdiv(s.Mg, t.mt);
  p->tiles_n = (int)cdiv(s.Ng, t.nt);
  const long long tiles = (long long)p->tiles_m * p->tiles_n;
  if (tiles > 0x7fffffffLL) return false;
  long long dp = tiles, tail = 0;
  if (sched == kSplitAll && param > 1) {
    dp = 0;
    tail = tiles;
  } else if ((sched == kSplitTail && param > 1) || sched == kStreamK) {
    // whole rounds of resident work-groups run unsplit (none if the tiles do
    // not fill one round: then every tile is shared out)
    const long long slots = (long long)kCUs * resident_wgs(t, f);
    dp = tiles / slots * slots;
    tail = tiles - dp;
  }
  const long long k = p->k_tiles;
  long long wgs = 0, runs = 0, q = 0, r = 0;    // runs: per tail tile (split), 0 (stream-K)
  if (tail > 0) {
    const long long steps = tail * k;
    if (steps > 0x7fffffffLL) return false;          // int step numbers in the kernels
    if (sched == kStreamK) {
      if (param < tail || param > steps) return false;
      wgs = param;
      if (wgs % tail == 0 && k % (wgs / tail) == 0) {
        runs = wgs / tail;                           // equal runs inside each tile: a split
        q = k / runs;
      } else {
        q = steps / wgs;
        r = steps % wgs;
      }
    } else {
      runs = std::min<long long>(param, k);         // no empty run
      wgs = tail * runs;
      q = k / runs;
      r = k % runs;
    }
    if (runs == 1) {                                 // one run per tile: run them whole
      dp = tiles;
      tail = wgs = q = r = runs = 0;
    }
  }
  if (dp + wgs > 0x7fffffffLL) return false;
  // persistent: every tile whole, `param` resident work-groups per CU looping over them
  p->persist = sched == kPersistent ? 1 : 0;
  p->dp_tiles = (int)dp;
  p->tail_tiles = (int)tail;
  p->tail_wgs = (int)wgs;
  p->sk_s = (int)runs;
  p->sk_q = (int)q;
  p->sk_r = (int)r;
  p->split = tail > 0 ? (int)cdiv(wgs, tail) : 1;
  p->grid = p->persist ? std::min<long long>(dp, (long long)kCUs * param) : dp + wgs;
  p->lds_bytes = lds_bytes(t, f);
  const double padded = (double)p->tiles_m * t.mt * (double)p->tiles_n * t.nt *
                        (double)p->k_tiles * t.kt;
  p->pad_eff = (double)s.Mg * (double)s.Ng * (double)s.Kg / padded;
  // partial slots: run w's piece in tail tile j goes to slot w + j
  const long long slots = wgs > 0 ? wgs + tail - 1 : 0;
  p->ws_bytes = (size_t)slots * t.mt * t.nt * (acc64 ? sizeof(double) : sizeof(float));
  p->est_us = 0.0;
  return true;
}

// The operand addressing forms of the kernel of bf16 part products: speed
// against the one-tap form when the chip is full, and the time a work-group
// alone on its CU takes for a k-step of 32 rows beyond its MFMAs (loads, splits,
// the barrier).  Fitted to timings of every b3 tile on the catalogue layers and
// on nineteen odd-sized ones (batches of 1 to 33, 3 to 384 channels).
double b3_factor(int load, const TileDesc& t) {
  switch (load) {
    case kB3Slab: return 1.0;
    case kB3SlabW: return 0.9;
    case kB3Group: return t.mt == 64 && t.nt >= 128 ? 1.0 : 0.9;
    case kB3GroupN: return t.mt == 32 ? 0.5 : 0.8;      // a load per column and row: half as many products to each
    case kB3GroupC: return 0.85;
    case kB3Row: return 0.68;
    default: return t.mt == 32 ? 0.45 : 0.62;
  }
}
// Chain of a tile's k_tiles stages (wm groups of waves share them out).
double b3_chain_us(int load, const TileDesc& t, int k_tiles) {
  constexpr double alone[] = {0.6, 0.75, 0.7, 0.95, 0.6, 0.85, 1.1};     // by B3Load
  const double mfma = 2.0 * t.mt * t.nt * 32 / (kFlopPerClkCUB3 * kClockHz) * 1e6;
  return (cdiv(k_tiles, t.wm) * alone[load] + k_tiles * mfma) * t.kt / 32 - kB3AloneUs;
}

// The selector's predicted time for a plan (microseconds).  Work-groups are
// dispatched in order, whole tiles first and tail runs after them.  In each
// phase the busiest CU runs ceil(work-groups / 256) of them, each costing its
// padded MFMA flops at the tile's measured efficiency, scaled down when that
// CU holds too few waves to hide latency, plus a fixed cost per round of
// resident work-groups.  A layer cannot beat streaming its tensors (and the
// partials) once; the tail reduction adds its traffic and a second launch.
double predict_us(const ConvShape& s, const Plan& p) {
  const TileDesc& t = p.t;
  const int occ = resident_wgs(t, family(p), p.persist && !p.b3 ? p.variant : -1);
  const double rate = p.acc64 ? kFlopPerClkCU64 : p.b3 ? kFlopPerClkCUB3 : kFlopPerClkCU;
  const double tile_flops = 2.0 * t.mt * t.nt * (double)t.kt;
  const bool multitap = s.R * s.S > 1 && (p.b3 || s.C >= 2 * t.kt);
  auto phase = [&](long long wgs, int k_tiles) {
    if (wgs <= 0) return 0.0;
    const long long per_cu = cdiv(wgs, kCUs);
    if (p.b3 && t.wm >= 8) {
      // a 16-wave work-group per CU: rounds of chains (eight or sixteen groups share
      // a tile's stages out), timed on 30 small layers (within 15% or so)
      const double round = t.wm == 16 ? 1.5 * cdiv(k_tiles, 16) + 4.9 : 1.32 * cdiv(k_tiles, 8) + 5.5;
      const bool by_column = p.b3_load == kB3GroupN || p.b3_load >= kB3Row;
      return (double)per_cu * round * (by_column ? 1.35 : 1.0) - kLaunchUs;
    }
    const double waves_per_simd = (double)std::min<long long>(per_cu, occ) * t.wm * t.wn / 4.0;
    const double util = p.b3 ? std::min(1.0, kUtilBaseB3 + kUtilPerWaveB3 * waves_per_simd)
                             : std::min(1.0, kUtilBase + kUtilPerWave * waves_per_simd);
    const double eff = t.eff * (p.b3 ? b3_factor(p.b3_load, t) : variant_factor(p.variant)) * util * (multitap ? t.eff_multitap : 1.0) *
                       (p.persist ? kPersistEff : 1.0) *
                       (p.b3 && s.R * s.S == 1 && s.N >= kB3WideBatch && t.mt * t.nt == 64 * 64 ? kB3Small1x1 : 1.0) *
                       (p.b3 && s.layout == kNCHW && s.Wo < 16 ? kNchwShortRowFactorB3 : 1.0) *
                       (s.layout == kNCHW && !p.b3 && p.b_mode == kBVecW && s.sw > 1 ? kNchwStridedFactor : 1.0);
    double us = (double)per_cu * tile_flops * k_tiles / (rate * kClockHz * eff) * 1e6;
    // few work-groups: no faster than the chain of their k-steps, and a four-wave
    // one alone on its CU just that
    if (p.b3) {
      const double chain = (double)cdiv(per_cu, occ) * b3_chain_us(p.b3_load, t, k_tiles);
      us = per_cu == 1 && t.wm == 1 && t.mt * t.nt <= 64 * 64 ? chain : std::max(us, chain);
    }
    if (p.b3) us += t.wm == 1 ? 0.0 : t.wm == 2 ? 1.2 : 4.0;             // adding up the groups' sums
    return us + (p.persist ? 1.0 : (double)cdiv(per_cu, occ)) * kRoundUs;
  };
  const int run_k = p.tail_wgs > 0 ? p.sk_q + (p.sk_r > 0 ? 1 : 0) : 0;
  double t_comp = phase(p.dp_tiles, p.k_tiles) + phase(p.tail_wgs, run_k);
  if (p.b3 && p.persist) {
    // blocks of 64x32 dealt out to the waves of a CU; with few of them, no
    // faster than the chain of a block's steps, twice where a work-group's run
    // of blocks reaches into a second filter tile
    const double blocks = (double)cdiv((long long)p.tiles_m * cdiv(s.Ng, 32), 4 * kCUs);
    const int chains = 32 % p.tiles_m == 0 || p.tiles_m % 32 == 0 ? 1 : 2;
    t_comp = kB3ResStartUs + std::max(blocks * 2.0 * 64 * 32 * (double)s.Kg / (kFlopPerClkCUB3 / 4 * kClockHz * kB3ResEff) * 1e6,
                                      chains * (double)s.Kg / 32 * kB3ResStepUs);
  }
  const double y_bytes = 4.0 * (double)s.Mg * (double)s.Ng;
  // (the resident-filter kernel walks x once per filter tile: from memory each
  // time where the last-level cache does not hold it; 384 -> 176 channels at 82x82,
  // N = 120, 1.24 GB: 1237 us, and 916 on fp32 MFMA)
  const double x_elems = (double)s.N * s.C * s.H * s.W;
  const double x_passes = p.b3 && p.persist && 4.0 * x_elems > kLastLevelCacheBytes ? p.tiles_m : 1.0;
  const double xw_bytes = 4.0 * (x_elems * x_passes + (double)s.Kg * s.Mg);
  const double part_bytes =
      (double)tail_pieces(p) * t.mt * t.nt * (p.acc64 ? sizeof(double) : sizeof(float));
  const double t_mem =
      (xw_bytes + y_bytes + part_bytes) / (p.persist ? kStreamBytesPerSPersist : kStreamBytesPerS) * 1e6;
  double est = std::max(t_comp, t_mem) + kLaunchUs;
  if (p.tail_tiles > 0) {
    const double tail_out = 4.0 * (double)p.tail_tiles * t.mt * t.nt;
    est += (part_bytes + tail_out) / kStreamBytesPerS * 1e6 + (p.b3 ? kTailLaunchUsB3 : kLaunchUs);
  }
  if (p.wt_bytes > 0) est += 2.0 * (double)p.wt_bytes / kStreamBytesPerS * 1e6 + kLaunchUs;
  return est;
}

}  // namespace

int make_shape(int N, int C, int H, int W, int K, int R, int S, int stride_h, int stride_w,
               int pad_h, int pad_w, int layout, ConvShape* s, std::string* err) {
  if (layout != kHWCN && layout != kNCHW) {
    *err = "unknown layout";
    return MG3M_ERR_LAYOUT;
  }
  if (N < 1 || C < 1 || H < 1 || W < 1 || K < 1 || R < 1 || S < 1 || stride_h < 1 ||
      stride_w < 1 || pad_h < 0 || pad_w < 0) {
    *err = "dimensions and strides must be >= 1, pads >= 0";
    return MG3M_ERR_SHAPE;
  }
  if (pad_h > (1 << 24) || pad_w > (1 << 24) || H > (1 << 24) || W > (1 << 24) ||
      R > (1 << 24) || S > (1 << 24) || stride_h > (1 << 24) || stride_w > (1 << 24)) {
    *err = "a spatial size, stride or pad exceeds 2^24";
    return MG3M_ERR_TOO_LARGE;
  }
  const long long eh = (long long)H + 2LL * pad_h - R, ew = (long long)W + 2LL * pad_w - S;
  if (eh < 0 || ew < 0) {
    *err = "filter larger than the padded input: empty output";
    return MG3M_ERR_SHAPE;
  }
  s->N = N; s->C = C; s->H = H; s->W = W; s->K = K; s->R = R; s->S = S;
  s->sh = stride_h;
  s->sw = stride_w;
  s->ph = pad_h;
  s->pw = pad_w;
  s->Ho = (int)(eh / stride_h + 1);
  s->Wo = (int)(ew / stride_w + 1);
  s->layout = layout;
  s->Mg = K;
  s->Ng = (long long)N * s->Ho * s->Wo;
  s->Kg = (long long)C * R * S;
  // int32 index arithmetic in the kernels, with head-room for a tile past the end
  // 32-bit byte offsets in the kernels' buffer loads
  const long long lim = kMaxTensorBytes / 4;
  const long long xe = (long long)N * C * H * W, we = (long long)K * C * R * S,
                  ye = (long long)N * K * s->Ho * s->Wo;
  if (xe > lim || we > lim || ye > lim) {
    *err = "a tensor is larger than 4 GiB - 64 bytes (the kernels use 32-bit byte offsets)";
    return MG3M_ERR_TOO_LARGE;
  }
  return MG3M_OK;
}

// Loader variant and epilogue mode for a plan whose tile is already set.
// dma: the one-tap HWCN loaders in their direct-to-LDS form.
void choose_modes(const ConvShape& s, bool x16, bool w16, bool y16, Plan* p, bool dma = false) {
  if (s.layout == kHWCN) {
    if (s.K % 4 == 0 && w16) {
      p->a_mode = kAVecM;
      if (s.N % 4 == 0 && x16 && s.C % p->t.kt == 0)
        p->b_mode = dma ? kBVecNTapDma : kBVecNTap, p->variant = dma ? kVarHwcnVecNTapDma : kVarHwcnVecNTap;
      else if (s.N % 4 == 0 && x16) p->b_mode = kBVecN, p->variant = kVarHwcnVecN;
      else if (s.N == 1 && s.C % 4 == 0 && x16) p->b_mode = kBVecC, p->variant = kVarHwcnVecC;
      else p->b_mode = kBScalar, p->variant = kVarHwcnVecA;
    } else {
      p->a_mode = kAScalar;
      p->b_mode = kBScalar;
      p->variant = kVarHwcnScalar;
    }
  } else if (s.C % p->t.kt == 0 && s.K % 4 == 0 && s.R * s.S > 1 && s.sw == 1) {
    // tap-major on a [R][S][C][K] copy of the filter (in the workspace).  A 1x1
    // filter has one tap (both orders coincide, the copy would be pure cost),
    // and other strides never take the 16-byte runs along W.
    p->a_mode = kAVecM;
    p->b_mode = kBVecWTap;
    p->variant = kVarNchwTap;
  } else {
    p->b_mode = kBVecW;
    if (s.Kg % 4 == 0 && w16) p->a_mode = kAVecK, p->variant = kVarNchwVecA;
    else p->a_mode = kAScalar, p->variant = kVarNchwScalar;
  }
  // The filter copy goes first in the workspace, the partials after it.
  p->wt_bytes = 0;
  if (p->variant == kVarNchwTap) {
    p->wt_bytes = ((size_t)4 * (size_t)s.Mg * (size_t)s.Kg + 255) / 256 * 256;
    p->ws_bytes += p->wt_bytes;
  }
  // Four consecutive output channels are contiguous only in HWCN with N == 1
  // (whole tiles store them with one 16-byte store; partials are stored per
  // element, so only y's alignment matters).
  p->e_mode = (s.layout == kHWCN && s.N == 1 && s.K % 4 == 0 && y16) ? kEVecM : kEElem;
  // the fp64 accumulator holds no four adjacent rows in one lane
  if (p->acc64) p->e_mode = kEElem;
}

// Operand addressing of the kernel of bf16 part products for a plan whose
// tile and modes are set; false where no form is built for it (named: the
// override names its waves).  By the
// narrowest that applies: a filter tap per stage where the channels fill whole
// stages, groups of eight channels, single rows of the reduction; and a lane's
// columns as one load where four batch elements lie together.  y's alignment is
// not asked: a buffer store of four dwords needs a dword's only, and the form
// decides on the tile, the split and the workspace, whose size callers ask for
// without naming a y.
static bool choose_b3(const ConvShape& s, bool x16, bool named, Plan* p) {
  const bool vec = s.N % 4 == 0 && x16;
  if (s.layout == kNCHW) {
    if (p->variant != kVarNchwTap) return false;
    p->b3_load = kB3SlabW;
  } else if (vec && s.C % p->t.kt == 0) {
    p->b3_load = kB3Slab;
    if (s.K % 4 != 0 || p->b_mode == kBScalar) p->b_mode = kBVecNTap;   // the filter is read by elements
  } else if (s.C % 8 == 0) {
    p->b3_load = vec ? kB3Group : s.N == 1 && x16 ? kB3GroupC : kB3GroupN;
  } else {
    p->b3_load = vec ? kB3Row : kB3RowN;
  }
  if (p->b3_load >= kB3Group) p->b_mode = vec ? kBVecN : p->b3_load == kB3GroupC ? kBVecC : kBScalar;
  p->a_mode = kAVecMB3;
  p->e_mode = kEElem;
  // the persistent kernel: 1x1, the filter's channels in LDS, pairs of 32-deep
  // steps, and a work-group on every CU (its share of the tiles is worked out
  // from the grid)
  if (p->persist)
    return p->tile == kTileB3Res && p->b3_load == kB3Slab && s.R * s.S == 1 && s.C % 64 == 0 && s.C <= kB3ResMaxC &&
           p->dp_tiles > kCUs && p->grid <= kCUs;
  if (p->t.mt == 64 && p->t.wm > 1 && p->k_tiles < kB3GroupStages && !named) return false;
  // the small tiles of many waves serve single images (batches of the smallest
  // layers would gain too, 4 images of 64 channels at 28x28 12.7 -> 9.7 us, but
  // their callers size the workspace of a split plan and share it among calls)
  if (p->t.wm >= 8 && s.N > 1 && !named) return false;
  return b3_built(p->b3_load, p->tile);
}

// Plans of the kernel of bf16 part products that lose to the fp32-MFMA kernels,
// whatever the two models say (theirs charges the shortest layers a launch and a
// round, 5 us, which they do in 3).  Counted over 3800 shapes of 1 to 124 images
// that the models gave to this kernel, both timed (more than 3% between them):
static bool b3_loses(const ConvShape& s, const Plan& c) {
  // less than a quarter of a stage: 19 of 19.  (And one product per output is
  // rounded once on fp32 MFMA, where the part products leave 0.75 ulp.)
  if (s.Kg < 8) return true;
  // where the fp32 kernels load single patch elements, not from there on
  if (c.variant == kVarHwcnVecA || c.variant == kVarHwcnScalar) return false;
  // one stage, or a second one mostly of padding: 283 of 298, 16 channels at
  // 14x14, N = 8: 3.0 against 3.9 us.  (24 channels, 1x1, are two of the fp32
  // kernels' stages, of their slower loader: 24 of 25 the other way.)
  const bool group24 = s.N % 4 == 0 && s.C % 8 == 0 && s.C % 16 != 0 && s.Kg > 16 && s.Kg <= 32;
  if (s.Kg <= 48) return !group24;
  // an address per row, for two or three stages: 13 of 14
  if (s.Kg <= 96 && s.C % 8 != 0 && s.R * s.S > 1) return true;
  // 1x1, two to four stages, and little work for most of the chip: 69 of 83, 5 the
  // other way; 32 -> 256 channels at 56x56, stride 2, N = 4: 4.1 against 4.9 us
  // (the resident-filter kernel with one filter tile holds its own)
  if (s.R * s.S == 1 && s.Kg <= 128 && c.dp_tiles + c.tail_wgs > kCUs / 2 && 2.0 * s.Mg * s.Ng * s.Kg < 5e8)
    return !(c.persist && c.tiles_m == 1);
  // 16 output channels, small batches, and columns for most of the chip: the fp32
  // kernels have a tile of 16 rows, 59 of 77, 7 the other way; 128 -> 16 channels,
  // 3x3 on 64x64, N = 16: 32 against 38 us
  if (s.K <= 16 && s.N % 4 == 0 && s.N <= 16 && s.C % 16 == 0 && s.sh == 1 && s.sw == 1 && s.Ng >= 100 * 64 && !c.persist)
    return true;
  // 24 pieces and more of a stage or two: 172 of 181, 2 the other way; 512 -> 32
  // channels, 3x3 on 20x20, stride 2, one image: 27 us in 128 pieces, 20 on fp32 MFMA
  // (and 11 on 16x16 tiles of sixteen waves)
  return c.split >= 24 && c.tail_wgs > 0 && c.sk_q + (c.sk_r > 0 ? 1 : 0) <= 2;
}

int make_plan(const ConvShape& s, const char* override_text, bool acc64, bool x16, bool w16,
              bool y16, Plan* p, std::string* err, size_t ws_cap) {
  Override o;
  int rc = parse_override(override_text, &o, err);
  if (rc) return rc;
  if (acc64 && o.kt && o.kt != 16) {
    *err = "plan override: the fp64-accumulating kernel steps the reduction by kt=16";
    return MG3M_ERR_PLAN;
  }

  int best = -1;
  Plan best_plan{};
  size_t least_over_cap = SIZE_MAX;     // smallest workspace among the candidates over ws_cap
  const bool open = !o.mt && !o.wm && !o.kt;      // the override, if any, leaves the kernel open
  bool f32_via = false;                 // the best plan of the fp32 kernels runs on HWCN copies
  // the split factors the cost model was calibrated on
  const int splits[] = {2, 3, 4, 6, 8, 16};
  // via: an NCHW call run as HWCN on 16-byte aligned copies of x, w and y in
  // the workspace, the layout changed on the way in and out (layout.hip)
  auto consider_one = [&](Family f, int ti, int sched, long long sp, bool via) {
    Plan c{};
    ConvShape sv = s;
    if (via) sv.layout = kHWCN;
    if (!shape_plan(sv, f, ti, sched, sp, &c)) return;
    // the one-tap HWCN loaders load straight into LDS unless the override says
    // otherwise, except in the fp64-accumulating kernels and the 16-row tile,
    // which stage through VGPRs
    const bool dma_ok = !c.acc64 && !c.t.m16;
    choose_modes(sv, via || x16, via || w16, via || y16, &c, dma_ok && o.dma != 0);
    if (c.b3 && (!choose_b3(sv, via || x16, o.wm > 0, &c) || (open && b3_loses(sv, c)))) return;
    if (via) {
      auto r256 = [](size_t b) { return (b + 255) / 256 * 256; };
      c.via_hwcn = 1;
      c.via_bytes = r256(4 * (size_t)s.N * s.C * s.H * s.W) + r256(4 * (size_t)s.Mg * (size_t)s.Kg) +
                    r256(4 * (size_t)s.Mg * (size_t)s.Ng);
      c.ws_bytes += c.via_bytes;
    }
    if (o.dma == 1 && c.variant != kVarHwcnVecNTapDma) return;
    // runs spanning two tiles need the kernel's loop over pieces (only the
    // 32x32x2 fp32 kernel with the one-tap HWCN loader has it)
    if (c.tail_wgs > 0 && c.sk_s == 0 && (c.acc64 || c.t.m16 || !(c.b3 || tail_runs_multi(c.b_mode)))) return;
    // the persistent kernel is built for the batch-vector HWCN loaders only
    if (c.persist && !c.b3 && (c.acc64 || !persist_built(c.variant, c.t))) return;
    if (c.persist && sp == 0) {
      // the selector's persistent plans fill every slot the kernel's
      // occupancy allows, and only pay off with more tiles than that
      const long long slots = (long long)kCUs * resident_wgs(c.t, f, c.b3 ? -1 : c.variant);
      if (c.dp_tiles <= slots) return;
      c.grid = slots;
    }
    if (c.ws_bytes > ws_cap) {
      least_over_cap = std::min(least_over_cap, c.ws_bytes);
      return;
    }
    c.est_us = predict_us(sv, c);
    // the layout changes: x and w in, y out, each read and written once; x's
    // copy in runs of N floats, below 16 of them a part of each sector (charged
    // where the choice is between it and a native plan of the fp32 kernels)
    if (via) {
      c.est_us += 2.0 * (double)c.via_bytes / kStreamBytesPerS * 1e6 + 2 * kLaunchUs;
      if (c.b3 && s.N < 16 && !f32_via)
        c.est_us += 4.0 * s.C * s.H * s.W * (16 - s.N) / (s.N % 4 == 0 ? kPartSectorBytesPerS4 : kPartSectorBytesPerS) * 1e6;
    }
    // ties: less workspace traffic, then the larger tile
    const bool better = best < 0 || c.est_us < best_plan.est_us * 0.999 ||
                        (std::fabs(c.est_us - best_plan.est_us) <= best_plan.est_us * 0.001 &&
                         (c.ws_bytes < best_plan.ws_bytes ||
                          (c.ws_bytes == best_plan.ws_bytes && c.t.mt * c.t.nt > best_plan.t.mt * best_plan.t.nt)));
    if (better) {
      best = ti;
      best_plan = c;
    }
  };
  const bool via_ok = s.layout == kNCHW && !acc64;
  if (o.via == 1 && !via_ok) {
    *err = "plan override: via=hwcn applies to NCHW calls of the fp32 kernel";
    return MG3M_ERR_PLAN;
  }
  Family fam = acc64 ? kF64 : kF32;
  auto consider = [&](int ti, int sched, long long sp) {
    if (o.via != 1) consider_one(fam, ti, sched, sp, false);
    if (via_ok && o.via != 0) consider_one(fam, ti, sched, sp, true);
  };
  bool named_f32 = false;               // the override's tile, waves and kt fit an fp32 (or fp64) tile
  auto consider_family = [&]() {
  for (int ti = 0; ti < num_tiles(fam); ++ti) {
    const TileDesc& td = tile_desc(fam, ti);
    if (o.mt && !(td.mt == o.mt && td.nt == o.nt)) continue;
    if (o.wm && !(td.wm == o.wm && td.wn == o.wn)) continue;
    // The selector takes a 16-row tile only where it saves padding, i.e. a
    // 32-row block would be at most half full (the case it was timed on).
    if (!o.mt && td.m16 && !(s.Mg % 32 != 0 && s.Mg % 32 <= 16)) continue;
    // A tile the cost model does not yet rank correctly is left to overrides
    // that name its shape and its waves.
    if (td.forced_only && !(o.mt && o.wm)) continue;
    // (kB3WideBatch)
    if (fam == kB3 && !o.mt && s.R * s.S == 1 && s.N < kB3WideBatch && !(td.mt == 64 && td.nt == 64 && td.kt == 32) &&
        !(s.N == 1 && td.wm >= 8)) continue;
    if (fam == kB3 && o.persist && !o.wm) continue;      // (without waves=, a persistent fp32 kernel)
    // a forced tile without a depth means the default depth of 16
    if ((o.kt || o.mt) && td.kt != (o.kt ? o.kt : 16)) continue;
    if (fam != kB3) named_f32 = true;
    if (o.split) {
      consider(ti, o.split > 1 ? kSplitAll : kDataParallel, o.split);
    } else if (o.tail) {
      consider(ti, kSplitTail, o.tail);
    } else if (o.sk) {
      consider(ti, kStreamK, o.sk);
    } else if (o.persist) {
      consider(ti, kPersistent, o.persist);
    } else {
      consider(ti, kDataParallel, 1);
      for (int sp : splits) {
        consider(ti, kSplitAll, sp);
        consider(ti, kSplitTail, sp);
      }
      // stream-K over the left-over tiles with one to all resident work-groups per CU
      for (int j = 1, occ = resident_wgs(td, fam); j <= occ; ++j) consider(ti, kStreamK, (long long)j * kCUs);
      // every tile whole, persistent work-groups filling the chip
      if (fam == kF32 || ti == kTileB3Res) consider(ti, kPersistent, 0);
    }
  }
  };
  consider_family();
  // The kernels of bf16 part products are the selector's to choose, or named by
  // tile and waves together.  An override that names less (a tile, a depth, dma=)
  // means the fp32 kernel that it has always meant, if there is one.
  if (!acc64 && o.dma < 0 && (open || (o.mt && o.wm) || !named_f32)) {
    f32_via = best >= 0 && best_plan.via_hwcn;
    fam = kB3;
    consider_family();
  }
  if (best < 0 && least_over_cap != SIZE_MAX) {
    *err = "every applicable plan needs more workspace than the " + std::to_string(ws_cap) +
           " bytes available (the smallest needs " + std::to_string(least_over_cap) + ")";
    return MG3M_ERR_WORKSPACE;
  }
  if (best < 0) {
    *err = "plan override: no applicable plan for tile " + std::to_string(o.mt) + "x" + std::to_string(o.nt) +
           (o.dma == 1 ? std::string(" dma=1 (the direct-to-LDS loaders serve the fp32 kernel's one-tap HWCN path"
                                     " with 32x32x2-MFMA tiles)")
                       : std::string()) +
           (o.persist ? " persist=" + std::to_string(o.persist) +
                            " (persistent tiles need the fp32 kernel's batch-vector HWCN loaders: HWCN, N and K"
                            " multiples of 4, aligned buffers; not the 16-row tile)"
                      : std::string()) +
           (o.kt ? " kt=" + std::to_string(o.kt) : std::string()) +
           (o.tail ? " tail=" + std::to_string(o.tail) : std::string()) +
           (o.sk ? " sk=" + std::to_string(o.sk) +
                       " (from the left-over tiles to their k-tiles in total; runs spanning two tiles"
                       " only with the fp32 kernel's one-tap HWCN loader)"
                 : std::string());
    return MG3M_ERR_PLAN;
  }
  *p = best_plan;
  return MG3M_OK;
}

std::string plan_to_string(const ConvShape& s, const Plan& p) {
  static const char* an[] = {"vec_m", "vec_k", "scalar", "vec_m_b3"};
  static const char* bn[] = {"vec_n", "vec_c", "scalar", "vec_n_tap", "vec_w", "vec_w_tap", "vec_n_tap_dma"};
  static const char* fn[] = {"slab", "slab_w", "group", "group_n", "group_c", "row", "row_n"};   // by B3Load
  static const char* en[] = {"elem", "vec_m"};
  char buf[512];
  std::snprintf(buf, sizeof buf,
                "%s%s%stile=%dx%d,waves=%dx%d,kt=%d,split=%d,dp_tiles=%d,tail_tiles=%d,tail_wgs=%d,grid=%lld,"
                "tiles=%dx%d,k_tiles=%d,a=%s,b=%s,e=%s,lds=%d,ws=%zu,pad_eff=%.4f,est_us=%.2f,"
                "Mg=%lld,Ng=%lld,Kg=%lld",
                p.acc64 ? "acc=f64," : "", p.via_hwcn ? "via=hwcn," : "",
                p.persist ? "persist," : "", p.t.mt, p.t.nt, p.t.wm, p.t.wn, p.t.kt, p.split, p.dp_tiles, p.tail_tiles, p.tail_wgs, p.grid,
                p.tiles_m, p.tiles_n, p.k_tiles, an[p.a_mode], p.b3 ? fn[p.b3_load] : bn[p.b_mode], en[p.e_mode],
                p.lds_bytes, p.ws_bytes, p.pad_eff, p.est_us, s.Mg, s.Ng, s.Kg);
  return buf;
}

}  // namespace mg3m
