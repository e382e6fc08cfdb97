// Host-only fuzz of libchunkft's C++ (planner, plan summary, schedule, argument validation,
// token-split and workspace logic), meant to be built with g++ -fsanitize=address,undefined
// from plan.cpp + api.cpp + shape.cpp.  The kernel launchers are replaced by stand-ins that
// launch nothing and instead check, on the host, what a kernel would have been handed: ranges
// inside the tensor, slabs that cover the tokens, partial sums that stay inside the caller's
// workspace.  No GPU, no HIP.  Exit code 0 and a line "ok ..." on success.

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "chunkft.h"
#include "internal.h"
#include "slab_offset.h"

namespace {
long g_launches = 0;
const char* g_fail = nullptr;
uintptr_t g_ws_lo = 0, g_ws_hi = 0;     // the workspace handed to the call under test

void expect(bool ok, const char* what) {
  if (!ok && !g_fail) g_fail = what;
}

void check_problem(const chunkft::WgradProblem& p) {
  expect(p.begin >= 0 && p.begin < p.end, "range order");
  expect(p.out > 0 && p.in > 0 && p.end <= p.out * p.in, "range inside the tensor");
  expect(p.T > 0 && p.S >= 1 && p.kslab > 0, "slab shape");
  expect((int64_t)p.S * p.kslab >= p.T && (int64_t)(p.S - 1) * p.kslab < p.T, "slabs cover the tokens, none empty");
}

void check_partials(const chunkft::WgradProblem& p, const chunkft::Sinks& s) {
  if (p.S <= 1) return;
  const int64_t E = p.end - p.begin;
  expect(s.ws_pitch >= E, "slab pitch");
  const uintptr_t lo = reinterpret_cast<uintptr_t>(s.ws);
  const uintptr_t hi = lo + 4u * (uintptr_t)((int64_t)(p.S - 1) * s.ws_pitch + E);
  expect(lo >= g_ws_lo && hi <= g_ws_hi, "partial sums inside the workspace");
}
}  // namespace

namespace chunkft {
int device_compute_units() { return kDefaultComputeUnits; }
int launch_wgrad_bf16_mfma(const WgradProblem& p, int mode, const Sinks& s, void*) {
  ++g_launches;
  check_problem(p);
  expect(mfma_path_ok(p), "MFMA path taken for a shape it cannot load");
  const RowSplit rs = split_rows(p);
  expect(rs.rb0 % 8 == 0 && rs.rb1 >= rs.rb0 && rs.rb1 <= p.out, "body rows");
  expect(rs.rb1 == rs.rb0 || (rs.rb0 * p.in >= p.begin && rs.rb1 * p.in <= p.end), "body rows lie inside the range");
  expect(rs.lead_base < 0 || (rs.lead_base % 8 == 0 && rs.lead_base + 8 == rs.rb0), "leading group");
  expect(rs.trail_row < rs.rb1 + 1 || rs.trail_row < p.out, "trailing row");
  if (mode == EMIT_PARTIAL) check_partials(p, s);
  return 0;
}
int launch_wgrad_ragged(const WgradProblem& p, int mode, const Sinks& s, void*) {
  ++g_launches;
  check_problem(p);
  if (mode == EMIT_PARTIAL) check_partials(p, s);
  return 0;
}
int launch_wgrad_f32(const WgradProblem& p, int mode, const Sinks& s, void* stream) { return launch_wgrad_ragged(p, mode, s, stream); }
int launch_colsum(const WgradProblem& p, int, int, const Sinks&, void*) { ++g_launches; check_problem(p); expect(p.S == 1, "vector split"); return 0; }
int launch_norm_wgrad(const WgradProblem& p, int, bool, float, float* stats, int, const Sinks&, void*) {
  ++g_launches;
  check_problem(p);
  const uintptr_t lo = reinterpret_cast<uintptr_t>(stats);
  expect(lo >= g_ws_lo && lo + 8u * (uintptr_t)p.T <= g_ws_hi, "statistics inside the workspace");
  return 0;
}
int launch_embed_wgrad(const WgradProblem& p, int, int, const Sinks&, void*) { ++g_launches; check_problem(p); expect(p.T <= kMaxEmbeddingTokens, "tokens per call"); return 0; }
int launch_reduce(const float* ws, int32_t S, int64_t E, int, const Sinks& s, void*, void*) {
  ++g_launches;
  const uintptr_t lo = reinterpret_cast<uintptr_t>(ws);
  expect(S >= 2 && E > 0 && s.ws_pitch >= E, "reduction shape");
  expect(lo >= g_ws_lo && lo + 4u * (uintptr_t)((int64_t)(S - 1) * s.ws_pitch + E) <= g_ws_hi, "reduction reads inside the workspace");
  return 0;
}
int launch_fused_group(const GroupSegment* segs, int n, bool, void*) {
  g_launches += n > 0;
  for (int i = 0; i < n; ++i) {
    check_problem(segs[i].p);
    expect(segs[i].p.S == 1, "grouped segment with a token split");
    expect(group_takes_segment(segs[i].p, segs[i].vector), "grouped segment the kernel cannot take");
    if (!segs[i].vector) expect(mfma_path_ok(segs[i].p), "grouped matrix segment off the MFMA path");
  }
  return 0;
}
int launch_adamw(const float*, int64_t n, const Sinks&, void*, void*) { ++g_launches; expect(n > 0, "adamw size"); return 0; }
}  // namespace chunkft

// Every load of every slab, as the kernels that fetch by slab_offset() cut it: slabs of `slab` tokens, loads of
// `tokens` tokens.  Each lane must name a token of the slab, its own one where that is there and the last one past the
// end, with both parts of the offset non-negative: their sum, taken without wrapping, is the address.
bool slab_offsets_ok(int slab, int tokens, unsigned column, unsigned token_bytes) {
  for (int left = 1; left <= slab + 1; ++left)
    for (int first = 0; first < slab; first += tokens)
      for (int k = 0; k < tokens; ++k) {
        const chunkft::LoadOffset o = chunkft::slab_offset(column, token_bytes, first, k, left, slab);
        const uint64_t token = first + k < left ? first + k : left - 1;
        if ((uint64_t)o.lane + o.scalar != column + token * token_bytes) {
          printf("slab of %d tokens, %d left, load of token %d, lane token %d: offset %llu, token %llu is at %llu\n", slab, left, first, k,
                 (unsigned long long)o.lane + o.scalar, (unsigned long long)token, (unsigned long long)(column + token * token_bytes));
          return false;
        }
      }
  return true;
}

// Which tile a chunk takes: what the large kernel cannot carry (no body row, edge rows beside a body of at most 128
// rows) goes to the small tiles whatever its size, and nothing else does beyond the line in tiles and tokens, however
// short its body is.
bool tile_rule_ok(std::mt19937_64& rng) {
  const int cus = chunkft::kDefaultComputeUnits;
  for (int it = 0; it < 200000; ++it) {
    chunkft::WgradProblem p{};
    p.in = 8 * (1 + (int64_t)(rng() % (rng() % 2 ? 600 : 20000)));
    p.T = 1 + (int64_t)(rng() % 16384);
    const int64_t r0 = (int64_t)(rng() % 300), rows = 1 + (int64_t)(rng() % (rng() % 2 ? 150 : 3000));
    p.begin = r0 * p.in;
    p.end = (r0 + rows) * p.in;
    if (rng() % 2) p.begin += (int64_t)(rng() % (uint64_t)p.in);                 // from mid-row
    if (rng() % 2) p.end -= (int64_t)(rng() % (uint64_t)(p.in - (rows == 1 ? p.begin % p.in : 0)));
    const chunkft::RowSplit rs = chunkft::split_rows(p);
    const int64_t body = rs.rb1 - rs.rb0;
    const bool edges = rs.lead_base >= 0 || rs.trail_row >= 0;
    const bool carried = body > 0 && (!edges || chunkft::edge_rows_folded(rs));
    const bool small = chunkft::takes_small_tiles(p.in, p.T, p.begin, p.end, cus);
    const int64_t tiles = ((p.end - 1) / p.in - p.begin / p.in / 8 * 8 + 1 + 63) / 64 * ((p.in + 63) / 64);
    const bool beyond = tiles > cus * 43 / 10 || tiles * p.T > cus * (body <= 64 ? 8600 : 4300);
    if (chunkft::plain_leaves_small_tiles(p, cus) && !carried) { printf("a gradient sent to a kernel that cannot carry it\n"); return false; }
    if (carried ? small == beyond : !small) {
      printf("[%ld, %ld) of %ld-wide rows, %ld tokens: body of %ld rows, %ld tiles, small tiles %d\n", (long)p.begin, (long)p.end, (long)p.in,
             (long)p.T, (long)body, (long)tiles, (int)small);
      return false;
    }
  }
  return true;
}

// The embedding gradient takes every number of row groups that a launch can count, in one part at least; never more.  Narrow
// tables of many groups are updated in one part, sparse gradients of many groups taken in one.
bool embed_parts_ok() {
  const int64_t most = chunkft::kMaxLaunchThreads / chunkft::kEmbedThreads;
  for (const bool update : {false, true})
    for (const int64_t groups : {(int64_t)1, (int64_t)1024, (int64_t)1025, most / 4 - 1, most / 4, most / 4 + 1, most - 1, most, most + 1, most * 2}) {
      const int parts = chunkft::embed_parts(update, groups, 64 * groups, 1024, 8192, 256);
      if ((parts != 0) != (groups <= most) || groups * parts * chunkft::kEmbedThreads > chunkft::kMaxLaunchThreads) {
        printf("embedding: %ld row groups in %d parts\n", (long)groups, parts);
        return false;
      }
    }
  const auto parts = [](bool update, int64_t rows, int64_t in, int64_t T) {
    return chunkft::embed_parts(update, (rows + 63) / 64 * ((in + 1023) / 1024), rows, in, T, 256);
  };
  if (parts(true, 400000, 176, 1) != 1 || parts(false, 29000, 1137, 4) != 1 || parts(false, 128256, 4096, 4096) != 1 ||
      parts(true, 128256, 4096, 4096) != 4 || parts(false, 4000, 8192, 4096) != 4 || parts(true, 8000, 64, 16) != 4) {
    printf("embedding: parts of a row group\n");
    return false;
  }
  return true;
}

// A run of countable_run() elements from the last column of a row, its first tile beginning up to 7 rows earlier, fits a launch.
bool countable_runs_ok(std::mt19937_64& rng) {
  for (int it = 0; it < 200000; ++it) {
    const int64_t in = 1 + (int64_t)(rng() >> (rng() % 64 < 20 ? 44 : 58 - rng() % 10)), bm = 32 << (rng() % 3), bn = 32 << (rng() % 4);
    const int32_t S = rng() % 2 ? 1 : 1 + (int32_t)(rng() % 64);
    const int threads = 256 << (rng() % 3);
    const int64_t run = chunkft::countable_run(in, S, bm, bn, threads);
    if (run < 0 || run % in != 0) { printf("run %ld of %ld-wide rows\n", (long)run, (long)in); return false; }
    if (run == 0) continue;
    const int64_t rows = run / in + (in > 1 ? 1 : 0) + 7, tiles = (rows + bm - 1) / bm * ((in + bn - 1) / bn);
    if ((tiles * S + 7) / 8 * 8 * threads > chunkft::kMaxLaunchThreads) {
      printf("%ld elements of %ld-wide rows in %ld x %ld tiles, %d slabs, %d threads: %ld tiles\n", (long)run, (long)in, (long)bm, (long)bn, S, threads,
             (long)tiles);
      return false;
    }
  }
  return chunkft::countable_run(1, 1, 32, 32, 1024) < ((int64_t)1 << 27) && chunkft::countable_run(4096, 1, 32, 64, 256) > ((int64_t)1 << 34);
}

// Gradients of more than four small tiles a compute unit go to the large ones, others stay.
bool plain_line_ok() {
  const auto leaves = [](int64_t rows, int64_t in, int64_t T, int64_t begin) {
    chunkft::WgradProblem p{};
    p.out = rows; p.in = p.ldx = in; p.lddy = rows; p.T = p.kslab = T; p.S = 1; p.begin = begin; p.end = rows * in;
    return chunkft::plain_leaves_small_tiles(p, 256);
  };
  const bool ok = leaves(280, 13408, 436, 0) && leaves(280, 13408, 700, 0) && leaves(1032, 4096, 700, 0) && !leaves(1024, 4096, 1000, 0) &&
                  !leaves(280, 13408, 200, 0) && leaves(1400, 2800, 700, 0) && !leaves(1024, 3016, 1400, 0) && !leaves(100, 70400, 1000, 8);
  if (!ok) printf("line of the plain gradient\n");
  return ok;
}

// The split that the small tiles' cost picks: long slabs are cut where that pays, and its partial sums always fit the library's
// static workspace.
bool small_splits_ok(std::mt19937_64& rng) {
  const auto split = [](int64_t rows, int64_t in, int64_t T) { return chunkft::pick_split(0, 1, rows, in, T, 0, rows * in, 0, true, 256).S; };
  if (split(256, 4104, 3000) != 2 || split(1000, 1000, 2500) != 2 || split(256, 4096, 3000) != 2 || split(256, 4096, 2500) != 1 || split(256, 4096, 1024) != 1) {
    printf("slabs of the small tiles\n");
    return false;
  }
  for (int it = 0; it < 100000; ++it) {
    const int64_t in = 8 * (1 + (int64_t)(rng() >> (rng() % 2 ? 54 : 46))), rows = 1 + (int64_t)(rng() % (rng() % 2 ? 150 : 4000)), T = 1 + (int64_t)(rng() % 20000);
    const int64_t begin = rng() % 2 ? 0 : (int64_t)(rng() % (uint64_t)in), end = rows * in;
    if (!chunkft::takes_small_tiles(in, T, begin, end, 256)) continue;
    const chunkft::Split s = chunkft::pick_split(0, 1, rows, in, T, begin, end, 0, true, 256);
    if (s.S > 1 && (int64_t)s.S * (end - begin + 32) * 4 > (int64_t)CHUNKFT_STATIC_WORKSPACE_BYTES) {
      printf("%ld x %ld, %ld tokens: %d slabs\n", (long)rows, (long)in, (long)T, s.S);
      return false;
    }
  }
  return true;
}

int main() {
  if (!embed_parts_ok()) return 1;
  // slabs of 32 and 64 tokens in loads of 8 are the kernel's; token strides up to the largest of the path (64 tokens below 4 GiB)
  for (const int slab : {8, 32, 64})
    for (const int tokens : {4, 8})
      for (const unsigned token_bytes : {16u, 8192u, 256512u, 66060288u})
        for (const unsigned column : {0u, 4080u})
          if (!slab_offsets_ok(slab, tokens, column, token_bytes)) return 1;
  std::mt19937_64 rule_rng(77);
  if (!tile_rule_ok(rule_rng) || !countable_runs_ok(rule_rng) || !small_splits_ok(rule_rng) || !plain_line_ok()) return 1;
  std::mt19937_64 rng(1234);
  long plans = 0, calls = 0, accepted = 0;
  // ---- planner, plan summary, schedule
  for (int it = 0; it < 60000; ++it) {
    const int n = rng() % 6;
    std::vector<chunkft_tensor_desc> t(n);
    for (auto& d : t) {
      d.rows = (rng() % 5 == 0) ? 0 : (int64_t)(rng() % 50);
      d.cols = (int64_t)(rng() % 40);
      if (rng() % 97 == 0) { d.rows = (int64_t)1 << (20 + rng() % 42); d.cols = (int64_t)1 << (rng() % 40); }
      d.dtype = rng() % 2;
      d.kind = rng() % 5;
    }
    int64_t budget = (int64_t)(rng() % 300);
    if (rng() % 31 == 0) budget = INT64_MAX - (int64_t)(rng() % 100);
    const uint32_t flags = rng() % 8;
    int64_t nc = -1, ns = -1;
    int r = chunkft_plan_cycle(t.data(), n, budget, flags, nullptr, 0, &nc, nullptr, 0, &ns);
    if (r == CHUNKFT_ERR_BUFFER_TOO_SMALL || r == CHUNKFT_OK) {
      if (nc > 200000 || ns > 200000) continue;
      std::vector<chunkft_chunk> c(nc + 1);
      std::vector<chunkft_segment> s(ns + 1);
      int64_t nc2 = 0, ns2 = 0;
      r = chunkft_plan_cycle(t.data(), n, budget, flags, c.data(), nc, &nc2, s.data(), ns, &ns2);
      if (r != CHUNKFT_OK || nc2 != nc || ns2 != ns) { printf("count-then-fill mismatch at %d\n", it); return 1; }
      std::vector<int64_t> pos(n, 0);
      for (int64_t i = 0; i < ns; ++i) {
        const auto& g = s[i];
        if (g.tensor < 0 || g.tensor >= n || g.begin != pos[g.tensor] || g.end <= g.begin) { printf("bad segment at %d\n", it); return 1; }
        pos[g.tensor] = g.end;
      }
      for (int i = 0; i < n; ++i) if (pos[i] != t[i].rows * t[i].cols) { printf("coverage at %d\n", it); return 1; }
      for (int64_t k = 0; k < nc; ++k) {
        if (c[k].cost_bytes <= 0 || c[k].cost_bytes > budget || c[k].seg_begin >= c[k].seg_end) { printf("chunk %ld at %d\n", (long)k, it); return 1; }
        int64_t numel = 0;
        for (int64_t i = c[k].seg_begin; i < c[k].seg_end; ++i) {
          if (s[i].chunk_off != numel) { printf("chunk_off at %d\n", it); return 1; }
          numel += s[i].end - s[i].begin;
        }
        if (numel != c[k].numel) { printf("numel at %d\n", it); return 1; }
      }
      if (nc > 0) {
        chunkft_plan_summary sum;
        if (chunkft_plan_stats(c.data(), nc, (int64_t)(rng() % 100000), &sum) != CHUNKFT_OK) { printf("stats at %d\n", it); return 1; }
        if (!(sum.jitter <= sum.jitter_bound * (1 + 1e-12) + 1e-300) || sum.imbalance_bytes < 0) { printf("jitter bound at %d\n", it); return 1; }
      }
      ++plans;
    }
    chunkft_schedule_entry e;
    chunkft_schedule_at((int64_t)(rng() >> (rng() % 64)), 1 + rng() % 9, 1 + (int64_t)(rng() >> (1 + rng() % 63)), &e);
  }
  // ---- device entry points with made-up addresses: validation, token split, workspace placement
  const uintptr_t base = 0x10000000u;
  for (int it = 0; it < 200000; ++it) {
    chunkft_layer L{};
    L.kind = (int32_t)(rng() % 6) - (rng() % 50 == 0);
    L.dtype = (int32_t)(rng() % 2) + (rng() % 60 == 0 ? 5 : 0);
    const bool wide = rng() % 40 == 0;
    L.out = wide ? (int64_t)(rng() >> (rng() % 64)) : (int64_t)(rng() % 3000) * (rng() % 3 ? 8 : 1);
    L.in = wide ? (int64_t)(rng() >> (rng() % 64)) : (int64_t)(rng() % 3000) * (rng() % 3 ? 8 : 1);
    if (L.kind == CHUNKFT_VECTOR || L.kind == CHUNKFT_RMSNORM || L.kind == CHUNKFT_LAYERNORM) L.out = rng() % 20 ? 1 : 2;
    L.T = (int64_t)(rng() % 20000) - (rng() % 80 == 0);
    L.ldx = L.in + (rng() % 4 ? 0 : (int64_t)(rng() % 64) - 8);
    L.lddy = (L.kind == CHUNKFT_LINEAR ? L.out : L.in) + (rng() % 4 ? 0 : (int64_t)(rng() % 64) - 8);
    L.X = rng() % 50 ? (const void*)(base + 16 * (rng() % 1000) + (rng() % 9 ? 0 : rng() % 16)) : nullptr;
    L.dY = rng() % 50 ? (const void*)(base + 16 * (rng() % 1000) + (rng() % 9 ? 0 : rng() % 16)) : nullptr;
    L.split_k = rng() % 3 ? 0 : (int32_t)(rng() % 70) - 2;
    L.reserved = rng() % 90 == 0;
    L.norm_eps = rng() % 70 ? 1e-6 : -1.0;
    const int64_t numel = (L.out > 0 && L.in > 0 && L.in < INT64_MAX / (L.out > 0 ? L.out : 1)) ? L.out * L.in : 1000;
    int64_t begin = (int64_t)(rng() % (uint64_t)(numel > 0 ? numel : 1));
    int64_t end = begin + 1 + (int64_t)(rng() % (uint64_t)(numel - begin > 0 ? numel - begin : 1));
    if (rng() % 60 == 0) end = begin;
    if (rng() % 60 == 0) end = numel + 1 + (int64_t)(rng() % 5);
    const size_t need = chunkft_workspace_bytes(&L, begin, end);
    const int S = chunkft_split_k(&L, begin, end);
    size_t have = need;
    if (rng() % 10 == 0 && need > 0) have = need - 1 - (size_t)(rng() % need);
    void* ws = have || rng() % 2 ? (void*)(base + 0x4000000u + 16 * (rng() % 64) + (rng() % 12 ? 0 : 4)) : nullptr;
    g_ws_lo = reinterpret_cast<uintptr_t>(ws);
    g_ws_hi = g_ws_lo + have;
    float* fp = (float*)(base + 0x2000000u + 4 * (rng() % 64));
    chunkft_adamw_hparams hp{1e-4, 0.9, 0.999, 1e-8, 0.01, (int64_t)(rng() % 5) - (rng() % 40 == 0)};
    const long before = g_launches;
    int r;
    if (rng() % 2) r = chunkft_chunk_wgrad(&L, begin, end, fp, (int)(rng() % 2), ws, have, nullptr);
    else r = chunkft_wgrad_adamw_fused(&L, begin, end, rng() % 2 ? (void*)fp : nullptr, fp, fp, fp, &hp, ws, have, nullptr);
    ++calls;
    if (r == CHUNKFT_OK) {
      ++accepted;
      if (S < 1) { printf("accepted call with split %d at %d\n", S, it); return 1; }
      if (g_launches == before) { printf("accepted call launched nothing at %d\n", it); return 1; }
    } else if (g_launches != before) {
      printf("rejected call (%d) reached a launcher at %d\n", r, it);
      return 1;
    }
    if (g_fail) { printf("launch check failed: %s (iteration %d)\n", g_fail, it); return 1; }
    if (rng() % 8 == 0) {
      const int64_t n = (int64_t)(rng() % 100000) - 3;
      const int ra = chunkft_adamw_chunk(fp, fp, fp, fp, rng() % 2 ? (void*)fp : nullptr, (int32_t)(rng() % 3), n, &hp, nullptr);
      if ((ra == CHUNKFT_OK) != (n > 0 && hp.step >= 1 && ra == 0)) { printf("adamw validation at %d\n", it); return 1; }
    }
  }
  // ---- grouped fused call: random groups of segments on made-up addresses
  long groups = 0, groups_ok = 0;
  for (int it = 0; it < 30000; ++it) {
    const int n = 1 + (int)(rng() % 20);
    std::vector<chunkft_group_segment> sg((size_t)n);
    for (auto& g : sg) {
      chunkft_layer& L = g.layer;
      L = chunkft_layer{};
      L.kind = rng() % 12 == 0 ? (int32_t)(rng() % 5) : (rng() % 4 == 0 ? CHUNKFT_VECTOR : CHUNKFT_LINEAR);
      L.dtype = rng() % 8 == 0 ? CHUNKFT_F32 : CHUNKFT_BF16;
      L.out = L.kind == CHUNKFT_LINEAR || L.kind == CHUNKFT_EMBEDDING ? 8 * (1 + (int64_t)(rng() % 600)) : 1;
      L.in = (rng() % 10 ? 8 : 1) * (1 + (int64_t)(rng() % 600));
      L.T = 1 + (int64_t)(rng() % 9000);
      if (L.kind == CHUNKFT_EMBEDDING && L.T > 8192) L.T = 8192;
      L.ldx = L.in;
      L.lddy = L.kind == CHUNKFT_LINEAR ? L.out : L.in;
      L.X = (const void*)(base + 16 * (rng() % 1000));
      L.dY = (const void*)(base + 16 * (rng() % 1000));
      L.split_k = rng() % 5 ? 0 : (int32_t)(rng() % 5);
      if (L.kind != CHUNKFT_LINEAR) L.split_k = 0;
      L.norm_eps = 1e-6;
      const int64_t numel = L.out * L.in;
      g.begin = (int64_t)(rng() % (uint64_t)numel);
      g.end = g.begin + 1 + (int64_t)(rng() % (uint64_t)(numel - g.begin));
      if (rng() % 400 == 0) g.end = g.begin;
      g.W = rng() % 2 ? (void*)(base + 0x1000000u) : nullptr;
      g.master = g.m = g.v = (float*)(base + 0x2000000u + 4 * (rng() % 64));
      if (rng() % 500 == 0) g.m = nullptr;
    }
    chunkft_adamw_hparams hp{1e-4, 0.9, 0.999, 1e-8, 0.01, 1 + (int64_t)(rng() % 5)};
    const size_t need = chunkft_group_workspace_bytes(sg.data(), n);
    size_t have = need;
    if (need > 0 && rng() % 10 == 0) have = need - 1;
    void* ws = have ? (void*)(base + 0x4000000u) : nullptr;
    g_ws_lo = reinterpret_cast<uintptr_t>(ws);
    g_ws_hi = g_ws_lo + have;
    const long before = g_launches;
    const int r = chunkft_wgrad_adamw_fused_group(sg.data(), n, &hp, ws, have, nullptr);
    ++groups;
    if (r == CHUNKFT_OK) {
      ++groups_ok;
      if (g_launches == before) { printf("accepted group launched nothing at %d\n", it); return 1; }
    } else if (g_launches != before) {
      printf("rejected group (%d) reached a launcher at %d\n", r, it);
      return 1;
    }
    if (g_fail) { printf("group launch check failed: %s (iteration %d)\n", g_fail, it); return 1; }
  }
  if (groups_ok < groups / 4) { printf("too few accepted groups: %ld of %ld\n", groups_ok, groups); return 1; }
  if (accepted < calls / 20) { printf("too few accepted calls: %ld of %ld\n", accepted, calls); return 1; }
  printf("ok: %ld plans, %ld device calls (%ld accepted), %ld grouped calls (%ld accepted), %ld stand-in launches\n", plans, calls,
         accepted, groups, groups_ok, g_launches);
  return 0;
}
