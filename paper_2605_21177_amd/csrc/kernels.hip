// gfx950 (CDNA4) kernels of the ChunkFT hot path.
//
//   wgrad_mfma_kernel   bf16 chunk-restricted weight gradient: LDS-staged dY and X
//                       token slabs, LDS transpose reads, 32x32x16 bf16 MFMA, fp32
//                       accumulators; epilogue stores g, a slab partial, or applies
//                       AdamW straight from the accumulators.
//   colsum_kernel       1-D scale-vector gradient sum_t dY[t,j] * X[t,j], X normalised by the
//                       caller or here (norm_stats_kernel: per-token mean and 1/std).
//   embed_wgrad_kernel  embedding table gradient: per table row the sum of the dY rows of
//                       the tokens that name it, in token order.
//   elementwise_kernel  AdamW over a chunk and/or the fixed-order sum of slab partials.
// fp32 layers are in wgrad_f32.hip, bf16 layers without 16-byte rows in wgrad_ragged.hip, chunks of few tiles in
// wgrad_small.hip.
//
// The operations are those of the paper's Section 3.1 (gradient of the active
// slices only, through the chunk-aware operators of Algorithm 1 line 8) and
// Algorithm 1 lines 19-21 (AdamW with the chunk's own counter).

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <cstdlib>

#include "device.h"
#include "internal.h"
#include "launch.h"

namespace chunkft {

// ---------------------------------------------------------------------------
// bf16 MFMA weight-gradient kernel
// ---------------------------------------------------------------------------
// Row decomposition of the chunk [begin, end) of W [out, in]:
//   body rows [rb0, rb1): complete rows, rb0 a multiple of 8 (16-byte dY loads),
//   computed by the MFMA kernel with no range mask beyond the row bound;
//   edge rows: the partial first row, the up-to-7 complete rows before rb0, and
//   the partial last row -- at most 9 of them.  The workgroups of the
//   first tile row, which stream every X column tile anyway, carry them as one
//   extra 32-row MFMA block.  (A chunk whose body has at most 128 rows does not come here.)
// Diagnostic build only (-DCHUNKFT_TIMELINE, a library of its own: libchunkft_timeline.so): every
// workgroup of the MFMA kernel notes when it starts, when the first fragments of its tile are in
// registers, when its loop ends and when its epilogue ends (the 100 MHz constant counter), and where
// it ran, in 8 words per work item of a buffer that the caller hands over with
// chunkft_timeline_buffer().  The product library has none of this.
#ifdef CHUNKFT_TIMELINE
static unsigned long long* g_timeline = nullptr;
static size_t g_timeline_words = 0;
extern "C" int chunkft_timeline_buffer(void* device_buffer, size_t bytes) {
  g_timeline = static_cast<unsigned long long*>(device_buffer);
  g_timeline_words = bytes / 8;
  return 0;
}
#define TIMELINE_STAMP(q, item, k)                                                                  \
  do {                                                                                              \
    if ((q).timeline && threadIdx.x == 0) (q).timeline[(size_t)(item) * 8 + (k)] = __builtin_amdgcn_s_memrealtime(); \
  } while (0)
#else
#define TIMELINE_STAMP(q, item, k) do { } while (0)
#endif

struct MfmaParams {
  WgradProblem p;
  int64_t rb0, rb1;
  int32_t tiles_m, tiles_n;
  int32_t n_tile_items;        // tiles_m * tiles_n * S
  int32_t group_m;
  int32_t stagger;             // start delay of every second resident workgroup, in units of 8128 cycles
  int32_t turned;              // XCD x begins x eighths into its run of tiles (runs_in_step)
  int64_t lead_base;           // edge rows folded into the first tile row (the 8-row group before rb0; -1: none)
  int64_t trail_row;
  Sinks s;
#ifdef CHUNKFT_TIMELINE
  unsigned long long* timeline;
#endif
};

// Tile configuration of the MFMA kernel: a (128 WM) x 256 output tile per workgroup
// of 4 WM waves (WM x 4, each wave 128 x 64 = 4 x 2 blocks of 32 x 32), tokens in
// slabs of 32, and a ring of NS slabs in LDS filled by global->LDS loads.
//   WM = 1, NS = 3: 128 x 256 tiles, 4 waves, 75 KB of LDS -- two workgroups share a
//   compute unit, so the store-bound epilogue of one runs under the MFMA loop of the other;
//   WM = 2, NS = 4: 256 x 256 tiles, 8 waves, 132 KB -- one workgroup per compute unit,
//   a third less operand traffic per flop.
template <int WM_, int NS_, int MI_ = 32, bool AHEAD_ = true>
struct RingCfg {
  static constexpr bool AHEAD = AHEAD_;               // how the update reads its state (tile_epilogue)
  static constexpr int WM = WM_, WN = 4, BM = 128 * WM, BN = 256, BK = 32, NS = NS_;
  static constexpr int MI = MI_;                      // MFMA shape: 32 (32x32x16) or 16 (16x16x32)
  static constexpr int NW = WM * WN, NT = 64 * NW;
  static constexpr int TM = BM / WM / MI, TN = BN / WN / MI;
  static constexpr int A_BYTES = BK * BM * 2, B_BYTES = BK * BN * 2;
  // edge block: per token 16 row values = the 8-row group of the leading edge rows and
  // the 8-row group that holds the trailing row (32 B per token, 1 KB per slab)
  static constexpr int E_BYTES = BK * 32;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES + E_BYTES;
  static constexpr int LA = A_BYTES / 1024 / NW;     // 1 KB wave-loads per wave per slab
  static constexpr int LB = B_BYTES / 1024 / NW;
  static constexpr int L = LA + LB;
  // epilogue staging: half a tile (BM / 2 rows x 256 columns of fp32) at a time; a row
  // pitch of 264 floats puts the two half-waves of a ds_write_b32 on disjoint banks
  // (with the 16 x 16 blocks of the other MFMA shape a write spans four row groups: 260 floats spread them)
  static constexpr int EPI_PITCH = MI == 32 ? BN + 8 : BN + 4;
  static constexpr size_t EPI_BYTES = (size_t)(BM / 2) * EPI_PITCH * 4;
  static constexpr size_t RING_BYTES = (size_t)NS * STAGE_BYTES;
  static constexpr size_t LDS_BYTES = RING_BYTES > EPI_BYTES ? RING_BYTES : EPI_BYTES;
  static constexpr int RA = BM * 2, RB = BN * 2;     // bytes of one token in the A / B image of a slab
  static_assert((MI == 32 || MI == 16) && TM * MI == 128 && TN * MI == 64 && (WM == 1 || WM == 2) && L >= 4 &&
                    L <= 6 && NS >= 3,
                "the main loops are written out for this shape");
};

#define WAIT_HALVES(h)                                                                                   \
  asm volatile("s_waitcnt lgkmcnt(0)"                                                                    \
               : "+v"(h[0]), "+v"(h[1]), "+v"(h[2]), "+v"(h[3]), "+v"(h[4]), "+v"(h[5]), "+v"(h[6]),     \
                 "+v"(h[7]), "+v"(h[8]), "+v"(h[9]), "+v"(h[10]), "+v"(h[11])::"memory")

#define WAIT_HALVES_E(h, he)                                                                             \
  asm volatile("s_waitcnt lgkmcnt(0)"                                                                    \
               : "+v"(h[0]), "+v"(h[1]), "+v"(h[2]), "+v"(h[3]), "+v"(h[4]), "+v"(h[5]), "+v"(h[6]),     \
                 "+v"(h[7]), "+v"(h[8]), "+v"(h[9]), "+v"(h[10]), "+v"(h[11]), "+v"(he[0]), "+v"(he[1])::"memory")

// Epilogue of one tile of the MFMA kernels.  Accumulator register v of a 32x32 block holds
// row (v / 4) * 8 + (lane / 32) * 4 + v % 4, column lane % 32 -- a layout that
// could only be stored 4 bytes per lane.  The tile is therefore staged through
// LDS (the ring is free by now), half of it at a time, and leaves as whole rows:
// a wave handles one row of 256 columns per trip, 16 bytes per lane, 1 KB per
// instruction, for the gradient as well as for the AdamW state.
// stage_half(h, stage, sft) writes the wave's share of half h into the staging area; emit_edge(E) emits
// the edge block's elements (both know the accumulator layout of the MFMA shape in use).
template <class C, int MODE, class StageHalf, class EmitEdge>
__device__ __forceinline__ void tile_epilogue(const MfmaParams& q, unsigned char* ldsb, int64_t row0, int64_t col0,
                                              int slab, int wave, int lane, int tid,
                                              StageHalf&& stage_half, EmitEdge&& emit_edge) {
  const WgradProblem& p = q.p;
  const int wn0 = (wave % C::WN) * (C::BN / C::WN);
  const int64_t E = p.end - p.begin;
  const int64_t origin = row0 * p.in + col0 - p.begin;             // chunk-local index of the tile corner
  const int rows_valid = (int)((q.rb1 - row0 < C::BM) ? q.rb1 - row0 : C::BM);
  const int cols_valid = (int)((p.in - col0 < C::BN) ? p.in - col0 : C::BN);
  float* const stage = reinterpret_cast<float*>(ldsb);
  const int wmi = wave / C::WN;
  constexpr int WR = C::BM / C::WM / 2;   // rows of one wave row in a staged half
  constexpr int HALF_ROWS = C::WM * WR;   // rows staged per pass
  float* const g_dst = MODE == EMIT_PARTIAL ? q.s.ws + (int64_t)slab * q.s.ws_pitch : q.s.g;
  // Groups of four columns start where the fp32 destination is 16-byte aligned:
  // at tile-local column delta (the same for every row, because in % 8 == 0).
  // The delta leading and 4 - delta trailing columns of a row that are left over
  // are taken one element per thread (128 rows x 4 = 512 of them per half tile).
  const float* const align_ref = MODE == EMIT_ADAMW ? q.s.master : g_dst;
  const int delta = (int)((4 - ((reinterpret_cast<uintptr_t>(align_ref) >> 2) + (uint64_t)origin) % 4) % 4);
  const int c4 = delta + lane * 4;
  const bool vec_lane = delta == 0 || lane < 63;
  // The staged copy of a row is shifted right by sft columns, so that the groups of four
  // that start at column delta sit on 16-byte boundaries in LDS too: one conflict-free
  // 16-byte read per lane (the row pitch leaves room for the shift).
  const int sft = (4 - delta) & 3;
  auto sink_at = [&](int64_t i) {
    Vec4Sink d;
    d.g = g_dst + i;
    d.master = q.s.master + i;
    d.m = q.s.m + i;
    d.v = q.s.v + i;
    d.W = (unsigned short*)q.s.W + i + p.begin;                    // a bf16 copy or none (the launchers refuse others)
    return d;
  };
  // Rows that are read before they are written.  AHEAD (the sum into g; the update on 256-row tiles, and on 128-row tiles over few tokens): batches
  // of RPT rows in a pipeline, the state of the next batch requested before the present one is finished, across the two
  // halves, the first before the tile is staged; a batch's stores are then younger than the next batch's loads.  The fp32
  // accesses are buffer forms whose range check drops what is not there (a row past the body, a group of four past the
  // row), so that no branch lies around them and the compiler counts what is in flight: the wait for a batch's loads leaves the stores of the batch
  // before it in flight.  (In the update the up to four bf16 stores of a batch do lie behind branches and are not counted; where they
  // were issued the last wait of the next batch takes in as many of the older fp32 stores.  Edge rows, one element at a time behind the
  // first request, wait for everything in flight.)  32 Mi elements of 4096-wide rows, fused call: 512 tokens
  // 176.8 -> 167.3 us, 1024 tokens 182.5 -> 179.5; sum into g, 24 Mi, 256 tokens 49.9 -> 42.5, 1024 tokens 79.4 -> 67.8.  Else (the
  // update of 128-row tiles over more tokens) a batch is requested, awaited and
  // finished: the loops decide there, and with twice the requests in flight the update takes more of the memory from
  // the loop beside it than it gains (2048 tokens 218 us, with the pipeline 223; 40 Mi of 14336-wide rows 309 against 326).
  constexpr bool AHEAD = MODE == EMIT_ACCUM || (MODE == EMIT_ADAMW && C::AHEAD);
  constexpr int RPT = MODE == EMIT_ACCUM ? 8 : 4, NB = HALF_ROWS / C::NW / RPT;
  static_assert(NB * RPT * C::NW == HALF_ROWS, "whole batches");
  constexpr int kNowhere = (int)0x80000000;                        // past every descriptor's end
  // (read once into scalar registers: a value that the compiler fetches again behind a lane-dependent branch makes
  // it treat the descriptors as lane-dependent too)
  auto scalar = [](uint64_t x) {
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)x), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(x >> 32));
    return hi << 32 | lo;
  };
  auto desc = [&](float* base) {     // a tile spans less than 255 rows of 2^21 elements: 2^31 bytes
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(scalar(reinterpret_cast<uint64_t>(base + origin))), 0, 0x7fffffff, 0x00020000);
  };
  const unsigned pitch = (unsigned)__builtin_amdgcn_readfirstlane((int)p.in);      // elements from row to row
  const bool low = MODE == EMIT_ADAMW && q.s.w_kind == W_BF16;
  auto* const low_copy = (GLOBAL_PTR(unsigned short))scalar(reinterpret_cast<uint64_t>((unsigned short*)q.s.W + p.begin + origin));   // the tile corner's
  const __amdgpu_buffer_rsrc_t first = desc(MODE == EMIT_ADAMW ? q.s.master : q.s.g);
  const __amdgpu_buffer_rsrc_t second = desc(q.s.m), third = desc(q.s.v);
  const int lane_off = vec_lane && c4 + 4 <= cols_valid ? c4 * 4 : kNowhere;
  auto batch_row = [&](int h, int j) {
    const int rr = j * C::NW + wave;                               // staged row, 0..HALF_ROWS-1
    return (rr / WR) * (2 * WR) + h * WR + rr % WR;
  };
  State4 ahead[2][RPT];
  auto request = [&](auto nc) {
    constexpr int n = decltype(nc)::value, h = n / NB;
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
      const int tile_row = batch_row(h, (n % NB) * RPT + u);
      const int vo = tile_row < rows_valid ? lane_off : kNowhere;
      const int so = (int)((unsigned)tile_row * pitch * 4u);
      auto get = [&](__amdgpu_buffer_rsrc_t from) { return __builtin_bit_cast(f32x4_u, __builtin_amdgcn_raw_buffer_load_b128(from, vo, so, kNonTemporal)); };
      State4& st = ahead[n & 1][u];
      st.th = get(first);
      if constexpr (MODE == EMIT_ADAMW) {
        st.mm = get(second);
        st.vv = get(third);
      }
    }
  };
  auto finish = [&](auto nc) {
    constexpr int n = decltype(nc)::value, h = n / NB;
    u32x2_a2 packed[RPT];
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
      const int j = (n % NB) * RPT + u, tile_row = batch_row(h, j);
      const int vo = tile_row < rows_valid ? (int)((unsigned)lane_off + (unsigned)tile_row * pitch * 4u) : kNowhere;
      auto put = [&](__amdgpu_buffer_rsrc_t to, f32x4_u x) {
        // The row goes into the lane offset, not into the scalar one: behind a 16-byte store with a register as its scalar
        // offset the compiler keeps no wait state, and where the next instruction wrote the first data register this
        // device stored the new value (every fourth m and v of the 256-row tile).
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, x), to, vo, 0, MODE == EMIT_ACCUM ? 0 : kNonTemporal);
      };
      const float4 q4 = *reinterpret_cast<const float4*>(stage + (j * C::NW + wave) * C::EPI_PITCH + sft + c4);
      const f32x4_u val = {q4.x, q4.y, q4.z, q4.w};
      State4& st = ahead[n & 1][u];
      if constexpr (MODE == EMIT_ACCUM) {
        st.th += val;
        put(first, st.th);
      } else {
        update4(val, st, q.s.c);
        put(first, st.th);
        put(second, st.mm);
        put(third, st.vv);
        packed[u] = pack_bf16(st.th);
      }
    }
    if constexpr (MODE == EMIT_ADAMW) {
      if (low && lane_off != kNowhere) {
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
          const int tile_row = batch_row(h, (n % NB) * RPT + u);
          if (tile_row < rows_valid)
            __builtin_nontemporal_store(packed[u], (GLOBAL_PTR(u32x2_a2))(low_copy + (unsigned)tile_row * pitch + c4));
        }
      }
    }
  };
  auto half = [&](int h, auto&& rows) __attribute__((always_inline)) {     // rows(): the staged rows of the half leave
    __syncthreads();                       // ring reads / previous half's row reads are done
    stage_half(h, stage + (wmi * WR) * C::EPI_PITCH + sft + wn0);
    __syncthreads();
    // The left-over element of this thread (delta != 0): in the fused call its state is requested
    // now and used after the row loop, so that this second round of loads costs no extra wait.
    bool lo_ok = false;
    int64_t lo_i = 0;
    float lo_val = 0.f, lo_th = 0.f, lo_m = 0.f, lo_v = 0.f;
    if (delta != 0) {
      static_assert(C::NT / 4 >= HALF_ROWS, "one thread per left-over element of a staged half tile");
      const int rr = tid >> 2, e = tid & 3;
      const int tile_row = (rr / WR) * (2 * WR) + h * WR + rr % WR;
      const int lc = e < delta ? e : cols_valid - 4 + e;      // cols_valid is a multiple of 8
      lo_ok = rr < HALF_ROWS && tile_row < rows_valid;
      if (lo_ok) {
        lo_i = origin + (int64_t)tile_row * p.in + lc;
        lo_val = stage[rr * C::EPI_PITCH + sft + lc];
        if constexpr (MODE == EMIT_ADAMW) {
          lo_th = q.s.master[lo_i];
          lo_m = q.s.m[lo_i];
          lo_v = q.s.v[lo_i];
        }
      }
    }
    rows();
    if (lo_ok) {
      if constexpr (MODE == EMIT_ADAMW) {
        adamw_update(lo_val, lo_th, lo_m, lo_v, q.s.c);
        q.s.master[lo_i] = lo_th;
        q.s.m[lo_i] = lo_m;
        q.s.v[lo_i] = lo_v;
        if (low) ((unsigned short*)q.s.W)[lo_i + p.begin] = f32_to_bf16_rne(lo_th);
      } else {
        emit<MODE>(q.s, E, slab, lo_i, lo_i + p.begin, lo_val);
      }
    }
  };
  if constexpr (AHEAD) {
    request(IntC<0>{});
    emit_edge(E);
    static_for<2>([&](auto hc) {
      half(decltype(hc)::value, [&] {
        static_for<NB>([&](auto bc) {
          constexpr int n = decltype(hc)::value * NB + decltype(bc)::value;
          if constexpr (n + 1 < 2 * NB) request(IntC<n + 1>{});
          finish(IntC<n>{});
        });
      });
    });
  } else {
    emit_edge(E);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      half(h, [&] {
        if (!(vec_lane && c4 + 4 <= cols_valid)) return;
        for (int j0 = 0; j0 < HALF_ROWS / C::NW; j0 += RPT) {
          Vec4Sink d[RPT];
          State4 st[RPT];
          bool ok[RPT];
#pragma unroll
          for (int u = 0; u < RPT; ++u) {
            const int tile_row = batch_row(h, j0 + u);
            ok[u] = tile_row < rows_valid;
            d[u] = sink_at(origin + (int64_t)tile_row * p.in + c4);
            if (ok[u]) st[u] = load_state4<MODE>(d[u]);
          }
#pragma unroll
          for (int u = 0; u < RPT; ++u) {
            if (ok[u]) {
              const float4 q4 = *reinterpret_cast<const float4*>(stage + ((j0 + u) * C::NW + wave) * C::EPI_PITCH + sft + c4);
              const f32x4_u val = {q4.x, q4.y, q4.z, q4.w};
              finish4<MODE>(d[u], low ? W_BF16 : W_NONE, q.s.c, val, st[u]);
            }
          }
        }
      });
  }
}

// One 256 x 256 tile of body rows over one slab of tokens.
//
// Data movement.  dY and X are [token][row] / [token][column]: both operands have
// the contraction index outermost, the opposite of what an MFMA lane wants (8
// consecutive tokens of one row).  A slab of 32 tokens x 256 rows is copied as it
// is (512 B per token) into LDS by buffer_load_dwordx4 ... lds -- no VGPR staging, up
// to NS-1 slabs in flight -- and transposed on the way out by ds_read_b64_tr_b16.
// A wave-load writes 1 KB = tokens 2j, 2j+1; lane l lands in token 2j + l/32,
// physical 16-byte slot l%32.  To keep the 8 tokens that one transpose read
// touches on different banks, slot s of token k holds logical slot
// s ^ (sw(k) << 2), sw(k) = (k & 3) | ((k >> 3 & 1) << 2): the swizzle is applied
// to the source offset each lane fetches from, LDS writes stay linear.
//
// Schedule.  Per 32-token slab a wave issues 16 MFMAs in two 16-token steps.
// The transpose reads of the NEXT step are issued behind the first three MFMAs
// of a step and the global->LDS loads of a later slab behind the last five of the
// second step, so their latency runs under MFMAs instead of in front of a wait.
// One s_barrier per slab, between its two steps: it publishes slab kt+1 (every
// wave waited for its own loads of it) and retires slab kt, whose ring slot the
// loads of slab kt+NS then overwrite -- the whole ring is in flight.
template <class C, int MODE>
__device__ __forceinline__ void mfma_tile(const MfmaParams& q, const int item, unsigned char* ldsb) {
  const WgradProblem& p = q.p;
  TIMELINE_STAMP(q, item, 0);
#ifdef CHUNKFT_TIMELINE
  // where: XCC_ID (hardware register 20) and HW_ID (4: wave, SIMD, compute unit, shader engine)
  if (q.timeline && threadIdx.x == 0)
    q.timeline[(size_t)item * 8 + 4] = ((unsigned long long)__builtin_amdgcn_s_getreg((32 - 1) << 11 | 20) << 32) |
                                       (unsigned)__builtin_amdgcn_s_getreg((32 - 1) << 11 | 4);
#endif

  // ---- which tile, which token slab
  const int n_tiles = q.tiles_m * q.tiles_n;
  const int slab = item / n_tiles;
  const int tile = item - slab * n_tiles;
  const int per_group = q.group_m * q.tiles_n;
  const int grp = tile / per_group;
  const int first_m = grp * q.group_m;
  const int gsz = (q.tiles_m - first_m < q.group_m) ? q.tiles_m - first_m : q.group_m;
  const int in_grp = tile - grp * per_group;
  const int tile_m = first_m + in_grp % gsz;
  const int tile_n = in_grp / gsz;
  const int64_t row0 = q.rb0 + (int64_t)tile_m * C::BM;
  const int64_t col0 = (int64_t)tile_n * C::BN;
  const int64_t k_begin = (int64_t)slab * p.kslab;
  const int64_t k_end = (k_begin + p.kslab < p.T) ? k_begin + p.kslab : p.T;
  const int klen = (int)(k_end - k_begin);
  const int nk = (klen + C::BK - 1) / C::BK;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave / C::WN) * (C::BM / C::WM);
  const int wn0 = (wave % C::WN) * (C::BN / C::WN);
  const unsigned short* dY = (const unsigned short*)p.dY;
  const unsigned short* X = (const unsigned short*)p.X;
  const unsigned lds_base = (unsigned)(uintptr_t)ldsb;

  // ---- global->LDS loads.  A load names its source as a uniform base (scalar registers:
  // the first row / column of the token the slab begins with, advanced one slab per fetch by
  // scalar adds) plus a per-lane byte offset that never changes -- the buffer form of the
  // load.  The form with a 64-bit per-lane address needs a vector add per load to advance,
  // and that add waits in the vector pipe behind the MFMAs: measured, every such load then
  // costs the matrix cores about 25 cycles, while the scalar-base form costs them nothing.
  // Rows / columns past the tensor are redirected to the tile's first ones (valid
  // memory, results masked in the epilogue); tokens past the end are clamped to
  // the last token and zeroed in the fragments of both operands (mask_halves).
  unsigned voa[C::LA], vob[C::LB];
  int ka[C::LA], kb[C::LB];
  const unsigned lddy2 = (unsigned)(p.lddy * 2), ldx2 = (unsigned)(p.ldx * 2);    // bytes per token
  // A wave-load writes 1 KB: 1024 / RA tokens, RA / 16 lanes (16-byte slots) per token.
  constexpr int LPT_A = C::RA / 16, TPL_A = 64 / LPT_A;
#pragma unroll
  for (int i = 0; i < C::LA; ++i) {
    const int k = TPL_A * (wave * C::LA + i) + lane / LPT_A;
    const int swk = C::WM == 2 ? ((k & 3) | (((k >> 3) & 1) << 2)) : (k & 3);
    const int lc = (lane % LPT_A) ^ (swk << 2);
    int64_t r = row0 + lc * 8;
    if (r >= p.out) r = row0;
    ka[i] = k;
    voa[i] = (unsigned)r * 2u + (unsigned)k * lddy2;
  }
#pragma unroll
  for (int i = 0; i < C::LB; ++i) {
    const int k = 2 * (wave * C::LB + i) + (lane >> 5);
    const int lc = (lane & 31) ^ (((k & 3) | (((k >> 3) & 1) << 2)) << 2);
    int64_t cc = col0 + lc * 8;
    if (cc >= p.in) cc = col0;
    kb[i] = k;
    vob[i] = (unsigned)cc * 2u + (unsigned)k * ldx2;
  }
  // row 0 / column 0 of the first token of slab `next_fetch`
  const unsigned char* ga = (const unsigned char*)(dY + k_begin * p.lddy);
  const unsigned char* gb = (const unsigned char*)(X + k_begin * p.ldx);
  const int64_t stepA = (int64_t)C::BK * p.lddy * 2, stepB = (int64_t)C::BK * p.ldx * 2;     // bytes per slab
  int next_fetch = 0;   // slab index the bases stand at
  auto load_to_lds = [&](const unsigned char* base, unsigned voff, unsigned dst) {
    // raw buffer over the whole address range behind `base`: the per-lane offsets are kept below 4 GB
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (LDS_PTR(void))(uintptr_t)dst, 16, (int)voff, 0, 0, 0);
  };
  auto next_slab = [&]() {
    ga += stepA;
    gb += stepB;
    ++next_fetch;
  };

  // ---- edge block (first tile row only).  One extra wave-load per slab, issued by
  // wave 0: lane l fetches, for token l/2, the 8-row group of the leading edge rows
  // (l even) or the one holding the trailing row (l odd); a missing group is
  // replaced by the tile's first rows (valid memory, masked in the epilogue).
  // With 8 waves, waves w and w + 4 share 64 columns and take one of the two 32-column
  // blocks each (workgroups of tile row 0); with 4 waves the workgroups of tile rows 0 and
  // 1 take one block each (the launcher folds the edge in only if there are two tile rows).
  const bool has_edge = (C::WM == 2 ? tile_m == 0 : tile_m < 2) && (q.lead_base >= 0 || q.trail_row >= 0);
  const int edge_blk = C::WM == 2 ? (wave >> 2) : tile_m;
  const int ke = lane >> 1;
  unsigned voe;
  {
    const int64_t lead = q.lead_base >= 0 ? q.lead_base : q.rb0;
    const int64_t trail = q.trail_row >= 0 ? (q.trail_row & ~(int64_t)7) : q.rb0;
    voe = (unsigned)((lane & 1) ? trail : lead) * 2u + (unsigned)ke * lddy2;
  }
  auto issue_edge = [&](auto stagec) {
    constexpr int STAGE = decltype(stagec)::value;
    const int stage = STAGE >= 0 ? STAGE : next_fetch % C::NS;
    const bool ragged = STAGE >= 0 ? false : (next_fetch + 1) * C::BK > klen;
    unsigned vo = voe;
    if (ragged) {      // the base stands at this slab: a token past the end steps back to the last one
      const int64_t over = k_begin + (int64_t)next_fetch * C::BK + ke - (p.T - 1);
      if (over > 0) vo -= (unsigned)over * lddy2;
    }
    load_to_lds(ga, vo, lds_base + stage * C::STAGE_BYTES + C::A_BYTES + C::B_BYTES);
  };
  // One of the L loads of slab `next_fetch`.  STAGE >= 0: the steady-state form, ring
  // slot known at compile time and the slab known to be complete; STAGE < 0: the general
  // form for the first and last slabs.
  auto issue_one = [&](auto idxc, auto stagec) {
    constexpr int idx = decltype(idxc)::value, STAGE = decltype(stagec)::value;
    const int stage = STAGE >= 0 ? STAGE : next_fetch % C::NS;
    const bool ragged = STAGE >= 0 ? false : (next_fetch + 1) * C::BK > klen;     // only the last slab can be
    if constexpr (idx < C::LA) {
      constexpr int i = idx;
      unsigned vo = voa[i];
      if (ragged) {
        const int64_t over = k_begin + (int64_t)next_fetch * C::BK + ka[i] - (p.T - 1);
        if (over > 0) vo -= (unsigned)over * lddy2;
      }
      load_to_lds(ga, vo, lds_base + stage * C::STAGE_BYTES + (wave * C::LA + i) * 1024);
    } else {
      constexpr int i = idx - C::LA;
      unsigned vo = vob[i];
      if (ragged) {
        const int64_t over = k_begin + (int64_t)next_fetch * C::BK + kb[i] - (p.T - 1);
        if (over > 0) vo -= (unsigned)over * ldx2;
      }
      load_to_lds(gb, vo, lds_base + stage * C::STAGE_BYTES + C::A_BYTES + (wave * C::LB + i) * 1024);
    }
  };

  // ---- transpose-read addressing.  In a block of 16 lanes, lane j reads 4
  // consecutive row indices of token (j / 4); the instruction hands lane i the 4
  // tokens of row index i.  Lanes 0-31 take tokens 0-7 of a 16-token step, lanes
  // 32-63 tokens 8-15: the operand layout of the 32x32x16 MFMA.  The swizzle
  // term of a lane is the same for every step: sw = (i16 / 4) | ((blk / 2) << 2).
  const int blk = lane >> 4, i16 = lane & 15;
  const int tr_k = (blk >> 1) * 8 + (i16 >> 2);
  const int swl = (i16 >> 2) | ((blk >> 1) << 2);
  const int low = (blk & 1) * 2 + ((i16 & 3) >> 1);     // low two bits of the 16-byte slot index
  const int sub = (i16 & 1) * 8;                        // byte offset inside the slot
  // Two bases 64 KB apart per block: with the ring slot known at compile time every
  // read then has an immediate offset (the field holds 16 bits) and costs no VALU add.
  unsigned addrA[C::TM], addrB[C::TN], addrA_hi[C::TM], addrB_hi[C::TN];
#pragma unroll
  for (int a = 0; a < C::TM; ++a) {
    addrA[a] = lds_base + tr_k * C::RA + ((((wm0 >> 3) + a * 4) ^ ((C::WM == 2 ? swl : (i16 >> 2)) << 2)) + low) * 16 + sub;
    addrA_hi[a] = addrA[a] + 65536;
  }
#pragma unroll
  for (int b = 0; b < C::TN; ++b) {
    addrB[b] = lds_base + C::A_BYTES + tr_k * C::RB + ((((wn0 >> 3) + b * 4) ^ (swl << 2)) + low) * 16 + sub;
    addrB_hi[b] = addrB[b] + 65536;
  }

  // Edge block reads: token t of a slab sits at byte 32 t, its 16 row values behind it.
  // Lanes 16-31 and 48-63 (MFMA rows 16-31) re-read rows 0-15; those output rows are dropped.
  const unsigned addrE = lds_base + C::A_BYTES + C::B_BYTES + tr_k * 32 + (i16 & 3) * 8;
  const unsigned addrE_hi = addrE + 65536;
  bf16x4 he0[2], he1[2];
  f32x16 acc_e;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc_e[v] = 0.f;
  auto read_edge = [&](bf16x4* he, unsigned so, auto ksc) {
    constexpr int ks = decltype(ksc)::value;
    he[0] = lds_tr_read<ks * 16 * 32>(addrE + so);
    he[1] = lds_tr_read<(ks * 16 + 4) * 32>(addrE + so);
  };
  auto read_edge_at = [&](bf16x4* he, auto stagec, auto ksc) {
    constexpr int st = decltype(stagec)::value, ks = decltype(ksc)::value;
    constexpr int so = st * C::STAGE_BYTES;
    constexpr int off = (so & 0xFFFF) + ks * 16 * 32;
    static_assert(off + 4 * 32 < 65536, "LDS offset field");
    he[0] = lds_tr_read<off>(so < 65536 ? addrE : addrE_hi);
    he[1] = lds_tr_read<off + 4 * 32>(so < 65536 ? addrE : addrE_hi);
  };
  // the edge MFMA of a wave uses one of its two B blocks
  // (the B block is picked by value, four selects, and not by a branch around two MFMAs: the
  // branch made the compiler keep two copies of the accumulator block and move 16 registers,
  // behind a full MFMA latency, in every step)
  auto edge_mma = [&](const bf16x4* he, const bf16x4* h) {
    const bf16x8 fe = __builtin_shufflevector(he[0], he[1], 0, 1, 2, 3, 4, 5, 6, 7);
    const u32x4_t b0 = __builtin_bit_cast(u32x4_t, __builtin_shufflevector(h[8], h[9], 0, 1, 2, 3, 4, 5, 6, 7));
    const u32x4_t b1 = __builtin_bit_cast(u32x4_t, __builtin_shufflevector(h[10], h[11], 0, 1, 2, 3, 4, 5, 6, 7));
    u32x4_t bs;
#pragma unroll
    for (int e = 0; e < 4; ++e) bs[e] = edge_blk == 0 ? b0[e] : b1[e];
    acc_e = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fe, __builtin_bit_cast(bf16x8, bs), acc_e, 0, 0, 0);
  };

  // Fragment halves: unit u < 8 is A block u/2 (tokens 0-3 | 8-11 if u is even,
  // 4-7 | 12-15 if odd), unit u >= 8 is B block (u-8)/2 likewise.
  bf16x4 h0[12], h1[12];
  auto read_unit = [&](bf16x4* h, unsigned so, auto ksc, auto uc) {
    constexpr int ks = decltype(ksc)::value, u = decltype(uc)::value;
    constexpr int off = (ks * 16 + (u & 1) * 4) * (u < 8 ? C::RA : C::RB);
    if constexpr (u < 8) h[u] = lds_tr_read<off>(addrA[u / 2] + so);
    else h[u] = lds_tr_read<off>(addrB[(u - 8) / 2] + so);
  };
  auto read_unit_at = [&](bf16x4* h, auto stagec, auto ksc, auto uc) {      // ring slot at compile time
    constexpr int st = decltype(stagec)::value, ks = decltype(ksc)::value, u = decltype(uc)::value;
    constexpr int so = st * C::STAGE_BYTES;
    constexpr int off = (so & 0xFFFF) + (ks * 16 + (u & 1) * 4) * (u < 8 ? C::RA : C::RB);
    static_assert(off < 65536, "LDS offset field");
    if constexpr (u < 8) h[u] = lds_tr_read<off>(so < 65536 ? addrA[u / 2] : addrA_hi[u / 2]);
    else h[u] = lds_tr_read<off>(so < 65536 ? addrB[(u - 8) / 2] : addrB_hi[(u - 8) / 2]);
  };
  auto frag = [&](const bf16x4* h, int u) {
    return __builtin_shufflevector(h[u], h[u + 1], 0, 1, 2, 3, 4, 5, 6, 7);
  };
  auto mask_halves = [&](bf16x4* h, bf16x4* he, int kt, int ks) {
    if (kt == nk - 1 && (klen % C::BK) != 0) {
      const int kv = klen - kt * C::BK - ks * 16 - (lane >> 5) * 8;   // valid tokens among this lane's 8
#pragma unroll
      for (int u = 0; u < 12; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((u & 1) * 4 + e >= kv) h[u][e] = (__bf16)0.f;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (u * 4 + e >= kv) he[u][e] = (__bf16)0.f;
    }
  };

  f32x16 acc[C::TM][C::TN];
#pragma unroll
  for (int a = 0; a < C::TM; ++a)
#pragma unroll
    for (int b = 0; b < C::TN; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

  // ---- prologue: the whole ring (NS slabs) in flight, first step of slab 0 in registers
#pragma unroll
  for (int s = 0; s < C::NS; ++s)
    if (s < nk) {
      static_for<C::L>([&](auto ic) { issue_one(ic, IntC<-1>{}); });
      if (has_edge && wave == 0) issue_edge(IntC<-1>{});
      next_slab();
    }
  // wave 0 of an edge workgroup has one more load per slab in flight than the others
  const bool five = has_edge && wave == 0;
  if (C::NS - 1 < nk) {
    if (five) wait_vmcnt<(C::NS - 1) * (C::L + 1)>(); else wait_vmcnt<(C::NS - 1) * C::L>();
  } else {
    wait_vmcnt<0>();
  }
  __builtin_amdgcn_s_barrier();
  static_for<12>([&](auto uc) { read_unit(h0, 0u, IntC<0>{}, uc); });
  he0[0] = he0[1] = he1[0] = he1[1] = bf16x4{};
  if (has_edge) read_edge(he0, 0u, IntC<0>{});
  WAIT_HALVES_E(h0, he0);
  mask_halves(h0, he0, 0, 0);
  TIMELINE_STAMP(q, item, 1);

  // One slab: sixteen MFMAs in two steps of eight, numbered i = 2a + b within a
  // step.  The twelve transpose reads of the next step follow MFMAs 0-2 (four
  // each), so the last of them has five MFMAs of time to return.  Between the two
  // steps sits the slab's one barrier: before it every wave has finished reading
  // ring slot kt (the reads of the second step were waited for) and has seen its
  // own loads of slab kt+1 land, so behind it slot kt is free -- the loads of
  // slab kt+NS go there, behind MFMAs 3-7 of the second step -- and slab kt+1 is
  // complete for the reads of that step.  A slab thus has NS-1 slab times to
  // arrive.  KM >= 0 is the steady-state form (kt mod NS known at compile time,
  // a later slab always fetched, nothing ragged): no branch, no address
  // arithmetic.  KM < 0 is the general form used for the last slabs.
  auto do_slab = [&](int kt, auto kmc, auto edgec) {
    constexpr int KM = decltype(kmc)::value;
    constexpr bool FAST = KM >= 0, EDGE = decltype(edgec)::value;
    const bool fetch = FAST || kt + C::NS < nk;
    const bool more = FAST || kt + 1 < nk;
    const unsigned so = (unsigned)((kt % C::NS) * C::STAGE_BYTES);
    const unsigned so_next = (unsigned)(((kt + 1) % C::NS) * C::STAGE_BYTES);
    constexpr int ST_FETCH = FAST ? KM : -1;
    static_for<8>([&](auto ic) {
      constexpr int i = decltype(ic)::value, a = i / 2, b = (a & 1) ? 1 - i % 2 : i % 2;
      __builtin_amdgcn_sched_barrier(0);
      acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(h0, 2 * a), frag(h0, 8 + 2 * b), acc[a][b], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (i < 3) {
        static_for<4>([&](auto jc) {
          constexpr int u = 4 * i + decltype(jc)::value;
          if constexpr (FAST) read_unit_at(h1, IntC<(KM >= 0 ? KM : 0)>{}, IntC<1>{}, IntC<u>{});
          else read_unit(h1, so, IntC<1>{}, IntC<u>{});
        });
      } else if constexpr (EDGE && i == 3) {
        if constexpr (FAST) read_edge_at(he1, IntC<(KM >= 0 ? KM : 0)>{}, IntC<1>{});
        else read_edge(he1, so, IntC<1>{});
      }
    });
    if constexpr (EDGE) edge_mma(he0, h0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (EDGE) WAIT_HALVES_E(h1, he1); else WAIT_HALVES(h1);
    if constexpr (!FAST) mask_halves(h1, he1, kt, 1);
    // slab kt+1 has landed once at most the NS-2 younger slabs are outstanding
    if (FAST || kt + C::NS - 1 < nk) {
      if (EDGE && wave == 0) wait_vmcnt<(C::NS - 2) * (C::L + 1)>(); else wait_vmcnt<(C::NS - 2) * C::L>();
    } else {
      wait_vmcnt<0>();
    }
    __builtin_amdgcn_s_barrier();
    static_for<8>([&](auto ic) {
      constexpr int i = decltype(ic)::value, a = i / 2, b = (a & 1) ? 1 - i % 2 : i % 2;
      __builtin_amdgcn_sched_barrier(0);
      acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(h1, 2 * a), frag(h1, 8 + 2 * b), acc[a][b], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (i < 3) {
        static_for<4>([&](auto jc) {
          constexpr int u = 4 * i + decltype(jc)::value;
          if constexpr (FAST) read_unit_at(h0, IntC<(KM >= 0 ? (KM + 1) % C::NS : 0)>{}, IntC<0>{}, IntC<u>{});
          else if (more) read_unit(h0, so_next, IntC<0>{}, IntC<u>{});
        });
      } else {
        if constexpr (EDGE && i == 3) {
          if constexpr (FAST) read_edge_at(he0, IntC<(KM >= 0 ? (KM + 1) % C::NS : 0)>{}, IntC<0>{});
          else if (more) read_edge(he0, so_next, IntC<0>{});
        }
        // loads of slab kt+NS: one behind each of MFMAs 3-6, the rest behind MFMA 7
        static_for<C::L>([&](auto lc) {
          constexpr int l = decltype(lc)::value;
          if constexpr ((l < 4 ? l + 3 : 7) == i) {
            if constexpr (FAST) issue_one(lc, IntC<ST_FETCH>{});
            else if (fetch) issue_one(lc, IntC<-1>{});
          }
        });
        if constexpr (EDGE && i == 7) {
          if (fetch && wave == 0) issue_edge(IntC<ST_FETCH>{});
        }
      }
    });
    if (fetch) next_slab();
    if constexpr (EDGE) edge_mma(he1, h1);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (EDGE) WAIT_HALVES_E(h0, he0); else WAIT_HALVES(h0);
    if constexpr (!FAST) mask_halves(h0, he0, kt + 1, 0);
  };

  // Steady state: slabs whose fetch (of slab kt + NS) exists and is complete, in
  // groups of NS so that the ring slot is a compile-time constant.
  const bool last_ragged = (klen % C::BK) != 0;
  const int n_fast_raw = (nk - C::NS - (last_ragged ? 1 : 0)) / C::NS * C::NS;
  const int n_fast = n_fast_raw > 0 ? n_fast_raw : 0;
  auto run_slabs = [&](auto edgec) {
    int kt = 0;
    for (; kt < n_fast; kt += C::NS)
      static_for<C::NS>([&](auto kmc) { do_slab(kt + decltype(kmc)::value, kmc, edgec); });
    for (; kt < nk; ++kt) do_slab(kt, IntC<-1>{}, edgec);
  };
  if (has_edge) run_slabs(IntC<1>{}); else run_slabs(IntC<0>{});
  TIMELINE_STAMP(q, item, 2);

  // accumulator register v of a 32 x 32 block: row (v / 4) * 8 + (lane / 32) * 4 + v % 4, column lane % 32
  auto stage_half = [&](int h, float* dst) {      // dst: the wave's first row and column in the staging area
    static_for<(C::TM / 2) * C::TN>([&](auto blk_c) {
      constexpr int a2 = decltype(blk_c)::value / C::TN, b = decltype(blk_c)::value % C::TN;
      float* base = dst + (a2 * 32 + (lane >> 5) * 4) * C::EPI_PITCH + b * 32 + (lane & 31);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float x = h == 0 ? acc[a2][b][v] : acc[C::TM / 2 + a2][b][v];
        base[((v >> 2) * 8 + (v & 3)) * C::EPI_PITCH] = x;
      }
    });
  };
  auto emit_edge = [&](int64_t E) {
    if (!has_edge) return;
    // Edge block: MFMA rows 0-7 are the leading group, 8-15 the group of the trailing row
    // (registers v = 0..7 of the block); one element at a time, masked by the chunk's range.
    const int64_t col = col0 + wn0 + edge_blk * 32 + (lane & 31);
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      const int r8 = (lane >> 5) * 4 + (v & 3);
      int64_t row;
      if (v < 4) row = q.lead_base >= 0 ? q.lead_base + r8 : -1;
      else row = (q.trail_row >= 0 && (q.trail_row & 7) == r8) ? q.trail_row : -1;
      const int64_t flat = row * p.in + col;
      if (row >= 0 && col < p.in && flat >= p.begin && flat < p.end)
        emit<MODE>(q.s, E, slab, flat - p.begin, flat, acc_e[v]);
    }
  };
  tile_epilogue<C, MODE>(q, ldsb, row0, col0, slab, wave, lane, tid, stage_half, emit_edge);
  TIMELINE_STAMP(q, item, 3);
}

// The same tile with the 16x16x32 MFMA (which holds a higher clock under the part's power limit).
// A wave's 128 x 64 sub-tile is 8 x 4 blocks of 16 x 16; an MFMA takes all 32 tokens of a slab, so
// a slab is 32 MFMAs in two halves of 16: the upper four row blocks, then the lower four, each against
// the slab's four column blocks.  Operand layout of the MFMA: lane l holds row (column) l % 16 and the
// 8 tokens 8 (l / 16) ... + 7; a transpose read hands a 16-lane block 4 tokens of 16 rows, so an
// operand block is two reads (tokens +0..3, +4..7).  A half-wave of such a read touches 8 tokens x 32
// bytes; the 16-byte slots of a token row are therefore XOR-swizzled in bits 1-3 by
// (k & 3) | ((k >> 3 & 1) << 2), which puts the 8 tokens on the 8 different 32-byte groups of the
// 256-byte bank window (applied to the source offsets of the global->LDS loads, as in the other form).
// Registers: the MFMAs of a half go column block by column block, so that in the lower half a
// column block's registers are free after its four MFMAs and take the next slab's block at once; the
// row blocks of one half are read while the other half's MFMAs run.  The ring keeps the A images of
// all slabs together, then the B images, then the edge blocks: every read of an operand block is then
// one base register plus an immediate offset, whatever the ring slot.
#define WAIT8(h)                                                                                         \
  asm volatile("s_waitcnt lgkmcnt(0)"                                                                    \
               : "+v"(h[0]), "+v"(h[1]), "+v"(h[2]), "+v"(h[3]), "+v"(h[4]), "+v"(h[5]), "+v"(h[6]),     \
                 "+v"(h[7])::"memory")
#define WAIT8_8_2(ha, hb, he)                                                                            \
  asm volatile("s_waitcnt lgkmcnt(0)"                                                                    \
               : "+v"(ha[0]), "+v"(ha[1]), "+v"(ha[2]), "+v"(ha[3]), "+v"(ha[4]), "+v"(ha[5]),           \
                 "+v"(ha[6]), "+v"(ha[7]), "+v"(hb[0]), "+v"(hb[1]), "+v"(hb[2]), "+v"(hb[3]),           \
                 "+v"(hb[4]), "+v"(hb[5]), "+v"(hb[6]), "+v"(hb[7]), "+v"(he[0]), "+v"(he[1])::"memory")
// all LDS reads but the last two issued (the next slab's last column block) have returned
#define WAIT8_6_2_BUT2(ha, hb, he)                                                                       \
  asm volatile("s_waitcnt lgkmcnt(2)"                                                                    \
               : "+v"(ha[0]), "+v"(ha[1]), "+v"(ha[2]), "+v"(ha[3]), "+v"(ha[4]), "+v"(ha[5]),           \
                 "+v"(ha[6]), "+v"(ha[7]), "+v"(hb[0]), "+v"(hb[1]), "+v"(hb[2]), "+v"(hb[3]),           \
                 "+v"(hb[4]), "+v"(hb[5]), "+v"(he[0]), "+v"(he[1])::"memory")
// the two reads issued before the last eight have returned
#define WAIT2_BEFORE8(hb) asm volatile("s_waitcnt lgkmcnt(8)" : "+v"(hb[6]), "+v"(hb[7])::"memory")

template <class C, int MODE>
__device__ __forceinline__ void mfma_tile16(const MfmaParams& q, const int item, unsigned char* ldsb) {
  static_assert(C::MI == 16 && C::TM == 8 && C::TN == 4, "written out for 8 x 4 blocks of 16 x 16 per wave");
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  const WgradProblem& p = q.p;
  TIMELINE_STAMP(q, item, 0);
#ifdef CHUNKFT_TIMELINE
  if (q.timeline && threadIdx.x == 0)
    q.timeline[(size_t)item * 8 + 4] = ((unsigned long long)__builtin_amdgcn_s_getreg((32 - 1) << 11 | 20) << 32) |
                                       (unsigned)__builtin_amdgcn_s_getreg((32 - 1) << 11 | 4);
#endif

  // ---- which tile, which token slab (as in mfma_tile)
  const int n_tiles = q.tiles_m * q.tiles_n;
  const int slab = item / n_tiles;
  const int tile = item - slab * n_tiles;
  const int per_group = q.group_m * q.tiles_n;
  const int grp = tile / per_group;
  const int first_m = grp * q.group_m;
  const int gsz = (q.tiles_m - first_m < q.group_m) ? q.tiles_m - first_m : q.group_m;
  const int in_grp = tile - grp * per_group;
  const int tile_m = first_m + in_grp % gsz;
  const int tile_n = in_grp / gsz;
  const int64_t row0 = q.rb0 + (int64_t)tile_m * C::BM;
  const int64_t col0 = (int64_t)tile_n * C::BN;
  const int64_t k_begin = (int64_t)slab * p.kslab;
  const int64_t k_end = (k_begin + p.kslab < p.T) ? k_begin + p.kslab : p.T;
  const int klen = (int)(k_end - k_begin);
  const int nk = (klen + C::BK - 1) / C::BK;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave / C::WN) * (C::BM / C::WM);
  const int wn0 = (wave % C::WN) * (C::BN / C::WN);
  const unsigned short* dY = (const unsigned short*)p.dY;
  const unsigned short* X = (const unsigned short*)p.X;
  const unsigned lds_base = (unsigned)(uintptr_t)ldsb;

  // ---- global->LDS loads (as in mfma_tile; the slot swizzle is the one described above)
  // A wave's loads of one operand name tokens 4 apart (A) or 2 apart (B); tokens 4 apart have the same
  // swizzle, so loads i and i + (4 tokens) share their per-lane offset and differ in a scalar offset.
  constexpr int LPT_A = C::RA / 16, TPL_A = 64 / LPT_A;
  constexpr int VA = TPL_A >= 4 ? 1 : (C::LA < 4 / TPL_A ? C::LA : 4 / TPL_A);   // distinct per-lane offsets
  constexpr int VB = C::LB < 2 ? C::LB : 2;
  unsigned voa[VA], vob[VB];
  const unsigned lddy2 = (unsigned)(p.lddy * 2), ldx2 = (unsigned)(p.ldx * 2);
  auto swz = [](int k) { return ((k & 3) | (((k >> 3) & 1) << 2)) << 1; };
  auto tok_a = [&](int i) { return TPL_A * (wave * C::LA + i) + lane / LPT_A; };
  auto tok_b = [&](int i) { return 2 * (wave * C::LB + i) + (lane >> 5); };
  static_assert((TPL_A * C::LA == 4 || TPL_A * C::LA == 8) && (2 * C::LB == 4 || 2 * C::LB == 8),
                "a wave's tokens of one operand are an aligned group of 4 or 8: tokens 4 apart share bit 3");
#pragma unroll
  for (int i = 0; i < VA; ++i) {
    const int k = tok_a(i);
    const int lc = (lane % LPT_A) ^ swz(k);
    int64_t r = row0 + lc * 8;
    if (r >= p.out) r = row0;
    voa[i] = (unsigned)r * 2u + (unsigned)k * lddy2;
  }
#pragma unroll
  for (int i = 0; i < VB; ++i) {
    const int k = tok_b(i);
    const int lc = (lane & 31) ^ swz(k);
    int64_t cc = col0 + lc * 8;
    if (cc >= p.in) cc = col0;
    vob[i] = (unsigned)cc * 2u + (unsigned)k * ldx2;
  }
  const unsigned char* ga = (const unsigned char*)(dY + k_begin * p.lddy);
  const unsigned char* gb = (const unsigned char*)(X + k_begin * p.ldx);
  const int64_t stepA = (int64_t)C::BK * p.lddy * 2, stepB = (int64_t)C::BK * p.ldx * 2;
  int next_fetch = 0;
  auto load_to_lds = [&](const unsigned char* base, unsigned voff, unsigned soff, unsigned dst) {
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (LDS_PTR(void))(uintptr_t)dst, 16, (int)voff, (int)soff, 0, 0);
  };
  auto next_slab = [&]() {
    ga += stepA;
    gb += stepB;
    ++next_fetch;
  };

  // ---- edge block: 16 rows per token (the 8-row group of the leading edge rows, the 8-row group of
  // the trailing row), one 16 x 16 row block.  The two workgroups (waves) that share 64 columns take
  // two of its four 16-column blocks each.
  const bool has_edge = (C::WM == 2 ? tile_m == 0 : tile_m < 2) && (q.lead_base >= 0 || q.trail_row >= 0);
  const int edge_blk = C::WM == 2 ? (wave >> 2) : tile_m;
  const int ke = lane >> 1;
  unsigned voe;
  {
    const int64_t lead = q.lead_base >= 0 ? q.lead_base : q.rb0;
    const int64_t trail = q.trail_row >= 0 ? (q.trail_row & ~(int64_t)7) : q.rb0;
    voe = (unsigned)((lane & 1) ? trail : lead) * 2u + (unsigned)ke * lddy2;
  }
  auto issue_edge = [&](auto stagec) {
    constexpr int STAGE = decltype(stagec)::value;
    const int stage = STAGE >= 0 ? STAGE : next_fetch % C::NS;
    const bool ragged = STAGE >= 0 ? false : (next_fetch + 1) * C::BK > klen;
    unsigned vo = voe;
    if (ragged) {
      const int64_t over = k_begin + (int64_t)next_fetch * C::BK + ke - (p.T - 1);
      if (over > 0) vo -= (unsigned)over * lddy2;
    }
    load_to_lds(ga, vo, 0u, lds_base + C::NS * (C::A_BYTES + C::B_BYTES) + stage * C::E_BYTES);
  };
  auto issue_one = [&](auto idxc, auto stagec) {
    constexpr int idx = decltype(idxc)::value, STAGE = decltype(stagec)::value;
    const int stage = STAGE >= 0 ? STAGE : next_fetch % C::NS;
    const bool ragged = STAGE >= 0 ? false : (next_fetch + 1) * C::BK > klen;
    if constexpr (idx < C::LA) {
      constexpr int i = idx;
      unsigned vo = voa[i % VA];
      if (ragged) {
        const int64_t over = k_begin + (int64_t)next_fetch * C::BK + tok_a(i) - (p.T - 1);
        if (over > 0) vo -= (unsigned)over * lddy2;
      }
      load_to_lds(ga, vo, (unsigned)(i / VA) * (unsigned)(TPL_A * VA) * lddy2,
                  lds_base + stage * C::A_BYTES + (wave * C::LA + i) * 1024);
    } else {
      constexpr int i = idx - C::LA;
      unsigned vo = vob[i % VB];
      if (ragged) {
        const int64_t over = k_begin + (int64_t)next_fetch * C::BK + tok_b(i) - (p.T - 1);
        if (over > 0) vo -= (unsigned)over * ldx2;
      }
      load_to_lds(gb, vo, (unsigned)(i / VB) * (unsigned)(2 * VB) * ldx2,
                  lds_base + C::NS * C::A_BYTES + stage * C::B_BYTES + (wave * C::LB + i) * 1024);
    }
  };

  // ---- transpose-read addressing
  const int blk = lane >> 4, i16 = lane & 15;
  const int tr_k = blk * 8 + (i16 >> 2);                     // first of the 4 + 4 tokens this lane's reads name
  const int swl = ((i16 >> 2) | ((blk & 1) << 2)) << 1;      // the swizzle of those tokens
  const int low = (i16 & 3) >> 1;
  const int sub = (i16 & 1) * 8;
  static_assert((C::NS - 1) * C::A_BYTES + 4 * C::RA < 65536 && (C::NS - 1) * C::B_BYTES + 4 * C::RB < 65536,
                "LDS offset field");
  unsigned addrA[C::TM], addrB[C::TN];
#pragma unroll
  for (int a = 0; a < C::TM; ++a)
    addrA[a] = lds_base + tr_k * C::RA + ((((wm0 >> 3) + a * 2) ^ swl) + low) * 16 + sub;
#pragma unroll
  for (int b = 0; b < C::TN; ++b)
    addrB[b] = lds_base + C::NS * C::A_BYTES + tr_k * C::RB + ((((wn0 >> 3) + b * 2) ^ swl) + low) * 16 + sub;
  const unsigned addrE = lds_base + C::NS * (C::A_BYTES + C::B_BYTES) + tr_k * 32 + (i16 & 3) * 8;

  // Fragment halves: unit u of a row half is row block u / 2 of that half (tokens +0..3 if u is
  // even, +4..7 if odd); unit u of the column set is column block u / 2 likewise.
  bf16x4 ha0[8], ha1[8], hb[8], he[2];
  // RH: which four row blocks (0: upper, 1: lower); st: ring slot
  auto read_a = [&](bf16x4* h, auto rhc, int st, auto uc) {
    constexpr int RH = decltype(rhc)::value, u = decltype(uc)::value;
    h[u] = lds_tr_read<(u & 1) * 4 * C::RA>(addrA[4 * RH + u / 2] + (unsigned)(st * C::A_BYTES));
  };
  auto read_a_at = [&](bf16x4* h, auto rhc, auto stagec, auto uc) {
    constexpr int RH = decltype(rhc)::value, st = decltype(stagec)::value, u = decltype(uc)::value;
    h[u] = lds_tr_read<st * C::A_BYTES + (u & 1) * 4 * C::RA>(addrA[4 * RH + u / 2]);
  };
  auto read_b = [&](int st, auto uc) {
    constexpr int u = decltype(uc)::value;
    hb[u] = lds_tr_read<(u & 1) * 4 * C::RB>(addrB[u / 2] + (unsigned)(st * C::B_BYTES));
  };
  auto read_b_at = [&](auto stagec, auto uc) {
    constexpr int st = decltype(stagec)::value, u = decltype(uc)::value;
    hb[u] = lds_tr_read<st * C::B_BYTES + (u & 1) * 4 * C::RB>(addrB[u / 2]);
  };
  auto read_e = [&](int st) {
    he[0] = lds_tr_read<0>(addrE + (unsigned)(st * C::E_BYTES));
    he[1] = lds_tr_read<4 * 32>(addrE + (unsigned)(st * C::E_BYTES));
  };
  auto read_e_at = [&](auto stagec) {
    constexpr int st = decltype(stagec)::value;
    he[0] = lds_tr_read<st * C::E_BYTES>(addrE);
    he[1] = lds_tr_read<st * C::E_BYTES + 4 * 32>(addrE);
  };
  auto frag = [&](const bf16x4* h, int u) {
    return __builtin_shufflevector(h[u], h[u + 1], 0, 1, 2, 3, 4, 5, 6, 7);
  };
  // tokens past the end of a ragged last slab: zero in the operands (units [U0, U1) of h)
  auto mask_units = [&](bf16x4* h, int kt, auto u0c, auto u1c) {
    if (kt == nk - 1 && (klen % C::BK) != 0) {
      const int kv = klen - kt * C::BK - blk * 8;            // valid tokens among this lane's 8
#pragma unroll
      for (int u = decltype(u0c)::value; u < decltype(u1c)::value; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((u & 1) * 4 + e >= kv) h[u][e] = (__bf16)0.f;
    }
  };
  auto mask_edge = [&](int kt) {
    if (kt == nk - 1 && (klen % C::BK) != 0) {
      const int kv = klen - kt * C::BK - blk * 8;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (u * 4 + e >= kv) he[u][e] = (__bf16)0.f;
    }
  };

  f32x4_t acc[C::TM][C::TN], acc_e[2];
#pragma unroll
  for (int a = 0; a < C::TM; ++a)
#pragma unroll
    for (int b = 0; b < C::TN; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[a][b][v] = 0.f;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc_e[j][v] = 0.f;

  // ---- prologue: the whole ring in flight, the operands of slab 0's upper half in registers
#pragma unroll
  for (int s = 0; s < C::NS; ++s)
    if (s < nk) {
      static_for<C::L>([&](auto ic) { issue_one(ic, IntC<-1>{}); });
      if (has_edge && wave == 0) issue_edge(IntC<-1>{});
      next_slab();
    }
  const bool five = has_edge && wave == 0;
  if (C::NS - 1 < nk) {
    if (five) wait_vmcnt<(C::NS - 1) * (C::L + 1)>(); else wait_vmcnt<(C::NS - 1) * C::L>();
  } else {
    wait_vmcnt<0>();
  }
  __builtin_amdgcn_s_barrier();
  static_for<8>([&](auto uc) { read_a(ha0, IntC<0>{}, 0, uc); });
  static_for<8>([&](auto uc) { read_b(0, uc); });
  he[0] = he[1] = bf16x4{};
  if (has_edge) read_e(0);
  WAIT8_8_2(ha0, hb, he);
  mask_units(ha0, 0, IntC<0>{}, IntC<8>{});
  mask_units(hb, 0, IntC<0>{}, IntC<8>{});
  mask_edge(0);
  TIMELINE_STAMP(q, item, 1);

  // the edge MFMAs of a wave use two of its four column blocks (picked by value, as in mfma_tile)
  auto edge_mma = [&]() {
    const bf16x8 fe = __builtin_shufflevector(he[0], he[1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const u32x4_t lo = __builtin_bit_cast(u32x4_t, __builtin_shufflevector(hb[2 * j], hb[2 * j + 1], 0, 1, 2, 3, 4, 5, 6, 7));
      const u32x4_t hi = __builtin_bit_cast(u32x4_t, __builtin_shufflevector(hb[4 + 2 * j], hb[5 + 2 * j], 0, 1, 2, 3, 4, 5, 6, 7));
      u32x4_t bs;
#pragma unroll
      for (int e = 0; e < 4; ++e) bs[e] = edge_blk == 0 ? lo[e] : hi[e];
      acc_e[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fe, __builtin_bit_cast(bf16x8, bs), acc_e[j], 0, 0, 0);
    }
  };

  // One slab.  Upper half: its 16 MFMAs (column block by column block), the reads of the lower row
  // blocks behind the first two; the last column block, whose reads were issued last in the slab
  // before, is waited for in front of its first MFMA.  Then the slab's one barrier (as in mfma_tile:
  // slot kt is consumed, slab kt+1 has landed).  Lower half: its 16 MFMAs; behind them the reads of
  // slab kt+1 -- upper row blocks and edge block first, each column block as soon as its four MFMAs
  // are issued -- and the loads of slab kt+NS.
  auto do_slab = [&](int kt, auto kmc, auto edgec) {
    constexpr int KM = decltype(kmc)::value;
    constexpr bool FAST = KM >= 0, EDGE = decltype(edgec)::value;
    const bool fetch = FAST || kt + C::NS < nk;
    const bool more = FAST || kt + 1 < nk;
    const int st = kt % C::NS, st_next = (kt + 1) % C::NS;
    constexpr int ST_FETCH = FAST ? KM : -1;
    constexpr int ST_NEXT = FAST ? (KM + 1) % C::NS : 0;
    static_for<16>([&](auto ic) {
      constexpr int i = decltype(ic)::value, b = i / 4, a = (b & 1) ? 3 - i % 4 : i % 4;
      if constexpr (i == 12) {
        WAIT2_BEFORE8(hb);                         // (nothing to wait for in slab 0: the prologue waited for everything)
        if constexpr (!FAST) mask_units(hb, kt, IntC<6>{}, IntC<8>{});
      }
      __builtin_amdgcn_sched_barrier(0);
      acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(ha0, 2 * a), frag(hb, 2 * b), acc[a][b], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (i < 2) {
        static_for<4>([&](auto jc) {
          constexpr int u = 4 * i + decltype(jc)::value;
          if constexpr (FAST) read_a_at(ha1, IntC<1>{}, IntC<(KM >= 0 ? KM : 0)>{}, IntC<u>{});
          else read_a(ha1, IntC<1>{}, st, IntC<u>{});
        });
      }
    });
    if constexpr (EDGE) edge_mma();
    __builtin_amdgcn_sched_barrier(0);
    WAIT8(ha1);
    if constexpr (!FAST) mask_units(ha1, kt, IntC<0>{}, IntC<8>{});
    if (FAST || kt + C::NS - 1 < nk) {
      if (EDGE && wave == 0) wait_vmcnt<(C::NS - 2) * (C::L + 1)>(); else wait_vmcnt<(C::NS - 2) * C::L>();
    } else {
      wait_vmcnt<0>();
    }
    __builtin_amdgcn_s_barrier();
    static_for<16>([&](auto ic) {
      constexpr int i = decltype(ic)::value, b = i / 4, a = (b & 1) ? 3 - i % 4 : i % 4;
      __builtin_amdgcn_sched_barrier(0);
      acc[4 + a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(ha1, 2 * a), frag(hb, 2 * b), acc[4 + a][b], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (i < 2) {
        static_for<4>([&](auto jc) {
          constexpr int u = 4 * i + decltype(jc)::value;
          if constexpr (FAST) read_a_at(ha0, IntC<0>{}, IntC<ST_NEXT>{}, IntC<u>{});
          else if (more) read_a(ha0, IntC<0>{}, st_next, IntC<u>{});
        });
      }
      if constexpr (EDGE && i == 2) {
        if constexpr (FAST) read_e_at(IntC<ST_NEXT>{});
        else if (more) read_e(st_next);
      }
      if constexpr (i % 4 == 3) {                  // column block b has had its last MFMA of this slab
        static_for<2>([&](auto jc) {
          constexpr int u = 2 * b + decltype(jc)::value;
          if constexpr (FAST) read_b_at(IntC<ST_NEXT>{}, IntC<u>{});
          else if (more) read_b(st_next, IntC<u>{});
        });
      }
      // loads of slab kt+NS: one behind each of MFMAs 4, 5, 6, 8, 9, 10
      static_for<C::L>([&](auto lc) {
        constexpr int l = decltype(lc)::value;
        if constexpr ((l < 3 ? 4 + l : 5 + l) == i) {
          if constexpr (FAST) issue_one(lc, IntC<ST_FETCH>{});
          else if (fetch) issue_one(lc, IntC<-1>{});
        }
      });
      if constexpr (EDGE && i == 12) {
        if (fetch && wave == 0) issue_edge(IntC<ST_FETCH>{});
      }
    });
    if (fetch) next_slab();
    __builtin_amdgcn_sched_barrier(0);
    WAIT8_6_2_BUT2(ha0, hb, he);
    if constexpr (!FAST) {
      mask_units(ha0, kt + 1, IntC<0>{}, IntC<8>{});
      mask_units(hb, kt + 1, IntC<0>{}, IntC<6>{});
      if constexpr (EDGE) mask_edge(kt + 1);
    }
  };

  // Steady state: slabs whose fetch (of slab kt + NS) exists and is complete, in groups of NS so that
  // the ring slot is a compile-time constant.
  const bool last_ragged = (klen % C::BK) != 0;
  const int n_fast_raw = (nk - C::NS - (last_ragged ? 1 : 0)) / C::NS * C::NS;
  const int n_fast = n_fast_raw > 0 ? n_fast_raw : 0;
  auto run_slabs = [&](auto edgec) {
    int kt = 0;
    for (; kt < n_fast; kt += C::NS)
      static_for<C::NS>([&](auto kmc) { do_slab(kt + decltype(kmc)::value, kmc, edgec); });
    for (; kt < nk; ++kt) do_slab(kt, IntC<-1>{}, edgec);
  };
  if (has_edge) run_slabs(IntC<1>{}); else run_slabs(IntC<0>{});
  TIMELINE_STAMP(q, item, 2);

  // accumulator register v of a 16 x 16 block: row (lane / 16) * 4 + v, column lane % 16
  auto stage_half = [&](int h, float* dst) {
    static_for<4 * C::TN>([&](auto blk_c) {
      constexpr int a = decltype(blk_c)::value / C::TN, b = decltype(blk_c)::value % C::TN;
      float* base = dst + (a * 16 + (lane >> 4) * 4) * C::EPI_PITCH + b * 16 + (lane & 15);
#pragma unroll
      for (int v = 0; v < 4; ++v) base[v * C::EPI_PITCH] = h == 0 ? acc[a][b][v] : acc[4 + a][b][v];
    });
  };
  auto emit_edge = [&](int64_t E) {
    if (!has_edge) return;
    // edge block rows 0-7 are the leading group, 8-15 the group of the trailing row
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t col = col0 + wn0 + (2 * edge_blk + j) * 16 + (lane & 15);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = (lane >> 4) * 4 + v;
        int64_t row;
        if (r < 8) row = q.lead_base >= 0 ? q.lead_base + r : -1;
        else row = (q.trail_row >= 0 && (q.trail_row & 7) == r - 8) ? q.trail_row : -1;
        const int64_t flat = row * p.in + col;
        if (row >= 0 && col < p.in && flat >= p.begin && flat < p.end)
          emit<MODE>(q.s, E, slab, flat - p.begin, flat, acc_e[j][v]);
      }
    }
  };
  tile_epilogue<C, MODE>(q, ldsb, row0, col0, slab, wave, lane, tid, stage_half, emit_edge);
  TIMELINE_STAMP(q, item, 3);
}

// Two workgroups share a compute unit.  Started together they run their MFMA loops
// together and then their HBM-bound epilogues together; with stagger > 0 the second
// one of each pair (workgroups are dealt to the 32 compute units of an XCD in order:
// the first 32 fill one slot each, the next 32 the other) starts late instead, so that
// one tends to be in its loop while the other is in its epilogue.
template <class C>
__device__ __forceinline__ void start_offset(int stagger) {
  const int j = (int)(blockIdx.x >> 3);
  if (C::WM == 1 && j >= 32 && j < 64)
    for (int i = 0; i < stagger; ++i) __builtin_amdgcn_s_sleep(127);
}

// The parameters stay in the kernel-argument memory and are read where they are used (the index
// below is always 0, which the compiler cannot know): taken by value they are all loaded into scalar
// registers up front, and the loop then runs out of registers (14 spilled vector registers in the
// 128 x 256 configuration against 2).
struct MfmaArgs {
  MfmaParams q[1];
};

template <class C, int MODE>
__global__ __launch_bounds__(C::NT, 2) void wgrad_mfma_kernel(const MfmaArgs args) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char ldsb[];
  const MfmaParams& q = args.q[blockIdx.y];
  const int n_items = q.n_tile_items;
  const int per_xcd = (n_items + 7) >> 3;
  const int xcd = (int)(blockIdx.x & 7), first = xcd * per_xcd;
  int j = (int)(blockIdx.x >> 3);
  if (first + j >= n_items) return;
  if (MODE == EMIT_ACCUM && q.turned) {
    const int run = n_items - first < per_xcd ? n_items - first : per_xcd;
    j += xcd * (run >> 3);
    if (j >= run) j -= run;
  }
  const int item = first + j;
  start_offset<C>(q.stagger);
  if constexpr (C::MI == 16) mfma_tile16<C, MODE>(q, item, ldsb);
  else mfma_tile<C, MODE>(q, item, ldsb);
}

// ---------------------------------------------------------------------------
// scale-vector gradient: g[j] = sum_t dY[t, j] * X[t, j]
// ---------------------------------------------------------------------------
// A block is CB columns over all tokens.  The tokens are dealt to 128 groups, group g = tokens g, g + 128, ...;
// a lane takes VE = 16 bytes / element size columns of a group, so that a wave's load is 1 KB of whole
// pieces (with one 2-byte column per lane, as this kernel had it, the loads were 128 bytes and a compute
// unit took in 3 bytes per clock).  The group sums meet in LDS, eight at a time and then the sixteen sums of
// eight, in group order: the result depends neither on CB nor on the number of threads.
// With NORM the operator normalises its input itself: X is the raw input and stats[2t],
// stats[2t+1] are the token's mean (0 for RMSNorm) and reciprocal standard deviation.
constexpr int kColsumGroups = 128;
constexpr int kColsumCols = 64;                // columns of a block in the grouped call
constexpr int kColsumUnroll = 4;               // tokens in flight per lane

template <typename T> struct Piece;            // 16 bytes of consecutive elements at any element
template <> struct Piece<float> {
  static constexpr int N = 4;
  f32x4_u v;
  __device__ __forceinline__ void load(const float* p) { v = *(const f32x4_u*)p; }
  __device__ __forceinline__ float at(int i) const { return v[i]; }
};
template <> struct Piece<unsigned short> {
  static constexpr int N = 8;
  typedef unsigned int raw_t __attribute__((ext_vector_type(4), aligned(2)));
  u32x4_t v;
  __device__ __forceinline__ void load(const unsigned short* p) { v = *(const raw_t*)p; }
  __device__ __forceinline__ float at(int i) const {
    return __uint_as_float(i & 1 ? v[i / 2] & 0xffff0000u : v[i / 2] << 16);
  }
};

template <int CB> constexpr size_t colsum_lds_floats = (size_t)(kColsumGroups + 16) * CB;

template <typename T, int MODE, int NORM, int NT, int CB>
__device__ __forceinline__ void colsum_block(const WgradProblem& p, const Sinks& s, const float* stats, int64_t block,
                                             float* red) {
  constexpr int VE = Piece<T>::N, LPG = CB / VE, NG = NT / LPG, U = kColsumUnroll;
  static_assert(CB % VE == 0 && kColsumGroups % NG == 0, "whole passes over the groups");
  const T* const dY = (const T*)p.dY;
  const T* const X = (const T*)p.X;
  const int l = threadIdx.x % LPG;
  const int64_t first = p.begin + block * CB + l * VE;        // the lane's columns, nominally
  // a piece that would reach past the row is moved back; a vector shorter than a piece goes by elements
  const bool pieces = p.in >= VE;
  const int64_t col = pieces ? (first + VE <= p.in ? first : p.in - VE) : first;
  for (int g = threadIdx.x / LPG; g < kColsumGroups; g += NG) {
    float acc[VE];
#pragma unroll
    for (int e = 0; e < VE; ++e) acc[e] = 0.f;
    if (first < p.end) {
      auto add = [&](int64_t t, const Piece<T>& x, const Piece<T>& d) {
        float mean = 0.f, rstd = 1.f;
        if constexpr (NORM) { mean = stats[2 * t]; rstd = stats[2 * t + 1]; }
#pragma unroll
        for (int e = 0; e < VE; ++e) {
          float v = x.at(e);
          if constexpr (NORM) v = (v - mean) * rstd;
          acc[e] = fmaf(d.at(e), v, acc[e]);
        }
      };
      if (pieces) {
        int64_t t = g;
        for (; t + (U - 1) * kColsumGroups < p.T; t += U * kColsumGroups) {
          Piece<T> x[U], d[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            x[u].load(X + (t + u * kColsumGroups) * p.ldx + col);
            d[u].load(dY + (t + u * kColsumGroups) * p.lddy + col);
          }
#pragma unroll
          for (int u = 0; u < U; ++u) add(t + u * kColsumGroups, x[u], d[u]);
        }
        for (; t < p.T; t += kColsumGroups) {
          Piece<T> x, d;
          x.load(X + t * p.ldx + col);
          d.load(dY + t * p.lddy + col);
          add(t, x, d);
        }
      } else {
        for (int64_t t = g; t < p.T; t += kColsumGroups)
          for (int e = 0; e < VE; ++e) {
            if (col + e >= p.in) break;
            float v = load_as_f32<T>(X + t * p.ldx + col + e);
            if constexpr (NORM) v = (v - stats[2 * t]) * stats[2 * t + 1];
            acc[e] = fmaf(load_as_f32<T>(dY + t * p.lddy + col + e), v, acc[e]);
          }
      }
    }
#pragma unroll
    for (int e = 0; e < VE; ++e) red[g * CB + l * VE + e] = acc[e];
  }
  __syncthreads();
  float* const red2 = red + kColsumGroups * CB;
  for (int o = threadIdx.x; o < 16 * CB; o += NT) {
    const int part = o / CB, c = o % CB;
    float sum = red[part * 8 * CB + c];
#pragma unroll
    for (int k = 1; k < 8; ++k) sum += red[(part * 8 + k) * CB + c];
    red2[o] = sum;
  }
  __syncthreads();
  if (threadIdx.x < CB) {
    const int lane = threadIdx.x / VE, e = threadIdx.x % VE;
    const int64_t nominal = p.begin + block * CB + lane * VE, j = nominal + e;
    if (j < p.end) {
      // in a piece that was moved back, column j sits that much further on
      const int64_t moved = pieces && nominal + VE > p.in ? nominal - (p.in - VE) : 0;
      const int c = (int)(lane * VE + e + moved);
      float sum = red2[c];
      for (int k = 1; k < 16; ++k) sum += red2[k * CB + c];
      emit<MODE>(s, p.end - p.begin, 0, j - p.begin, j, sum);
    }
  }
}

// one group per LPG lanes
template <typename T, int CB> constexpr int kColsumThreads = kColsumGroups * CB / Piece<T>::N;

template <typename T, int MODE, int NORM, int CB>
__global__ __launch_bounds__((kColsumThreads<T, CB>)) void colsum_kernel(const WgradProblem p, const Sinks s, const float* stats,
                                                                         int blocks) {
  __shared__ float red[colsum_lds_floats<CB>];
  const int block = xcd_work_item(blocks);
  if (block < 0) return;
  colsum_block<T, MODE, NORM, kColsumThreads<T, CB>, CB>(p, s, stats, block, red);
}

// ---------------------------------------------------------------------------
// one launch for all segments of a chunk (fused call only)
// ---------------------------------------------------------------------------
// The work items of up to kGroupMax segments are laid end to end: the tiles of each bf16 matrix
// segment (parameters as for wgrad_mfma_kernel) and, for a bf16 scale-vector segment (tiles_m = 0),
// blocks of kColsumCols elements.  A workgroup finds its segment by its item number and then does exactly
// what the single-segment kernels do, in the same order, so the results are theirs bit for bit.
constexpr int kGroupMax = 12;

struct GroupParams {
  int32_t n_segs, n_items, stagger, reserved;
  int32_t item_start[kGroupMax + 1];     // first work item of each segment; [n_segs] = n_items
  MfmaParams seg[kGroupMax];
};
static_assert(sizeof(GroupParams) <= 4096, "the table travels as a kernel argument");

template <class C>
__global__ __launch_bounds__(C::NT, 2) void wgrad_group_kernel(const GroupParams gp) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char ldsb[];
  const int item = xcd_work_item(gp.n_items);
  if (item < 0) return;
  start_offset<C>(gp.stagger);
  int si = 0;
  while (si + 1 < gp.n_segs && item >= gp.item_start[si + 1]) ++si;
  const MfmaParams& q = gp.seg[si];
  const int local = item - gp.item_start[si];
  if (q.tiles_m == 0)
    colsum_block<unsigned short, EMIT_ADAMW, 0, C::NT, kColsumCols>(q.p, q.s, nullptr, local, reinterpret_cast<float*>(ldsb));
  else if constexpr (C::MI == 16) mfma_tile16<C, EMIT_ADAMW>(q, local, ldsb);
  else mfma_tile<C, EMIT_ADAMW>(q, local, ldsb);
}

// Per-token statistics of RMSNorm (SUB = 0) or LayerNorm (SUB = 1): one wave per token, two
// passes over the row (mean first, then the centred sum of squares), fp32, 16 bytes per lane.
template <typename T, int SUB>
__global__ __launch_bounds__(256) void norm_stats_kernel(const T* X, int64_t ldx, int64_t n, int64_t tokens,
                                                         float eps, float* stats) {
  constexpr int VE = Piece<T>::N, U = 4;
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= tokens) return;
  const T* row = X + t * ldx;
  auto row_sum = [&](auto term) {                             // sum of term(x) over the row
    float s[2] = {0.f, 0.f};
    int64_t j = lane * VE;
    for (; j + (U - 1) * 64 * VE + VE <= n; j += U * 64 * VE) {
      Piece<T> x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u].load(row + j + u * 64 * VE);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < VE; ++e) s[e & 1] = term(x[u].at(e), s[e & 1]);
    }
    for (; j + VE <= n; j += 64 * VE) {
      Piece<T> x;
      x.load(row + j);
#pragma unroll
      for (int e = 0; e < VE; ++e) s[e & 1] = term(x.at(e), s[e & 1]);
    }
    for (; j < n; ++j) {                                      // the one lane whose piece the row's end cuts
      s[0] = term(load_as_f32<T>(row + j), s[0]);
      if ((j + 1) % VE == 0) break;
    }
    float v = s[0] + s[1];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
  };
  float mean = 0.f;
  if constexpr (SUB) mean = row_sum([](float x, float s) { return s + x; }) / (float)n;
  const float var = row_sum([&](float x, float s) { return fmaf(x - mean, x - mean, s); }) / (float)n;
  if (lane == 0) {
    stats[2 * t] = mean;
    stats[2 * t + 1] = 1.0f / sqrtf(var + eps);
  }
}

// ---------------------------------------------------------------------------
// embedding table gradient: g[r, :] = sum over the tokens t with ids[t] = r of dY[t, :]
// ---------------------------------------------------------------------------
// A group is kEmbRows = 64 consecutive table rows and a block of 1024 columns; a workgroup of 8 waves takes
// it, or one of its PARTS runs of rows.  It first turns the token ids into "which of the group's rows, if
// any" in LDS (every wave a run of the tokens, counted and then written behind the hits of the waves
// before it), the short list of hits in token order.  Every wave then takes rows in turn: it looks through
// the list 64 entries at a time (a ballot per 64; entry by entry, as it was, the walk was a chain of LDS
// latencies as long as the list: 154 us for a 8000 x 512 table at 1024 tokens, now 38) and adds the dY rows
// of its row in ascending token order -- no atomics, the order of the sum is fixed.  The loads of four
// tokens are issued before their additions, so a row that several
// tokens name does not cost one memory latency per token; a row that very many name (token
// frequencies are heavy-tailed: the commonest token can be a tenth of a batch, and common tokens
// can be neighbours in the table) is summed by all eight waves together, wave w taking every eighth hit,
// and the eight partial sums are added in wave order -- still a fixed order.  A lane holds the columns
// 256 i + 4 lane + e (i < kEmbIter, e < 4), so loads and
// stores of a wave are 1 KB (fp32) pieces.  HBM-bound: the rows are written (or updated)
// once, whether any token names them or not -- except when the result is added to g
// (accumulation over micro-batches), where only the named rows are touched.  Fused call, 128 Mi elements of
// 128256 x 4096 at 4096 tokens: 635 us = 5.5 TB/s (710 with one part, the walk and two shared rows a group at most).
constexpr int kEmbWaves = 8;
constexpr int kEmbRows = 64;       // rows of a group
constexpr int kEmbIter = 4;        // 256-column pieces per workgroup
constexpr int kEmbTok = 8192;      // most tokens per call (their list lives in LDS)
constexpr int kEmbHot = 32;        // hits from which a row is summed by all waves together
static_assert(kEmbRows == 64, "a row is a bit of a ballot");
static_assert(64 * kEmbWaves == kEmbedThreads, "embed_parts counts the threads of a launch");

template <typename T> __device__ __forceinline__ void load4_as_f32(const T* p, int valid, float (&o)[4]);
template <> __device__ __forceinline__ void load4_as_f32<float>(const float* p, int valid, float (&o)[4]) {
  if (valid >= 4) {
    const f32x4_u v = *(const f32x4_u*)p;
    o[0] = v[0]; o[1] = v[1]; o[2] = v[2]; o[3] = v[3];
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = e < valid ? p[e] : 0.f;
  }
}
template <> __device__ __forceinline__ void load4_as_f32<unsigned short>(const unsigned short* p, int valid,
                                                                         float (&o)[4]) {
  if (valid >= 4) {
    const u32x2_a2 v = *(const u32x2_a2*)p;
    o[0] = __uint_as_float(v[0] << 16); o[1] = __uint_as_float(v[0] & 0xffff0000u);
    o[2] = __uint_as_float(v[1] << 16); o[3] = __uint_as_float(v[1] & 0xffff0000u);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = e < valid ? bf16_bits_to_f32(p[e]) : 0.f;
  }
}

template <typename T, int MODE, int PARTS>
__global__ __launch_bounds__(64 * kEmbWaves) void embed_wgrad_kernel(const WgradProblem p, const Sinks s) {
  constexpr int kPartRows = kEmbRows / PARTS;
  __shared__ int list[kEmbTok];
  __shared__ unsigned char row_of[kEmbTok];
  __shared__ int wave_hits[kEmbWaves], hits_of[kEmbRows];
  __shared__ __attribute__((aligned(16))) float part[kEmbWaves][256 * kEmbIter];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // column blocks of one group of rows are neighbours in the launch order, so that a row's
  // pieces are touched at about the same time
  const int n_cblk = (int)((p.in + 256 * kEmbIter - 1) / (256 * kEmbIter));
  const int part_id = (int)(blockIdx.x / n_cblk % PARTS);
  const int64_t row_base = p.begin / p.in + (int64_t)(blockIdx.x / n_cblk / PARTS) * kEmbRows;
  const int64_t row_last = (p.end - 1) / p.in;
  const int64_t cbase = (int64_t)(blockIdx.x % n_cblk) * (256 * kEmbIter);
  const int64_t* ids = (const int64_t*)p.X;
  const T* dY = (const T*)p.dY;
  const int n = (int)p.T;                                   // <= kEmbTok, checked by the launcher
  // every wave takes a run of whole 64s of the tokens: notes which of the rows each names and counts its hits, then
  // writes them behind those of the waves before it as entries (token << 6 | row), so that token order is kept
  const int run = (n + 64 * kEmbWaves - 1) / (64 * kEmbWaves) * 64, t_begin = wave * run;
  const int t_end = t_begin + run < n ? t_begin + run : n;
  int count = 0;
#pragma unroll 4
  for (int t0 = t_begin; t0 < t_end; t0 += 64) {
    const int64_t d = t0 + lane < t_end ? ids[t0 + lane] - row_base : -1;
    const bool hit = d >= 0 && d < kEmbRows;
    row_of[t0 + lane] = hit ? (unsigned char)d : (unsigned char)255;
    count += __popcll(__ballot(hit));
  }
  if (lane == 0) wave_hits[wave] = count;
  __syncthreads();
  int at = 0, len = 0;
#pragma unroll
  for (int w = 0; w < kEmbWaves; ++w) {
    if (w == wave) at = len;
    len += wave_hits[w];
  }
  if (count > 0) {
#pragma unroll 4
    for (int t0 = t_begin; t0 < t_end; t0 += 64) {
      const int r = row_of[t0 + lane];
      const unsigned long long hits = __ballot(r != 255);
      if (r != 255) list[at + __popcll(hits & ((1ull << lane) - 1ull))] = ((t0 + lane) << 6) | r;
      at += __popcll(hits);
    }
  }
  __syncthreads();
  const int64_t E = p.end - p.begin;
  // adding to g: rows that no token names stay as they are, their traffic is saved
  if (MODE == EMIT_ACCUM && len == 0) return;               // the same for every thread

  // NT tokens at a time into `into`: all their loads, then their additions in token order
  auto add_tokens = [&](float (&into)[kEmbIter][4], auto ntc, int ta, int tb, int tc, int td) {
    constexpr int NT = decltype(ntc)::value;
    const int tok[4] = {ta, tb, tc, td};
    float x[NT][kEmbIter][4];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const T* src = dY + (int64_t)tok[k] * p.lddy;
#pragma unroll
      for (int i = 0; i < kEmbIter; ++i) {
        const int64_t c = cbase + i * 256 + 4 * lane;
        if (c < p.in) load4_as_f32<T>(src + c, (int)(p.in - c < 4 ? p.in - c : 4), x[k][i]);
        else x[k][i][0] = x[k][i][1] = x[k][i][2] = x[k][i][3] = 0.f;
      }
    }
#pragma unroll
    for (int k = 0; k < NT; ++k)
#pragma unroll
      for (int i = 0; i < kEmbIter; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) into[i][e] += x[k][i][e];
  };
  // Sum of the hits of local row `r` that `mine(ordinal)` selects, ordinal = 0, 1, ... in token order.
  auto gather = [&](float (&into)[kEmbIter][4], int r, auto mine) {
    int q0 = 0, q1 = 0, q2 = 0, pending = 0, ordinal = 0;     // the last tokens found, oldest in q2
    for (int j0 = 0; j0 < len; j0 += 64) {
      const int e = j0 + lane < len ? list[j0 + lane] : -1;
      unsigned long long found = __ballot(e >= 0 && (e & 63) == r);
      for (; found != 0; found &= found - 1) {
        if (!mine(ordinal++)) continue;
        const int t = __builtin_amdgcn_readlane(e, __builtin_ctzll(found)) >> 6;
        if (pending == 3) {
          add_tokens(into, IntC<4>{}, q2, q1, q0, t);
          pending = 0;
        } else {
          q2 = q1; q1 = q0; q0 = t;
          ++pending;
        }
      }
    }
    if (pending == 3) { add_tokens(into, IntC<2>{}, q2, q1, 0, 0); add_tokens(into, IntC<1>{}, q0, 0, 0, 0); }
    else if (pending == 2) add_tokens(into, IntC<2>{}, q1, q0, 0, 0);
    else if (pending == 1) add_tokens(into, IntC<1>{}, q0, 0, 0, 0);
  };

  // which rows of the group have hits, and very many: a bit each, the same in every wave (a look at a row's count in
  // LDS where it is asked for was a latency per row and pass: 3 us a workgroup, as much as all its work on a narrow table)
  unsigned long long named = 0, hot = 0;
  if (len > 0) {                                            // the same for every thread
    for (int i = threadIdx.x; i < kEmbRows; i += 64 * kEmbWaves) hits_of[i] = 0;
    __syncthreads();
    for (int j = threadIdx.x; j < len; j += 64 * kEmbWaves) atomicAdd(&hits_of[list[j] & 63], 1);
    __syncthreads();
    const int hits = hits_of[lane];
    named = __ballot(hits > 0);
    hot = __ballot(hits >= kEmbHot);
  }

  // One row of the part: where its pieces go, their state requested; and the update from the sums in `acc`.
  struct Row {
    Vec4Sink d[kEmbIter];
    State4 st[kEmbIter];
    bool whole[kEmbIter];
  };
  auto request = [&](Row& w, int64_t row) {
#pragma unroll
    for (int i = 0; i < kEmbIter; ++i) {
      const int64_t c = cbase + i * 256 + 4 * lane;
      const int64_t flat = row * p.in + c;
      w.whole[i] = c + 4 <= p.in && flat >= p.begin && flat + 4 <= p.end;
      const int64_t k = flat - p.begin;
      w.d[i].g = s.g + k;
      w.d[i].master = s.master + k;
      w.d[i].m = s.m + k;
      w.d[i].v = s.v + k;
      w.d[i].W = s.w_kind == W_BF16 ? (void*)((unsigned short*)s.W + flat) : (void*)((float*)s.W + flat);
      if (w.whole[i]) w.st[i] = load_state4<MODE>(w.d[i]);
    }
  };
  auto finish = [&](Row& w, int64_t row, const float (&acc)[kEmbIter][4]) {
#pragma unroll
    for (int i = 0; i < kEmbIter; ++i) {
      const int64_t c = cbase + i * 256 + 4 * lane;
      if (c >= p.in) continue;
      const int64_t flat = row * p.in + c;
      if (w.whole[i]) {
        const f32x4_u val = {acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
        finish4<MODE>(w.d[i], s.w_kind, s.c, val, w.st[i]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (c + e < p.in && flat + e >= p.begin && flat + e < p.end)
            emit<MODE>(s, E, 0, flat + e - p.begin, flat + e, acc[i][e]);
      }
    }
  };

  // ---- rows with very many hits: summed by all waves together, updated by one of them
  constexpr unsigned long long kPartMask = kPartRows == 64 ? ~0ull : (1ull << kPartRows) - 1ull;
  for (unsigned long long left = hot & (kPartMask << (part_id * kPartRows)); left != 0; left &= left - 1) {
    const int local = __builtin_ctzll(left);
    float acc[kEmbIter][4];
#pragma unroll
    for (int i = 0; i < kEmbIter; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][e] = 0.f;
    gather(acc, local, [&](int ordinal) { return (ordinal & (kEmbWaves - 1)) == wave; });
#pragma unroll
    for (int i = 0; i < kEmbIter; ++i) *(float4*)&part[wave][i * 256 + 4 * lane] = float4{acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
    __syncthreads();
    if (wave == (local & (kEmbWaves - 1))) {
      Row w;
      request(w, row_base + local);
#pragma unroll
      for (int i = 0; i < kEmbIter; ++i) {
        float4 sum = *(const float4*)&part[0][i * 256 + 4 * lane];
#pragma unroll
        for (int k = 1; k < kEmbWaves; ++k) {
          const float4 x = *(const float4*)&part[k][i * 256 + 4 * lane];
          sum.x += x.x; sum.y += x.y; sum.z += x.z; sum.w += x.w;
        }
        acc[i][0] = sum.x; acc[i][1] = sum.y; acc[i][2] = sum.z; acc[i][3] = sum.w;
      }
      finish(w, row_base + local, acc);
    }
    __syncthreads();
  }

  for (int sub = 0; sub < kPartRows / kEmbWaves; ++sub) {
    const int local = part_id * kPartRows + sub * kEmbWaves + wave;     // consecutive rows go to different waves
    const int64_t row = row_base + local;
    if (row > row_last) break;
    const bool is_named = (named >> local & 1) != 0;
    if ((hot >> local & 1) != 0 || (MODE == EMIT_ACCUM && !is_named)) continue;
    float acc[kEmbIter][4];
#pragma unroll
    for (int i = 0; i < kEmbIter; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][e] = 0.f;
    Row w;
    request(w, row);                                        // travels while the hit list is walked
    if (is_named) gather(acc, local, [](int) { return true; });
    finish(w, row, acc);
  }
}

// ---------------------------------------------------------------------------
// element-wise pass: AdamW and/or the sum of slab partials (HBM-bound)
// ---------------------------------------------------------------------------
struct ElemParams {
  const float* src;     // g (S = 0) or the slab partials, slab sl at src + sl * pitch
  int32_t S;            // 0: src is g itself
  int64_t n;
  int64_t pitch;
  int64_t head;         // elements before the first 4-element group (at most 31)
  float* g_out;         // EMIT_STORE / EMIT_ACCUM
  float* master;
  float* m;
  float* v;
  void* W;              // already offset to element 0, or nullptr
  int32_t w_kind;
  AdamWConsts c;
};

template <int MODE>
__device__ __forceinline__ void elem_one(const ElemParams& q, int64_t i) {
  float val;
  if (q.S == 0) {
    val = q.src[i];
  } else {
    val = q.src[i];
    for (int32_t sl = 1; sl < q.S; ++sl) val += q.src[(int64_t)sl * q.pitch + i];
  }
  if constexpr (MODE == EMIT_STORE) {
    q.g_out[i] = val;
  } else if constexpr (MODE == EMIT_ACCUM) {
    q.g_out[i] += val;
  } else {
    float th = q.master[i], mm = q.m[i], vv = q.v[i];
    adamw_update(val, th, mm, vv, q.c);
    q.master[i] = th;
    q.m[i] = mm;
    q.v[i] = vv;
    if (q.w_kind == W_BF16) ((unsigned short*)q.W)[i] = f32_to_bf16_rne(th);
    else if (q.w_kind == W_F32) ((float*)q.W)[i] = th;
  }
}

template <int MODE, int U = 1>
__global__ __launch_bounds__(256) void elementwise_kernel(const ElemParams q) {
  const int64_t nvec = (q.n - q.head) >> 2;
  if (blockIdx.x == 0 && threadIdx.x < 36) {
    // the few elements before (at most 31) and after (at most 3) the 4-element groups
    const int64_t tail0 = q.head + (nvec << 2);
    const int64_t i = threadIdx.x < 32 ? (int64_t)threadIdx.x : tail0 + (threadIdx.x - 32);
    const bool ok = threadIdx.x < 32 ? (i < q.head) : (i < q.n);
    if (ok) elem_one<MODE>(q, i);
  }
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  // U 4-element groups per trip, all loads ahead of the arithmetic
  for (int64_t j0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j0 < nvec; j0 += U * stride) {
    Vec4Sink d[U];
    State4 st[U];
    f32x4_u val[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t j = j0 + u * stride;
      ok[u] = j < nvec;
      const int64_t i = q.head + (j << 2);
      d[u].g = q.g_out + i;
      d[u].master = q.master + i;
      d[u].m = q.m + i;
      d[u].v = q.v + i;
      d[u].W = q.w_kind == W_BF16 ? (void*)((unsigned short*)q.W + i) : (void*)((float*)q.W + i);
      if (ok[u]) {
        val[u] = __builtin_nontemporal_load((const f32x4_u*)(q.src + i));
        for (int32_t sl = 1; sl < q.S; ++sl)
          val[u] += __builtin_nontemporal_load((const f32x4_u*)(q.src + (int64_t)sl * q.pitch + i));
        st[u] = load_state4<MODE>(d[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (ok[u]) finish4<MODE>(d[u], q.w_kind, q.c, val[u], st[u]);
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
namespace {

// Start delay (units of 8128 cycles) of the second workgroup of each compute unit in the fused call, single or grouped, whose
// epilogue is long and HBM-bound; the plain gradient gains nothing.  In us at delays of 0 / 2 / 4 / 6.  With the state requested
// ahead, 2: 32 Mi elements, 1024 tokens 183.7 / 179.5 / 180.8 / 182.5; groups at 1024 tokens, two 1024 x 14336 183.3 / 179.7 /
// 182.5 / 183.8, a 1024-wide block 84.1 / 86.3 / 89.7 / 90.1, a 2048-wide one 327 / 325 / 329 / 330 (without the state ahead, at 6:
// 180.5, 91.9, 343).  A launch of less than a round would rather have none (12 Mi, 82.3 / 84.6 / 87.4 / 88.6, and the
// 1024-wide block).  Without, 6: 2048 tokens 225.6 / 221.4 / 219.0 / 218.5; 40 Mi of 14336-wide rows 325 / 320 / 313 / 309.  The
// 256-row tile, one workgroup per compute unit, starts together: every second unit late by 10 was no faster (64 Mi, 8192
// tokens 1018 us against 1016; 32 Mi, 6400 tokens 447 against 439).
template <class C> constexpr int kStaggerAdamW = C::WM == 2 ? 0 : C::AHEAD ? 2 : 6;
// 256 x 256 tiles, four slabs of 33 KB in LDS, one workgroup per compute unit: both waves of a SIMD are in
// the loop together, which the 16x16x32 MFMA needs (a wave then issues one MFMA per 32 cycles; alone
// on its SIMD it would have to issue one per 16 cycles beside its reads and loads, and cannot)
using MainCfg = RingCfg<2, 4, 16>;
// 128 x 256 tiles, three slabs of 25 KB, two workgroups per compute unit: while its partner is in its
// epilogue a workgroup's waves are alone on their SIMDs, so this one keeps the 32x32x16 MFMA (with the
// other shape its loops were 10 % slower).  The two shapes give the same bits: the hardware adds the
// tokens of either in the same order.
using FusedCfg = RingCfg<1, 3, 32>;         // (the fused call, and plain gradients with few tiles)
using FusedLongCfg = RingCfg<1, 3, 32, false>;   // the fused call over more tokens (update_requests_ahead)

template <class C, int MODE>
int launch_mfma_mode(const MfmaParams& q, int grid, hipStream_t st) {
  const int err = raise_lds_limit<&wgrad_mfma_kernel<C, MODE>>(C::LDS_BYTES);
  if (err != 0) return err;
  MfmaArgs args;
  args.q[0] = q;
#ifdef CHUNKFT_TIMELINE
  args.q[0].timeline = g_timeline_words >= (size_t)q.n_tile_items * 8 ? g_timeline : nullptr;
#endif
  hipLaunchKernelGGL((wgrad_mfma_kernel<C, MODE>), dim3(grid), dim3(C::NT), C::LDS_BYTES, st, args);
  return (int)hipGetLastError();
}

}  // namespace

static_assert(MainCfg::BM == kMainTileM && MainCfg::BN == kMainTileN && MainCfg::BK == kMainTileK,
              "the token split is chosen from these tile sizes");

// Compute units of the current device, asked once per device (a launch-shape input: how many
// workgroups fill the part).  Without a device -- the host-only size queries on a machine
// that has none -- the count of the MI355X this library is written for.
int device_compute_units() {
  static std::atomic<int> cached[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) { (void)hipGetLastError(); return kDefaultComputeUnits; }
  if (dev < kMaxDevices) {
    const int c = cached[dev].load(std::memory_order_relaxed);
    if (c > 0) return c;
  }
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
    (void)hipGetLastError();
    return kDefaultComputeUnits;
  }
  if (dev < kMaxDevices) cached[dev].store(cus, std::memory_order_relaxed);
  return cus;
}

// Whether the tiles that the XCDs start with, one run of tiles each, lie a power of two of at least 8 MiB (16 on the 256-row
// tile) apart in g, or nearly, on rows of a power of two of at least 16 KB: the XCDs then walk over the same address bits in step, and the
// sum into g, which requests its rows ahead, holds up a part of the channels.  Each XCD then begins an eighth of its run
// further on than the one before.  g of 4096-wide rows in us, in step / turned (one batch at a time, in step): 16 Mi elements 16 tokens
// 32.9 / 25.1 (28.7), 128 tokens 34.7 / 26.5 (32.6), 512 tokens 38.0 / 32.7 (41.7); 32 Mi 16 tokens 59.6 / 44.3 (52.4),
// 1024 tokens, 256-row tile, 101.7 / 85.1 (109.2); 8192-wide 32 Mi 128 tokens 61.7 / 50.2 (70.7).  Elsewhere turning only breaks up the groups of
// tile rows: 4096-wide 20 Mi 1024 tokens 58.8 / 61.0, 40 Mi 102.5 / 107.3, 14336-wide 8 Mi 512 tokens 25.4 / 28.6; and so it does over more than
// 2048 tokens, where the loop decides (32 Mi 4096 tokens, 4096-wide 225 / 213, 16384-wide 212 / 219; 128 Mi of 8192-wide rows 6000
// tokens 1240 / 1273).
bool runs_in_step(int64_t in, int64_t tokens, int64_t items) {
  const int64_t per_xcd = (items + 7) / 8;
  int64_t top = 1;
  while (top * 2 <= per_xcd) top *= 2;
  return tokens <= 2048 && in >= 4096 && (in & (in - 1)) == 0 && per_xcd >= 64 && per_xcd - top <= per_xcd / 32;
}

// Parameters of the MFMA kernel for a call.  False if the work items cannot be counted in 32 bits.
template <class C>
bool fill_mfma_params(const WgradProblem& p, int mode, const Sinks& s, const RowSplit& rs, MfmaParams& q) {
  const bool folded = edge_rows_folded(rs);
  q = MfmaParams{};
  q.p = p;
  q.s = s;
  q.rb0 = rs.rb0;
  q.rb1 = rs.rb1;
  q.lead_base = folded ? rs.lead_base : -1;
  q.trail_row = folded ? rs.trail_row : -1;
  const int64_t tiles_m = ceil_div(rs.rb1 - rs.rb0, C::BM), tiles_n = ceil_div(p.in, C::BN);
  if (tiles_m > 0x3fffffff || tiles_n > 0x3fffffff || tiles_m * tiles_n > 0x3fffffff / p.S) return false;
  q.tiles_m = (int32_t)tiles_m;
  q.tiles_n = (int32_t)tiles_n;
  q.n_tile_items = (int32_t)(tiles_m * tiles_n * p.S);
  // Order of the tiles inside an XCD's run of work items: groups of 8 tile rows (4 of the fused
  // call's smaller tiles), column tile by column tile, so that X tiles stay in that L2.  Measured
  // for the fused call on 4096 x 14336 at T = 4096: 571 us in groups of 4 against 736 us row-major;
  // on 14336 x 4096 at T = 1024: 313 against 335 us.
  q.group_m = mode == EMIT_ADAMW ? 4 : 8;
  q.stagger = mode == EMIT_ADAMW ? kStaggerAdamW<C> : 0;
  q.turned = mode == EMIT_ACCUM && runs_in_step(p.in, p.T, q.n_tile_items);
  return true;
}

template <class C>
int launch_update_cfg(const WgradProblem& p, const Sinks& s, hipStream_t st) {
  MfmaParams q;
  if (!fill_mfma_params<C>(p, EMIT_ADAMW, s, split_rows(p), q)) return (int)hipErrorInvalidValue;   // work items are counted in 32 bits
  return launch_mfma_mode<C, EMIT_ADAMW>(q, (q.n_tile_items + 7) / 8 * 8, st);
}

template <class C>
int launch_mfma_cfg(const WgradProblem& p, int mode, const Sinks& s, hipStream_t st) {
  if (mode == EMIT_ADAMW) return launch_update_cfg<C>(p, s, st);
  MfmaParams q;
  if (!fill_mfma_params<C>(p, mode, s, split_rows(p), q)) return (int)hipErrorInvalidValue;
  const int grid = (q.n_tile_items + 7) / 8 * 8;
  switch (mode) {
    case EMIT_STORE: return launch_mfma_mode<C, EMIT_STORE>(q, grid, st);
    case EMIT_ACCUM: return launch_mfma_mode<C, EMIT_ACCUM>(q, grid, st);
    default: return launch_mfma_mode<C, EMIT_PARTIAL>(q, grid, st);
  }
}

int launch_wgrad_bf16_mfma(const WgradProblem& p, int mode, const Sinks& s, void* stream) {
  if (mode == EMIT_ADAMW && (s.w_kind == W_F32 || p.S > 1)) return (int)hipErrorInvalidValue;   // bf16 weights; slabs are summed first
  if (takes_small_tiles(p.in, p.T, p.begin, p.end, device_compute_units()) &&
      (mode == EMIT_ADAMW || !plain_leaves_small_tiles(p, device_compute_units())))
    return launch_wgrad_small(p, mode, s, stream);
  // The plain gradient (short epilogue) is a little faster on the large tile; the fused call,
  // whose epilogue moves 26 bytes per element, gains from two workgroups per compute unit.
  if (mode == EMIT_ADAMW) {
    if (fused_takes_large_tile(p, device_compute_units())) return launch_mfma_cfg<MainCfg>(p, mode, s, (hipStream_t)stream);
    if (update_requests_ahead(p.in, p.T)) return launch_mfma_cfg<FusedCfg>(p, mode, s, (hipStream_t)stream);
    return launch_update_cfg<FusedLongCfg>(p, s, (hipStream_t)stream);
  }
  // The plain gradient takes whichever tile is faster for its number of tiles and tokens
  // (plain_takes_large_tile, csrc/shape.cpp); every element is summed over the tokens in the same
  // order either way.
  const RowSplit rs = split_rows(p);
  const int64_t big_tiles = ceil_div(rs.rb1 - rs.rb0, MainCfg::BM) * ceil_div(p.in, MainCfg::BN) * p.S;
  const int64_t slab_tokens = p.S > 1 ? p.kslab : p.T;
  if (!plain_takes_large_tile(big_tiles, slab_tokens, device_compute_units()))
    return launch_mfma_cfg<FusedCfg>(p, mode, s, (hipStream_t)stream);
  return launch_mfma_cfg<MainCfg>(p, mode, s, (hipStream_t)stream);
}

// ---- grouped fused call
template <class C>
static int launch_group_cfg(const GroupSegment* segs, int n, hipStream_t st) {
  const int lds_err = raise_lds_limit<&wgrad_group_kernel<C>>(C::LDS_BYTES);
  if (lds_err != 0) return lds_err;
  for (int first = 0; first < n; first += kGroupMax) {
    const int count = n - first < kGroupMax ? n - first : kGroupMax;
    GroupParams gp{};
    int64_t items = 0;
    for (int i = 0; i < count; ++i) {
      const GroupSegment& g = segs[first + i];
      MfmaParams& q = gp.seg[i];
      gp.item_start[i] = (int32_t)items;
      if (g.vector) {
        q = MfmaParams{};
        q.p = g.p;
        q.s = g.s;
        q.tiles_m = 0;
        items += ceil_div(g.p.end - g.p.begin, kColsumCols);
      } else {
        if (!fill_mfma_params<C>(g.p, EMIT_ADAMW, g.s, split_rows(g.p), q)) return (int)hipErrorInvalidValue;
        items += q.n_tile_items;
      }
      if (items > 0x3fffffff) return (int)hipErrorInvalidValue;
    }
    gp.stagger = kStaggerAdamW<C>;
    gp.item_start[count] = (int32_t)items;
    gp.n_segs = count;
    gp.n_items = (int32_t)items;
    const int grid = (gp.n_items + 7) / 8 * 8;
    hipLaunchKernelGGL((wgrad_group_kernel<C>), dim3(grid), dim3(C::NT), C::LDS_BYTES, st, gp);
    const int err = (int)hipGetLastError();
    if (err != 0) return err;
  }
  return 0;
}

int launch_fused_group(const GroupSegment* segs, int n, bool large_tile, void* stream) {
  if (n <= 0) return 0;
  for (int i = 0; i < n; ++i)
    if (!segs[i].vector && (segs[i].s.w_kind == W_F32 || segs[i].p.S > 1)) return (int)hipErrorInvalidValue;
  if (large_tile) return launch_group_cfg<MainCfg>(segs, n, (hipStream_t)stream);
  bool ahead = true;
  for (int i = 0; i < n; ++i) ahead = ahead && (segs[i].vector || group_requests_ahead(segs[i].p.T));
  return ahead ? launch_group_cfg<FusedCfg>(segs, n, (hipStream_t)stream)
               : launch_group_cfg<FusedLongCfg>(segs, n, (hipStream_t)stream);
}

template <typename T, int NORM, int CB>
static int launch_colsum_cb(const WgradProblem& p, int mode, const Sinks& s, const float* stats, hipStream_t st) {
  // vectors of more blocks than a launch can count (2^27 fp32 or 2^28 bf16 elements) go in pieces
  constexpr int64_t most = kMaxLaunchThreads / kColsumThreads<T, CB> / 8 * 8 * CB;
  if (p.end - p.begin > most)
    return in_pieces(p, s, most, [&](const WgradProblem& q, const Sinks& to) { return launch_colsum_cb<T, NORM, CB>(q, mode, to, stats, st); });
  const int64_t blocks = ceil_div(p.end - p.begin, CB);
  const dim3 grid((unsigned)((blocks + 7) / 8 * 8)), threads((kColsumThreads<T, CB>));
  const int n = (int)blocks;
  switch (mode) {
    case EMIT_STORE: hipLaunchKernelGGL((colsum_kernel<T, EMIT_STORE, NORM, CB>), grid, threads, 0, st, p, s, stats, n); break;
    case EMIT_ACCUM: hipLaunchKernelGGL((colsum_kernel<T, EMIT_ACCUM, NORM, CB>), grid, threads, 0, st, p, s, stats, n); break;
    default: hipLaunchKernelGGL((colsum_kernel<T, EMIT_ADAMW, NORM, CB>), grid, threads, 0, st, p, s, stats, n); break;
  }
  return (int)hipGetLastError();
}

// What a block takes of every token: a whole 128-byte line, half of one or a quarter, the widest that still leaves no
// compute unit with a second block.  A compute unit takes in about 27 bytes per clock in whole lines, so narrow vectors
// want more units (the parts of a line meet in one XCD's L2: its blocks are neighbours there) and wide ones whole
// lines.  Line / half / quarter, fused RMSNorm and LayerNorm calls in us: bf16 1024 wide, 16384 tokens 78 / 69 / 52;
// 4096 wide, 4096 tokens 28.8 / 26.4 / 24.1; 8192 wide, 16384 tokens 183 / 174 / 255; 16384 wide, 4096 tokens
// 67 / 73 / 87;  fp32 2048 wide, 4096 tokens 29.4 / 26.5 / 24.4; 4096 wide 48.4 / 45.5 / 50.2; 8192 wide 83 / 87 / 100.
template <typename T, int NORM>
static int launch_colsum_t(const WgradProblem& p, int mode, const Sinks& s, const float* stats, hipStream_t st) {
  constexpr int LINE = 128 / sizeof(T);
  const int64_t n = p.end - p.begin, cus = device_compute_units();
  if (ceil_div(n, LINE / 4) <= cus) return launch_colsum_cb<T, NORM, LINE / 4>(p, mode, s, stats, st);
  if (ceil_div(n, LINE / 2) <= cus) return launch_colsum_cb<T, NORM, LINE / 2>(p, mode, s, stats, st);
  return launch_colsum_cb<T, NORM, LINE>(p, mode, s, stats, st);
}

int launch_colsum(const WgradProblem& p, int dtype, int mode, const Sinks& s, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  return dtype == 0 ? launch_colsum_t<float, 0>(p, mode, s, nullptr, st)
                    : launch_colsum_t<unsigned short, 0>(p, mode, s, nullptr, st);
}

int launch_norm_wgrad(const WgradProblem& p, int dtype, bool subtract_mean, float eps, float* stats, int mode,
                      const Sinks& s, void* stream) {
  const int64_t sgrid = ceil_div(p.T, 4);
  if (sgrid > 0x7fffffff) return (int)hipErrorInvalidValue;
  hipStream_t st = (hipStream_t)stream;
  if (dtype == 0) {
    if (subtract_mean) hipLaunchKernelGGL((norm_stats_kernel<float, 1>), dim3((int)sgrid), dim3(256), 0, st, (const float*)p.X, p.ldx, p.in, p.T, eps, stats);
    else hipLaunchKernelGGL((norm_stats_kernel<float, 0>), dim3((int)sgrid), dim3(256), 0, st, (const float*)p.X, p.ldx, p.in, p.T, eps, stats);
  } else {
    if (subtract_mean) hipLaunchKernelGGL((norm_stats_kernel<unsigned short, 1>), dim3((int)sgrid), dim3(256), 0, st, (const unsigned short*)p.X, p.ldx, p.in, p.T, eps, stats);
    else hipLaunchKernelGGL((norm_stats_kernel<unsigned short, 0>), dim3((int)sgrid), dim3(256), 0, st, (const unsigned short*)p.X, p.ldx, p.in, p.T, eps, stats);
  }
  const int err = (int)hipGetLastError();
  if (err != 0) return err;
  return dtype == 0 ? launch_colsum_t<float, 1>(p, mode, s, stats, st)
                    : launch_colsum_t<unsigned short, 1>(p, mode, s, stats, st);
}

template <typename T, int MODE>
static int launch_embed_mode(const WgradProblem& p, int64_t groups, const Sinks& s, hipStream_t st) {
  const dim3 threads(64 * kEmbWaves);
  const int parts = embed_parts(MODE == EMIT_ADAMW, groups, p.out, p.in, p.T, device_compute_units());
  if (parts == 1) hipLaunchKernelGGL((embed_wgrad_kernel<T, MODE, 1>), dim3((unsigned)groups), threads, 0, st, p, s);
  else if (parts == 4) hipLaunchKernelGGL((embed_wgrad_kernel<T, MODE, 4>), dim3((unsigned)groups * 4), threads, 0, st, p, s);
  else return (int)hipErrorInvalidValue;
  return (int)hipGetLastError();
}

int launch_embed_wgrad(const WgradProblem& p, int dtype, int mode, const Sinks& s, void* stream) {
  const int64_t rows = (p.end - 1) / p.in - p.begin / p.in + 1;
  const int64_t gx = ceil_div(rows, kEmbRows), gy = ceil_div(p.in, 256 * kEmbIter);
  if (gy > 65535 || gx > 0x7fffffff / gy || p.T > kEmbTok) return (int)hipErrorInvalidValue;
  const hipStream_t st = (hipStream_t)stream;
  switch (mode) {
    case EMIT_STORE: return dtype == 0 ? launch_embed_mode<float, EMIT_STORE>(p, gx * gy, s, st) : launch_embed_mode<unsigned short, EMIT_STORE>(p, gx * gy, s, st);
    case EMIT_ACCUM: return dtype == 0 ? launch_embed_mode<float, EMIT_ACCUM>(p, gx * gy, s, st) : launch_embed_mode<unsigned short, EMIT_ACCUM>(p, gx * gy, s, st);
    default: return dtype == 0 ? launch_embed_mode<float, EMIT_ADAMW>(p, gx * gy, s, st) : launch_embed_mode<unsigned short, EMIT_ADAMW>(p, gx * gy, s, st);
  }
}

static int launch_elem(ElemParams& q, int mode, hipStream_t st) {
  // the first 4-element group starts where the fp32 arrays are 128-byte aligned (judged by the
  // master weights for the update, by the output gradient otherwise): the 1 KB a wave requests
  // per array is then eight whole lines; at a 16-byte phase inside a line it is nine, and the
  // pass 14 % slower (measured)
  const void* ref = mode == EMIT_ADAMW ? (const void*)q.master : (const void*)q.g_out;
  int64_t head = ((128 - (reinterpret_cast<uintptr_t>(ref) & 127u)) & 127u) / 4;
  if (head > q.n) head = q.n;
  q.head = head;
  const int64_t nvec = (q.n - head) >> 2;
  int64_t blocks = ceil_div(nvec, 256);
  // One block of 256 threads per CU, one group of four elements per thread in flight: the
  // seven streams of the update then reach 5.9 - 6.0 TB/s; with twice the blocks, or twice the
  // groups per trip, HBM efficiency drops to 5.3 - 5.4 TB/s (measured sweep: 16 Mi elements 87 us against 92).
  // Short passes wait for latency instead: AdamW on 1 / 2 / 4 Mi elements 7.2 / 12.1 / 23.7 us with one block per CU,
  // 6.4 / 10.8 / 22.8 with two, and the sum of slabs, whose slab loads add to the chain, takes four (fused call
  // with 3 slabs, 2 / 4 Mi elements at 4096 tokens: 47.4 / 79.3 us with one, 43.6 / 70.7 with two, 42.7 / 68.2 with four).
  const int64_t short_pass = int64_t(4) << 20;
  const int64_t cap = (int64_t)device_compute_units() * (q.n > short_pass ? 1 : q.S > 1 ? 4 : 2);
  if (blocks > cap) blocks = cap;
  if (blocks < 1) blocks = 1;
  switch (mode) {
    case EMIT_STORE: hipLaunchKernelGGL((elementwise_kernel<EMIT_STORE>), dim3((int)blocks), dim3(256), 0, st, q); break;
    case EMIT_ACCUM: hipLaunchKernelGGL((elementwise_kernel<EMIT_ACCUM>), dim3((int)blocks), dim3(256), 0, st, q); break;
    default: hipLaunchKernelGGL((elementwise_kernel<EMIT_ADAMW>), dim3((int)blocks), dim3(256), 0, st, q); break;
  }
  return (int)hipGetLastError();
}

int launch_reduce(const float* ws, int32_t S, int64_t E, int mode, const Sinks& s, void* W_at_begin,
                  void* stream) {
  ElemParams q{};
  q.src = ws;
  q.S = S;
  q.n = E;
  q.pitch = s.ws_pitch;
  q.g_out = s.g;
  q.master = s.master;
  q.m = s.m;
  q.v = s.v;
  q.W = W_at_begin;
  q.w_kind = W_at_begin ? s.w_kind : W_NONE;
  q.c = s.c;
  return launch_elem(q, mode, (hipStream_t)stream);
}

int launch_adamw(const float* g, int64_t n, const Sinks& s, void* W_at_begin, void* stream) {
  ElemParams q{};
  q.src = g;
  q.S = 0;
  q.n = n;
  q.master = s.master;
  q.m = s.m;
  q.v = s.v;
  q.W = W_at_begin;
  q.w_kind = W_at_begin ? s.w_kind : W_NONE;
  q.c = s.c;
  return launch_elem(q, EMIT_ADAMW, (hipStream_t)stream);
}

}  // namespace chunkft
