// Step 1 of the eviction path: the task-guided key score of Eq. 1 (Sec. 3.2).
//
// For every (sequence b, layer l, KV head h) segment the guide rows are the R*G_b
// (query head, guide token) pairs of the GQA group; the score of context token i is
//   raw_i   = (1/R) sum_rows exp(scale*<q_row, k_i> - lse_row)        (softmax over context)
//   s_key_i = (1/K) sum_{|t|<=K/2} raw_{i+t}                           (zero-padded pooling)
// The exact per-row normaliser lse_row needs every logit of the row, so the logits are
// produced twice (never stored): pass 1 keeps an online (max, sum) per row and chunk,
// a small kernel (or, in small calls, pass 2) merges the chunks into lse, and pass 2 recomputes
// the logits and sums the normalised weights per token.  Everything is kept in the log2 domain:
// x' = x * scale * log2(e), exp2(x' - lse2).
//
// The contraction over d runs on v_mfma_f32_32x32x16_bf16.  Pass 1 puts tokens on M and
// guide rows on N, so each lane owns one row and 16 tokens (row statistics reduce inside
// the lane); pass 2 swaps the operands, so each lane owns one token and 16 rows (the
// token's sum over rows reduces inside the lane).  The same register fragments serve both
// orientations because the A and B operand layouts of the instruction coincide.
//
// A workgroup (8 waves, one per CU) takes one chunk of 256 to 16384 tokens (plan_chunk) and one
// group of <= 256 guide rows.  The group's queries sit in LDS for the whole chunk.  Each wave
// streams its own 32-token K sub-tiles: an asynchronous global->LDS copy into the wave's private
// staging buffer runs while the wave computes from registers, so no barrier is needed inside
// the main loop and the K fragments take no prefetch registers.
//
// A wave holds two K tiles (a and b) and walks the group's row blocks in a circle, each query
// fragment it reads from LDS serving both tiles.  The tiles are half a revolution apart: the
// sub-tile that replaces a enters at row block 0, the one that replaces b at row block NP of
// 2 NP, and each leaves after a whole revolution.  So one staging buffer per wave serves both
// (two buffers would not fit beside the queries), a copy has half a revolution, 2 NP tile
// products, to land, and the query reads from LDS are half of what one tile at a time takes.
// They bound the passes next to the vector ALU and the power-limited clock.  tp_evict at 262144
// tokens, 48 layers of 16q/2kv heads, 256 guide tokens: 27.3 ms with one tile at a time, 26.6 with
// two, 25.5 with the copies' addresses out of the vector ALU as well (dma_whole).
// Inside a half the wave is software-pipelined: the MFMAs of one row block run while the vector
// ALU does the softmax work of the previous one.
#include <math.h>

#include <algorithm>

#include "tile_common.h"
#include "tp_internal.h"

namespace tp {
namespace {

constexpr double kCus = 256.0;      // score-pass workgroups in flight: one per CU
constexpr uint32_t kLongContext = 65536;
constexpr double kWgTokens = 350.0; // a workgroup's fixed work (5 us: query staging, merge) in tokens of a 256-row chunk

struct Work {
  int b, seg, l, h, rg, chunk;
  int64_t n0, nb, c0, c1, g0;
  int gb, rows, row0, nrows, nchunk;
};


// Workgroup -> (sequence, row group, chunk, segment).  Each sequence owns a contiguous range
// of workgroup ids (wg_off).  Within it the work units (segment, chunk) are numbered
// consecutively and dealt round-robin to the 8 XCDs, as consecutive workgroup ids are, so
// every XCD gets an even share whatever the number of chunks; the row groups of one unit get
// ids 8 apart, so they land on the same XCD and share the chunk's K through its L2.
__device__ inline bool decode(const GuideArgs& a, Work& w) {
  const int x = blockIdx.x;
  int b = 0;
  while (b + 1 < a.bt.batch && x >= a.wg_off[b + 1]) ++b;
  w.b = b;
  const int xb = x - a.wg_off[b];
  w.n0 = a.bt.ctx_off[b];
  w.nb = a.bt.ctx_off[b + 1] - w.n0;
  w.g0 = a.bt.g_off[b];
  w.gb = (int)(a.bt.g_off[b + 1] - w.g0);
  w.rows = a.R * w.gb;
  const int nrg = (w.rows + kRowsPerGroup - 1) / kRowsPerGroup;
  const int csize = seq_chunk(w.nb, a.chunk);
  const int nchunk = (int)(((uint32_t)w.nb + (uint32_t)csize - 1u) / (uint32_t)csize);
  w.nchunk = nchunk;
  const int xcd = xb & 7, slot = xb >> 3;
  w.rg = slot % nrg;
  const int64_t unit = (int64_t)(slot / nrg) * 8 + xcd;
  if (unit >= (int64_t)a.L * a.Hkv * nchunk) return false;  // padding to a multiple of 8
  w.seg = (int)(unit / nchunk);
  w.chunk = (int)(unit % nchunk);
  w.l = w.seg / a.Hkv;
  w.h = w.seg % a.Hkv;
  w.c0 = (int64_t)w.chunk * csize;
  w.c1 = w.c0 + csize < w.nb ? w.c0 + csize : w.nb;
  w.row0 = w.rg * kRowsPerGroup;
  w.nrows = w.rows - w.row0 < kRowsPerGroup ? w.rows - w.row0 : kRowsPerGroup;
  return true;
}

// Global row id (index into q_guide rows, stats and lse) of guide row rho of the segment.
__device__ inline int64_t grow_of(const GuideArgs& a, const Work& w, int rho) {
  const int r = rho / w.gb, j = rho - r * w.gb;
  const int64_t qh = (int64_t)w.h * a.R + r;
  return ((int64_t)w.l * a.Hq + qh) * a.g_tot + w.g0 + j;
}

// The row group's guide queries in LDS: local row rr at rr * kStride bytes.  The 16-byte pad
// per row makes 16 consecutive rows start on different bank groups, so the fragment reads
// below are conflict-free, and every fragment address is one per-lane base plus a constant.
// Rows past the group's end repeat its last row (finite data, discarded later).
// All of a thread's loads are issued before the first is written to LDS: one memory latency per
// workgroup instead of one per 32 rows.
template <int D, int NB>
__device__ inline void stage_q(const GuideArgs& a, const Work& w, char* qs) {
  using C = Cfg<D>;
  constexpr int kRows = kGuideThreads / C::kPieces;  // rows per sweep of the workgroup
  constexpr int kSweeps = (NB * 32 + kRows - 1) / kRows;
  const int rr0 = threadIdx.x / C::kPieces, p = threadIdx.x % C::kPieces;
  uint4 v[kSweeps];
#pragma unroll
  for (int i = 0; i < kSweeps; ++i) {
    const int rr = rr0 + i * kRows;
    const int src_row = rr < w.nrows ? rr : w.nrows - 1;
    v[i] = *(const uint4*)(a.q + grow_of(a, w, w.row0 + src_row) * D + p * 8);
  }
#pragma unroll
  for (int i = 0; i < kSweeps; ++i) {
    const int rr = rr0 + i * kRows;
    if (NB * 32 % kRows == 0 || rr < NB * 32) *(uint4*)(qs + rr * C::kStride + p * 16) = v[i];
  }
}

// k-steps [S0, S1) of the Q fragment of local row block rb: row 32 rb + lane%32, the d-columns of
// this half-wave.
template <int D, int S0, int S1>
__device__ inline void read_qfrag(const char* qs, int rb, Frag (&qf)[Cfg<D>::kSteps]) {
  using C = Cfg<D>;
  const int lane = threadIdx.x & 63;
  const char* base = qs + (lane & 31) * C::kStride + (lane >> 5) * C::kRowBytes / 2 + rb * 32 * C::kStride;
#pragma unroll
  for (int s = S0; s < S1; ++s) qf[s].u = *(const uint4*)(base + 16 * s);
}

// Issue the copy of the sub-tile starting at chunk token t0 into `kbuf`: each instruction
// moves 1 KB of consecutive K rows (coalesced); lane i fills slot i of that kilobyte, so it
// fetches the piece that the swizzle assigns to that slot.  Tokens past the chunk's `ntok`
// repeat its last token (finite data that pass 1 masks and pass 2 never stores).
template <int D>
__device__ inline void dma_subtile(const char* kchunk, int t0, int ntok, char* kbuf) {
  using C = Cfg<D>;
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int j = 0; j < 32 / C::kTokPerKB; ++j) {
    const int tl = j * C::kTokPerKB + lane / C::kPieces;
    const int p = (lane % C::kPieces) ^ swz<D>(tl);
    const int tok = min(t0 + tl, ntok - 1);
    const char* src = kchunk + (uint32_t)tok * C::kRowBytes + p * 16;
    __builtin_amdgcn_global_load_lds((const void*)src, (__attribute__((address_space(3))) void*)(kbuf + j * 1024), 16,
                                     0, 0);
  }
}

// The same for a sub-tile whose 32 tokens all exist: copy j reads from a wave-uniform base and the
// lane's fixed offset, whose swizzle differs between copies only in piece bit 2, 3 or both
// (j * kTokPerKB enters swz there), so a whole sub-tile takes a few vector instructions instead
// of about ninety.  Inline assembly for the scalar-base form; completion is tracked by
// wait_copies.  One wait state separates the M0 write from the copy that reads it; the base comes from
// scalar instructions, whose results a copy may use at once (a vector instruction's would need
// five wait states here, which the compiler does not add before inline assembly).
template <int D>
__device__ inline void dma_whole(const char* kchunk, int t0, uint32_t kbuf_lds) {
  using C = Cfg<D>;
  const int lane = threadIdx.x & 63;
  const int tl0 = lane / C::kPieces;
  const uint32_t off0 = (uint32_t)(tl0 * C::kRowBytes + ((lane % C::kPieces) ^ swz<D>(tl0)) * 16);
  const char* base = kchunk + (int64_t)t0 * C::kRowBytes;
#pragma unroll
  for (int j = 0; j < 32 / C::kTokPerKB; ++j) {
    const uint32_t flip = (uint32_t)swz<D>(j * C::kTokPerKB) * 16;
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off0 ^ flip),
                 "s"(base + j * 1024), "s"(kbuf_lds + (uint32_t)j * 1024u)
                 : "memory", "m0");
  }
}

// Issue-priority balancing of the two waves that share a SIMD (waves w and w ^ 4).  With equal
// priority the older wave wins most issue slots, finishes its sub-tiles early and leaves
// the other to run alone at the end of the workgroup.  After each sub-tile a wave publishes
// its count and raises its priority while it is behind its partner.  This changes only the
// timing, never which wave computes what.
__device__ inline void balance_issue(int* progress, int wave, int done) {
  if ((threadIdx.x & 63) == 0) progress[wave] = done;
  const int other = uniform(progress[wave ^ 4]);
  if (done < other)
    __builtin_amdgcn_s_setprio(2);
  else if (done == other)
    __builtin_amdgcn_s_setprio(1);
  else
    __builtin_amdgcn_s_setprio(0);
}

// The staging buffer has landed (the wave's copies are complete).  The memory clobber keeps
// the compiler from moving LDS reads of the buffer above the wait.
__device__ inline void wait_copies() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// The fragment reads of the buffer are complete, so it may be overwritten.  The builtin tells the
// compiler so, which then adds no wait of its own at the fragments' first uses (there it would
// also wait for the query reads issued since).
__device__ inline void wait_lds_reads() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// Which of the wave's two K tiles a step computes: both, or one (the wave's first and last half
// revolutions).
constexpr int kBothTiles = 0, kOnlyA = 1, kOnlyB = 2;

// One row block against the wave's K tiles a and b: two independent MFMA chains that share the
// query fragment.  The chains start from `init`; a tile left out gives -inf (an empty slot).
template <int KS, bool Q_IS_A, int TILES>
__device__ inline void mfma_tiles(const Frag (&q)[KS], const Frag (&ka)[KS], const Frag (&kb)[KS], const f32x16& init,
                                  f32x16& c0, f32x16& c1) {
  c0 = init;
  c1 = init;
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    if (TILES != kOnlyB)
      c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Q_IS_A ? q[s].v : ka[s].v, Q_IS_A ? ka[s].v : q[s].v, c0, 0, 0, 0);
    if (TILES != kOnlyA)
      c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Q_IS_A ? q[s].v : kb[s].v, Q_IS_A ? kb[s].v : q[s].v, c1, 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if (TILES == kOnlyB) c0[i] = -INFINITY;
    if (TILES == kOnlyA) c1[i] = -INFINITY;
  }
}

// The last kLateQ k-steps of a row block's query fragment are read after the first MFMAs of its own
// step, the others during the step before, each once its predecessor has been consumed: the
// first MFMA of a step waits for every LDS read issued before it, so none may be issued late.
constexpr int kLateQ = 2;

// Instruction order of one pipeline step: each MFMA followed by an even share of the vector work of
// the previous step (NV plain, NT transcendental, counted separately because the scheduler
// classes them separately) and by LDS reads: the late query reads, the next step's query
// fragment as this one's is consumed and, with Z, its four start values (pass 2).  The matrix
// core, the vector ALU and the LDS stay busy together, and the LDS latency is covered.
template <int KS, int NMFMA, int NV, int NT, bool Z>
__device__ inline void step_schedule() {
  constexpr int kPer = NMFMA / KS;  // MFMAs per query fragment
#pragma unroll
  for (int i = 0; i < NMFMA; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, NV, 0);
    __builtin_amdgcn_sched_group_barrier(0x400, NT, 0);
    if (i < kLateQ) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    const bool refill = (i + 1) % kPer == 0 && (i + 1) / kPer < KS - kLateQ;
    if (refill || i == kPer * (KS - kLateQ)) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    if (Z && i % kPer == 0 && i >= kPer && i <= 4 * kPer) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
}

// Keeps the vector work of a pipeline step inside the step: without a use here the
// compiler sinks it past the loop's branches, away from the MFMAs it should overlap.
__device__ inline void pin(float a, float b, float c, float d) { asm volatile("" ::"v"(a), "v"(b), "v"(c), "v"(d)); }

// ---------------------------------------------------------------------------- pass 1
// Online (max, sum) of one unit (32 tokens x 32 rows): acc[i] is the logit of token
// (i/4)*8 + (lane/32)*4 + i%4 and row lane%32.  c > 0, so max(x) * c = max(x * c).
__device__ inline void stats_update(const f32x16& acc, float c, float& m, float& s) {
  const float mn = fmaxf(m, max16(acc) * c);
  float e[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) e[j] = __builtin_amdgcn_exp2f(fmaf(acc[j], c, -mn));
#pragma unroll
  for (int i = 4; i < 16; i += 4)
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] += __builtin_amdgcn_exp2f(fmaf(acc[i + j], c, -mn));
  s = fmaf(s, __builtin_amdgcn_exp2f(m - mn), (e[0] + e[1]) + (e[2] + e[3]));
  m = mn;
}

// The unit's terms exp2(x*c - m) against the lane's current maximum m, summed.
__device__ inline float unit_sum(const f32x16& acc, float c, float m) {
  float e[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) e[j] = __builtin_amdgcn_exp2f(fmaf(acc[j], c, -m));
#pragma unroll
  for (int i = 4; i < 16; i += 4)
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] += __builtin_amdgcn_exp2f(fmaf(acc[i + j], c, -m));
  return (e[0] + e[1]) + (e[2] + e[3]);
}

// Lazily updated maximum: the pair's terms are summed against the lanes' current maxima
// and accepted while a unit's sum stays below 2^64, i.e. while no logit exceeds m by more
// than about 60 (log2 domain); s then holds sum exp2(x*c - m) for an m that is a logit
// already seen, which is all the normaliser needs.  A larger sum (the first unit of a row,
// whose m is still the empty value kNoMax, or a new extreme) is discarded and the unit is
// redone by the exact online update, which raises m.  This drops the per-logit max and the
// rescaling from the common case.
constexpr float kLazyLimit = 18446744073709551616.0f;  // 2^64

// Half a revolution of pass 1 (see the head of the file): row blocks H NP .. H NP + NP - 1
// against the wave's two K tiles.  Step p issues the MFMAs of its row block (query fragment q,
// fetched during the previous step) while the vector ALU turns the pending results (the row block
// before, both tiles) into row statistics and the LDS delivers the next block's query fragment.
template <int D, int NP, int H, int TILES>
__device__ inline void stats_half(const char* qs, const Frag (&ka)[Cfg<D>::kSteps], const Frag (&kb)[Cfg<D>::kSteps],
                                  Frag (&q)[Cfg<D>::kSteps], f32x16& p0, f32x16& p1, float (&sm)[2 * NP],
                                  float (&ss)[2 * NP], float c) {
  constexpr int KS = Cfg<D>::kSteps;
  constexpr int NM = TILES == kBothTiles ? 2 * KS : KS;  // MFMAs per step
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    f32x16 n0, n1;
    read_qfrag<D, KS - kLateQ, KS>(qs, H * NP + p, q);
    mfma_tiles<KS, false, TILES>(q, ka, kb, (f32x16){}, n0, n1);
    read_qfrag<D, 0, KS - kLateQ>(qs, (H * NP + p + 1) % (2 * NP), q);
    const int rb = (H * NP + p + 2 * NP - 1) % (2 * NP);
    const float t = unit_sum(p0, c, sm[rb]) + unit_sum(p1, c, sm[rb]);
    const bool big = !(t < kLazyLimit);
    ss[rb] += big ? 0.f : t;
    pin(ss[rb], t, t, t);
    // 2 x (16 fma + 15 add) + compare, select and adds; 32 exp2
    step_schedule<KS, NM, (66 + NM - 1) / NM, 32 / NM, false>();
    if (__builtin_amdgcn_ballot_w64(big)) {  // rare: exact update of those units
      if (big) {
        stats_update(p0, c, sm[rb], ss[rb]);
        stats_update(p1, c, sm[rb], ss[rb]);
      }
    }
    p0 = n0;
    p1 = n1;
  }
}

// The ragged last sub-tile of a chunk: tokens at or past `nvalid` get logit -inf.
template <int D, int NP>
__device__ inline void stats_tail(const char* qs, const Frag (&kf)[Cfg<D>::kSteps], int nvalid, float (&sm)[2 * NP],
                                  float (&ss)[2 * NP], float c) {
  using C = Cfg<D>;
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int rb = 0; rb < 2 * NP; ++rb) {
    Frag q[C::kSteps];
    read_qfrag<D, 0, C::kSteps>(qs, rb, q);
    f32x16 x, none;
    mfma_tiles<C::kSteps, false, kOnlyA>(q, kf, kf, (f32x16){}, x, none);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int tok = (i >> 2) * 8 + (lane >> 5) * 4 + (i & 3);
      x[i] = tok < nvalid ? x[i] : -INFINITY;
    }
    stats_update(x, c, sm[rb], ss[rb]);
  }
}

template <int D, int NP>
__global__ __launch_bounds__(kGuideThreads, 1) void k_guide_stats(GuideArgs a) {
  Work w;
  if (!decode(a, w)) return;
  using C = Cfg<D>;
  constexpr int NB = 2 * NP;  // 32-row blocks staged (rows past the group repeat its last row)
  __shared__ __attribute__((aligned(1024))) char qs[NB * 32 * C::kStride];
  __shared__ __attribute__((aligned(1024))) char kst[kGuideWaves * C::kStageBytes];
  const int lane = threadIdx.x & 63;
  const int wave = uniform(threadIdx.x >> 6);
  char* kbuf = kst + wave * C::kStageBytes;
  const uint32_t kbuf_lds = (uint32_t)uniform((int)(uintptr_t)(__attribute__((address_space(3))) char*)kbuf);
  const char* kchunk = (const char*)(a.k + ((int64_t)w.seg * a.n_tot + w.n0 + w.c0) * D);
  const int ntok = (int)(w.c1 - w.c0);
  const int nfull = ntok / 32;
  int st = wave;
  if (st < nfull) dma_subtile<D>(kchunk, 32 * st, ntok, kbuf);
  stage_q<D, NB>(a, w, qs);
  __syncthreads();

  float sm[NB], ss[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    sm[i] = kNoMax;
    ss[i] = 0.f;
  }
  // full sub-tiles st = wave, wave + 8, ..., into tiles a and b in turn
  Frag ka[C::kSteps], kb[C::kSteps], q[C::kSteps];
  f32x16 p0, p1;
#pragma unroll
  for (int i = 0; i < 16; ++i) p0[i] = p1[i] = -INFINITY;  // empty pipeline slot
  read_qfrag<D, 0, C::kSteps - kLateQ>(qs, 0, q);
  __shared__ int progress[kGuideWaves];
  if (threadIdx.x < kGuideWaves) progress[threadIdx.x] = 0;
  __syncthreads();
  int done = 0;
  const auto next_tile = [&](Frag(&kf)[C::kSteps]) {
    wait_copies();
    read_kfrag<D>(kbuf, kf);
    wait_lds_reads();
    st += kGuideWaves;
    if (st < nfull) dma_whole<D>(kchunk, 32 * st, kbuf_lds);
    __builtin_amdgcn_sched_barrier(0);  // the step's LDS slots are for the query fragments
  };
  if (st < nfull) {
    next_tile(ka);
    stats_half<D, NP, 0, kOnlyA>(qs, ka, kb, q, p0, p1, sm, ss, a.c);
    balance_issue(progress, wave, ++done);
    while (st + kGuideWaves < nfull) {  // two more tiles
      next_tile(kb);
      stats_half<D, NP, 1, kBothTiles>(qs, ka, kb, q, p0, p1, sm, ss, a.c);
      balance_issue(progress, wave, ++done);
      next_tile(ka);
      stats_half<D, NP, 0, kBothTiles>(qs, ka, kb, q, p0, p1, sm, ss, a.c);
      balance_issue(progress, wave, ++done);
    }
    if (st < nfull) {
      next_tile(kb);
      stats_half<D, NP, 1, kBothTiles>(qs, ka, kb, q, p0, p1, sm, ss, a.c);
      balance_issue(progress, wave, ++done);
      stats_half<D, NP, 0, kOnlyB>(qs, ka, kb, q, p0, p1, sm, ss, a.c);
      stats_update(p1, a.c, sm[NP - 1], ss[NP - 1]);
    } else {
      asm volatile("" : "+v"(sm[NP - 1]));  // keeps the branches' common first terms out of registers before them
      stats_half<D, NP, 1, kOnlyA>(qs, ka, kb, q, p0, p1, sm, ss, a.c);
      stats_update(p0, a.c, sm[NB - 1], ss[NB - 1]);
    }
  }
  __builtin_amdgcn_s_setprio(0);
  if (ntok > 32 * nfull && wave == nfull % kGuideWaves) {
    dma_subtile<D>(kchunk, 32 * nfull, ntok, kbuf);
    wait_copies();
    read_kfrag<D>(kbuf, ka);
    stats_tail<D, NP>(qs, ka, ntok - 32 * nfull, sm, ss, a.c);
  }

  // merge the half-waves (same rows, other tokens), then the waves, through LDS (the query
  // buffer is free now)
  __syncthreads();
  float2* xch = (float2*)qs;  // [wave][NB * 32]
  static_assert(kGuideWaves * NB * 32 * sizeof(float2) <= sizeof(qs), "exchange buffer");
#pragma unroll
  for (int rb = 0; rb < NB; ++rb) {
    merge_stats(sm[rb], ss[rb], __shfl_xor(sm[rb], 32), __shfl_xor(ss[rb], 32));
    if (lane < 32) xch[wave * NB * 32 + rb * 32 + lane] = make_float2(sm[rb], ss[rb]);
  }
  __syncthreads();
  const int64_t growtot = (int64_t)a.L * a.Hq * a.g_tot;
  for (int t = threadIdx.x; t < w.nrows; t += kGuideThreads) {
    float mm = xch[t].x, s2 = xch[t].y;
#pragma unroll
    for (int q = 1; q < kGuideWaves; ++q) merge_stats(mm, s2, xch[q * NB * 32 + t].x, xch[q * NB * 32 + t].y);
    a.stats[(int64_t)w.chunk * growtot + grow_of(a, w, w.row0 + t)] = make_float2(mm, s2);
  }
}

// ---------------------------------------------------------------------------- guide keys
// With the guide's own keys (the paper-literal slice of the causal attention over context +
// appended guide, Sec. 3.2), guide row j's normaliser also takes the logits of guide keys
// 0..j.  One workgroup takes up to kKeyRows guide rows of a (sequence, layer, KV head); the
// guide keys of that head are staged in LDS kGuideKeyTile at a time, and kKeyLanes adjacent
// lanes per row (its query in the registers of each) take every kKeyLanes-th key, so a wave reads
// kKeyLanes key rows at once (broadcasts from different banks: rows are padded by 16 bytes).
// The row's (max, sum) over its keys t <= j goes to the extra statistics slot nchunk_max,
// which the merge below treats as one more chunk.  Bound by a lane's serial chain over its
// keys: with one lane per row the separate calls on 24 segments of 7 to 33 guide tokens took
// 68.6 us, with four 62.7.
constexpr int kGuideKeyTile = 64;
constexpr int kKeyLanes = 4;
constexpr int kKeyRows = 256 / kKeyLanes;

template <int D>
__global__ __launch_bounds__(256) void k_guide_key_stats(GuideArgs a) {
  const int b = blockIdx.z, seg = blockIdx.y;
  const int64_t g0 = a.bt.g_off[b];
  const int gb = (int)(a.bt.g_off[b + 1] - g0);
  const int rows = a.R * gb;
  const int rho = blockIdx.x * kKeyRows + threadIdx.x / kKeyLanes;  // guide row of the segment: (r, j)
  const int part = threadIdx.x % kKeyLanes;
  if ((int)blockIdx.x * kKeyRows >= rows) return;  // the whole block has no rows
  const int64_t l = seg / a.Hkv, h = seg % a.Hkv;
  const bool live = rho < rows;
  const int r = live ? rho / gb : 0, j = live ? rho % gb : -1;
  const int64_t grow = ((l * a.Hq + h * a.R + r) * a.g_tot) + g0 + (live ? j : 0);
  __shared__ uint4 keys[kGuideKeyTile][D / 8 + 1];
  uint4 qv[D / 8];  // the row's query, bf16 pairs
  {
    const uint4* qrow = (const uint4*)(a.q + grow * D);
#pragma unroll
    for (int p = 0; p < D / 8; ++p) qv[p] = qrow[p];
  }
  // the block's rows need keys 0 .. max j; its last row has the largest j unless it wraps
  const int last = min(rows, (int)(blockIdx.x + 1) * kKeyRows) - 1;
  const int nkeys = ((int)blockIdx.x * kKeyRows) / gb == last / gb ? last % gb + 1 : gb;
  const uint4* kg = (const uint4*)(a.kg + ((l * a.Hkv + h) * a.g_tot + g0) * D);
  float m = kNoMax, s = 0.f;
  for (int t0 = 0; t0 < nkeys; t0 += kGuideKeyTile) {
    const int nt = min(kGuideKeyTile, nkeys - t0);
    __syncthreads();
    for (int i = threadIdx.x; i < nt * (D / 8); i += 256) keys[i / (D / 8)][i % (D / 8)] = kg[(int64_t)(t0 + i / (D / 8)) * (D / 8) + i % (D / 8)];
    __syncthreads();
    const int tend = min(nt, j - t0 + 1);  // keys t0 .. j of this tile (none for idle lanes)
    for (int t = part; t < tend; t += kKeyLanes) {
      // fp32 dot product of bf16 pairs (v_dot2_f32_bf16), four independent partial sums
      float dot[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int p = 0; p < D / 8; ++p) {
        const uint4 u = keys[t][p];
        const uint32_t kw[4] = {u.x, u.y, u.z, u.w};
        const uint32_t qw[4] = {qv[p].x, qv[p].y, qv[p].z, qv[p].w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          dot[e] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, qw[e]),
                                                   __builtin_bit_cast(bf16x2, kw[e]), dot[e], false);
      }
      merge_stats(m, s, ((dot[0] + dot[1]) + (dot[2] + dot[3])) * a.c, 1.0f);
    }
  }
#pragma unroll
  for (int o = 1; o < kKeyLanes; o <<= 1) merge_stats(m, s, __shfl_xor(m, o), __shfl_xor(s, o));
  if (live && part == 0) a.stats[(int64_t)a.nchunk_max * ((int64_t)a.L * a.Hq * a.g_tot) + grow] = make_float2(m, s);
}

// ---------------------------------------------------------------------------- lse merge
// One thread per guide row: merge the row's per-chunk (max, sum) pairs (and, with guide
// keys, the guide-key slot) into lse2.
template <int D>
__global__ __launch_bounds__(256) void k_guide_lse(GuideArgs a) {
  const int b = blockIdx.y;
  const int64_t g0 = a.bt.g_off[b];
  const int gb = (int)(a.bt.g_off[b + 1] - g0);
  const int64_t nb = a.bt.ctx_off[b + 1] - a.bt.ctx_off[b];
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)a.L * a.Hq * gb) return;
  const int64_t per_layer = (int64_t)a.Hq * gb;
  const int64_t l = idx / per_layer, rem = idx - l * per_layer;
  const int64_t qh = rem / gb, j = rem - qh * gb;
  const int64_t grow = (l * a.Hq + qh) * a.g_tot + g0 + j;
  const int64_t growtot = (int64_t)a.L * a.Hq * a.g_tot;
  const int nch = chunks_of(nb, a.chunk);
  float m = kNoMax, s = 0.f;
  for (int c = 0; c < nch; ++c) {
    const float2 v = a.stats[(int64_t)c * growtot + grow];
    merge_stats(m, s, v.x, v.y);
  }
  if (a.kg != nullptr) {
    const float2 v = a.stats[(int64_t)a.nchunk_max * growtot + grow];
    merge_stats(m, s, v.x, v.y);
  }
  a.lse2[grow] = m + log2f(s);
}

// ---------------------------------------------------------------------------- pass 2
// The MFMA chains of pass 2 start from -lse2/c instead of zero, so a unit's accumulator
// holds x - lse2/c and the normalised weight is exp2(acc * c).  acc[i] belongs to row
// (i/4)*8 + (lane/32)*4 + i%4 and token lane%32; the lane sums its 16 rows.
__device__ inline float attn_sum(const f32x16& acc, float c) {
  float e[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) e[j] = __builtin_amdgcn_exp2f(acc[j] * c);
#pragma unroll
  for (int i = 4; i < 16; i += 4)
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] += __builtin_amdgcn_exp2f(acc[i + j] * c);
  return (e[0] + e[1]) + (e[2] + e[3]);
}

// Accumulator start values of row block rb: -lse2/c of the lane's 16 rows.
__device__ inline void read_lz(const float* lz_s, int rb, f32x16& acc) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const float4 v = *(const float4*)(lz_s + rb * 32 + g * 8 + (lane >> 5) * 4);
    acc[4 * g + 0] = v.x;
    acc[4 * g + 1] = v.y;
    acc[4 * g + 2] = v.z;
    acc[4 * g + 3] = v.w;
  }
}

// The row group's accumulator start values -lse2/c in LDS, from whichever form the row
// normalisers are in: the caller's natural logs, the merged lse2, or (fold_lse) the chunks'
// statistics, which P adjacent lanes per row merge here.  Every workgroup of a row merges in
// the same order, so all use the same value.
template <int NB>
__device__ inline void stage_lz(const GuideArgs& a, const Work& w, float* lz_s) {
  if (a.fold_lse) {
    constexpr int P = NB * 32 <= 64 ? 8 : (NB * 32 <= 128 ? 4 : 2);
    static_assert(NB * 32 * P <= kGuideThreads, "a row's lanes fit one sweep of the workgroup");
    const int t = threadIdx.x / P, part = threadIdx.x % P;
    const int64_t growtot = (int64_t)a.L * a.Hq * a.g_tot;
    const bool live = t < w.nrows;
    const float2* st = a.stats + (live ? grow_of(a, w, w.row0 + t) : 0);
    float m = kNoMax, s = 0.f;
    if (live) {
#pragma unroll 4
      for (int c = part; c < w.nchunk; c += P) {
        const float2 v = st[(int64_t)c * growtot];
        merge_stats(m, s, v.x, v.y);
      }
      if (part == 0 && a.kg != nullptr) {
        const float2 v = st[(int64_t)a.nchunk_max * growtot];
        merge_stats(m, s, v.x, v.y);
      }
    }
#pragma unroll
    for (int o = 1; o < P; o <<= 1) merge_stats(m, s, __shfl_xor(m, o), __shfl_xor(s, o));
    if (part == 0 && t < NB * 32) lz_s[t] = live ? -(m + log2f(s)) / a.c : -INFINITY;
    return;
  }
  for (int t = threadIdx.x; t < NB * 32; t += kGuideThreads) {  // padding rows: exp2(-inf) = 0
    float z = -INFINITY;
    if (t < w.nrows) {
      const int64_t grow = grow_of(a, w, w.row0 + t);
      const float lse2 = a.lse_in ? (float)((double)a.lse_in[grow] * 1.4426950408889634) : a.lse2[grow];
      z = -lse2 / a.c;
    }
    lz_s[t] = z;
  }
}

// The sum over rows is finished for a sub-tile once its last pair has been summed: add the
// other half-wave's rows and store the token's value.
__device__ inline void attn_flush(float part, float* raw_out, int tok0, int ntok) {
  const int lane = threadIdx.x & 63;
  const float v = part + __shfl_xor(part, 32);
  const int tok = tok0 + lane;
  if (tok0 >= 0 && lane < 32 && tok < ntok) raw_out[tok] = v;
}

// Half a revolution of pass 2, pipelined like pass 1.  `parta` and `partb` carry the partial row
// sums of tiles a and b.  The tile that entered with this half (a for H = 0, b for H = 1) has
// replaced one whose last row block is summed in the half's first step, which then stores that
// tile's tokens (from chunk token `prev` on).  z holds the start values of the next row block.
template <int D, int NP, int H, int TILES>
__device__ inline void attn_half(const char* qs, const float* lz_s, const Frag (&ka)[Cfg<D>::kSteps],
                                 const Frag (&kb)[Cfg<D>::kSteps], Frag (&q)[Cfg<D>::kSteps], f32x16& z, f32x16& p0,
                                 f32x16& p1, float& parta, float& partb, int prev, float* raw_out, int ntok, float c) {
  constexpr int KS = Cfg<D>::kSteps;
  constexpr int NM = TILES == kBothTiles ? 2 * KS : KS;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    f32x16 n0, n1;
    read_qfrag<D, KS - kLateQ, KS>(qs, H * NP + p, q);
    mfma_tiles<KS, true, TILES>(q, ka, kb, z, n0, n1);
    const int rn = (H * NP + p + 1) % (2 * NP);
    read_qfrag<D, 0, KS - kLateQ>(qs, rn, q);
    read_lz(lz_s, rn, z);
    parta += attn_sum(p0, c);
    partb += attn_sum(p1, c);
    pin(parta, partb, parta, partb);
    // 2 x (16 multiplies + 15 adds) + 2 adds; 32 exp2
    step_schedule<KS, NM, 64 / NM, 32 / NM, true>();
    if (p == 0) {
      float& part = H == 0 ? parta : partb;
      attn_flush(part, raw_out, prev, ntok);
      part = 0.f;
    }
    p0 = n0;
    p1 = n1;
  }
}

template <int D, int NP>
__global__ __launch_bounds__(kGuideThreads, 1) void k_guide_attn(GuideArgs a) {
  Work w;
  if (!decode(a, w)) return;
  using C = Cfg<D>;
  constexpr int NB = 2 * NP;
  __shared__ __attribute__((aligned(1024))) char qs[NB * 32 * C::kStride];
  __shared__ __attribute__((aligned(1024))) char kst[kGuideWaves * C::kStageBytes];
  __shared__ __attribute__((aligned(16))) float lz_s[NB * 32];
  const int wave = uniform(threadIdx.x >> 6);
  char* kbuf = kst + wave * C::kStageBytes;
  const uint32_t kbuf_lds = (uint32_t)uniform((int)(uintptr_t)(__attribute__((address_space(3))) char*)kbuf);
  const int64_t tok0 = (int64_t)w.seg * a.n_tot + w.n0 + w.c0;  // first token row of the chunk
  const char* kchunk = (const char*)(a.k + tok0 * D);
  const int ntok = (int)(w.c1 - w.c0);
  // every sub-tile, the ragged last one included: its repeated tokens are never stored
  const int nsub = (ntok + 31) / 32;
  int st = wave;
  if (st < nsub) dma_subtile<D>(kchunk, 32 * st, ntok, kbuf);
  stage_q<D, NB>(a, w, qs);
  stage_lz<NB>(a, w, lz_s);
  __syncthreads();

  float* raw_out = a.raw + ((int64_t)w.rg * a.L * a.Hkv + w.seg) * a.n_tot + w.n0 + w.c0;
  Frag ka[C::kSteps], kb[C::kSteps], q[C::kSteps];
  f32x16 p0, p1, z;
#pragma unroll
  for (int i = 0; i < 16; ++i) p0[i] = p1[i] = -INFINITY;  // empty pipeline slot: sums to 0
  float parta = 0.f, partb = 0.f;
  int preva = -1, prevb = -1;  // first chunk token of the tile held in a and b (none yet)
  read_qfrag<D, 0, C::kSteps - kLateQ>(qs, 0, q);
  read_lz(lz_s, 0, z);
  __shared__ int progress[kGuideWaves];
  if (threadIdx.x < kGuideWaves) progress[threadIdx.x] = 0;
  __syncthreads();
  int done = 0;
  const auto next_tile = [&](Frag(&kf)[C::kSteps]) {
    wait_copies();
    read_kfrag<D>(kbuf, kf);
    wait_lds_reads();
    st += kGuideWaves;
    if (32 * (st + 1) <= ntok)
      dma_whole<D>(kchunk, 32 * st, kbuf_lds);
    else if (st < nsub)
      dma_subtile<D>(kchunk, 32 * st, ntok, kbuf);
    __builtin_amdgcn_sched_barrier(0);  // the step's LDS slots are for the query fragments
  };
  if (st < nsub) {
    next_tile(ka);
    attn_half<D, NP, 0, kOnlyA>(qs, lz_s, ka, kb, q, z, p0, p1, parta, partb, preva, raw_out, ntok, a.c);
    preva = 32 * (st - kGuideWaves);
    balance_issue(progress, wave, ++done);
    while (st + kGuideWaves < nsub) {  // two more tiles
      next_tile(kb);
      attn_half<D, NP, 1, kBothTiles>(qs, lz_s, ka, kb, q, z, p0, p1, parta, partb, prevb, raw_out, ntok, a.c);
      prevb = 32 * (st - kGuideWaves);
      balance_issue(progress, wave, ++done);
      next_tile(ka);
      attn_half<D, NP, 0, kBothTiles>(qs, lz_s, ka, kb, q, z, p0, p1, parta, partb, preva, raw_out, ntok, a.c);
      preva = 32 * (st - kGuideWaves);
      balance_issue(progress, wave, ++done);
    }
    if (st < nsub) {
      next_tile(kb);
      attn_half<D, NP, 1, kBothTiles>(qs, lz_s, ka, kb, q, z, p0, p1, parta, partb, prevb, raw_out, ntok, a.c);
      prevb = 32 * (st - kGuideWaves);
      balance_issue(progress, wave, ++done);
      attn_half<D, NP, 0, kOnlyB>(qs, lz_s, ka, kb, q, z, p0, p1, parta, partb, preva, raw_out, ntok, a.c);
      attn_flush(partb + attn_sum(p1, a.c), raw_out, prevb, ntok);
    } else {
      attn_half<D, NP, 1, kOnlyA>(qs, lz_s, ka, kb, q, z, p0, p1, parta, partb, prevb, raw_out, ntok, a.c);
      attn_flush(parta + attn_sum(p0, a.c), raw_out, preva, ntok);
    }
  }
}

// ---------------------------------------------------------------------------- pooling
// s_key = (1/(R K)) * sum over the window of the raw sums of all row groups (zero outside the
// sequence).  A block stages TILE + 2*half raw values (summed over row groups) in LDS
// with coalesced loads, then each thread sums its windows from LDS; windows wider than
// kPoolMaxHalf use the direct loop.
constexpr int kPoolTile = 4096;      // calls of many tiles, bound by bytes
// Calls whose 4096-token tiles leave CUs idle are bound by one block's latency (four rounds of loads
// and sixteen windows a thread): 24 segments of up to 4097 tokens, the whole sequence of separate
// calls 76.2 -> 68.8 us.  The line is one block per CU.
constexpr int kPoolTileFew = 1024;
constexpr int kPoolFewBlocks = 256;
constexpr int kPoolMaxHalf = 512;

__device__ inline float raw_at(const GuideArgs& a, const float* raw, int nrg, int64_t j) {
  const int64_t lh = (int64_t)a.L * a.Hkv;
  float v = 0.f;
  for (int rg = 0; rg < nrg; ++rg) v += raw[rg * lh * a.n_tot + j];
  return v;
}

template <int TILE>
__global__ __launch_bounds__(256) void k_guide_pool(GuideArgs a) {
  __shared__ float buf[TILE + 2 * kPoolMaxHalf];
  const int seg = blockIdx.y, b = blockIdx.z;
  const int64_t n0 = a.bt.ctx_off[b];
  const int64_t nb = a.bt.ctx_off[b + 1] - n0;
  const int64_t i0 = (int64_t)blockIdx.x * TILE;
  if (i0 >= nb) return;
  const int gb = (int)(a.bt.g_off[b + 1] - a.bt.g_off[b]);
  const int nrg = (a.R * gb + kRowsPerGroup - 1) / kRowsPerGroup;
  const float* raw = a.raw + (int64_t)seg * a.n_tot + n0;
  float* out = a.s_key + (int64_t)seg * a.n_tot + n0;
  const int half = a.pool_half;
  if (half > kPoolMaxHalf) {  // wide windows: direct sums
    for (int u = 0; u < TILE / 256; ++u) {
      const int64_t i = i0 + threadIdx.x + 256 * u;
      if (i >= nb) break;
      float acc = 0.f;
      for (int t = -half; t <= half; ++t)
        if (i + t >= 0 && i + t < nb) acc += raw_at(a, raw, nrg, i + t);
      out[i] = acc * a.pool_inv;
    }
    return;
  }
  const int nstage = TILE + 2 * half;
  for (int t0 = 0; t0 < nstage; t0 += 256 * 8) {  // eight loads in flight per thread
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int t = t0 + 256 * e + threadIdx.x;
      const int64_t j = i0 - half + t;
      v[e] = (t < nstage && j >= 0 && j < nb) ? raw_at(a, raw, nrg, j) : 0.f;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int t = t0 + 256 * e + threadIdx.x;
      if (t < nstage) buf[t] = v[e];
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < TILE / 256; ++u) {
    const int l = threadIdx.x + 256 * u;
    if (i0 + l >= nb) break;
    float acc = 0.f;
    for (int t = 0; t <= 2 * half; ++t) acc += buf[l + t];
    out[i0 + l] = acc * a.pool_inv;
  }
}

template <int D, int NP>
hipError_t launch_pass(const GuideArgs& a, bool attn, hipStream_t stream) {
  const unsigned nwg = (unsigned)a.wg_off[a.bt.batch];
  if (nwg == 0) return hipSuccess;
  if (attn) {
    hipLaunchKernelGGL((k_guide_attn<D, NP>), dim3(nwg), dim3(kGuideThreads), 0, stream, a);
  } else {
    hipLaunchKernelGGL((k_guide_stats<D, NP>), dim3(nwg), dim3(kGuideThreads), 0, stream, a);
  }
  return hipGetLastError();
}

// One launch per class of sequences that need the same number NP of staged row-block pairs
// (NP = ceil(min(R G_b, 256) / 64)), so short guides do not pay for 256 rows; each class's
// arguments give the other sequences empty workgroup ranges.  Three pairs are padded to four where
// the call has a class of four anyway and this one is small (at most kPadWgs workgroups of
// kPadTokens tokens): the fourth pair then costs less than a launch in each pass (tp_guide_scores of
// two sequences of 1000 tokens, 192 and 256 rows, one layer 44 -> 26 us, 64 layers 72.5 -> 67.8;
// four of 4000 tokens, 192 rows but the last, 32 layers 246 apart, 253 padded).
constexpr int64_t kPadWgs = 256, kPadTokens = 2048;

template <int D>
hipError_t launch_d(const GuideArgs& a, hipStream_t stream, hipEvent_t* ev, GuideBetween between, void* ctx) {
  static_assert(kChunkUnit % (32 * kGuideWaves) == 0, "every wave owns whole sub-tiles of a chunk");
  int64_t max_nb = 0, max_gb = 0;
  // per class NP (1..4 staged row-block pairs) the launch arguments, with the other classes'
  // sequences given empty workgroup ranges
  GuideArgs cls[4];
  int64_t wg[4] = {0, 0, 0, 0};
  for (int c = 0; c < 4; ++c) {
    cls[c] = a;
    cls[c].wg_off[0] = 0;
  }
  const auto pairs_of = [&](int b) {
    const int64_t rows = (int64_t)a.R * (a.bt.g_off[b + 1] - a.bt.g_off[b]);
    return (int)(((rows < kRowsPerGroup ? rows : kRowsPerGroup) + 63) / 64);
  };
  int64_t wg3 = 0, longest3 = 0;
  bool four = false;
  for (int b = 0; b < a.bt.batch; ++b) {
    const int64_t nb = a.bt.ctx_off[b + 1] - a.bt.ctx_off[b];
    four = four || pairs_of(b) == 4;
    if (pairs_of(b) != 3) continue;
    wg3 += ((int64_t)a.L * a.Hkv * chunks_of(nb, a.chunk) + 7) / 8 * 8;
    longest3 = std::max(longest3, std::min<int64_t>(nb, seq_chunk(nb, a.chunk)));
  }
  const bool pad3 = four && wg3 <= kPadWgs && longest3 <= kPadTokens;
  for (int b = 0; b < a.bt.batch; ++b) {
    const int64_t nb = a.bt.ctx_off[b + 1] - a.bt.ctx_off[b];
    const int64_t gb = a.bt.g_off[b + 1] - a.bt.g_off[b];
    if (nb > max_nb) max_nb = nb;
    if (gb > max_gb) max_gb = gb;
    const int64_t rows = (int64_t)a.R * gb;
    const int np = pairs_of(b) == 3 && pad3 ? 4 : pairs_of(b);
    const int64_t units = (int64_t)a.L * a.Hkv * chunks_of(nb, a.chunk);
    const int64_t seq_wg = (units + 7) / 8 * 8 * ((rows + kRowsPerGroup - 1) / kRowsPerGroup);
    wg[np - 1] += seq_wg;
    for (int c = 0; c < 4; ++c) cls[c].wg_off[b + 1] = (int32_t)wg[c];
  }
  for (int pass = 0; pass < 2; ++pass) {  // the large classes first: shorter tail
    if (pass == 0 && a.lse_in) {  // normalisers given: no pass 1
      hipError_t e = ev ? hipEventRecord(ev[0], stream) : hipSuccess;
      if (e == hipSuccess && ev) e = hipEventRecord(ev[1], stream);
      if (e == hipSuccess && between) e = between(ctx);
      if (e != hipSuccess) return e;
      continue;
    }
    hipError_t e = launch_pass<D, 4>(cls[3], pass == 1, stream);
    if (e == hipSuccess) e = launch_pass<D, 3>(cls[2], pass == 1, stream);
    if (e == hipSuccess) e = launch_pass<D, 2>(cls[1], pass == 1, stream);
    if (e == hipSuccess) e = launch_pass<D, 1>(cls[0], pass == 1, stream);
    if (e == hipSuccess && ev) e = hipEventRecord(ev[pass == 0 ? 0 : 2], stream);
    if (e != hipSuccess) return e;
    if (pass == 0) {
      if (a.kg != nullptr) {
        const dim3 kgrid((unsigned)((a.R * max_gb + kKeyRows - 1) / kKeyRows), (unsigned)(a.L * a.Hkv), (unsigned)a.bt.batch);
        hipLaunchKernelGGL(k_guide_key_stats<D>, kgrid, dim3(256), 0, stream, a);
      }
      if (!a.fold_lse) {
        const dim3 lgrid((unsigned)((a.L * a.Hq * max_gb + 255) / 256), (unsigned)a.bt.batch);
        hipLaunchKernelGGL(k_guide_lse<D>, lgrid, dim3(256), 0, stream, a);
      }
      e = hipGetLastError();
      if (e == hipSuccess && ev) e = hipEventRecord(ev[1], stream);
      if (e == hipSuccess && between) e = between(ctx);
      if (e != hipSuccess) return e;
    }
  }
  if (a.skip_pool) return hipSuccess;  // the selection pools the raw sums itself
  const auto pgrid = [&](int tile) {
    return dim3((unsigned)((max_nb + tile - 1) / tile), (unsigned)(a.L * a.Hkv), (unsigned)a.bt.batch);
  };
  const dim3 wide = pgrid(kPoolTile);
  if ((int64_t)wide.x * wide.y * wide.z < kPoolFewBlocks)
    hipLaunchKernelGGL(k_guide_pool<kPoolTileFew>, pgrid(kPoolTileFew), dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL(k_guide_pool<kPoolTile>, wide, dim3(256), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && ev && ev[3]) e = hipEventRecord(ev[3], stream);
  return e;
}

}  // namespace

// The call's target chunk.  The usual one is 16384 when every sequence has 65536 tokens or more
// (the query staging and the statistics merge are spread over more tokens), else 8192 (short
// and ragged sequences; 32 layers at 32768 tokens, the whole tp_evict: 1844 us at 8192, 1880 at
// 16384, whose last round ends later).  Calls that give it fewer than three rounds of workgroups
// take the candidate with the least estimated pass time, the sum over the launches (row-block
// classes) of rounds over the CUs x (a workgroup's fixed work + its tokens), where that is 3 %
// less.  Both passes together, us at 8192 and at the target chosen: one layer of 32q/8kv heads
// with 64 guide tokens at 32768 tokens 200 -> 64 (1024), four layers 208 -> 164 (4096), three
// layers at 131072 tokens 524 -> 505 (4096), seven segments of 3924 tokens 108 -> 33 (256).
// Chunks of which the statistics would exceed `max_slots` are not planned.
static int32_t plan_chunk(int32_t L, int32_t Hq, int32_t Hkv, const int64_t* ctx_off, const int64_t* g_off,
                          int32_t batch, int64_t max_slots) {
  static const int32_t kTargets[] = {16384, 14336, 12288, 10240, 8192, 7168, 6144, 5120, 4096, 3584, 3072,
                                     2560,  2048,  1792,  1536,  1280, 1024, 768,  512,  256};
  // by staged row-block pairs: K's bytes bound few rows.  One round of 8192-token chunks at head_dim
  // 128, us per pass: 107, 110, 128, 138 (and 4096-token ones, half of K in the caches, 47, 51, 59,
  // 73; at head_dim 64 49, 57, 75, 94).
  static const double kTokenCost[4] = {0.75, 0.75, 0.8, 1.0};
  const int64_t R = Hq / Hkv, segs = (int64_t)L * Hkv;
  struct Seq {
    uint32_t n;  // context tokens
    int cls;     // row-block class
    double rg;   // row groups
  } seq[TP_MAX_BATCH];
  for (int b = 0; b < batch; ++b) {
    const int64_t rows = R * (g_off[b + 1] - g_off[b]);
    seq[b].n = (uint32_t)(ctx_off[b + 1] - ctx_off[b]);
    seq[b].cls = (int)(((rows < kRowsPerGroup ? rows : kRowsPerGroup) + 63) / 64) - 1;
    seq[b].rg = (double)((rows + kRowsPerGroup - 1) / kRowsPerGroup);
  }
  bool all_long = true;
  uint32_t most_n = 0;
  for (int b = 0; b < batch; ++b) {
    all_long = all_long && seq[b].n >= kLongContext;
    most_n = std::max(most_n, seq[b].n);
  }
  const int32_t usual = all_long ? 16384 : 8192;
  struct Cost {
    double time, rounds;
  };
  auto cost_of = [&](int32_t target) {
    double wgs[4] = {0, 0, 0, 0};
    uint32_t longest[4] = {0, 0, 0, 0};
    for (int b = 0; b < batch; ++b) {
      const uint32_t c = (uint32_t)seq_chunk(seq[b].n, target);
      wgs[seq[b].cls] += (double)((segs * ((seq[b].n + c - 1u) / c) + 7) / 8 * 8) * seq[b].rg;
      longest[seq[b].cls] = std::max(longest[seq[b].cls], std::min(c, seq[b].n));
    }
    Cost cost{0.0, 0.0};
    for (int i = 0; i < 4; ++i) {
      if (wgs[i] <= 0) continue;
      // a partly filled last round costs half its length and half its share: its workgroups have the
      // HBM and the power budget to themselves (4096-token chunks of 256 rows in 1, 1.25, 1.5, 1.75
      // and 2 rounds 73, 127, 133, 141, 149 us, of 64 rows 47, 79, 89, 98, 110)
      const double whole = ceil(wgs[i] / kCus), r = whole > 1.0 ? 0.5 * (whole + wgs[i] / kCus) : 1.0;
      cost.rounds += r;
      cost.time += r * (kWgTokens + kTokenCost[i] * longest[i]);
    }
    return cost;
  };
  const Cost at_usual = cost_of(usual);
  if (at_usual.rounds >= 3.0) return usual;
  int32_t best = usual;
  double least = at_usual.time * 0.97;
  for (const int32_t target : kTargets) {
    if (((int64_t)most_n + target - 1) / target > max_slots) break;
    const Cost c = cost_of(target);
    if (c.time < least) {
      best = target;
      least = c.time;
    }
    if (c.rounds >= 16.0) break;  // shorter chunks only add fixed work from here on
  }
  return best;
}

// Room for the chunks' statistics: what chunks of 8192 tokens need or, where shorter ones may be
// planned, what 4352 workgroups of 256 rows write (16 rounds of the chip and a little, 8.9 MB), at
// most what kChunkUnit needs.  Not the planned chunk's own need, which falls where a longer call
// takes longer chunks.
constexpr int64_t kStatsPlanRows = 4352 * 256;

GuideWorkspace guide_workspace_layout(int32_t L, int32_t Hq, int32_t Hkv, const int64_t* ctx_off,
                                      const int64_t* g_off, int32_t batch) {
  int64_t max_nb = 0, max_gb = 0;
  for (int b = 0; b < batch; ++b) {
    if (ctx_off[b + 1] - ctx_off[b] > max_nb) max_nb = ctx_off[b + 1] - ctx_off[b];
    if (g_off[b + 1] - g_off[b] > max_gb) max_gb = g_off[b + 1] - g_off[b];
  }
  const int64_t n_tot = ctx_off[batch], g_tot = g_off[batch];
  const int64_t R = Hq / Hkv, rows = (int64_t)L * Hq * g_tot;
  const int64_t nrg = (R * max_gb + kRowsPerGroup - 1) / kRowsPerGroup;
  // slots of per-chunk statistics, and one for the guide keys
  const int64_t whole = (max_nb + kChunkWhole - 1) / kChunkWhole + 1, fine = (max_nb + kChunkUnit - 1) / kChunkUnit + 1;
  const int64_t entries = std::max(whole * rows, (double)fine * (double)rows < (double)kStatsPlanRows ? fine * rows
                                                                                                     : kStatsPlanRows);
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  GuideWorkspace w;
  w.chunk = plan_chunk(L, Hq, Hkv, ctx_off, g_off, batch, entries / rows - 1);
  w.stats_off = 0;
  w.lse_off = up((size_t)entries * sizeof(float2));
  w.raw_off = w.lse_off + up((size_t)rows * sizeof(float));
  w.total = w.raw_off + up((size_t)nrg * L * Hkv * n_tot * sizeof(float));
  return w;
}

hipError_t launch_guide_scores(const GuideArgs& a, int head_dim, hipStream_t stream, hipEvent_t* ev,
                               GuideBetween between, void* ctx) {
  if (head_dim == 128) return launch_d<128>(a, stream, ev, between, ctx);
  return launch_d<64>(a, stream, ev, between, ctx);
}

}  // namespace tp
