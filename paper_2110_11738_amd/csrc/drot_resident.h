// The resident iteration: whole iterations of Algorithm 1 with the plan and
// the cost held on the chip.
//
// A problem is cut into R x S tiles, one workgroup (one compute unit) each.
// A workgroup of eight waves loads its tile of X and of rho C once, keeps
// both in registers (the largest tiles keep half of rho C in LDS) for up to
// thousands of iterations, and writes X back at the end.  What crosses
// workgroups in an iteration is O(rows + columns) per tile: the tile's row
// and column partials and a few scalars, exchanged through memory.  256
// compute units hold 128 MB of registers, so float32 problems up to
// 4096 x 4096 (float64: up to 2048 x 4096) fit.
//
// The exchange.  Every workgroup owns one message per phase: its row
// partials, its column partials and its scalars as 8-byte words, written with
// device-scope stores (which bypass the per-XCD L2 caches) and polled with
// device-scope loads by the workgroups of the same tile row and tile column
// (everybody reads the scalar words).  A word that has not been written holds
// the sentinel, so data and readiness travel together: one memory trip, no
// flags, no fences, no atomic counters.  Message s lives in phase s mod 4.
// Having published s, a workgroup puts the sentinel back into its words of
// phase (s + 2) mod 4, i.e. of message s - 2, which every reader has consumed:
// it published s - 1 after reading s - 2.  That reset is complete (vmcnt 0 and
// a barrier) before s + 1 is published, so whoever has seen s + 1 and polls
// for s + 2 cannot see message s - 2 any more.
//
// All workgroups have to be on the chip together.  The launch is cooperative,
// which does not keep other processes' kernels away: so each workgroup reports
// as it starts, the last one gives the word to go, and one that has polled for
// it kResGatePolls times calls the launch off.  Which of the two it is one
// compare-and-swap decides for all.  A launch that is called off has touched
// nothing: it adds its iterations to DevState::missed, and the host makes them
// up with sweeps.  Once all are there nothing keeps one of them away, and a poll
// of a message that runs dry all the same ends the kernel with an error state
// instead of spinning on.
//
// Every workgroup of a tile row adds the same row partials in the same order
// (columns likewise), so the row's duals are computed redundantly and
// identically; the total of X, which gives beta, comes from the scalar words.
//
// The stopping test needs sums over all rows and columns of quantities that
// follow from this exchange, so it trails: workgroup 0 tests iteration k
// while it waits for the words of iteration k + 2, and announces a stop in
// its next message.
// By then X has moved on; the workgroups load the last saved state and repeat
// the iterations up to the stopping one (everything is deterministic), so the
// result is exactly X at the stopping iteration.  A state is saved when two
// exchanges of scalar words have told everybody that no test up to it ended
// the solve: after kResSaves[1] iterations of the solve (kResSaves[0] beyond 32
// tile rows, where an iteration costs more than half of the sweeps'), then
// each time they have doubled, then every kResSaves[2].  A save takes about two
// iterations' time and the write of X, 8 us at 517 x 483 and 25 at 4096 x 4096.
//
// What bounds it: up to about 2000 x 2000 latency.  In 9.8 k clocks at
// 517 x 483, 2.9 go to the sweep and its reductions (two waves share a SIMD),
// 0.8 to publishing, 2.5 to 3.8 to the words' trip through memory, 1.3 to the
// total and the scalar step, 1.0 to steps 5-8.  Beyond that the vector units:
// nine operations per entry, 64 lanes per clock and compute unit, make 13.1 k
// of the 18.5 k clocks at 4096 x 4096.  So nothing is spilled inside the
// iteration loop (with spills: 12.4 us instead of 7.7 at 4096 x 4096): values
// that depend on the thread number are made again in each step instead of
// being kept, and the words of a poll are loaded without branches, all in
// flight together (a branch and a wait per word: 5.1 us instead of 4.3 at
// 517 x 483).
// Measured per iteration against sweep + aux launches, float32: 4.1 us (10.6)
// at 517 x 483, 4.2 (13.5) at 1000^2, 4.85 (17) at 2000^2, 7.0 at 3000^2, 7.65
// (36.5) at 4096^2, 10.6 (17.3) at 16384 x 64; float64: 4.3 (14) at 700 x 901,
// 5.35 at 2000^2, 9.3 at 2800^2; and per launch 35 to 85 us more, of which the
// gate takes 3 to 5.
#pragma once

#include "drot_device.h"
#include "drot_internal.h"

namespace drot {
namespace {

typedef unsigned long long u64;
constexpr u64 kSent = ~0ull;
constexpr int kResSpins = 1 << 22;  // polls of one word before giving up (seconds)
constexpr int kResScal = 16;        // scalar words of a message
// Scalar words: <rho C, X>, sum [t]_+^2, total of the tile, stop iteration
// (workgroup 0), and of the previous iteration sum r^2, sum p phi~ (tile
// column 0), sum s^2, sum q psi~ (tile row 0).  Float64 problems have the total
// in two words (see split_sum), in one line of memory, and the stop iteration
// in the last word.
enum ResWord : int { kRwS0 = 0, kRwS1, kRwTot, kRwLow, kRwR2, kRwPphi, kRwS2, kRwQpsi, kRwLast };
// A message: column words, row words, scalar words.

// Messages are global memory (the address space is spelled out because the
// pointers come out of a record in memory).
typedef __attribute__((address_space(1))) u64* Msg;
typedef __attribute__((address_space(1))) char* MsgByte;
// A word by wave-uniform base and 32-bit offset in bytes.
__device__ __forceinline__ Msg word_at(Msg base, uint32_t off) { return (Msg)((MsgByte)base + off); }
__device__ __forceinline__ u64 ld_word(Msg base, uint32_t off) {
  return __hip_atomic_load(word_at(base, off), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_word(Msg base, uint32_t off, u64 v) {
  __hip_atomic_store(word_at(base, off), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A message word of T: two floats or one double.  The sentinel is a NaN
// pattern per value; a value that has it (a NaN) is replaced by another NaN.
// gap() folds a word into a running maximum, which is all ones if and only if
// a word was missing.
template <typename T>
struct WordOf;
template <>
struct WordOf<float> {
  static __device__ __forceinline__ uint32_t gap(uint32_t g, u64 w) {
    const uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32);
    const uint32_t t = lo > hi ? lo : hi;
    return g > t ? g : t;
  }
  static __device__ __forceinline__ uint32_t half(float v) {
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    return u == 0xffffffffu ? 0x7fc00000u : u;
  }
  static __device__ __forceinline__ u64 pack(float x, float y) {
    return ((u64)half(y) << 32) | half(x);
  }
  static __device__ __forceinline__ void add(u64 w, double (&s)[2]) {
    s[0] += (double)__builtin_bit_cast(float, (uint32_t)w);
    s[1] += (double)__builtin_bit_cast(float, (uint32_t)(w >> 32));
  }
};
__device__ __forceinline__ u64 pack_double(double v) {
  const u64 u = __builtin_bit_cast(u64, v);
  return u == kSent ? 0x7ff8000000000000ull : u;
}
template <>
struct WordOf<double> {
  static __device__ __forceinline__ uint32_t gap(uint32_t g, u64 w) {
    const uint32_t t = (uint32_t)w & (uint32_t)(w >> 32);
    return g > t ? g : t;
  }
  static __device__ __forceinline__ void add(u64 w, double (&s)[1]) {
    s[0] += __builtin_bit_cast(double, w);
  }
};

// Sums over the wave of G values at once (G = 8 or 4): lane l gets the sum of
// value l / (64 / G).  Each folding step halves the registers, so eight sums
// cost 18 operations instead of 48.
template <typename V>
__device__ __forceinline__ V wave_fold(V (&r)[8], int lane) {
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = fold32(r[i], r[i + 4]);
#pragma unroll
  for (int i = 0; i < 2; ++i) r[i] = fold16(r[i], r[i + 2]);
  const bool up = lane & 8;
  const V keep = up ? r[1] : r[0], send = up ? r[0] : r[1];
  V v = keep + dpp<0x128>(send);  // row_ror:8
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  return v;
}
template <typename V>
__device__ __forceinline__ V wave_fold(V (&r)[4], int) {
#pragma unroll
  for (int i = 0; i < 2; ++i) r[i] = fold32(r[i], r[i + 2]);
  V v = fold16(r[0], r[1]);
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  v += dpp<0x140>(v);
  return v;
}

// beta is the small difference of two sums of about sum p, so a float64 problem
// takes it from sums without rounding errors of their size: every row sum and every
// p_i is split into a multiple of 2^-24 sum p, whose sums are exact, and the rest,
// whose sums' errors are 2^-24 times smaller.  (With beta from the rounded total
// less sum p, alpha gathers its errors: nu of 8000 x 40 was 2.8 times as far from
// the exact iterate after 1000 iterations as with the sweeps, which add residuals.
// It costs 0.13 us of 4.2 per iteration at 700 x 901, 0.3 of 5.05 at 2000 x 2000,
// 0.4 of 8.8 at 2800 x 2800; with the second words read by a wave of their own,
// from lines of their own, 0.25, 0.65 and 0.45.)
__device__ __forceinline__ double split_magic(double sum_p) {
  const uint64_t e = ((__builtin_bit_cast(uint64_t, sum_p) >> 52) & 0x7ffu) + 28;
  return __builtin_bit_cast(double, (e < 2046 ? e : 2046) << 52 | (uint64_t)1 << 51);  // 1.5 2^52 multiples
}
__device__ __forceinline__ void split_sum(double v, double magic, double (&sum)[2]) {
  const double big = (v + magic) - magic;
  sum[0] += big;
  sum[1] += v - big;
}

// Keeps the compiler from carrying `p` (and addresses made from it) in
// registers from an earlier use: the plan takes most of them.
template <typename P>
__device__ __forceinline__ P* fresh(P* p) {
  asm volatile("" : "+s"(p));
  return p;
}

// Wave-uniform values, held in scalar registers.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename P>
__device__ __forceinline__ P* uni(P* p) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  return reinterpret_cast<P*>(((uint64_t)(uint32_t)uni((int)(u >> 32)) << 32) | (uint32_t)uni((int)u));
}
__device__ __forceinline__ int64_t uni(int64_t v) {
  return (int64_t)(((uint64_t)(uint32_t)uni((int)(v >> 32)) << 32) | (uint32_t)uni((int)v));
}

// The same for a value whose comparisons are not worth a register.
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+s"(v));
  return v;
}
template <typename V>
__device__ __forceinline__ V fresh_lane(V v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The gate of a launch (one thread of each workgroup): report, the last of
// `blocks` giving the word; wait for the word or call the launch off; and, off,
// leave, true for the last one, which clears the words for the next launch.
__device__ __forceinline__ void res_say(ResSync* g, uint32_t v) {
  uint32_t open = 0;
  __hip_atomic_compare_exchange_strong(&g->verdict, &open, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t res_count(uint32_t* word) {
  return __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
}
__device__ __forceinline__ uint32_t res_verdict(ResSync* g) {
  return __hip_atomic_load(&g->verdict, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// False for the whole workgroup where the launch is off.
__device__ __forceinline__ bool res_gate(ResSync* g, int blocks, int polls, int& go) {
  if (threadIdx.x == 0) {
    uint32_t v = 0;
    if (res_count(&g->arrived) == (uint32_t)blocks) res_say(g, kResGo);
    for (int k = 0; k < polls && (v = res_verdict(g)) == 0; ++k) __builtin_amdgcn_s_sleep(2);
    if (v == 0) {
      res_say(g, kResOff);
      v = res_verdict(g);
    }
    go = v == kResGo;
  }
  __syncthreads();
  return uni(go);
}
__device__ __forceinline__ void res_clear(ResSync* g) { g->arrived = g->verdict = g->left = 0; }
__device__ __forceinline__ bool res_leave(ResSync* g, int blocks) {
  if (res_count(&g->left) != (uint32_t)blocks) return false;
  res_clear(g);
  return true;
}

// Shared state of a workgroup outside the sums.
struct ResShared {
  double wsum[4][kResWaves];  // <rho C,X>, sum [t]_+^2, total (float64: in two) per wave
  double psum[2][4];          // float64, first tile column: sum of p_i in two, per wave
  double total[2][2];         // float64: the total less sum p in two, by waves 7 and 2
  double magic;
  double esum[2][kResWaves];  // sum r^2 (or s^2), sum p phi~ (or q psi~) per wave
  double bc[4][3];            // cphi, cpsi, alpha after iteration k, at k mod 4
  double inv[3];              // 1 / n, 1 / m, 1 / (m + n)
  double mon[2][6][kWave];    // workgroup 0: a step's test sums per lane, by step parity
  double prev[2];             // workgroup 0: <rho C,X> and sum [t]_+^2 one iteration back
  double rec[6];              // workgroup 0: the latest tested iteration
  StateIn sv;
  double rhoT, wall_rate;
  double* trace;
  double ctl;                 // workgroup 0: stop iteration to announce
  int trace_mask;
  double base[3];             // cphi, cpsi, alpha of the saved state
  int rec_k, rec_status, rec_done;
  int stop_at, dead, go;
};

// Four words of a lane, `count` of them wanted (the rest repeats the last
// one, so that all loads go out together without a branch).
__device__ __forceinline__ void res_load4(u64 (&w)[4], Msg cur, uint32_t off, int stride, int count) {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int q = u < count ? u : count > 0 ? count - 1 : 0;
    w[u] = ld_word(cur, off + (uint32_t)(q * stride));
  }
}
// ... again until none is missing, and their sum; false when the spins run out.
__device__ __forceinline__ bool res_sum4(u64 (&w)[4], Msg cur, uint32_t off, int stride, int count,
                                         double& sum) {
  bool fine = false;
  for (int spin = 0; spin < kResSpins; ++spin) {
    uint32_t g = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) g = WordOf<double>::gap(g, w[u]);
    fine = g != 0xffffffffu || count < 1;
    if (fine) break;
    res_load4(w, cur, off, stride, count);
  }
  sum = 0.0;
#pragma unroll
  for (int u = 0; u < 4; ++u) sum += u < count ? __builtin_bit_cast(double, w[u]) : 0.0;
  return fine;
}

// Read and add a thread's column words (nc of them, the same for its wave,
// stride sc) and row words (nr, stride sr), NC and NR at a time; nq rounds.
// All loads of a round are in flight together, and so are the repeats.
template <typename T, int NC, int NR, int PW>
__device__ __forceinline__ bool res_read(Msg pcol, uint32_t ocol, int sc, int nc, Msg prow,
                                         uint32_t orow, int sr, int nr, int nq, double (&cs)[PW],
                                         double (&rs)[PW]) {
  using Wd = WordOf<T>;
  bool fine = true;
  for (int q = 0; q < nq; ++q) {
    u64 wc[NC], wr[NR];
    bool ok = false;
    for (int spin = 0; spin < kResSpins; ++spin) {
#pragma unroll
      for (int u = 0; u < NC; ++u) {
        const int i = q * NC + u < nc ? q * NC + u : nc > 0 ? nc - 1 : 0;
        wc[u] = ld_word(word_at(pcol, (uint32_t)(i * sc)), ocol);
      }
#pragma unroll
      for (int u = 0; u < NR; ++u) {
        const int i = q * NR + u < nr ? q * NR + u : nr > 0 ? nr - 1 : 0;
        wr[u] = ld_word(prow, orow + (uint32_t)(i * sr));
      }
      uint32_t g = 0;
#pragma unroll
      for (int u = 0; u < NC; ++u) g = Wd::gap(g, wc[u]);
#pragma unroll
      for (int u = 0; u < NR; ++u) g = Wd::gap(g, wr[u]);
      ok = g != 0xffffffffu;
      if (ok) break;
    }
    fine = fine && ok;
    if (!fine) break;
#pragma unroll
    for (int u = 0; u < NC; ++u)
      if (q * NC + u < nc) Wd::add(wc[u], cs);
#pragma unroll
    for (int u = 0; u < NR; ++u)
      if (q * NR + u < nr) Wd::add(wr[u], rs);
  }
  return fine;
}

// The four sums of iteration kt that waves 3 (rows) and 4 (columns) of
// workgroup 0 read: even lanes hold the first word's, odd lanes the second's.
__device__ __forceinline__ void res_keep(double (&mon)[6][kWave], int wave, int lane, double v) {
  mon[2 * wave - 4][lane] = lane & 1 ? 0.0 : v;
  mon[2 * wave - 3][lane] = lane & 1 ? v : 0.0;
}

// Workgroup 0, one wave: the test of iteration kt (of this launch; none if
// kt < 1) with the sums that the step of iteration kt + 1 (or the closing
// step) brought into sh.mon: <rho C,X> and sum [t]_+^2 of that step's own
// iteration, kept for the next call, and the other four of iteration kt.
__device__ __forceinline__ void res_test(ResShared& sh, const double (&mon)[6][kWave], int kt,
                                         int lane) {
  // lane 8 q + s adds eight entries of sum q, then its row of eight lanes
  double v = 0.0;
  if (lane < 48) {
    const double* const p = &mon[0][0] + (lane >> 3) * kWave + (lane & 7);
#pragma unroll
    for (int u = 0; u < 8; ++u) v += p[8 * u];
  }
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  double w[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) w[q] = read_lane(v, 8 * q);
  if (lane != 0) return;
  if (kt >= 1 && sh.ctl == 0.0) {
    ScalarStep f;
    f.cphi = sh.bc[kt & 3][0];
    f.cpsi = sh.bc[kt & 3][1];
    f.alpha = sh.bc[kt & 3][2];
    f.k = sh.sv.iter + kt;
    const double ws[8] = {0.0, w[2], w[3], 0.0, w[4], w[5], sh.prev[0] / sh.rhoT, sh.prev[1]};
    scalar_tests(f, sh.sv, ws, false);
    double* const tr = sh.trace + (((int)f.k - 1) & sh.trace_mask) * kTraceWidth;
    trace_record(tr, f, sh.sv.t_start, wall_clock64(), sh.wall_rate);
    sh.rec[0] = f.pobj;
    sh.rec[1] = f.dobj;
    sh.rec[2] = f.rp;
    sh.rec[3] = f.rd;
    sh.rec[4] = f.gap;
    sh.rec[5] = f.test;
    sh.rec_k = kt;
    sh.rec_done = f.done;
    sh.rec_status = f.status;
    if (f.done) sh.ctl = (double)kt;
  }
  sh.prev[0] = w[0];
  sh.prev[1] = w[1];
}

// The scalar step of iteration k + 1 from the total of X less sum p (one wave).
__device__ __forceinline__ void res_scalars(ResShared& sh, int k, int lane, double excess, double alpha,
                                            double dn, double dm, const double (&inv)[3]) {
  const double beta = div_by(excess, dm + dn, inv[2]);
  const double cc = 2.0 * beta - alpha;
  const double nphi = div_by(cc, dn, inv[0]), npsi = div_by(cc, dm, inv[1]);
  if (lane == 0) {
    sh.bc[(k + 1) & 3][0] = nphi;
    sh.bc[(k + 1) & 3][1] = npsi;
    sh.bc[(k + 1) & 3][2] = alpha - beta;
  }
}

// RPW rows per wave (tiles of 8 RPW rows), of which the last CL keep rho C in
// LDS.  `map`: the (team, workgroup) of each block, or null for the one team
// teams[0].
//
// FINE (float32): column sums cross tiles unrounded where a plan has few columns
// or few rows.  Such a side sums many entries into few duals, and a float rounding
// of every tile's sum shows in them: nu of a plan of 4096 x 26 is 1.4 times as far
// off after 500 iterations as with sweeps over blocks of eight rows, 0.96 times
// here.  With at most half a tile's columns (`slim`) each has a whole word, for
// the sum as a float and what that leaves out; with one tile row (`lone`) the
// tile's sums are the totals and are taken as they are.  A lane's column sum is
// float32 over four rows, not eight, and a row's sum is formed in float64 across
// the lanes and has a whole word too: a flat plan's few rows sum as many entries.
// It costs 0.6 us of 5.8 per iteration there, 0.9 of 9.7 at 16384 x 64, and would
// cost the other plans 0.1 of 4.1.
template <typename T, int RPW, int CL, bool FINE>
__global__ __launch_bounds__(kResBlock, 2) void resident_kernel(const ResTeam* teams,
                                                                const uint2* map, int64_t iters,
                                                                int gate_polls) {
  constexpr int VEC = 16 / sizeof(T);
  constexpr int W = kWave * VEC;             // tile columns
  constexpr int TR = kResWaves * RPW;        // tile rows
  constexpr int PW = 8 / sizeof(T);          // values per message word
  // Rows in full (see FINE): a word for each, their sums over the wave in float64.
  constexpr bool kRows64 = FINE && PW == 2;
  using RowSum = typename std::conditional<kRows64, double, T>::type;
  constexpr int WR = kRows64 ? TR : TR / PW, WC = W / PW;  // row and column words
  constexpr int MSG = WR + WC + kResScal;
  constexpr int GC = kResBlock / WC;         // peers read side by side, columns
  constexpr int GR = kResBlock / WR;         // and rows
  constexpr int G = FINE || RPW < 8 ? 4 : 8;  // rows whose sums are folded together
  constexpr int kHeld = RPW - CL;            // rows with rho C in registers
  constexpr int kBuf = kResWaves * W > GC * W + GR * WR * PW ? kResWaves * W : GC * W + GR * WR * PW;
  // Row words in flight per thread: all of them for the usual team shapes.
  constexpr int NR = sizeof(T) == 4 ? (kRows64 ? 2 : RPW == 4 ? 1 : RPW <= 16 ? 2 : 4)
                                    : (RPW == 4 ? 2 : RPW <= 16 ? 4 : 8);
  static_assert(RPW % G == 0 && TR <= 256 && W <= 256 && MSG <= kResBlock, "thread roles");
  static_assert(WC == 128, "message layout");
  using Wd = WordOf<T>;

  __shared__ double buf[kBuf];  // column sums of the waves, then the peers' sums
  // rho C of the last CL rows; before that (and where CL = 0) the staging area
  // of rows on their way between memory and registers, SR rows per wave.
  constexpr int SR = CL > 0 ? CL : RPW < 8 ? RPW : 8;
  static_assert(RPW % SR == 0 && (CL == 0 || SR == CL), "staging");
  __shared__ __align__(16) T cl[kResWaves * SR * W];
  __shared__ __align__(16) T rowsh[TR];
  __shared__ __align__(16) T colsh[W];
  __shared__ __align__(16) RowSum rowp[TR];
  __shared__ double accs[kResBlock];  // a_i, b_j of the thread's row or column
  __shared__ ResShared sh;

  if (iters <= 0) return;  // see resident_warm(): nothing is there to be read
  const uint2 who = map ? map[blockIdx.x] : uint2{0u, blockIdx.x};
  const ResTeam* const tm = teams + uni((int)who.x);
  const int b = uni((int)who.y);
  DevState* const st = uni(tm->a.st);
  if (uni(st->done)) return;
  const int64_t left = uni(st->max_iter - st->iter);
  int limit = (int)(iters < left ? iters : left);
  if (limit <= 0) return;

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int R = uni(tm->R), S = uni(tm->S);
  const int ti = uni(b / S), tj = b - ti * S;
  const int m = uni((int)tm->a.g.m), n = uni((int)tm->a.g.n);
  const bool slim = FINE && PW == 2 && n <= WC && R > 1;
  const bool lone = FINE && R == 1;
  if (!res_gate(uni(tm->sync), R * S, gate_polls, sh.go)) {
    if (tid == 0 && res_leave(uni(tm->sync), R * S)) st->missed += (uint32_t)limit;
    return;
  }
  int seq = uni((int)uni(tm->sync)->seq);
  const Msg xch = (Msg)uni(tm->xch);
  const int phase = R * S * MSG;

  // Roles: thread t < TR finishes row t of the tile, thread 256 + c column c.
  const int row0 = ti * TR, col0 = tj * W;
  const int cc0 = tid - 256;
  const bool is_row = tid < TR, is_col = cc0 >= 0 && cc0 < W;
  const int gid = is_row ? row0 + tid : col0 + cc0;  // row or column index
  const bool own_r = is_row && gid < m, own_c = is_col && gid < n;
  // The tile's entries of this lane: rows wr0 + r, columns jl .. jl + VEC - 1.
  const int wr0 = row0 + wave * RPW;
  const int jl = col0 + lane * VEC;
  const int nv = n - jl >= VEC ? VEC : n > jl ? n - jl : 0;

  // Words of the peers' messages that a thread reads: column word tid mod WC
  // of the tile column's workgroups csub, csub + GC, ... (nc0 of them), and
  // row word tid mod WR of the tile row's.  Only scalars are kept; what depends
  // on the thread is made again in every step, which costs a few operations
  // where keeping it would cost registers that the plan needs.
  const int csub = uni(tid / WC);
  const int nc0 = csub < R && !lone ? (R - csub + GC - 1) / GC : 0;
  const int ocol = 8 * ((csub < R ? csub : 0) * S + tj) * MSG;
  const int nqr = (S + GR * NR - 1) / (GR * NR);  // rounds for the row words
  // Scalar words that a wave reads, up to four per lane: word ox + (lane mod
  // (1 << xsh)) of every xstep-th byte from lane >> xsh on, xcnt of them.
  // Every workgroup: wave 7 the totals, wave 2 the stop word; float64: wave 7
  // the totals' two words by two lanes, of the first kHalf workgroups, wave 2 of
  // the others, wave 1 the stop word.  Workgroup 0:
  // waves 5 and 6 <rho C,X> and the dual sums of all tiles, wave 3 the row sums
  // (first tile column), wave 4 the column sums (first tile row), two words
  // of a workgroup by two lanes.
  int xcnt = R * S, xstep = 8 * MSG, xsh = 0, xw = kRwTot;
  constexpr bool kSplit = sizeof(T) == 8;
  constexpr int kCtlWave = kSplit ? 1 : 2, kRwCtl = kSplit ? kRwLast : kRwLow;
  constexpr int kRwCount = kRwLast + kSplit, kHalf = 2 * kWave;
  static_assert(kRwCount <= kResScal, "scalar words");
  if (kSplit && wave == 7) xsh = 1, xcnt = xcnt < kHalf ? xcnt : kHalf;
  if (kSplit && wave == 2) xsh = 1, xcnt -= kHalf, xw += kHalf * MSG;
  if (wave == kCtlWave) xcnt = 1, xstep = 0, xw = kRwCtl;
  if (wave == 3) xcnt = R, xstep = 8 * MSG * S, xsh = 1, xw = kRwR2;
  if (wave == 4) xcnt = S, xsh = 1, xw = kRwS2;
  if (wave == 5) xw = kRwS0;
  if (wave == 6) xw = kRwS1;
  const bool totals = wave == 7 || (kSplit && wave == 2 && xcnt > 0);
  const bool extra = wave == kCtlWave || totals || (b == 0 && wave > 2);
  // Words of its own message that a thread writes: column and row words by
  // number, the scalar words in the last wave, which has no others.
  static_assert(WC + WR <= kResBlock - kWave, "the last wave writes the scalar words");
  static_assert(WC % kWave == 0, "a wave holds words of one kind and of one peer");

  T marg = (T)0;
  if (own_r) marg = static_cast<const T*>(tm->a.p)[gid];
  if (own_c) marg = static_cast<const T*>(tm->a.q)[gid];
  T xr[RPW][VEC], pc[kHeld][VEC];
  const T rhoT = (T)st->rho;
  T* const stage = cl + (wave * SR * kWave + lane) * VEC;  // + u * W: row u of the wave
  if (tid == 0) {
    sh.sv = load_state(st);
    sh.inv[0] = 1.0 / (double)n;
    sh.inv[1] = 1.0 / (double)m;
    sh.inv[2] = 1.0 / ((double)m + (double)n);
    sh.rhoT = (double)rhoT;
    sh.wall_rate = tm->a.wall_rate;
    sh.trace = tm->a.trace;
    sh.trace_mask = (int)tm->a.trace_cap - 1;
    sh.ctl = 0.0;
    sh.magic = split_magic(sh.sv.sum_p);
    sh.total[1][0] = sh.total[1][1] = 0.0;
    sh.dead = 0;
    sh.rec_k = sh.rec_done = sh.rec_status = 0;
  }

  // The state is saved between segments of the launch (kResSaves says when).
  const int seg0 = R > 32 ? kResSaves[0] : kResSaves[1];
  bool replay = false;
  int base = 0, k = 0;  // iterations of this launch in the saved state, and done
  auto saved = [&]() {  // this thread's accs[] and shift in the saved state
    return reinterpret_cast<double*>((uintptr_t)(xch + kResPhases * phase)) +
           2 * (b * kResBlock + fresh_lane(tid));
  };
  // X to memory.
  auto store_x = [&]() {
    const ResTeam* const t3 = fresh(tm);
    const int ws0 = fresh(wr0), nvs = fresh_lane(nv);
    T* const X = uni(static_cast<T*>(t3->a.X));
    const int64_t ldx = uni(t3->a.g.ldx);
    const bool vec = uni(t3->vec_x) != 0;
    if (vec && nvs == VEC) {
#pragma unroll
      for (int r = 0; r < RPW; ++r)
        if (ws0 + r < m) store_chunk<T, VEC, false>(X + (int64_t)(ws0 + r) * ldx + jl, xr[r]);
    }
    if (!vec || n % VEC != 0) {  // the other chunks, element by element
      const int ne = vec && nvs == VEC ? 0 : nvs;
      if constexpr (CL > 0) {  // the staging area holds rho C
        T* const Xl = X + jl;
#pragma unroll
        for (int r = 0; r < RPW; ++r)
          if (ws0 + r < m)
#pragma unroll
            for (int e = 0; e < VEC; ++e)
              if (e < ne) Xl[(int64_t)(ws0 + r) * ldx + e] = xr[r][e];
      } else {
#pragma unroll
        for (int g = 0; g < RPW / SR; ++g) {
#pragma unroll
          for (int u = 0; u < SR; ++u) store_chunk<T, VEC, false>(stage + u * W, xr[g * SR + u]);
#pragma unroll 1
          for (int u = 0; u < SR; ++u) {
            const int i = ws0 + g * SR + u;
#pragma unroll
            for (int e = 0; e < VEC; ++e)
              if (i < m && e < ne) X[i * ldx + jl + e] = stage[u * W + e];
          }
        }
      }
    }
  };
  // An exchange of the scalar words alone, with workgroup 0's stop word.
  // Workgroup 0 reads the sums of iteration k too.
  auto exchange = [&]() {
    const Msg cur = xch + (seq & 3) * phase;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const Msg dst = word_at(cur, 8 * b * MSG);
    const Msg clr = word_at(xch + ((seq + 2) & 3) * phase, 8 * b * MSG);
    if (wave == kResWaves - 1) {
      if (lane < kRwCount) {
        const double* src = &sh.esum[lane & 1][lane >= kRwS2 ? 4 : 0];
        double v = lane >= kRwR2 && lane <= kRwQpsi ? (src[0] + src[1]) + (src[2] + src[3]) : 0.0;
        if (lane == kRwCtl) v = sh.ctl;
        st_word(dst, 8 * (WC + WR + lane), pack_double(v));
        st_word(clr, 8 * (WC + WR + lane), kSent);
      }
    } else if (tid < WC + WR) {
      st_word(clr, 8 * tid, kSent);
    }
    // Wave 7 (and 2) waits for everybody's word, as in an iteration: whoever has
    // it is done with the message before, which the next step clears.
    if (wave == kCtlWave || totals || (b == 0 && (wave == 3 || wave == 4))) {
      const int xl = lane >> xsh;
      const int nx = xcnt > xl ? (xcnt - xl + (kWave >> xsh) - 1) >> (6 - xsh) : 0;
      const uint32_t ox = 8 * (WC + WR + xw + (lane & xsh)) + (nx > 0 ? xl * xstep : 0);
      const int sx = xstep << (6 - xsh);
      u64 wx[4];
      double v = 0.0;
      res_load4(wx, cur, ox, sx, nx);
      if (!res_sum4(wx, cur, ox, sx, nx, v)) sh.dead = 1;
      if (wave == 3 || wave == 4) res_keep(sh.mon[seq & 1], wave, lane, v);
      else if (wave == kCtlWave && lane == 0) sh.stop_at = (int)v;
    }
    __syncthreads();
    ++seq;
  };
  for (;;) {  // from the saved state on: the iterations, and after a stop once more up to it
    const ResTeam* const t2 = fresh(tm);
    const int wl0 = fresh(wr0), nvl = fresh_lane(nv);
    {
      // X, then rho C.  Chunks of 16 bytes straight to registers where the
      // layout allows (a chunk that straddles column n stays inside the row's
      // leading dimension); else element by element through the staging area.
      const T* const X = uni(static_cast<const T*>(t2->a.X));
      const int64_t ldx = uni(t2->a.g.ldx);
      if (uni(t2->vec_x)) {
        const int jc = nvl > 0 ? jl : 0;
#pragma unroll
        for (int r = 0; r < RPW; ++r)
          load_chunk<T, VEC, false>(X + (int64_t)(wl0 + r < m ? wl0 + r : m - 1) * ldx + jc, xr[r]);
      } else {
#pragma unroll
        for (int g = 0; g < RPW / SR; ++g) {
#pragma unroll 4
          for (int u = 0; u < SR; ++u) {
            const int i = wl0 + g * SR + u < m ? wl0 + g * SR + u : m - 1;
#pragma unroll
            for (int e = 0; e < VEC; ++e)
              stage[u * W + e] = X[i * ldx + (e < nvl ? jl + e : 0)];
          }
#pragma unroll
          for (int u = 0; u < SR; ++u) load_chunk<T, VEC, false>(stage + u * W, xr[g * SR + u]);
        }
      }
      if (row0 + TR > m || col0 + W > n) {
#pragma unroll
        for (int r = 0; r < RPW; ++r)
#pragma unroll
          for (int e = 0; e < VEC; ++e) xr[r][e] = wl0 + r < m && e < nvl ? xr[r][e] : (T)0;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      // rho c outside the matrix: such entries stay 0
      const T kFar = std::is_same<T, float>::value ? (T)3e38f : (T)1e300;
      const int64_t ldc = uni(t2->a.g.ldc);
      const int wc0 = fresh(wr0), nvc = fresh_lane(nv);
      if (uni(t2->vec_c)) {
        const T* const C = uni(static_cast<const T*>(t2->a.C));
        const int jc = nvc > 0 ? jl : 0;
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
          T c[VEC];
          load_chunk<T, VEC, false>(C + (int64_t)(wc0 + r < m ? wc0 + r : m - 1) * ldc + jc, c);
#pragma unroll
          for (int e = 0; e < VEC; ++e)
            c[e] = wc0 + r < m && e < nvc ? mul_rounded<T>(rhoT, c[e]) : kFar;
          if (r < kHeld) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) pc[r < kHeld ? r : 0][e] = c[e];
          } else {
            store_chunk<T, VEC, false>(stage + (r - kHeld) * W, c);
          }
        }
      } else {
        const int kind = uni(t2->a.cost_kind), dim = uni(t2->a.dim);
        const float cscale = (float)st->cscale;
#pragma unroll
        for (int g = 0; g < RPW / SR; ++g) {
#pragma unroll 1
          for (int u0 = 0; u0 < SR; u0 += 4) {
            T c[4][VEC];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int64_t i = wc0 + g * SR + u0 + u < m ? wc0 + g * SR + u0 + u : m - 1;
#pragma unroll
              for (int e = 0; e < VEC; ++e) {
                const int64_t j = e < nvc ? jl + e : 0;
                if (kind == kCostDense) {
                  c[u][e] = static_cast<const T*>(t2->a.C)[i * ldc + j];
                } else if (kind == kCostBF16) {
                  c[u][e] = (T)__builtin_bit_cast(
                      float, (uint32_t)static_cast<const uint16_t*>(t2->a.C)[i * ldc + j] << 16);
                } else {
                  float s = 0.f;
                  for (int d = 0; d < dim; ++d) {
                    const float df = t2->a.xs[i * dim + d] - t2->a.xt[j * dim + d];
                    s += df * df;
                  }
                  c[u][e] = (T)(s * cscale);
                }
              }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
              for (int e = 0; e < VEC; ++e)
                stage[(u0 + u) * W + e] = wc0 + g * SR + u0 + u < m && e < nvc
                                              ? mul_rounded<T>(rhoT, c[u][e]) : kFar;
          }
          if (g * SR < kHeld) {
#pragma unroll
            for (int u = 0; u < SR; ++u)
              load_chunk<T, VEC, false>(stage + u * W, pc[g * SR < kHeld ? g * SR + u : 0]);
          }
        }
      }
    }
    if (base == 0) {
      accs[tid] = own_r ? t2->a.a[gid] : own_c ? t2->a.b[gid] : 0.0;
      if (is_row) rowsh[tid] = own_r ? static_cast<const T*>(t2->a.phiT)[gid] : (T)0;
      if (is_col) colsh[cc0] = own_c ? static_cast<const T*>(t2->a.psiT)[gid] : (T)0;
      if (tid == 0) {
        sh.base[0] = st->cphi;
        sh.base[1] = st->cpsi;
        sh.base[2] = st->alpha;
      }
    } else {
      const double* const v = saved();
      accs[tid] = v[0];
      if (is_row) rowsh[tid] = (T)v[1];
      if (is_col) colsh[cc0] = (T)v[1];
    }
    if (tid == 0) {
#pragma unroll
      for (int q = 0; q < 3; ++q) sh.bc[base & 3][q] = sh.base[q];
      sh.stop_at = 0;
    }
    if (tid < 2 * kResWaves) sh.esum[tid & 1][tid >> 1] = 0.0;
    if constexpr (kSplit) {
      if (wave < 4) {
        double ps[2] = {0.0, 0.0};
        if (own_r && tj == 0) split_sum((double)marg, split_magic(st->sum_p), ps);
        wave_sum_n(ps);
        if (lane == 0) sh.psum[0][wave] = ps[0], sh.psum[1][wave] = ps[1];
      }
    }
    __syncthreads();

    k = base;
    for (;;) {  // segments
      const int start = k;
      int end = limit;
      if (!replay) {
        const int64_t total = uni(sh.sv.iter) + k;
        const int len = total < seg0 ? seg0 : total < kResSaves[2] ? (int)total : kResSaves[2];
        if (limit - k > len) end = k + len;
      }
      while (k < end) {  // sweep iteration k + 1, exchange, steps 5-8
        const Msg cur = xch + (seq & 3) * phase;
        // Step 4 on the held entries, with the row and column sums of step 5
        // and the stopping-test sums.  Of a float32 problem a lane's column sums
        // are float32 over 8 rows (FINE: 4), its <rho C,X> and sum [t]_+^2 over
        // their 32 (16) entries, a row's sum over 4 entries and then, but for
        // FINE, over the wave; a tile's row and column sums are rounded once more
        // for their way to the other tiles (FINE: see there).  Every other sum
        // is float64.
        {
          const int lane = fresh_lane(tid) & (kWave - 1);
          const T shift = (T)(sh.bc[k & 3][0] + sh.bc[k & 3][1]);
          T* const held = cl + (wave * SR * kWave + lane) * VEC;
          T colv[VEC];
#pragma unroll
          for (int e = 0; e < VEC; ++e) colv[e] = colsh[lane * VEC + e];
          double cd[VEC], s0d = 0.0, s1d = 0.0, rtot[2] = {0.0, 0.0};
          const double magic = kSplit ? sh.magic : 0.0;
#pragma unroll
          for (int e = 0; e < VEC; ++e) cd[e] = 0.0;
#pragma unroll
          for (int g = 0; g < RPW / G; ++g) {
            T ca[VEC], s0 = (T)0, s1 = (T)0;
            RowSum rs[G];
#pragma unroll
            for (int u = 0; u < G; ++u) {
              const int r = g * G + u;
              const T rowv = rowsh[wave * RPW + r] + shift;
              T c[VEC];
              if (r < kHeld) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) c[e] = pc[r < kHeld ? r : 0][e];
              } else {
                load_chunk<T, VEC, false>(held + (r - kHeld) * W, c);
              }
              T rsum = (T)0;
#pragma unroll
              for (int e = 0; e < VEC; ++e) {
                const T t = rowv + colv[e] - c[e];
                const T tp = relu_of(t);
                s1 += tp * tp;
                const T x = relu_of(xr[r][e] + t);
                xr[r][e] = x;
                rsum = e == 0 ? x : rsum + x;
                ca[e] = u == 0 ? x : ca[e] + x;
                s0 += c[e] * x;
              }
              rs[u] = (RowSum)rsum;
            }
#pragma unroll
            for (int e = 0; e < VEC; ++e) cd[e] += (double)ca[e];
            s0d += (double)s0;
            s1d += (double)s1;
            const RowSum v = wave_fold(rs, lane);
            rowp[wave * RPW + g * G + lane / (kWave / G)] = v;  // its 64 / G lanes agree
            if constexpr (kSplit) split_sum((double)v, magic, rtot);
            else rtot[0] += (double)v;
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int e = 0; e < VEC; ++e) buf[wave * W + lane * VEC + e] = cd[e];
          // rtot holds G distinct values, each in 64 / G neighbouring lanes
#pragma unroll
          for (int h = 0; h < (kSplit ? 2 : 1); ++h) {
            if (G == 8) rtot[h] += dpp<0x128>(rtot[h]);
            rtot[h] += dpp<0x142, 0xA>(rtot[h]);
            rtot[h] += dpp<0x143, 0xC>(rtot[h]);
          }
          double sx = fold32(s0d, s1d);  // lanes < 32: s0, others: s1
          sx += dpp<0xB1>(sx);
          sx += dpp<0x4E>(sx);
          sx += dpp<0x141>(sx);
          sx += dpp<0x140>(sx);
          sx += dpp<0x142, 0xA>(sx);
          if (lane == 63) {
            sh.wsum[kRwTot][wave] = rtot[0];
            sh.wsum[kRwS1][wave] = sx;
            if (kSplit) sh.wsum[kRwLow][wave] = rtot[1];
          }
          if (lane == 31) sh.wsum[kRwS0][wave] = sx;
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();

        // Publish, then clear the words for the step after the next.
        double own[PW];
#pragma unroll
        for (int e = 0; e < PW; ++e) own[e] = 0.0;
        {
          const int t = fresh_lane(tid);
          const Msg dst = word_at(cur, 8 * b * MSG);
          const Msg clr = word_at(xch + ((seq + 2) & 3) * phase, 8 * b * MSG);
          if (wave < WC / kWave) {
            double v[PW];
            const double* const src = buf + (slim ? t : t * PW);
#pragma unroll
            for (int e = 0; e < PW; ++e) v[e] = src[e];
#pragma unroll
            for (int q = 1; q < kResWaves; ++q)
#pragma unroll
              for (int e = 0; e < PW; ++e) v[e] += src[q * W + e];
            if (lone)
#pragma unroll
              for (int e = 0; e < PW; ++e) own[e] = v[e];
            if (slim) {  // the column's sum as a float and what that leaves out
              const double rest = v[0] - (double)(float)v[0];
              v[PW - 1] = rest - rest == 0.0 ? rest : 0.0;
            }
            if constexpr (PW == 2) st_word(dst, 8 * t, Wd::pack((float)v[0], (float)v[PW - 1]));
            else st_word(dst, 8 * t, pack_double(v[0]));
            st_word(clr, 8 * t, kSent);
          } else if (wave == kResWaves - 1) {
            // the sum of eight (or four) LDS values from `src` on
            const int q = t & (kWave - 1);
            if (q < kRwCount) {
              const bool sums = q <= kRwLow;  // of the eight waves
              const double* src = sums ? sh.wsum[q] : &sh.esum[q & 1][q >= kRwS2 ? 4 : 0];
              double v = (src[0] + src[1]) + (src[2] + src[3]);
              if (sums) v += (src[4] + src[5]) + (src[6] + src[7]);
              if (kSplit && (q == kRwTot || q == kRwLow)) {
                const double* const ps = sh.psum[q == kRwLow];
                v -= (ps[0] + ps[1]) + (ps[2] + ps[3]);
              }
              if (q == kRwCtl) v = sh.ctl;
              st_word(dst, 8 * (WC + WR + q), pack_double(v));
              st_word(clr, 8 * (WC + WR + q), kSent);
            }
          } else if (t < WC + WR) {
            const int w = t - WC;
            if constexpr (kRows64) {
              const double v = rowp[w], rest = v - (double)(float)v;
              st_word(dst, 8 * t, Wd::pack((float)v, rest - rest == 0.0 ? (float)rest : 0.f));
            } else if constexpr (PW == 2) st_word(dst, 8 * t, Wd::pack(rowp[2 * w], rowp[2 * w + 1]));
            else st_word(dst, 8 * t, pack_double((double)rowp[w]));
            st_word(clr, 8 * t, kSent);
          }
        }
        __syncthreads();  // `buf` changes its use

        // While the peers' words are on their way: the test of iteration k - 1.
        // (A segment begins with both iterations before it tested.)
        if (b == 0 && wave == 6 && !replay && k > start)
          res_test(sh, sh.mon[(seq - 1) & 1], k - 1 > start ? k - 1 : 0, lane);

        // Read the peers' words.  All loads of a batch are in flight together,
        // and so are the repeats of those that came too early.
        bool fine = true;
        {
          const int t = fresh_lane(tid), nc = fresh(nc0);
          const int rsub = t / WR;
          const int nr = rsub < GR && rsub < S ? (S - rsub + GR - 1) / GR : 0;
          const uint32_t orow = 8 * ((nr > 0 ? rsub : 0) * MSG + t % WR);
          const int sc = 8 * GC * S * MSG, sr = 8 * GR * MSG;
          const Msg pcol = word_at(cur, ocol), prow = word_at(cur, 8 * (ti * S * MSG + WC));
          const uint32_t vcol = 8 * (t & (WC - 1));
          const int xl = (t & (kWave - 1)) >> xsh;  // which workgroup's word
          const int nx = xcnt > xl ? (xcnt - xl + (kWave >> xsh) - 1) >> (6 - xsh) : 0;
          const uint32_t ox = 8 * (WC + WR + xw + (t & xsh)) + (nx > 0 ? xl * xstep : 0);
          const int sx = xstep << (6 - xsh);
          double cs[PW], rsu[PW];
          u64 wx[4];
#pragma unroll
          for (int e = 0; e < PW; ++e) cs[e] = rsu[e] = 0.0;
          // wave 7's scalar step: everything but the total, ready beforehand
          double sum_p = 0.0, alpha = 0.0, dn = 0.0, dm = 0.0, inv[3] = {0.0, 0.0, 0.0};
          auto scalars = [&]() {
            sum_p = sh.sv.sum_p;
            alpha = sh.bc[k & 3][2];
            dn = (double)fresh_lane(n);
            dm = (double)fresh_lane(m);
#pragma unroll
            for (int q = 0; q < 3; ++q) inv[q] = sh.inv[q];
          };
          if (!kSplit && RPW <= 16 && wave == 7) scalars();
          if (extra) res_load4(wx, cur, ox, sx, nx);
          auto rounds = [&](int rc) { return rc > nqr ? rc : nqr; };
          if (RPW >= 24 || (R > 2 * GC && R <= 4 * GC))
            fine = res_read<T, 4, NR>(pcol, vcol, sc, nc, prow, orow, sr, nr, rounds((R + 4 * GC - 1) / (4 * GC)), cs, rsu);
          else if (R <= 2 * GC)
            fine = res_read<T, 2, NR>(pcol, vcol, sc, nc, prow, orow, sr, nr, rounds(1), cs, rsu);
          else
            fine = res_read<T, 8, NR>(pcol, vcol, sc, nc, prow, orow, sr, nr, rounds((R + 8 * GC - 1) / (8 * GC)), cs, rsu);
#pragma unroll
          for (int e = 0; e < PW; ++e) buf[t * PW + e] = lone ? own[e] : cs[e];  // [csub][column]
          if (t < GR * WR)
#pragma unroll
            for (int e = 0; e < PW; ++e) buf[GC * W + t * PW + e] = rsu[e];  // [rsub][row]
          if (extra) {
            double v = 0.0;
            if (fine) fine = res_sum4(wx, cur, ox, sx, nx, v);
            if (kSplit && totals) {
              v += dpp<0x4E>(v);   // even lanes the first words, odd lanes the second
              v += dpp<0x124>(v);  // row_ror:4
              v += dpp<0x128>(v);
              const double hi = (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
              const double lo = (read_lane(v, 1) + read_lane(v, 17)) + (read_lane(v, 33) + read_lane(v, 49));
              if (lane == 0) sh.total[wave == 2][0] = hi, sh.total[wave == 2][1] = lo;
            } else if (wave == 7) {
              v = wave_sum(v);
              if (RPW > 16) scalars();
              res_scalars(sh, k, lane, v - sum_p, alpha, dn, dm, inv);
            } else if (wave == kCtlWave) {
              if (lane == 0 && !replay) sh.stop_at = (int)v;
            } else if (wave >= 5) {
              sh.mon[seq & 1][wave - 5][lane] = v;
            } else {
              res_keep(sh.mon[seq & 1], wave, lane, v);
            }
          }
        }
        if (!fine) sh.dead = 1;
        __syncthreads();
        if (uni(sh.dead)) break;

        if (kSplit && wave == 7) {  // it has no columns; the next sweep is two barriers away
          double inv[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) inv[q] = sh.inv[q];
          res_scalars(sh, k, lane, (sh.total[0][0] + sh.total[1][0]) + (sh.total[0][1] + sh.total[1][1]), sh.bc[k & 3][2], (double)fresh_lane(n),
                      (double)fresh_lane(m), inv);
        }
        // Steps 5-8 of this tile's rows and columns.
        {
          const int tid = fresh_lane((int)threadIdx.x), cc0 = tid - 256;
          const bool is_row = tid < TR, is_col = cc0 >= 0 && cc0 < W;
          const int gid = is_row ? row0 + tid : col0 + cc0;
          const bool own_r = is_row && gid < m, own_c = is_col && gid < n;
          double tot = 0.0;
          if (is_row) {
            for (int q = 0; q < GR && q < S; q += 4) {
              // the peers' sums in order, zeros where there is no peer
#pragma unroll
              for (int u = 0; u < 4; ++u)
                if (q + u < GR) {
                  if constexpr (kRows64) {
                    const double* const v = buf + GC * W + ((q + u) * WR + tid) * 2;
                    tot += v[0] + v[1];
                  } else {
                    tot += buf[GC * W + (q + u) * TR + tid];
                  }
                }
            }
          } else if (is_col) {
#pragma unroll
            for (int q = 0; q < GC; ++q)
              tot += slim ? buf[q * W + 2 * (cc0 & (WC - 1))] + buf[q * W + 2 * (cc0 & (WC - 1)) + 1]
                          : buf[q * W + cc0];
          }
          double e[2] = {0.0, 0.0};
          if (own_r || own_c) {
            const double mg = (double)fresh_lane(marg), acc = accs[tid];
            const double res = tot - mg;
            const int len = is_row ? n : m;
            const double dual = div_by(acc - 2.0 * res, (double)fresh_lane(len), sh.inv[is_row ? 0 : 1]);
            accs[tid] = acc - res;
            if (is_row) rowsh[tid] = (T)dual;
            else colsh[cc0] = (T)dual;
            e[0] = res * res;
            e[1] = mg * dual;
            // phi~ and psi~ in full, of what may be the last iteration
            if (k + 1 == end) {
              const ResTeam* const t4 = fresh(tm);
              if (is_row && tj == 0) t4->a.phi64[gid] = dual;
              if (!is_row && ti == 0) t4->a.psi64[gid] = dual;
            }
          }
          __syncthreads();
          // The sums that the test needs, from the first tile column and row
          // (waves 0-3 hold rows, 4-7 columns).
          if (!replay && ((wave < 4 && tj == 0) || (wave >= 4 && ti == 0))) {
            double v = fold32(e[0], e[1]);  // lanes < 32: e[0], others: e[1]
            v += dpp<0xB1>(v);
            v += dpp<0x4E>(v);
            v += dpp<0x141>(v);
            v += dpp<0x140>(v);
            v += dpp<0x142, 0xA>(v);
            if (lane == 31) sh.esum[0][wave] = v;
            if (lane == 63) sh.esum[1][wave] = v;
          }
        }
        ++seq;
        ++k;
        if (uni(sh.stop_at) > 0) break;
      }
      if (uni(sh.dead) || replay || uni(sh.stop_at) > 0) break;
      // The end of a segment: an exchange for the last two tests.
      if (b == 0 && wave == 6)
        res_test(sh, sh.mon[(seq - 1) & 1], k - 1 > start ? k - 1 : 0, lane);
      exchange();
      if (uni(sh.dead) || uni(sh.stop_at) > 0) break;
      if (b == 0 && wave == 6)
        res_test(sh, sh.mon[(seq - 1) & 1], k, lane);
      if (k == limit) break;
      // Another one for the word that the launch goes on, and the state is saved.
      __syncthreads();  // every thread has read stop_at
      exchange();
      if (uni(sh.dead) || uni(sh.stop_at) > 0) break;
      store_x();
      double* const v = saved();
      v[0] = accs[tid];
      v[1] = is_row ? (double)rowsh[tid] : is_col ? (double)colsh[cc0] : 0.0;
      if (tid == 0)
#pragma unroll
        for (int q = 0; q < 3; ++q) sh.base[q] = sh.bc[k & 3][q];
      base = k;
    }
    const int stop = uni(sh.stop_at);
    if (uni(sh.dead) || replay || stop == 0 || stop == k) break;
    limit = stop;
    replay = true;
    __syncthreads();  // every thread has read stop_at
  }
  if (uni(sh.dead)) {  // a peer never published: report instead of hanging
    if (tid == 0) {
      st->done = 1;
      st->status = -5;
    }
    return;
  }

  // Write back X, the vectors and the state.
  store_x();
  const ResTeam* const t3 = fresh(tm);
  if (own_r && tj == 0) {
    t3->a.a[gid] = accs[tid];
    static_cast<T*>(t3->a.phiT)[gid] = rowsh[tid];
  }
  if (own_c && ti == 0) {
    t3->a.b[gid] = accs[tid];
    static_cast<T*>(t3->a.psiT)[gid] = colsh[cc0];
  }
  if (b == 0 && tid == 6 * kWave) {
    const uint64_t now = wall_clock64();
    t3->sync->seq = (uint32_t)seq;
    res_clear(t3->sync);  // everybody is past the gate: their messages have been read
    st->cphi = sh.bc[k & 3][0];
    st->cpsi = sh.bc[k & 3][1];
    st->alpha = sh.bc[k & 3][2];
    st->iter = sh.sv.iter + k;
    if (replay) st->repeated += (uint32_t)(k - base);
    st->t_last = now;
    st->pobj = sh.rec[0];
    st->dobj = sh.rec[1];
    st->rp = sh.rec[2];
    st->rd = sh.rec[3];
    st->gap = sh.rec[4];
    st->test = sh.rec[5];
    if (sh.rec_done) {
      st->done = 1;
      st->status = sh.rec_status;
      st->stop_iter = sh.sv.iter + sh.rec_k;
      st->t_stop = now;
    }
  }
}

// Plans with few rows (one row of the smallest tiles) or columns (half a tile's).
inline bool resident_fine(int64_t m, int64_t n) {
  return m <= kResWaves * kResRpw[0] || n <= kResBlock / 4;
}

template <typename T, bool FINE>
const void* resident_entry(int rpw) {
  switch (rpw) {
    case 4: return reinterpret_cast<const void*>(&resident_kernel<T, 4, 0, FINE>);
    case 8: return reinterpret_cast<const void*>(&resident_kernel<T, 8, 0, FINE>);
    case 16: return reinterpret_cast<const void*>(&resident_kernel<T, 16, 0, FINE>);
    case 24: return reinterpret_cast<const void*>(&resident_kernel<T, 24, 0, FINE>);
    case 32: return reinterpret_cast<const void*>(&resident_kernel<T, 32, 16, FINE>);
  }
  return nullptr;
}

// Launch `blocks` workgroups of teams with `rpw` rows per wave.  Cooperative:
// the workgroups wait for each other, so they have to be on the chip together.
// `fine`: one of them has a plan that resident_fine() names.
hipError_t launch_resident(int dtype, int rpw, bool fine, const ResTeam* teams, const uint2* map,
                           int blocks, int64_t iters, int gate_polls, hipStream_t s) {
  const void* f = dtype != 0 ? resident_entry<double, false>(rpw)
                  : fine     ? resident_entry<float, true>(rpw)
                             : resident_entry<float, false>(rpw);
  if (!f || blocks < 1) return hipErrorInvalidValue;
  void* args[] = {(void*)&teams, (void*)&map, (void*)&iters, (void*)&gate_polls};
  return hipLaunchCooperativeKernel(f, dim3((unsigned)blocks), dim3(kResBlock), args, 0, s);
}

// A process's first cooperative launch sets up a queue, loads these kernels and
// takes their scratch memory, 17 ms in all: an empty launch pays for it when a
// context is made, not the first solve.  False where there are none.
bool resident_warm(int blocks, hipStream_t s) {
  for (int dtype = 0; dtype < 2; ++dtype)
    if (launch_resident(dtype, kResRpw[4], false, nullptr, nullptr, blocks, 0, 0, s) != hipSuccess)
      return false;
  return hipStreamSynchronize(s) == hipSuccess;
}

}  // namespace
}  // namespace drot
