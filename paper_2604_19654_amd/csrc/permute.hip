// Permute: group the rank's token rows by static / dynamic expert group
// (paper Section 2.2 Phase 1: tokens are permuted by expert where they will be
// computed; Section 2.3: static vs dynamic experts).
//
// The row order is fully determined (groups in table order, ascending flat
// assignment inside a group), so no atomics may decide a row position.  It is a
// stable counting sort over the flat assignments a = t*k + j.  A workgroup owns a
// run of them, a wavefront of it a shorter run:
//   - per expert, the occurrences ahead of the run and in all of the batch, from
//     one of three sources (below); inside the run LDS histograms per wavefront
//   - sizes of the ordinal windows -> offsets[G+1], and per-expert chains of groups
//   - each wavefront walks its run 64 assignments at a time; the ordinal inside the
//     slice comes from a ballot-based match of equal experts, the running ordinal
//     per expert lives in LDS; the window that contains the ordinal gives the row
// Where the occurrences outside the run come from:
//   COUNTED  every workgroup counts the whole batch for itself: one launch
//   TABLE    chunk_hist has written every run's histogram, every workgroup adds them up
//   SCANNED  chunk_scan has turned the histograms into prefix sums (large batches, many experts)
// gather_rows: Xp[r,:] = X[row_src[r] / k, :], one wavefront per row, 16-byte lanes
// (pure HBM traffic: 2*R*d*2 bytes)
#include "common.h"

namespace {

constexpr int WAVES = 4;             // wavefronts per block of chunk_scan
constexpr int BLOCK = WAVES * 64;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct GroupTable {
  feplb_group g[FEPLB_MAX_GROUPS];
};

// LDS histograms that a whole workgroup adds to come in copies, one for each residue of the lane: the lanes of a wavefront
// hold neighbouring assignments, and a popular expert is in many of them.
constexpr int RUN_MAX_E = 512;   // 16 histograms, the copies and the tables in 64 KB of LDS; above it half as many wavefronts, no copies
constexpr int copies_for(int E) { return E <= RUN_MAX_E ? 4 : 1; }

constexpr int HIST_THREADS = 1024;
__global__ __launch_bounds__(HIST_THREADS) void chunk_hist_kernel(const int* __restrict__ ids, long long A, int E, int chunk,
                                                                  int* __restrict__ chunk_hist) {
  extern __shared__ int lds[];
  const int copies = copies_for(E), mine = threadIdx.x % copies * E;
  for (int i = threadIdx.x; i < copies * E; i += HIST_THREADS) lds[i] = 0;
  __syncthreads();
  const long long a0 = (long long)blockIdx.x * chunk;
  const int n = (int)min((long long)chunk, A - a0);
  for (int i = threadIdx.x; i < n; i += HIST_THREADS) {
    const int e = ids[a0 + i];
    if ((unsigned)e < (unsigned)E) atomicAdd(&lds[mine + e], 1);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += HIST_THREADS) {
    int v = 0;
    for (int c = 0; c < copies; ++c) v += lds[c * E + e];
    chunk_hist[(long long)blockIdx.x * E + e] = v;
  }
}

// One wavefront per expert; lane l owns a contiguous run of chunks.
__global__ __launch_bounds__(BLOCK) void chunk_scan_kernel(int* __restrict__ chunk_hist, int E,
                                                           int nchunks, int* __restrict__ total) {
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int e = blockIdx.x * WAVES + wave;
  if (e >= E) return;
  const int per = (nchunks + 63) / 64;
  const int c0 = lane * per;
  const int c1 = min(c0 + per, nchunks);
  int sum = 0;
  for (int c = c0; c < c1; ++c) sum += chunk_hist[(long long)c * E + e];
  int incl = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(incl, d, 64);
    if (lane >= d) incl += o;
  }
  int run = incl - sum;
  for (int c = c0; c < c1; ++c) {
    const int v = chunk_hist[(long long)c * E + e];
    chunk_hist[(long long)c * E + e] = run;
    run += v;
  }
  if (lane == 63) total[e] = incl;
}

// LDS tables of the groups: the groups of expert e are the chain head[e], next[.] in table order (end: G or more)
struct GroupTables {
  int *head, *next, *lo, *hi, *start, *sums;   // [E], 4 x [G], [2]; row = start + ordinal
  static __host__ __device__ int ints(int E, int G) { return E + 4 * G + 2; }
  __device__ GroupTables(int* lds, int E, int G)
      : head(lds), next(head + E), lo(next + G), hi(lo + G), start(hi + G), sums(start + G) {}
};

// Made by every workgroup for itself, by all its threads (at least FEPLB_MAX_GROUPS): in a launch of its own the
// tables cost a launch and a trip through memory, and one thread linked the chains (the whole permutation inside a graph:
// T = 8192, k = 8, G = 16 18.1 -> 14.8 us; T = 32768, G = 32 30.8 -> 25.7 us).  total[e]: occurrences of expert e; base: first row; offsets: written if given.
__device__ __forceinline__ void make_group_tables(const GroupTable& tab, int G, int E, const int* total, int base,
                                                  const GroupTables& t, int* offsets, bool append) {
  static_assert(FEPLB_MAX_GROUPS == 128, "one group per thread of two wavefronts");
  const int g = threadIdx.x, lane = g % 64;
  for (int i = g; i < E; i += blockDim.x) t.head[i] = G;
  int lo = 0, hi = 0, e = -1, size = 0;
  if (g < G) {
    e = tab.g[g].expert;
    lo = tab.g[g].ord_lo;
    hi = tab.g[g].ord_hi;
    const int n = total[e];   // the host has checked every e
    size = max(0, min(hi, n) - min(lo, n));
  }
  int incl = size;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(incl, d, 64);
    if (lane >= d) incl += o;
  }
  if (g < FEPLB_MAX_GROUPS && lane == 63) t.sums[g / 64] = incl;
  __syncthreads();
  if (g < G) {
    const int end = base + incl + (g >= 64 ? t.sums[0] : 0), off = end - size;
    t.lo[g] = lo;
    t.hi[g] = hi;
    t.start[g] = off - lo;
    atomicMin(&t.head[e], g);
    int next = G;
    for (int h = G - 1; h >= 0; --h)
      if (h > g && tab.g[h].expert == e) next = h;
    t.next[g] = next;
    if (offsets) {
      if (g > 0 || !append) offsets[g] = off;   // appending: offsets[0] is the base, it stays
      if (g == G - 1) offsets[G] = end;
    }
  }
  if (G == 0 && g == 0 && offsets && !append) offsets[0] = base;
  __syncthreads();
}

// rows of 64 consecutive assignments, one per lane (e < 0: none); run[e]: the wavefront's next ordinal of expert e
__device__ __forceinline__ int next_row(int e, int nbits, int G, volatile int* run, const GroupTables& t) {
  const int lane = threadIdx.x % 64;
  const bool valid = e >= 0;
  unsigned long long same = __ballot(valid);
  for (int b = 0; b < nbits; ++b) {
    const bool bit = (e >> b) & 1;
    const unsigned long long m = __ballot(bit);
    same &= bit ? m : ~m;
  }
  int row = -1;
  if (valid) {
    const int base = run[e];
    const int o = base + __popcll(same & ((1ull << lane) - 1ull));
    if ((same >> lane) == 1ull) run[e] = base + __popcll(same);  // highest lane of the set
    for (int g = t.head[e]; g < G; g = t.next[g])
      if (o >= t.lo[g] && o < t.hi[g]) {
        row = t.start[g] + o;
        break;
      }
  }
  __builtin_amdgcn_wave_barrier();
  return row;
}

__device__ __forceinline__ int bits_for(int E) { return E > 1 ? 32 - __builtin_clz(E - 1) : 0; }

enum Source { COUNTED, TABLE, SCANNED };

// Measured inside a graph, E = 128 unless said otherwise, 16 local experts (three launches, runs of 256 or 1024 assignments and bases
// from a scan, as before all of this: 12.0 us at 8192 assignments, 14.7 at 65536, 24.4 at 262144, 38.7 at 1048576):
//   counting the batch in every workgroup (8192: 6.9 us; 16384: 8.5; E = 1024 11.7; 49728, E = 128: 14.6) against a table of histograms by
//   a launch of its own (16392: 8.7; E = 1024 12.4; 49728: 9.8): the line lies between 10004 and 49728.  Above RUN_MAX_E experts there is
//   one copy of a workgroup's histogram, and a batch that is all one expert adds to one word of it, lane by lane: E = 600, 16384
//   assignments 11.4 us drawn evenly, 12.5 half of them one expert, 19.2 all; from scanned bases 11.0, 11.2 and 11.3 (10240: 9.1, 9.8 and 13.9,
//   scanned 10.9 to 11.4): the line lies at 10240;
//   runs of 1024 against 4096 assignments: 11.0 against 13.8 us at 262144, where there are 256 or 64 workgroups to walk them;
//   at 1048576 runs of 4096 take 18.4 us (from scanned bases).
// Every workgroup reads the whole table, runs x E words, which saves the launch of the scan until reading takes longer.  Table against
// scan, us: in runs of 1024, 32768 words (E = 128, 262144) 11.0 and 12.9, 49152 words (E = 256, 196608) 12.4 and 12.8, 65536 words (E = 256,
// 262144) 14.0 and 13.8, 131072 words (E = 512, 262144) 19.8 and 14.8; in runs of 4096, 4096 words (E = 64, 262152) 12.3 and 13.7, 8320
// words (E = 128) 13.8 and 13.9, 16640 words (E = 256) 16.4 and 14.3, 262144 words (E = 512, 2097152) 126 and 33.  Above RUN_MAX_E experts a
// workgroup has half as many threads for longer rows, and the scan is ahead everywhere (16392, E = 520: 11.1 and 10.8; 1048576,
// E = 1024: 271 and 28).
constexpr long long SHORT_RUNS_MAX = 262144, COUNTED_MAX = 16384, COUNTED_MAX_ONE_COPY = 10240, TABLE_WORDS_SHORT = 49152, TABLE_WORDS_LONG = 8192;

// in_place: the rows replace the assignments (inv == topk_ids).  A workgroup that counts the batch reads other runs' assignments, which
// those replace meanwhile; the other sources read them in launches ahead, and each run's own before its rows are written.
Source pick_source(long long A, int E, long long runs, bool short_runs, bool in_place) {
  if (A <= (copies_for(E) > 1 ? COUNTED_MAX : COUNTED_MAX_ONE_COPY) && (runs == 1 || !in_place)) return COUNTED;
  return E <= RUN_MAX_E && runs * E <= (short_runs ? TABLE_WORDS_SHORT : TABLE_WORDS_LONG) ? TABLE : SCANNED;
}

// LDS: run[RUN_WAVES][E] | before[copies][E] | after[copies][E] | total[E] | group tables
size_t permute_lds_bytes(int waves, int E, int G) {
  return ((size_t)(waves + 2 * copies_for(E) + 1) * E + GroupTables::ints(E, G)) * sizeof(int);
}

// A workgroup owns RUN_WAVES * 64 * SLICES assignments; they stay in registers between the counting and the walk, which takes
// about 0.9 us per slice.
template <int RUN_WAVES, int SLICES>
__global__ __launch_bounds__(RUN_WAVES * 64) void permute_kernel(GroupTable tab, const int* ids, long long A, int E, int G,
                                                                 int nchunks, int source, const int* __restrict__ chunk_hist,
                                                                 const int* __restrict__ totals, int R_cap, int* offsets,
                                                                 int* __restrict__ row_src, int* inv, int append) {
  extern __shared__ int lds[];
  constexpr int THREADS = RUN_WAVES * 64;
  constexpr int COPIES = copies_for(RUN_WAVES == 16 ? RUN_MAX_E : RUN_MAX_E + 1);
  const bool alone = gridDim.x == 1;   // nothing outside the only run
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  int* const before = lds + RUN_WAVES * E;
  int* const after = before + COPIES * E;
  int* const total = after + COPIES * E;
  const GroupTables t(total + E, E, G);
  const int c = blockIdx.x;
  const long long run0 = (long long)c * (THREADS * SLICES);
  const long long a0 = run0 + wave * (64 * SLICES);
  int e[SLICES];
#pragma unroll
  for (int i = 0; i < SLICES; ++i) {
    const long long a = a0 + i * 64 + lane;
    e[i] = a < A ? ids[a] : -1;
    if ((unsigned)e[i] >= (unsigned)E) e[i] = -1;
  }
  const int base = append ? offsets[0] : 0;   // offsets[0] is not written when appending
  for (int i = threadIdx.x; i < (RUN_WAVES + (alone ? 0 : 2 * COPIES)) * E; i += THREADS) lds[i] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < SLICES; ++i)
    if (e[i] >= 0) atomicAdd(&lds[wave * E + e[i]], 1);
  if (alone) {
  } else if (source == COUNTED) {
    const int n = (int)A, mine = lane % COPIES * E;
    for (int i = threadIdx.x; i < n; i += THREADS) {
      if (i >= run0 && i < run0 + THREADS * SLICES) continue;   // (whole slices of the loop: the run is a multiple of THREADS)
      const int x = ids[i];
      if ((unsigned)x < (unsigned)E) atomicAdd((i < run0 ? before : after) + mine + x, 1);
    }
  } else if (source == TABLE) {
    const int rows = max(1, THREADS / E);   // rows of the table in work at a time
    for (int x = threadIdx.x; x < rows * E; x += THREADS) {
      const int ex = x % E;
      int nb = 0, na = 0;
#pragma unroll 8
      for (int r = x / E; r < nchunks; r += rows) {
        const int v = chunk_hist[(long long)r * E + ex];
        nb += r < c ? v : 0;
        na += r > c ? v : 0;
      }
      atomicAdd(&before[ex], nb);
      atomicAdd(&after[ex], na);
    }
  } else {
    for (int x = threadIdx.x; x < E; x += THREADS) before[x] = chunk_hist[(long long)c * E + x];
  }
  __syncthreads();
  for (int x = threadIdx.x; x < E; x += THREADS) {
    int sum = 0, rest = 0;
    if (!alone) {
#pragma unroll
      for (int i = 0; i < COPIES; ++i) {
        sum += before[i * E + x];
        rest += after[i * E + x];
      }
    }
    int n[RUN_WAVES];
#pragma unroll
    for (int w = 0; w < RUN_WAVES; ++w) n[w] = lds[w * E + x];
#pragma unroll
    for (int w = 0; w < RUN_WAVES; ++w) {
      lds[w * E + x] = sum;
      sum += n[w];
    }
    total[x] = source == SCANNED ? totals[x] : sum + rest;
  }
  __syncthreads();
  // appending: the rows of these groups follow those of an earlier call, whose end is offsets[0]
  make_group_tables(tab, G, E, total, base, t, c == 0 ? offsets : nullptr, append);
  const int nbits = bits_for(E);
#pragma unroll
  for (int i = 0; i < SLICES; ++i) {
    const long long a = a0 + i * 64 + lane;
    if (a - lane >= A) break;   // uniform across the wave
    const int row = next_row(e[i], nbits, G, lds + wave * E, t);
    if (a < A) {
      if (!append || row >= 0) inv[a] = row;   // appending leaves the other calls' entries alone
      if (row >= 0 && row < R_cap) row_src[row] = (int)a;
    }
  }
}

// One wavefront per row and per workgroup: measured against 2, 4 and 8 rows per workgroup at
// d = 6144, single-wave workgroups copy 2 % faster (5.60 against 5.48 TB/s).
template <int UNROLL>
__global__ __launch_bounds__(64) void gather_rows_kernel(const u32x4* __restrict__ X,
                                                            const int* __restrict__ row_src,
                                                            const int* __restrict__ offsets, int G,
                                                            int k, int nvec, int R_cap,
                                                            u32x4* __restrict__ Xp) {
  const int lane = threadIdx.x;
  const long long r = blockIdx.x;
  const int R = min(offsets[G], R_cap);
  if (r < offsets[0] || r >= R) return;   // offsets[0] > 0 only for an appending call
  const long long t = row_src[r] / k;
  const u32x4* src = X + t * nvec;
  u32x4* dst = Xp + r * nvec;
  for (int v0 = 0; v0 < nvec; v0 += 64 * UNROLL) {
    u32x4 p[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int v = v0 + u * 64 + lane;
      if (v < nvec) p[u] = __builtin_nontemporal_load(src + v);
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int v = v0 + u * 64 + lane;
      if (v < nvec) {
        __builtin_nontemporal_store(p[u], dst + v);   // written once, read by a later kernel
      }
    }
  }
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct Layout {
  size_t hist_off, total_off, bytes;
};

// Callers size and share workspaces by this formula: a histogram for every 256 assignments (1024 in larger batches), the totals and
// group tables, which the kernels have made in LDS since.  The runs are at least as long.
Layout layout(long long A, int E, int G) {
  Layout L;
  const int unit = A <= (1ll << 18) ? 256 : 1024;
  const long long units = (A + unit - 1) / unit;
  size_t off = 0;
  L.hist_off = off;
  off = align_up(off + (size_t)(units > 0 ? units : 1) * E * sizeof(int), 256);
  L.total_off = off;
  off = align_up(off + (size_t)E * sizeof(int), 256);
  off = align_up(off + ((size_t)E + 4 * (size_t)(G > 0 ? G : 1)) * sizeof(int), 256);
  L.bytes = off;
  return L;
}

}  // namespace

extern "C" size_t feplb_permute_workspace_bytes(int32_t T, int32_t k, int32_t E, int32_t G) {
  if (T < 0 || k < 1 || E < 1 || G < 0) return 0;
  return layout((long long)T * k, E, G).bytes;
}

namespace {
int32_t permute_impl(const int32_t* topk_ids, int32_t T, int32_t k, int32_t E,
                     const feplb_group* groups, int32_t G, const void* X, int32_t d,
                     void* Xp, int32_t R_cap, int32_t* offsets, int32_t* row_src,
                     int32_t* inv, void* ws, size_t ws_bytes, void* stream, int append) {
  FEPLB_REQUIRE(T >= 0 && k >= 1 && E >= 1 && G >= 0 && R_cap >= 0 && d >= 0, FEPLB_EINVAL,
                "permute: negative size");
  FEPLB_REQUIRE(E <= FEPLB_MAX_EXPERTS && G <= FEPLB_MAX_GROUPS && k <= FEPLB_MAX_TOPK,
                FEPLB_ESHAPE, "permute: E=%d G=%d k=%d above the limits", E, G, k);
  const long long A = (long long)T * k;
  FEPLB_REQUIRE(A < (1ll << 31), FEPLB_ESHAPE, "permute: T*k does not fit int32");
  FEPLB_REQUIRE(offsets, FEPLB_EINVAL, "permute: null offsets");
  FEPLB_REQUIRE(groups || G == 0, FEPLB_EINVAL, "permute: null groups");
  FEPLB_REQUIRE((topk_ids && inv) || A == 0, FEPLB_EINVAL, "permute: null ids/inv");
  FEPLB_REQUIRE(row_src || R_cap == 0, FEPLB_EINVAL, "permute: null row_src");
  FEPLB_REQUIRE(X || !Xp || A == 0 || d == 0, FEPLB_EINVAL, "permute: Xp given without X");
  if (X && Xp) {
    FEPLB_REQUIRE(d % 8 == 0, FEPLB_ESHAPE, "permute: d=%d not a multiple of 8", d);
    FEPLB_REQUIRE(feplb::aligned16(X) && feplb::aligned16(Xp), FEPLB_EALIGN,
                  "permute: X/Xp not 16-byte aligned");
  }
  GroupTable tab;
  for (int g = 0; g < G; ++g) {
    FEPLB_REQUIRE(groups[g].ord_lo >= 0 && groups[g].ord_hi >= groups[g].ord_lo, FEPLB_EINVAL,
                  "permute: group %d has window [%d,%d)", g, groups[g].ord_lo, groups[g].ord_hi);
    FEPLB_REQUIRE(groups[g].expert >= 0 && groups[g].expert < E, FEPLB_EINVAL,
                  "permute: group %d names expert %d", g, groups[g].expert);
    for (int h = 0; h < g; ++h)
      if (groups[h].expert == groups[g].expert) {
        const bool apart =
            groups[h].ord_hi <= groups[g].ord_lo || groups[g].ord_hi <= groups[h].ord_lo;
        FEPLB_REQUIRE(apart, FEPLB_EINVAL, "permute: groups %d and %d overlap on expert %d", h, g,
                      groups[g].expert);
      }
    tab.g[g] = groups[g];
  }
  const Layout L = layout(A, E, G);
  FEPLB_REQUIRE(ws && ws_bytes >= L.bytes, FEPLB_EWORKSPACE, "permute: workspace %zu < %zu",
                ws_bytes, L.bytes);
  FEPLB_REQUIRE(feplb::aligned16(ws), FEPLB_EALIGN, "permute: workspace not 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  char* base = (char*)ws;
  int* hist = (int*)(base + L.hist_off);
  int* total = (int*)(base + L.total_off);
  const int waves = E <= RUN_MAX_E ? 16 : 8;
  const bool short_runs = A <= SHORT_RUNS_MAX;
  const int chunk = waves * 64 * (short_runs ? 1 : 4);
  const long long runs = A > 0 ? (A + chunk - 1) / chunk : 1;   // none: the offsets alone
  const Source source = pick_source(A, E, runs, short_runs, inv == topk_ids);
  if (source != COUNTED) {
    hipLaunchKernelGGL(chunk_hist_kernel, dim3((unsigned)runs), dim3(HIST_THREADS), (size_t)copies_for(E) * E * sizeof(int), s, topk_ids, A, E,
                       chunk, hist);
    FEPLB_LAUNCH_CHECK("chunk_hist_kernel");
  }
  if (source == SCANNED) {
    hipLaunchKernelGGL(chunk_scan_kernel, dim3((E + WAVES - 1) / WAVES), dim3(BLOCK), 0, s, hist, E, (int)runs, total);
    FEPLB_LAUNCH_CHECK("chunk_scan_kernel");
  }
#define FEPLB_PERMUTE(W, S)                                                                                                     \
  hipLaunchKernelGGL((permute_kernel<W, S>), dim3((unsigned)runs), dim3(W * 64), permute_lds_bytes(W, E, G), s, tab, topk_ids, A, E, G, \
                     (int)runs, source, hist, total, R_cap, offsets, row_src, inv, append)
  if (waves == 16) {
    if (short_runs) FEPLB_PERMUTE(16, 1);
    else FEPLB_PERMUTE(16, 4);
  } else {
    if (short_runs) FEPLB_PERMUTE(8, 1);
    else FEPLB_PERMUTE(8, 4);
  }
#undef FEPLB_PERMUTE
  FEPLB_LAUNCH_CHECK("permute_kernel");
  if (X && Xp && R_cap > 0 && d > 0) {
    hipLaunchKernelGGL((gather_rows_kernel<4>), dim3(R_cap), dim3(64), 0, s, (const u32x4*)X,
                       row_src, offsets, G, k, d / 8, R_cap, (u32x4*)Xp);
    FEPLB_LAUNCH_CHECK("gather_rows_kernel");
  }
  return FEPLB_OK;
}
}  // namespace

extern "C" int32_t feplb_permute(const int32_t* topk_ids, int32_t T, int32_t k, int32_t E,
                                 const feplb_group* groups, int32_t G, const void* X, int32_t d,
                                 void* Xp, int32_t R_cap, int32_t* offsets, int32_t* row_src,
                                 int32_t* inv, void* ws, size_t ws_bytes, void* stream) {
  return permute_impl(topk_ids, T, k, E, groups, G, X, d, Xp, R_cap, offsets, row_src, inv, ws,
                      ws_bytes, stream, 0);
}

extern "C" int32_t feplb_permute_append(const int32_t* topk_ids, int32_t T, int32_t k, int32_t E,
                                        const feplb_group* groups, int32_t G, const void* X,
                                        int32_t d, void* Xp, int32_t R_cap, int32_t* offsets,
                                        int32_t* row_src, int32_t* inv, void* ws, size_t ws_bytes,
                                        void* stream) {
  return permute_impl(topk_ids, T, k, E, groups, G, X, d, Xp, R_cap, offsets, row_src, inv, ws,
                      ws_bytes, stream, 1);
}

