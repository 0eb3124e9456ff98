// Permute: group the rank's token rows by static / dynamic expert group
// (paper Section 2.2 Phase 1: tokens are permuted by expert where they will be
// computed; Section 2.3: static vs dynamic experts).
//
// The row order is fully determined (groups in table order, ascending flat
// assignment inside a group), so no atomics may decide a row position.  It is a
// stable counting sort over the flat assignments a = t*k + j, split in chunks
// of 256 or 1024 assignments (by batch size), one wavefront per chunk:
//   1. chunk_hist : per-chunk, per-expert counts (LDS histogram per wave)
//   2. chunk_scan : per expert, exclusive prefix over chunks -> the ordinal of
//                   the first occurrence in each chunk, and the expert's total
//   3. assign_rows: sizes of the ordinal windows -> offsets[G+1], and per-expert
//                   chains of groups; then per chunk, walk 64 assignments at a
//                   time; the ordinal inside the slice comes from a ballot-based
//                   match of equal experts, the running ordinal per expert lives
//                   in LDS; the window that contains the ordinal gives the row
// (small batches: all three in one workgroup, permute_one_kernel)
//   4. gather_rows: Xp[r,:] = X[row_src[r] / k, :], one wavefront per row,
//                   16-byte lanes (pure HBM traffic: 2*R*d*2 bytes)
#include "common.h"

namespace {

// assignments per wavefront: small batches get shorter chunks, i.e. more wavefronts for the
// serial walk of assign_rows (a multiple of 64 either way)
int chunk_for(long long A) { return A <= (1ll << 18) ? 256 : 1024; }
constexpr int WAVES = 4;             // wavefronts per block
constexpr int BLOCK = WAVES * 64;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct GroupTable {
  feplb_group g[FEPLB_MAX_GROUPS];
};

__global__ __launch_bounds__(BLOCK) void chunk_hist_kernel(const int* __restrict__ ids,
                                                           long long A, int E, int nchunks, int chunk,
                                                           int* __restrict__ chunk_hist) {
  extern __shared__ int lds[];
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  int* h = lds + wave * E;
  const int c = blockIdx.x * WAVES + wave;
  for (int e = lane; e < E; e += 64) h[e] = 0;
  __builtin_amdgcn_wave_barrier();
  if (c < nchunks) {
    const long long a0 = (long long)c * chunk;
    for (int i = lane; i < chunk; i += 64) {
      const long long a = a0 + i;
      if (a < A) {
        const int e = ids[a];
        if ((unsigned)e < (unsigned)E) atomicAdd(&h[e], 1);
      }
    }
  }
  __syncthreads();
  if (c < nchunks)
    for (int e = lane; e < E; e += 64) chunk_hist[(long long)c * E + e] = h[e];
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

__global__ __launch_bounds__(BLOCK) void assign_rows_kernel(
    GroupTable tab, const int* __restrict__ ids, long long A, int E, int G, int nchunks, int chunk,
    const int* __restrict__ chunk_base, const int* __restrict__ total, int R_cap, int* offsets,
    int* __restrict__ row_src, int* __restrict__ inv, int append) {
  extern __shared__ int lds[];
  // LDS: run[WAVES][E] | group tables
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int c = blockIdx.x * WAVES + wave;
  volatile int* run = lds + wave * E;
  if (c < nchunks)
    for (int e = lane; e < E; e += 64) run[e] = chunk_base[(long long)c * E + e];
  const GroupTables t(lds + WAVES * E, E, G);
  // appending: the rows of these groups follow those of an earlier call, whose end is offsets[0]
  make_group_tables(tab, G, E, total, append ? offsets[0] : 0, t, blockIdx.x == 0 ? offsets : nullptr, append);
  if (c >= nchunks) return;
  const int nbits = bits_for(E);
  const long long a0 = (long long)c * chunk;
  for (int i = 0; i < chunk; i += 64) {
    const long long a = a0 + i + lane;
    if (a0 + i >= A) break;  // uniform across the wave
    int e = -1;
    if (a < A) {
      e = ids[a];
      if ((unsigned)e >= (unsigned)E) e = -1;
    }
    const int row = next_row(e, nbits, G, run, t);
    if (a < A) {
      if (!append || row >= 0) inv[a] = row;   // appending leaves the other calls' entries alone
      if (row >= 0 && row < R_cap) row_src[row] = (int)a;
    }
  }
}

// All of it in one workgroup, for batches of at most ONE_WAVES * 64 * SLICES assignments: wavefront w owns a run of
// 64 SLICES assignments, kept in registers between the counting and the walk, so the batch is read once and the
// histograms and bases never leave LDS.  Bound by latency: the walk takes about 0.9 us
// per slice.  Inside a graph, against the launches one after the other: T = 96, k = 8, E = 128 14.3 -> 4.8 us;
// T = 512, k = 2, E = 8 12.2 -> 4.3 us; T = 512, k = 8, E = 128 15.1 -> 7.9 us.
constexpr int ONE_WAVES = 16;
constexpr int ONE_MAX_E = 512;       // 16 histograms, the totals and the tables in 64 KB of LDS
constexpr int ONE_MAX_A = ONE_WAVES * 64 * 4;
template <int SLICES>
__global__ __launch_bounds__(ONE_WAVES * 64) void permute_one_kernel(GroupTable tab, const int* __restrict__ ids, int A,
                                                                     int E, int G, int R_cap, int* offsets,
                                                                     int* __restrict__ row_src, int* __restrict__ inv,
                                                                     int append) {
  extern __shared__ int lds[];
  // LDS: run[ONE_WAVES][E] | total[E] | group tables
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  int* const total = lds + ONE_WAVES * E;
  const GroupTables t(total + E, E, G);
  const int a0 = wave * (64 * SLICES) + lane;
  int e[SLICES];
#pragma unroll
  for (int i = 0; i < SLICES; ++i) {
    const int a = a0 + i * 64;
    e[i] = a < A ? ids[a] : -1;
    if ((unsigned)e[i] >= (unsigned)E) e[i] = -1;
  }
  const int base = append ? offsets[0] : 0;   // offsets[0] is not written when appending
  for (int i = threadIdx.x; i < ONE_WAVES * E; i += ONE_WAVES * 64) lds[i] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < SLICES; ++i)
    if (e[i] >= 0) atomicAdd(&lds[wave * E + e[i]], 1);
  __syncthreads();
  for (int x = threadIdx.x; x < E; x += ONE_WAVES * 64) {
    int n[ONE_WAVES];
#pragma unroll
    for (int w = 0; w < ONE_WAVES; ++w) n[w] = lds[w * E + x];
    int sum = 0;
#pragma unroll
    for (int w = 0; w < ONE_WAVES; ++w) {
      lds[w * E + x] = sum;
      sum += n[w];
    }
    total[x] = sum;
  }
  __syncthreads();
  make_group_tables(tab, G, E, total, base, t, offsets, append);
  const int nbits = bits_for(E);
#pragma unroll
  for (int i = 0; i < SLICES; ++i) {
    const int a = a0 + i * 64;
    if (a - lane >= A) break;   // uniform across the wave
    const int row = next_row(e[i], nbits, G, lds + wave * E, t);
    if (a < A) {
      if (!append || row >= 0) inv[a] = row;
      if (row >= 0 && row < R_cap) row_src[row] = a;
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
  int nchunks, chunk;
  size_t hist_off, total_off, bytes;
};

Layout layout(long long A, int E, int G) {
  Layout L;
  L.chunk = chunk_for(A);
  L.nchunks = (int)((A + L.chunk - 1) / L.chunk);
  size_t off = 0;
  L.hist_off = off;
  off = align_up(off + (size_t)(L.nchunks > 0 ? L.nchunks : 1) * E * sizeof(int), 256);
  L.total_off = off;
  off = align_up(off + (size_t)E * sizeof(int), 256);
  // the group tables' place: callers size and share workspaces by this formula, so it stays in the sum
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
  // One workgroup up to 4096 assignments, where it takes 8.6 us (E = 512) and the three launches 14.9; with 16 slices
  // per wavefront it took 16.7 us at 6018 assignments and 21.8 at 16384 (three launches: 12 to 15.7).
  if (A <= ONE_MAX_A && E <= ONE_MAX_E) {
    const size_t lds = ((size_t)(ONE_WAVES + 1) * E + GroupTables::ints(E, G)) * sizeof(int);
#define FEPLB_PERMUTE_ONE(S)                                                                             \
  hipLaunchKernelGGL((permute_one_kernel<S>), dim3(1), dim3(ONE_WAVES * 64), lds, s, tab, topk_ids, (int)A, E, G, \
                     R_cap, offsets, row_src, inv, append)
    if (A <= ONE_WAVES * 64) FEPLB_PERMUTE_ONE(1);
    else FEPLB_PERMUTE_ONE(4);
#undef FEPLB_PERMUTE_ONE
    FEPLB_LAUNCH_CHECK("permute_one_kernel");
  } else {
    const int blocks = L.nchunks > 0 ? (L.nchunks + WAVES - 1) / WAVES : 1;   // no chunk: the offsets alone
    if (L.nchunks > 0) {
      hipLaunchKernelGGL(chunk_hist_kernel, dim3(blocks), dim3(BLOCK), (size_t)WAVES * E * sizeof(int), s, topk_ids, A,
                         E, L.nchunks, L.chunk, hist);
      FEPLB_LAUNCH_CHECK("chunk_hist_kernel");
    }
    hipLaunchKernelGGL(chunk_scan_kernel, dim3((E + WAVES - 1) / WAVES), dim3(BLOCK), 0, s, hist, E,
                       L.nchunks, total);
    FEPLB_LAUNCH_CHECK("chunk_scan_kernel");
    const size_t lds = ((size_t)WAVES * E + GroupTables::ints(E, G)) * sizeof(int);
    hipLaunchKernelGGL(assign_rows_kernel, dim3(blocks), dim3(BLOCK), lds, s, tab, topk_ids, A, E, G,
                       L.nchunks, L.chunk, hist, total, R_cap, offsets, row_src, inv, append);
    FEPLB_LAUNCH_CHECK("assign_rows_kernel");
  }
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

