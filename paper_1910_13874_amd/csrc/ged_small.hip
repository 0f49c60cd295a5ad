// Small graphs: a whole chain per workgroup, its level vector in LDS.
//
// On a graph of some thousand vertices a step kernel moves a few hundred
// kilobytes and takes 4 to 11 us whatever it does (launch, two memory round
// trips, drain), and a score is a dozen of them in a row.  Here one workgroup
// of 16 wavefronts runs all levels of one chain (Section 3.1.1) on its own:
// the vector x (FP64, up to 18,000 vertices in the CU's 160 KiB) stays in LDS,
// the arcs stream from the caches as 16-bit ids, and a level ends with a
// workgroup barrier instead of a launch.  Groups of a batch and candidates of
// a greedy round are independent chains, one workgroup each, so 256 of them
// fill the device.
//
// Rows are cut into chunks of at most L arcs, sorted by length and dealt 64
// to a slice; lane l of a slice owns its l-th chunk, and the slice's sources
// are stored four per lane and step (8 bytes, coalesced), padded with the id
// n, whose x is 0.  Slices are dealt to the wavefronts round robin.  A row in
// one chunk is finished by its lane; the sums of a longer row go through LDS
// and eight lanes add them.
//
// The level loop is bound by the LDS gathers (one random 8-byte read per arc:
// ER n = 10^4, 80 K arcs, 256 groups of 12 levels 119 us, about 13 cycles per
// 64 reads) or, for a single group, by the chain of a level's latencies (ER
// n = 1000: 21 us for 12 levels, whose members' values are requested ahead;
// the step kernels took 65 us, 83 us per call against 36 us now).  The first
// such call of a process also loads this file's kernels (0.7 ms).
#include <algorithm>
#include <cstring>
#include <numeric>

#include "ged_internal.h"

namespace ged {

constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
// Most slices per wavefront.  A pass holds its row, slot, accumulator and
// gathered sum, six registers; 16 wavefronts on a CU leave 128 per lane, so
// from ten passes on the compiler spills some to scratch (the score kernels 20
// of them at 10, 67 at 14, 147 at 18; with weights 30, 77, 177).
constexpr int kSmallPasses = 18;
constexpr int kSmallGreedyPasses = 10;  // ... of a graph whose greedy runs here
constexpr int kSmallChunk = 32;    // most arcs of a chunk
constexpr int kSmallTinyChunk = 16;            // ... of a graph of at most
constexpr int64_t kSmallTinyArcs = 32 << 10;   // this many arcs
constexpr size_t kSmallLds = 160 * 1024 - 1024;
constexpr int kSmallGrid = 1 << 20;  // groups per launch (a grid holds fewer than 2^32 threads)

// One direction of a small graph in slices.
struct SmallSide {
  const ushort4 *col = nullptr;   // [steps * 64] sources, four per lane and step
  const double4 *w = nullptr;     // their weights (weighted graphs)
  const int *off = nullptr;       // [n_slices + 1] first step of each slice
  const int *crow = nullptr;      // [n_slices * 64] row of a chunk, -1 past the last
  const int *cslot = nullptr;     // its slot in the partial sums, -1: the row's only chunk
  const int *mrow = nullptr;      // [n_multi] rows of several chunks
  const int *mfirst = nullptr;    // [n_multi + 1] their first slot
  int n_slices = 0, n_multi = 0, n_slots = 0, n = 0;
};

struct SmallGraph {
  int n = 0, passes = 0;
  size_t lds = 0;
  bool ok = false, tiny = false;
  DBuf buf[2][7];
  DBuf new_id;  // int [n]: internal id of a caller id
  SmallSide side[2];
};

struct SmallArgs {
  SmallSide s;
  double alpha = 0;
  int levels = 0;            // a: levels run
  int mode = 0;              // how the column total is formed (kSum ..)
  const double *inj = nullptr;   // score: t_i at i*n (value of a member at level i);
                                 // gain: miss levels m_i at i*n (value of the candidate)
  const double *tr = nullptr;    // [n] sum_{c<=r} t_c (quad: + 2 t_{b+1}); gain: sum m_c
  const int64_t *offs = nullptr; // score: group g's members are mem[offs[g] .. offs[g+1])
  const int *mem = nullptr;
  double *out = nullptr;         // [groups] totals
  // gain: the candidates; score: one group of n_inline >= 0 members in place
  // of offs and mem
  int cand[kSmallInline];
  int n_inline = -1;
  // gain: candidate c is the c-th pair (bound, caller id) of a selection of
  // n_sel; the first workgroup copies the pairs to sel_key_host / sel_id_host
  const double *sel_key = nullptr;
  const int *sel_id = nullptr, *new_id = nullptr;
  int n_sel = 0;
  double *sel_key_host = nullptr;
  int *sel_id_host = nullptr;
  // gain: S, and what a round keeps of an evaluated candidate
  const uint32_t *smask = nullptr;
  double *stale = nullptr, *ub = nullptr, *host = nullptr;
  int *done = nullptr;
  int round = 0;
};

// Miss chains of S (+ join): levels 1 .. levels to M (level i at i*n) and on
// undirected graphs Mr = sum_{c<=r} m_c; workgroup 1 the reverse graph's.
struct SmallMissArgs {
  SmallSide s[2];
  double *M[2] = {nullptr, nullptr};
  double *Mr = nullptr;
  int r = 0;
  double alpha = 0;
  int levels = 0;
  uint32_t *smask = nullptr;
  int join = -1;  // a vertex whose bit is not in smask yet
};

// Column totals: every level summed (directed graphs); the walk split at even
// and odd lengths; the quadratic form of odd lengths (see combine_quad; here
// over every arc, so the product counts once).
enum : int { kSum = 0, kEven = 1, kOdd = 2, kQuad = 3 };

struct SmallLds {
  double *x, *part, *qm, *red;
  uint32_t *bits;
};

__device__ __forceinline__ SmallLds small_lds(const SmallSide &s) {
  extern __shared__ double sh[];
  SmallLds l;
  l.x = sh;
  l.part = l.x + s.n + 1;
  l.qm = l.part + s.n_slots;
  l.red = l.qm + s.n_multi;
  l.bits = reinterpret_cast<uint32_t *>(l.red + kSmallWaves);
  return l;
}

// The sources of a lane's chunks held in registers for the whole chain (J > 0:
// chunks of at most 4J arcs), so that a level of a tiny graph waits for LDS
// alone.  At four passes 45 of a score kernel's registers spill, and it is
// still the better variant: directed n = 3,000, 24 K arcs 81 us against 88
// with streamed sources and a greedy 1.56 ms against 1.88, ER n = 3,000 54 us
// either way (greedy 0.94 and 1.06 ms); BA n = 3,000 36 us against 33.
template <int P, int J>
struct SmallCols {
  ushort4 c[P][J > 0 ? J : 1];
  int steps[P];  // of the wavefront's slices
  __device__ __forceinline__ void load(const SmallSide &s) {
    if constexpr (J > 0) {
      const int lane = threadIdx.x & 63;
      const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const int sl = wave + kSmallWaves * p;
        const int o = sl < s.n_slices ? s.off[sl] : 0;
        steps[p] = (sl < s.n_slices ? s.off[sl + 1] : 0) - o;
#pragma unroll
        for (int j = 0; j < J; ++j)
          if (j < steps[p]) c[p][j] = s.col[(size_t)(o + j) * 64 + lane];
      }
    }
  }
};

// y[p] = sum of x over the arcs of this lane's chunk in its p-th slice.
template <int P, int J, bool WGT>
__device__ __forceinline__ void small_gather(const SmallSide &s, const SmallCols<P, J> &cols,
                                             const double *x, double (&y)[P]) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int p = 0; p < P; ++p) {
    double a0 = 0.0, a1 = 0.0;
    if constexpr (J > 0) {
#pragma unroll
      for (int j = 0; j < J; ++j) {
        if (j >= cols.steps[p]) break;  // uniform over the wavefront
        const ushort4 c = cols.c[p][j];
        a0 += x[c.x];
        a1 += x[c.y];
        a0 += x[c.z];
        a1 += x[c.w];
      }
    } else {
      const int sl = wave + kSmallWaves * p;
      y[p] = 0.0;
      if (sl >= s.n_slices) continue;
      const int o = s.off[sl], e = s.off[sl + 1];
      if (o < e) {
        // the next step's sources are requested before this step's are used
        ushort4 c = s.col[(size_t)o * 64 + lane];
        for (int j = o; j < e; ++j) {
          const ushort4 d = s.col[(size_t)min(j + 1, e - 1) * 64 + lane];
          if constexpr (WGT) {
            const double4 w = s.w[(size_t)j * 64 + lane];
            a0 += w.x * x[c.x];
            a1 += w.y * x[c.y];
            a0 += w.z * x[c.z];
            a1 += w.w * x[c.w];
          } else {
            a0 += x[c.x];
            a1 += x[c.y];
            a0 += x[c.z];
            a1 += x[c.w];
          }
          c = d;
        }
      }
    }
    y[p] = a0 + a1;
  }
}

// Sum of a value over the workgroup, in thread 0 (fixed order).
__device__ __forceinline__ double small_sum(double v, double *red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < kSmallWaves; ++w) r += red[w];
  return r;
}

// One level over all rows: gathers from x, then f(row, sum, q) for each row
// once all gathers have finished -- q is the row's accumulator, kept by the
// thread (or, for a row of several chunks, in LDS).
template <int P, int J, bool WGT, class F>
__device__ __forceinline__ void small_level(const SmallSide &s, const SmallCols<P, J> &cols,
                                            const SmallLds &l, const int (&row)[P], const int (&slot)[P],
                                            double (&q)[P], F &&f) {
  double y[P];
  small_gather<P, J, WGT>(s, cols, l.x, y);
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (slot[p] >= 0) l.part[slot[p]] = y[p];
  __syncthreads();
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (row[p] >= 0 && slot[p] < 0) f(row[p], y[p], q[p]);
  // rows of several chunks: eight lanes each
  const int t = threadIdx.x, k = t & 7;
  for (int m = t >> 3; m < s.n_multi; m += kSmallThreads / 8) {
    double a = 0.0;
    for (int i = s.mfirst[m] + k; i < s.mfirst[m + 1]; i += 8) a += l.part[i];
    for (int o = 4; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
    if (k == 0) f(s.mrow[m], a, l.qm[m]);
  }
  __syncthreads();
}

template <int P>
__device__ __forceinline__ void small_rows(const SmallSide &s, const SmallLds &l, int (&row)[P],
                                           int (&slot)[P], double (&q)[P]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int sl = wave + kSmallWaves * p;
    row[p] = sl < s.n_slices ? s.crow[sl * 64 + lane] : -1;
    slot[p] = sl < s.n_slices ? s.cslot[sl * 64 + lane] : -1;
    q[p] = 0.0;
  }
  for (int m = threadIdx.x; m < s.n_multi; m += kSmallThreads) l.qm[m] = 0.0;
}

// Score of group blockIdx.x (GAIN false) or gain of candidate blockIdx.x.
template <int P, int J, bool WGT, bool GAIN>
__global__ __launch_bounds__(kSmallThreads) void k_small_chain(SmallArgs a) {
  const SmallSide &s = a.s;
  const SmallLds l = small_lds(s);
  const int t = threadIdx.x, n = s.n;
  int row[P], slot[P];
  double q[P];
  SmallCols<P, J> cols;
  cols.load(s);
  small_rows<P>(s, l, row, slot, q);
  const int words = (n + 31) / 32;
  int x0 = -1;
  if constexpr (GAIN) {
    if (blockIdx.x == 0 && t < a.n_sel) {
      a.sel_key_host[t] = a.sel_key[t];
      a.sel_id_host[t] = a.sel_id[t];
    }
    const int id = a.sel_id[blockIdx.x];
    if (id < 0 || id >= n) return;  // fewer candidates than workgroups (all threads)
    x0 = a.new_id[id];
  }
  for (int v = t; v <= n; v += kSmallThreads) l.x[v] = v == x0 ? 1.0 : 0.0;
  for (int w = t; w < words; w += kSmallThreads) l.bits[w] = GAIN ? a.smask[w] : 0u;
  __syncthreads();
  if (!GAIN && a.n_inline >= 0) {
    if (t < a.n_inline) {
      const int v = a.cand[t];
      atomicOr(&l.bits[v >> 5], 1u << (v & 31));
      l.x[v] = 1.0;
    }
    __syncthreads();
  } else if (!GAIN) {
    for (int64_t j = a.offs[blockIdx.x] + t; j < a.offs[blockIdx.x + 1]; j += kSmallThreads) {
      const int v = a.mem[j];
      atomicOr(&l.bits[v >> 5], 1u << (v & 31));
      l.x[v] = 1.0;
    }
    __syncthreads();
  }
  auto bit = [&](int v) { return (l.bits[v >> 5] >> (v & 31)) & 1u; };
  // rows whose level value is read (members; the candidate): the thread's
  // first one is requested ahead of the level's gathers
  auto fixed = [&](int v) { return GAIN ? v == x0 : (bool)bit(v); };
  int vm = -1;
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (vm < 0 && row[p] >= 0 && slot[p] < 0 && fixed(row[p])) vm = row[p];
  double tv = 0.0;
  // the level's value at a row, given the gathered sum
  auto value = [&](int i, int v, double sum) -> double {
    if (GAIN && bit(v)) return 0.0;
    if (fixed(v)) return v == vm ? tv : a.inj[(size_t)i * n + v];
    return a.alpha * sum;
  };
  for (int i = 1; i < a.levels; ++i) {
    if (vm >= 0) tv = a.inj[(size_t)i * n + vm];
    small_level<P, J, WGT>(s, cols, l, row, slot, q, [&](int v, double sum, double &qv) {
      const double y = value(i, v, sum);
      l.x[v] = y;
      qv += y;
    });
  }
  double total = 0.0;
  const int L = a.levels;
  if (vm >= 0) tv = a.inj[(size_t)L * n + vm];
  small_level<P, J, WGT>(s, cols, l, row, slot, q, [&](int v, double sum, double &qv) {
    const bool inS = bit(v);
    if (a.mode == kSum) {
      total += qv + value(L, v, sum);
    } else if (a.mode == kQuad) {
      const double hb = l.x[v], tb = a.inj[(size_t)(L - 1) * n + v];
      total += (qv + hb * a.tr[v]) + (inS ? 0.0 : (tb - hb) * qv) - hb * (a.alpha * sum);
    } else {
      const double y = value(L, v, sum), ta = a.inj[(size_t)L * n + v];
      const double rs = a.mode == kEven ? qv + y : qv;
      total += ((qv + y) + y * a.tr[v]) + (!GAIN && inS ? 0.0 : (ta - y) * rs);
    }
  });
  const double r = small_sum(total, l.red);
  if (t == 0) {
    if constexpr (GAIN) {
      a.host[blockIdx.x] = r;
      a.stale[x0] = r;
      a.ub[x0] = r;
      a.done[x0] = a.round;
    } else {
      a.out[blockIdx.x] = r;
    }
  }
}

template <int P, int J, bool WGT>
__global__ __launch_bounds__(kSmallThreads) void k_small_miss(SmallMissArgs a) {
  const bool rev = blockIdx.x == 1;
  const SmallSide &s = rev ? a.s[1] : a.s[0];
  double *M = rev ? a.M[1] : a.M[0];
  const SmallLds l = small_lds(s);
  const int t = threadIdx.x, n = s.n;
  int row[P], slot[P];
  double q[P];
  SmallCols<P, J> cols;
  cols.load(s);
  small_rows<P>(s, l, row, slot, q);
  for (int w = t; w < (n + 31) / 32; w += kSmallThreads) {
    uint32_t b = a.smask[w];
    if (a.join >= 0 && (a.join >> 5) == w) {
      b |= 1u << (a.join & 31);
      if (!rev) a.smask[w] = b;  // both workgroups may read either value: same bits
    }
    l.bits[w] = b;
  }
  __syncthreads();
  auto bit = [&](int v) { return (l.bits[v >> 5] >> (v & 31)) & 1u; };
  for (int v = t; v <= n; v += kSmallThreads) l.x[v] = v < n && !bit(v) ? 1.0 : 0.0;
  __syncthreads();
  for (int i = 1; i <= a.levels; ++i)
    small_level<P, J, WGT>(s, cols, l, row, slot, q, [&](int v, double sum, double &qv) {
      const double y = bit(v) ? 0.0 : a.alpha * sum;
      l.x[v] = y;
      M[(size_t)i * n + v] = y;
      if (i <= a.r) qv += y;
      if (i == a.levels && a.Mr) a.Mr[v] = qv;
    });
}

// ------------------------------------------------------------------ host --

static void small_build(ged_graph *g, bool reverse, SmallGraph &sg, int L,
                        std::vector<int> &ci, const std::vector<double> &w) {
  const std::vector<int> &rp = reverse ? g->h_rp_r : g->h_rp;
  const int n = (int)g->n;
  struct Chunk {
    int row, j0, len, slot;
  };
  std::vector<Chunk> ch;
  std::vector<int> mrow, mfirst;
  int slots = 0;
  for (int v = 0; v < n; ++v) {
    const int d = rp[v + 1] - rp[v];
    if (d <= L) {
      ch.push_back({v, rp[v], d, -1});
      continue;
    }
    mrow.push_back(v);
    mfirst.push_back(slots);
    for (int j = rp[v]; j < rp[v + 1]; j += L)
      ch.push_back({v, j, std::min(L, rp[v + 1] - j), slots++});
  }
  mfirst.push_back(slots);
  std::stable_sort(ch.begin(), ch.end(),
                   [](const Chunk &x, const Chunk &y) { return x.len > y.len; });
  const int ns = ((int)ch.size() + 63) / 64;
  std::vector<int> off((size_t)ns + 1, 0), crow((size_t)ns * 64, -1), cslot((size_t)ns * 64, -1);
  for (int s = 0; s < ns; ++s) off[(size_t)s + 1] = off[s] + (ch[(size_t)s * 64].len + 3) / 4;
  std::vector<uint16_t> col((size_t)off[ns] * 256, (uint16_t)n);
  std::vector<double> wt(w.empty() ? 0 : col.size(), 0.0);
  for (size_t c = 0; c < ch.size(); ++c) {
    const size_t s = c / 64, lane = c % 64;
    crow[c] = ch[c].row;
    cslot[c] = ch[c].slot;
    for (int j = 0; j < ch[c].len; ++j) {
      const size_t at = (((size_t)off[s] + j / 4) * 64 + lane) * 4 + j % 4;
      col[at] = (uint16_t)ci[(size_t)ch[c].j0 + j];
      if (!wt.empty()) wt[at] = w[(size_t)ch[c].j0 + j];
    }
  }
  DBuf *b = sg.buf[reverse ? 1 : 0];
  SmallSide &sd = sg.side[reverse ? 1 : 0];
  auto up = [](DBuf &d, const void *p, size_t bytes) -> void * {
    d.ensure(std::max<size_t>(bytes, 256));
    if (bytes) GED_HIP(hipMemcpy(d.p, p, bytes, hipMemcpyHostToDevice));
    return d.p;
  };
  sd.col = static_cast<const ushort4 *>(up(b[0], col.data(), 2 * col.size()));
  sd.off = static_cast<const int *>(up(b[1], off.data(), 4 * off.size()));
  sd.crow = static_cast<const int *>(up(b[2], crow.data(), 4 * crow.size()));
  sd.cslot = static_cast<const int *>(up(b[3], cslot.data(), 4 * cslot.size()));
  sd.mrow = static_cast<const int *>(up(b[4], mrow.data(), 4 * mrow.size()));
  sd.mfirst = static_cast<const int *>(up(b[5], mfirst.data(), 4 * mfirst.size()));
  if (!wt.empty()) sd.w = static_cast<const double4 *>(up(b[6], wt.data(), 8 * wt.size()));
  sd.n_slices = ns;
  sd.n_multi = (int)mrow.size();
  sd.n_slots = slots;
  sd.n = n;
  sg.passes = std::max(sg.passes, (ns + kSmallWaves - 1) / kSmallWaves);
  sg.lds = std::max(sg.lds, sizeof(double) * ((size_t)n + 1 + slots + mrow.size() + kSmallWaves) +
                                sizeof(uint32_t) * (((size_t)n + 31) / 32));
}

enum SmallKind { kScoreChain, kGainChain, kMissChain };

template <int P, int J, bool WGT>
static void small_launch(const void *args, SmallKind kind, int grid, size_t lds,
                         hipStream_t st) {
  if constexpr (P > kSmallGreedyPasses) {
    if (kind != kScoreChain) throw HipError{GED_ERR_ARG, "greedy chain of too many passes"};
    hipLaunchKernelGGL((k_small_chain<P, J, WGT, false>), dim3(grid), dim3(kSmallThreads), lds, st,
                       *static_cast<const SmallArgs *>(args));
  } else if (kind == kMissChain)
    hipLaunchKernelGGL((k_small_miss<P, J, WGT>), dim3(grid), dim3(kSmallThreads), lds, st,
                       *static_cast<const SmallMissArgs *>(args));
  else if (kind == kGainChain)
    hipLaunchKernelGGL((k_small_chain<P, J, WGT, true>), dim3(grid), dim3(kSmallThreads), lds, st,
                       *static_cast<const SmallArgs *>(args));
  else
    hipLaunchKernelGGL((k_small_chain<P, J, WGT, false>), dim3(grid), dim3(kSmallThreads), lds, st,
                       *static_cast<const SmallArgs *>(args));
}

// args: SmallMissArgs for kMissChain, else SmallArgs.
template <bool WGT>
static void small_run(const SmallGraph &sg, const void *a, SmallKind gain, int grid,
                      hipStream_t st) {
  const int p = sg.passes;
  // sources in registers: up to four chunks of kSmallTinyChunk arcs per lane
  constexpr int JR = WGT ? 0 : kSmallTinyChunk / 4;
  if (p <= 1 && sg.tiny)
    small_launch<1, JR, WGT>(a, gain, grid, sg.lds, st);
  else if (p <= 2 && sg.tiny)
    small_launch<2, JR, WGT>(a, gain, grid, sg.lds, st);
  else if (p <= 4 && sg.tiny)
    small_launch<4, JR, WGT>(a, gain, grid, sg.lds, st);
  else if (p <= 6)
    small_launch<6, 0, WGT>(a, gain, grid, sg.lds, st);
  else if (p <= 10)
    small_launch<10, 0, WGT>(a, gain, grid, sg.lds, st);
  else if (p <= 14)
    small_launch<14, 0, WGT>(a, gain, grid, sg.lds, st);
  else
    small_launch<kSmallPasses, 0, WGT>(a, gain, grid, sg.lds, st);
  GED_HIP(hipGetLastError());
}

// The slices of a graph (built once); ok is false where they do not fit.
static SmallGraph &small_graph(ged_graph *g) {
  if (g->small) return *g->small;
  auto sg = std::make_shared<SmallGraph>();
  sg->n = (int)g->n;
  // shorter chunks where a level is one latency chain
  sg->tiny = g->nnz <= kSmallTinyArcs;
  const int L = sg->tiny ? kSmallTinyChunk : kSmallChunk;
  for (int r = 0; r < (g->flags == GED_DIRECTED ? 2 : 1); ++r) {
    std::vector<int> ci((size_t)g->nnz);
    std::vector<double> w(g->weighted ? (size_t)g->nnz : 0);
    if (g->nnz > 0) {
      GED_HIP(hipMemcpy(ci.data(), (r ? g->ci_r : g->ci).p, 4 * ci.size(), hipMemcpyDeviceToHost));
      if (g->weighted)
        GED_HIP(hipMemcpy(w.data(), (r ? g->w_r : g->w).p, 8 * w.size(), hipMemcpyDeviceToHost));
    }
    small_build(g, r == 1, *sg, L, ci, w);
  }
  sg->new_id.ensure(sizeof(int) * (size_t)g->n);
  GED_HIP(hipMemcpy(sg->new_id.p, g->new_id.data(), sizeof(int) * (size_t)g->n,
                    hipMemcpyHostToDevice));
  sg->ok = sg->passes <= kSmallPasses && sg->lds <= kSmallLds;
  g->small = sg;
  return *g->small;
}

bool small_batch_ok(ged_graph *g) {
  return g->n <= kSmallVertices && g->nnz <= kSmallBatchArcs && small_graph(g).ok;
}

bool small_score_ok(ged_graph *g) {
  return g->n <= (g->weighted ? kSmallScoreWeighted : kSmallScoreVertices) &&
         g->nnz <= kSmallScoreArcs && small_graph(g).ok;
}

bool small_greedy_ok(ged_graph *g) {
  return g->n <= kSmallGreedyVertices && g->nnz <= kSmallScoreArcs && small_graph(g).ok &&
         small_graph(g).passes <= kSmallGreedyPasses;
}

size_t small_bytes(const ged_graph *g) {
  if (!g->small) return 0;
  size_t b = g->small->new_id.bytes;
  for (const auto &side : g->small->buf)
    for (const DBuf &d : side) b += d.bytes;
  return b;
}

void small_scores(ged_graph *g, const int64_t *offs, const int *mem, int groups, double *out,
                  hipStream_t st, int n_inline) {
  const SmallGraph &sg = small_graph(g);
  const PrepCache &pc = g->prep;
  SmallArgs a;
  a.s = sg.side[0];
  a.alpha = pc.alpha;
  a.inj = pc.t_levels.as<const double>();
  a.levels = pc.ell;
  if (split_ok(g)) {
    SplitPlan pl = split_plan(g, pc.ell);
    split_tables(g, pl, st);
    a.levels = pl.a;
    a.mode = pl.even ? kEven : pl.quad ? kQuad : kOdd;
    a.tr = pc.tr.as<const double>();
  }
  if (n_inline >= 0)
    std::copy(mem, mem + n_inline, a.cand);
  else
    a.mem = mem;
  a.n_inline = n_inline;
  for (int g0 = 0; g0 < groups; g0 += kSmallGrid) {
    const int grid = std::min(groups - g0, kSmallGrid);
    a.offs = offs ? offs + g0 : nullptr;
    a.out = out + g0;
    if (g->weighted)
      small_run<true>(sg, &a, kScoreChain, grid, st);
    else
      small_run<false>(sg, &a, kScoreChain, grid, st);
  }
}

void small_miss(ged_graph *g, int levels, int r, uint32_t *smask, int join, double *M, double *Mb,
                double *Mr, hipStream_t st) {
  const SmallGraph &sg = small_graph(g);
  SmallMissArgs a;
  const bool directed = g->flags == GED_DIRECTED;
  a.s[0] = sg.side[0];
  a.s[1] = sg.side[directed ? 1 : 0];
  a.M[0] = M;
  a.M[1] = Mb;
  a.Mr = directed ? nullptr : Mr;
  a.r = r;
  a.alpha = g->prep.alpha;
  a.levels = levels;
  a.smask = smask;
  a.join = join;
  if (g->weighted)
    small_run<true>(sg, &a, kMissChain, directed ? 2 : 1, st);
  else
    small_run<false>(sg, &a, kMissChain, directed ? 2 : 1, st);
}

void small_gains(ged_graph *g, const SmallGains &b, hipStream_t st) {
  const SmallGraph &sg = small_graph(g);
  SmallArgs a;
  a.s = sg.side[0];
  a.alpha = g->prep.alpha;
  a.levels = b.ell;
  a.mode = kSum;
  if (split_ok(g)) {
    a.levels = (b.ell + 1) / 2;
    a.mode = b.ell % 2 == 0 ? kEven : kOdd;
  }
  a.inj = b.M;
  a.tr = b.Mr;
  a.sel_key = b.sel_key;
  a.sel_id = b.sel_id;
  a.new_id = sg.new_id.as<const int>();
  a.n_sel = b.n_sel;
  a.sel_key_host = b.sel_key_host;
  a.sel_id_host = b.sel_id_host;
  a.smask = b.smask;
  a.stale = b.stale;
  a.ub = b.ub;
  a.done = b.done;
  a.round = b.round;
  a.host = b.gains_host;
  if (g->weighted)
    small_run<true>(sg, &a, kGainChain, b.width, st);
  else
    small_run<false>(sg, &a, kGainChain, b.width, st);
}

}  // namespace ged
