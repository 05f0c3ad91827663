// Memory pass of the 32-bit path for graphs whose gap table fits one CU's LDS
// (gfx950): per-device peaks of the residency intervals (Sec. 3.3.2) and the
// violation verdict, one workgroup per candidate, with no interval record in
// global memory.
//
// A device's ops run one at a time in dispatch order, so their starts
// S[0..m) are sorted and cut the device's time into gaps 0..m.  Every event
// falls into one gap:
//   own output of rank k    allocated at S[k], counted as opening gap k + 1
//   copy allocated at t     gap #{k : S[k] < t}
//   free at t               gap #{k : S[k] < t}
// (frees precede allocations at equal times: intervals are half-open).  A free
// at the finish of a local op of rank k has gap k + 1; a copy is allocated at
// or before the start of its first consumer, of rank k, so its gap is searched
// downwards from k; a transfer-bound free of an op of rank k upwards from
// k + 1.  With A[g] the bytes allocated and F[g] the bytes freed in gap g,
//   L[g] = sum_{g' <= g} A[g'] - F[g']
// is the live bytes before own g, so L[k] + own_k is exact at every own start,
// and U[g] = L[g] + F[g] bounds the live bytes inside gap g.  Only a "hard"
// gap, whose U exceeds the best exact value of its device, has its events
// collected and swept in time order (0 to 4 events per gap and about three
// such gaps per device with every op placed at random; one or two gaps per
// candidate when a candidate moves a few ops of a partition).
//
// All devices of a candidate share one flat index space of N + D entries
// (device d from gb[d], m + 1 entries), 12 bytes an entry with 32-bit byte
// sums, so a workgroup walks the ops in index order with full lanes whatever
// the devices' loads, the prefix sum is one block scan, and the only traffic
// beyond the placement and finish rows is a two-byte rank and a two-byte gap
// per op, which stay in the CU's caches.
//
// Bound: the latency of each pass over the ops at 16 to 24 waves a CU (fewer on
// graphs with wide successors whose table nearly fills the LDS), then LDS
// access.  It takes the place of interval records in global memory, bucketed
// per device and evaluated one device at a time in a wave of its own, whose
// fixed cost per device was most of the pass on small graphs; the two passes
// before and this one: 65,536 candidates of 322 ops 2.8 and 0.73 ms, 100,003 of
// 2,052 ops 11.5 and 3.2 ms, 131,072 of 10,000 ops 38.2 and 17.5 ms, 32,771 of
// a 2,001-op graph with 34 consumers of some outputs 16.5 and 3.9 ms.  Graphs
// that do not fit keep the records.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "peaks.h"

namespace {

constexpr int kWave = 64;
constexpr uint32_t kInf32 = 0xFFFFFFFFu;
constexpr uint32_t kNoGap = 0xFFFFu;  // gap table: no own free (never freed, or the op is on the list)
constexpr int kMaxFlat = 0xFFFF;      // flat gaps a table entry can hold

__device__ __forceinline__ uint32_t umax32(uint32_t a, uint32_t b) { return a > b ? a : b; }

__device__ __forceinline__ uint32_t link_bit(const GmgView &G, uint32_t a, uint32_t b) {
  return (G.link_bits[a * G.link_words + (b >> 5)] >> (b & 31)) & 1u;
}

__device__ __forceinline__ uint32_t xfer_of(const GmgView &G, int u, int du, int d) {
  const int K = G.n_link;
  if (K == 1) return G.xfer32[u];
  if (K == 2) return G.xfer32[2 * u + (int)link_bit(G, (uint32_t)du, (uint32_t)d)];
  return G.xfer32[u * K + G.link_class[du * G.n_dev + d]];
}

// Orders a wave's LDS accesses (they complete in issue order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// #{k : S[k] < t} given that it is at most hi: the answer is hi itself for
// about 85% of the copies and within three of it for nearly all others.
__device__ __forceinline__ int gap_down(const uint32_t *S, int hi, uint32_t t) {
  int g = hi;
  for (int i = 0; i < 4; ++i) {
    if (g == 0 || S[g - 1] < t) return g;
    --g;
  }
  int lo = 0;  // the answer lies in [lo, g]
  while (lo < g) {
    const int mid = (lo + g) >> 1;
    if (S[mid] < t)
      lo = mid + 1;
    else
      g = mid;
  }
  return lo;
}

// #{k : S[k] < t} given that it is at least lo (S[m] is a sentinel above every t).
__device__ __forceinline__ int gap_up(const uint32_t *S, int lo, int m, uint32_t t) {
  int g = lo;
  for (int i = 0; i < 4; ++i) {
    if (S[g] >= t) return g;
    ++g;
  }
  int hi = m;
  while (g < hi) {
    const int mid = (g + hi) >> 1;
    if (S[mid] < t)
      g = mid + 1;
    else
      hi = mid;
  }
  return g;
}

__device__ __forceinline__ void lds_add(uint32_t *p, uint32_t v) { atomicAdd(p, v); }
__device__ __forceinline__ void lds_add(int64_t *p, int64_t v) {
  atomicAdd(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v);
}
__device__ __forceinline__ void lds_max(uint32_t *p, uint32_t v) { atomicMax(p, v); }
__device__ __forceinline__ void lds_max(int64_t *p, int64_t v) {
  atomicMax(reinterpret_cast<long long *>(p), (long long)v);
}
__device__ __forceinline__ uint32_t shfl_up(uint32_t x, int o) { return (uint32_t)__shfl_up((int)x, o, kWave); }
__device__ __forceinline__ int64_t shfl_up(int64_t x, int o) { return __shfl_up(x, o, kWave); }

__device__ __forceinline__ uint64_t wave_max64(uint64_t x) {
  for (int o = kWave / 2; o >= 1; o >>= 1) {
    const uint64_t y = __shfl_xor(x, o, kWave);
    x = y > x ? y : x;
  }
  return x;
}

// A wave's per-device arrays for ops with many successors: lowest consumer
// rank (kInf32: none) and latest consumer (finish << 32 | rank).
struct WideLds {
  uint64_t *last;
  uint32_t *low;
};
constexpr int kWide = 8;  // successors a lane walks alone (three nested walks of them); more are walked by the wave

// An op's fields, and its successors' (absent ones repeat the op itself).
struct OpIn {
  uint32_t d, rv, f, b, s2;
};
struct SuccIn {
  uint32_t dx0, dx1, fx0, fx1, rx0, rx1;
};

template <bool kCsr>
__device__ __forceinline__ OpIn load_op(const GmgView &G, const uint8_t *prow, const uint32_t *frow,
                                        const uint16_t *rk, int v) {
  return OpIn{prow[v], rk[v], frow[v], G.bytes32[v], kCsr ? 0u : G.succ2[v]};
}

template <bool kCsr>
__device__ __forceinline__ SuccIn load_succ(const uint8_t *prow, const uint32_t *frow, const uint16_t *rk,
                                            const OpIn &a, int v) {
  if (kCsr) return SuccIn{};
  const uint32_t i0 = a.s2 & 0xFFFFu, i1 = a.s2 >> 16;
  const int y0 = i0 != 0xFFFFu ? (int)i0 : v, y1 = i1 != 0xFFFFu ? (int)i1 : v;
  return SuccIn{prow[y0], prow[y1], frow[y0], frow[y1], rk[y0], rk[y1]};
}

// The residency events of op v, passed to `ev` (an op per lane):
//   ev.own_free(d, q, t, b)      the own output's free on v's device, flat gap q
//   ev.copy(e, qa, ta, qf, tf, b)  a copy on device e: allocated in gap qa, freed in qf (from any lane)
//   ev.copied()                  v has a copy
// kCsr: any graph, successors from the CSR.  Otherwise at most two successors
// per op, one device class and at most two link classes: with kShift the link class comes from the device ids.  kPorts:
// arrivals of the transfers per predecessor edge in arow.
template <bool kCsr, bool kShift, bool kPorts, class Ev>
__device__ __forceinline__ void op_events(const GmgView &G, const uint8_t *prow, const uint32_t *frow,
                                          const uint16_t *rk, const uint32_t *arow, int v, bool act, const OpIn &op,
                                          const SuccIn &su, int sh, const uint32_t *S, const int *gb,
                                          const WideLds &wl, Ev &&ev) {
  const uint32_t d = op.d, rv = op.rv, f = op.f, b = op.b >> sh;
  if (kCsr) {
    const int x0 = G.succ_ptr[v], x1 = act ? G.succ_ptr[v + 1] : x0;
    const int qd = gb[d];
    if (x1 > x0 && x1 - x0 <= kWide) {  // (without consumers: kept for ever)
      uint32_t L = f, A = 0, rl = rv;
      bool remote = false;
      for (int q = x0; q < x1; ++q) {
        const int x = G.succ_idx[q];
        const uint32_t dx = prow[x];
        if (dx == d) {
          if (frow[x] > L) {
            L = frow[x];
            rl = rk[x];
          }
        } else {
          remote = true;
          A = umax32(A, f + xfer_of(G, v, (int)d, (int)dx));
        }
      }
      const bool arrive = A > L;
      const int g = arrive ? gap_up(S + qd, (int)rv + 1, gb[d + 1] - qd - 1, A) : (int)rl + 1;
      ev.own_free((int)d, qd + g, arrive ? A : L, b);
      if (remote && b != 0) {
        ev.copied();
        for (int q = x0; q < x1; ++q) {
          const int xf = G.succ_idx[q];
          const uint32_t e = prow[xf];
          if (e == d) continue;
          bool first = true;
          for (int q2 = x0; q2 < q; ++q2)
            if (prow[G.succ_idx[q2]] == e) first = false;
          if (!first) continue;
          // allocated before the consumer on e that starts first (lowest
          // rank), freed by the one that finishes last
          int y = xf, ra = rk[xf];
          for (int q2 = q + 1; q2 < x1; ++q2) {
            const int x = G.succ_idx[q2];
            if (prow[x] == e) {
              if (frow[x] > frow[y]) y = x;
              ra = min(ra, (int)rk[x]);
            }
          }
          const int qe = gb[e];
          ev.copy((int)e, qe + gap_down(S + qe, ra, f), f, qe + (int)rk[y] + 1, frow[y], b);
        }
      }
    }
    // ops with more successors: the wave walks them together, one op at a time
    const int lane = threadIdx.x % kWave;
    for (uint64_t wide = __ballot(x1 - x0 > kWide); wide; wide &= wide - 1) {
      const int src = __ffsll((unsigned long long)wide) - 1;
      const int u = __builtin_amdgcn_readlane(v, src);
      const uint32_t du = (uint32_t)__builtin_amdgcn_readlane((int)d, src);
      const uint32_t fu = (uint32_t)__builtin_amdgcn_readlane((int)f, src);
      const uint32_t ru = (uint32_t)__builtin_amdgcn_readlane((int)rv, src);
      const uint32_t bu = (uint32_t)__builtin_amdgcn_readlane((int)b, src);
      const int e1 = G.succ_ptr[u + 1];
      uint64_t loc = (uint64_t)fu << 32 | ru;
      uint32_t A = 0;
      for (int q = G.succ_ptr[u] + lane; q < e1; q += kWave) {
        const int x = G.succ_idx[q];
        const uint32_t dx = prow[x];
        const uint64_t key = (uint64_t)frow[x] << 32 | rk[x];
        if (dx == du) {
          loc = key > loc ? key : loc;
        } else {
          A = umax32(A, fu + xfer_of(G, u, (int)du, (int)dx));
          atomicMin(&wl.low[dx], (uint32_t)key);
          atomicMax(reinterpret_cast<unsigned long long *>(&wl.last[dx]), (unsigned long long)key);
        }
      }
      loc = wave_max64(loc);
      A = (uint32_t)wave_max64(A);
      wave_lds_fence();
      if (lane == src) {
        const int qu = gb[du];
        const uint32_t L = (uint32_t)(loc >> 32);
        const bool arrive = A > L;
        const int g = arrive ? gap_up(S + qu, (int)ru + 1, gb[du + 1] - qu - 1, A) : (int)(uint32_t)loc + 1;
        ev.own_free((int)du, qu + g, arrive ? A : L, bu);
        if (A != 0 && bu != 0) ev.copied();  // A is at least fu > 0 with a remote consumer
      }
      for (int e = lane; e < G.n_dev; e += kWave) {
        const uint32_t ra = wl.low[e];
        if (ra == kInf32) continue;
        const uint64_t last = wl.last[e];
        const int qe = gb[e];
        if (bu != 0)
          ev.copy(e, qe + gap_down(S + qe, (int)ra, fu), fu, qe + (int)(uint32_t)last + 1, (uint32_t)(last >> 32), bu);
        wl.low[e] = kInf32;
        wl.last[e] = 0;
      }
      wave_lds_fence();
    }
  } else {
    // an op with a consumer on another device
    const bool has0 = act && (op.s2 & 0xFFFFu) != 0xFFFFu, has1 = act && (op.s2 >> 16) != 0xFFFFu;
    const uint32_t dx0 = su.dx0, dx1 = su.dx1, fx0 = su.fx0, fx1 = su.fx1, rx0 = su.rx0, rx1 = su.rx1;
    const bool loc0 = dx0 == d, loc1 = dx1 == d;
    const bool rem0 = has0 && !loc0, rem1 = has1 && !loc1;
    if (!__any(has0)) return;
    // own output: until the local consumer that finishes last (an absent
    // successor repeats v itself, whose finish is f)
    uint32_t L = f, rl = rv;
    rl = loc0 && fx0 > L ? rx0 : rl;
    L = loc0 && fx0 > L ? fx0 : L;
    rl = loc1 && fx1 > L ? rx1 : rl;
    L = loc1 && fx1 > L ? fx1 : L;
    const int qd = gb[d];
    int g = (int)rl + 1;
    uint32_t F = L;
    auto cls = [&](uint32_t to) -> uint32_t {
      if (!kShift) return link_bit(G, d, to);
      const uint32_t s = (uint32_t)G.link_shift, same = (uint32_t)G.link_same;
      return (d >> s) == (to >> s) ? same : 1u - same;
    };
    const int K = G.n_link;
    const uint32_t xa = G.xfer32[v * K], xb = G.xfer32[v * K + K - 1];
    const uint32_t X0 = cls(dx0) ? xb : xa, X1 = cls(dx1) ? xb : xa;
    uint32_t T0 = f + X0, T1 = f + X1;  // arrivals
    if (kPorts) {
      const uint32_t pe = G.succ2_pe[v], e0 = pe & 0xFFFFu, e1 = pe >> 16;
      T0 = arow[e0 == 0xFFFFu ? 0u : e0];  // (an absent one's is not used)
      T1 = arow[e1 == 0xFFFFu ? 0u : e1];
    }
    // two successors on one remote device share the first one's transfer
    uint32_t A = rem0 ? T0 : 0u;
    A = rem1 ? umax32(A, T1) : A;
    if (A > L) {
      F = A;
      g = gap_up(S + qd, (int)rv + 1, gb[d + 1] - qd - 1, A);
    }
    if (has0) ev.own_free((int)d, qd + g, F, b);
    const bool same = has1 && dx1 == dx0;
    if (rem0 && b != 0) {
      const bool late1 = same && fx1 > fx0;
      const int ra = same ? (int)min(rx0, rx1) : (int)rx0;
      const uint32_t st = kPorts ? T0 - X0 : f;  // the transfer's start
      const int qe = gb[dx0];
      ev.copy((int)dx0, qe + gap_down(S + qe, ra, st), st, qe + (int)(late1 ? rx1 : rx0) + 1, late1 ? fx1 : fx0, b);
    }
    if (rem1 && !same && b != 0) {
      const uint32_t st = kPorts ? T1 - X1 : f;
      const int qe = gb[dx1];
      ev.copy((int)dx1, qe + gap_down(S + qe, (int)rx1, st), st, qe + (int)rx1 + 1, fx1, b);
    }
  }
}

// First walk: bytes allocated and freed per gap.
template <class Acc>
struct Accumulate {
  Acc *A, *F;
  uint32_t gap;  // of this op's own free
  bool remote;   // it has copies
  __device__ void own_free(int, int q, uint32_t, uint32_t b) {
    lds_add(&F[q], (Acc)b);
    gap = (uint32_t)q;
  }
  __device__ void copy(int, int qa, uint32_t, int qf, uint32_t, uint32_t b) {
    lds_add(&A[qa], (Acc)b);
    lds_add(&F[qf], (Acc)b);
  }
  __device__ void copied() { remote = true; }
};

// Second walk: the events of hard gaps, as a list per gap whose head replaces
// the gap's sum in A.  Node: {time, bytes, flat gap | device << 16 |
// allocation << 24, next}.
constexpr uint32_t kEmpty = 0xFFFFFFFFu;  // head of a hard gap without events yet
constexpr uint32_t kEasy = 0xFFFFFFFEu;   // a gap that is not hard
template <class Acc>
struct Collect {
  Acc *A;
  uint4 *node;
  uint32_t *count;
  uint32_t cap;
  __device__ void push(int d, int q, uint32_t t, uint32_t b, uint32_t alloc) {
    uint32_t *head = reinterpret_cast<uint32_t *>(&A[q]);
    if (*head == kEasy) return;
    const uint32_t at = atomicAdd(count, 1u);
    if (at >= cap) return;
    const uint32_t next = atomicExch(head, at);
    node[at] = make_uint4(t, b, (uint32_t)q | (uint32_t)d << 16 | alloc << 24, next);
  }
  __device__ void own_free(int d, int q, uint32_t t, uint32_t b) { push(d, q, t, b, 0); }
  __device__ void copy(int e, int qa, uint32_t ta, int qf, uint32_t tf, uint32_t b) {
    push(e, qa, ta, b, 1);
    push(e, qf, tf, b, 0);
  }
  __device__ void copied() {}
};

template <bool kCsr, bool kGiven, bool kShift, bool kPorts, bool kNarrow>
__global__ __launch_bounds__(1024) void lds_peaks(const GmgView G, const uint8_t *__restrict__ P,
                                                  const uint32_t *__restrict__ fin, int64_t fpitch,
                                                  const uint32_t *__restrict__ arr, uint16_t *__restrict__ rank_all,
                                                  uint16_t *__restrict__ gap_all, uint16_t *__restrict__ list_all,
                                                  uint4 *__restrict__ node_all,
                                                  int64_t node_cap, int lds_nodes, int64_t nb,
                                                  uint32_t *__restrict__ ticket, int64_t *__restrict__ peak,
                                                  uint8_t *__restrict__ violation) {
  using Acc = typename std::conditional<kNarrow, uint32_t, int64_t>::type;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int D = G.n_dev, N = G.n_ops, C = G.n_class, n = N + D;
  const int E = kPorts ? G.pred_ptr[N] : 0;
  const int T = blockDim.x, W = T / kWave, tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
  const int n4 = (n + 3) & ~3;
  Acc *A = reinterpret_cast<Acc *>(lds_raw);                 // [n4]
  Acc *F = A + n4;                                           // [n4]
  uint32_t *S = reinterpret_cast<uint32_t *>(F + n4);        // [n4]
  uint4 *s_node = reinterpret_cast<uint4 *>(S + n4);         // [lds_nodes]
  Acc *best = reinterpret_cast<Acc *>(s_node + lds_nodes);   // [D]
  Acc *sb = best + D;                                        // [D] prefix sum before the device's first gap
  Acc *wsum = sb + D;                                        // [16] sums of the waves' runs
  int *gb = reinterpret_cast<int *>(wsum + 16);              // [D + 1] first flat entry of the device
  uint32_t *misc = reinterpret_cast<uint32_t *>(gb + D + 1);  // [0] ticket, [1] hard gaps, [2] events, [3] violated, [4] listed ops
  WideLds wl{nullptr, nullptr};
  if (kCsr) {  // [W][D] each
    unsigned char *p = reinterpret_cast<unsigned char *>((reinterpret_cast<uintptr_t>(misc + 5) + 7) & ~uintptr_t(7));
    wl.last = reinterpret_cast<uint64_t *>(p) + (size_t)w * D;
    wl.low = reinterpret_cast<uint32_t *>(p + (size_t)W * D * 8) + (size_t)w * D;
    for (int d = lane; d < D; d += kWave) {
      wl.last[d] = 0;
      wl.low[d] = kInf32;
    }
  }
  // while the ranks are made: op counts [W][D] on A and F, lane masks [W][D] past them
  uint64_t *mask = reinterpret_cast<uint64_t *>(A) + (size_t)w * D;
  uint32_t *hist = reinterpret_cast<uint32_t *>(reinterpret_cast<uint64_t *>(A) + (size_t)W * D);
  uint32_t *whist = hist + (size_t)w * D;
  const int sh = kNarrow ? G.peak_shift : 0;
  uint16_t *gap_of = gap_all + (int64_t)blockIdx.x * N;
  uint16_t *list = list_all + (int64_t)blockIdx.x * N;  // ops with a consumer on another device
  const int seg = ((N + T - 1) / T) * kWave;  // ops of a wave while ranks are made

  // Candidates: kPeakTickets contiguous ranges, each with its share of the
  // workgroups and a counter on a line of its own (one counter for all took
  // 14 ns a candidate, as long as a small candidate's work over the chip);
  // a workgroup's first candidate needs none, the next is fetched meanwhile.
  const int n_cls = min(kPeakTickets, (int)gridDim.x), cls = blockIdx.x % n_cls;
  const int64_t c_hi = nb * (cls + 1) / n_cls, c_lo = nb * cls / n_cls;
  const int64_t c_rest = c_lo + ((int)gridDim.x - cls + n_cls - 1) / n_cls;  // past the first ones
  int64_t c_next = c_lo + blockIdx.x / n_cls;
  for (;;) {
    __syncthreads();  // the last candidate's LDS state has been read
    if (tid == 0) {
      misc[0] = (uint32_t)(c_next < c_hi ? c_next : nb);
      misc[1] = misc[2] = misc[3] = misc[4] = 0;
      c_next = c_rest < c_hi ? c_rest + atomicAdd(&ticket[cls * kTicketPitch], 1u) : nb;
    }
    for (int d = lane; d < D; d += kWave) {
      whist[d] = 0;
      mask[d] = 0;
    }
    __syncthreads();
    const int64_t c = misc[0];
    if (c >= nb) return;
    if (violation[c] & (SS_VIOLATION_INVALID | SS_VIOLATION_RETRY)) {
      if (peak)
        for (int d = tid; d < D; d += T) peak[c * D + d] = 0;
      continue;
    }
    const uint8_t *prow = P + c * N;
    const uint32_t *frow = fin + c * fpitch;
    const uint32_t *arow = kPorts ? arr + c * E : nullptr;
    uint16_t *rk = rank_all + (kGiven ? c : (int64_t)blockIdx.x) * N;

    // Each wave counts its segment's ops per device; with index ranks it ranks
    // them too, among the segment's: the lanes of a chunk on one device come
    // from a lane mask per device, and the lowest of them moves the count on
    // (many lanes of a chunk share a device where a request's ops follow each
    // other on it, and an atomic from each would take its turn).
    const int v_lo = min(w * seg, N), v_hi = min(v_lo + seg, N);
    if (v_lo < v_hi) {
      uint32_t dn = prow[min(v_lo + lane, v_hi - 1)];
      for (int v0 = v_lo; v0 < v_hi; v0 += kWave) {
        const int v = v0 + lane;
        const bool act = v < v_hi;
        const uint32_t d = dn;
        dn = prow[min(v + kWave, v_hi - 1)];  // the next chunk's, in flight meanwhile
        if (act) atomicOr(reinterpret_cast<unsigned long long *>(&mask[d]), 1ull << lane);
        wave_lds_fence();
        const uint64_t peers = mask[d];
        const uint32_t before = whist[d];
        wave_lds_fence();
        const uint32_t below =
            __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
        if (act) {
          if (below == 0) {
            mask[d] = 0;
            whist[d] = before + (uint32_t)__popcll(peers);
          }
          if (!kGiven) rk[v] = (uint16_t)(before + below);
        }
        wave_lds_fence();
      }
    }
    __syncthreads();
    for (int d = tid; d < D; d += T) {
      uint32_t s = 0;
      for (int k = 0; k < W; ++k) {
        const uint32_t t = hist[(size_t)k * D + d];
        hist[(size_t)k * D + d] = s;
        s += t;
      }
      gb[d] = (int)s + 1;
    }
    __syncthreads();
    if (w == 0) {  // counts to first flat entries
      int carry = 0;
      for (int d0 = 0; d0 < D; d0 += kWave) {
        const int d = d0 + lane, x = d < D ? gb[d] : 0;
        int s = x;
        for (int o = 1; o < kWave; o <<= 1) {
          const int y = __shfl_up(s, o, kWave);
          if (lane >= o) s += y;
        }
        if (d < D) {
          gb[d] = carry + s - x;
          S[carry + s - 1] = kInf32;  // sentinel past the device's last start
        }
        carry += __shfl(s, kWave - 1, kWave);
      }
      if (lane == 0) gb[D] = carry;
    }
    __syncthreads();
    // every op's rank on its device and its start
    if (v_lo < v_hi) {
      auto load = [&](int v, uint32_t &d, uint32_t &r, uint32_t &f, uint32_t &w_) {
        v = min(v, v_hi - 1);
        d = prow[v];
        r = rk[v];
        f = frow[v];
        w_ = !kCsr || C == 1 ? G.dur32[v] : 0u;
      };
      uint32_t dn, rn, fn, wn;
      load(v_lo + lane, dn, rn, fn, wn);
      for (int v0 = v_lo; v0 < v_hi; v0 += kWave) {
        const int v = v0 + lane;
        const uint32_t d = dn, f = fn;
        uint32_t r = rn, dur = wn;
        load(v + kWave, dn, rn, fn, wn);  // in flight meanwhile
        if (v < v_hi) {
          if (!kGiven) {
            r += whist[d];
            rk[v] = (uint16_t)r;
          }
          if (kCsr && C != 1) dur = G.dur32[(int64_t)v * C + G.dev_class[d]];
          S[gb[d] + r] = f - dur;
        }
      }
    }
    __syncthreads();
    for (int q = tid; q < n; q += T) {
      A[q] = 0;
      F[q] = 0;
    }
    __syncthreads();

    // bytes allocated and freed per gap: ops whose consumers are all local at
    // once; those with a remote one, whose gaps take searches, go to a list and
    // are taken from it with full lanes (a candidate that moves a few ops has
    // one or two of them in every chunk)
    for (int v0 = w * kWave; v0 < N; v0 += T) {
      const int v = v0 + lane, vc = min(v, N - 1);
      const bool act = v < N;
      const OpIn op = load_op<kCsr>(G, prow, frow, rk, vc);
      const uint32_t b = op.b >> sh;
      uint32_t gap = kNoGap;
      bool listed;
      if (kCsr) {
        Accumulate<Acc> ev{A, F, kNoGap, false};
        op_events<kCsr, kShift, kPorts>(G, prow, frow, rk, arow, vc, act, op, SuccIn{}, sh, S, gb, wl, ev);
        listed = act && ev.remote;
        gap = listed ? kNoGap : ev.gap;
      } else {
        const SuccIn su = load_succ<kCsr>(prow, frow, rk, op, vc);
        const bool has0 = act && (op.s2 & 0xFFFFu) != 0xFFFFu;
        // (absent successors repeat the op itself)
        listed = act && (su.dx0 != op.d || su.dx1 != op.d);
        if (has0 && !listed) {
          gap = (uint32_t)(gb[op.d] + (int)(su.fx1 > su.fx0 ? su.rx1 : su.rx0) + 1);
          lds_add(&F[gap], (Acc)b);
        }
      }
      const uint64_t m = __ballot(listed);
      if (m) {
        int at = lane == 0 ? (int)atomicAdd(&misc[4], (uint32_t)__popcll(m)) : 0;
        at = __builtin_amdgcn_readfirstlane(at);
        if (listed) list[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
            (uint16_t)v;
      }
      if (act) {
        lds_add(&A[gb[op.d] + op.rv + 1], (Acc)b);  // the own output opens gap rank + 1
        gap_of[v] = (uint16_t)gap;
      }
    }
    __syncthreads();
    const int n_list = (int)misc[4];
    // the listed ops' events, passed to ev (CSR graphs: in the second walk only)
    auto walk_list = [&](auto ev) {
      for (int i0 = w * kWave; i0 < n_list; i0 += T) {
        const bool act = i0 + lane < n_list;
        const int v = list[min(i0 + lane, n_list - 1)];
        const OpIn op = load_op<kCsr>(G, prow, frow, rk, v);
        op_events<kCsr, kShift, kPorts>(G, prow, frow, rk, arow, v, act, op, load_succ<kCsr>(prow, frow, rk, op, v), sh,
                                        S, gb, wl, ev);
      }
    };
    if (!kCsr) {
      walk_list(Accumulate<Acc>{A, F, kNoGap, false});
      __syncthreads();
    }
    // prefix sums over the flat entries (modulo 2^32 with 32-bit sums): each
    // thread a run, of odd length so that the lanes' accesses spread over the banks
    {
      const int per = ((n + T - 1) / T) | 1, lo = min(tid * per, n), hi = min(lo + per, n);
      Acc s = 0;
      for (int q = lo; q < hi; ++q) s += A[q] - F[q];
      Acc incl = s;
      for (int o = 1; o < kWave; o <<= 1) {
        const Acc y = shfl_up(incl, o);
        if (lane >= o) incl += y;
      }
      if (lane == kWave - 1) wsum[w] = incl;
      __syncthreads();
      Acc run = incl - s;
      for (int k = 0; k < w; ++k) run += wsum[k];
      for (int q = lo; q < hi; ++q) {
        run += A[q] - F[q];
        A[q] = run;
      }
    }
    __syncthreads();
    for (int d = tid; d < D; d += T) {
      sb[d] = d > 0 ? A[gb[d] - 1] : (Acc)0;
      best[d] = 0;
    }
    __syncthreads();
    // the exact values: live bytes at every own start
    // (few raise their device's best: reading it first spares the atomic)
    for (int v0 = tid; v0 < N; v0 += 4 * T) {
      uint32_t d[4], r[4], b[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int v = min(v0 + k * T, N - 1);
        d[k] = prow[v];
        r[k] = rk[v];
        b[k] = G.bytes32[v] >> sh;
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {  // (the last op again past the end)
        const Acc live = A[gb[d[k]] + r[k]] - sb[d[k]] + (Acc)b[k];
        if (live > best[d[k]]) lds_max(&best[d[k]], live);
      }
    }
    __syncthreads();
    // hard gaps: their bound replaces their frees, an empty list their sum
    for (int d = w; d < D; d += W) {
      const Acc base = sb[d], top = best[d];
      const int q1 = gb[d + 1];
      bool any = false;
      for (int q = gb[d] + lane; q < q1; q += kWave) {
        const Acc U = A[q] - base + F[q];
        const bool hard = U > top;
        F[q] = U;
        *reinterpret_cast<uint32_t *>(&A[q]) = hard ? kEmpty : kEasy;
        any |= hard;
      }
      if (any) misc[1] = 1;
    }
    __syncthreads();
    if (misc[1]) {
      // the events of the hard gaps: own frees that fall into one, and the
      // listed ops'
      auto collect = [&](uint4 *node, uint32_t cap) {
        Collect<Acc> ev{A, node, &misc[2], cap};
        for (int v0 = w * kWave; v0 < N; v0 += T) {
          const int v = v0 + lane, vc = min(v, N - 1);
          const uint32_t q = gap_of[vc];
          const bool act = v < N && q != kNoGap && *reinterpret_cast<const uint32_t *>(&A[q]) != kEasy;
          if (!__any(act)) continue;
          const OpIn op = load_op<kCsr>(G, prow, frow, rk, vc);
          op_events<kCsr, kShift, kPorts>(G, prow, frow, rk, arow, vc, act, op, load_succ<kCsr>(prow, frow, rk, op, vc),
                                          sh, S, gb, wl, ev);
        }
        walk_list(ev);
        __syncthreads();
      };
      // live bytes at each collected allocation: the gap's bound less the
      // copies allocated later and the frees at or before it
      auto sweep = [&](const uint4 *node, uint32_t cnt) {
        for (uint32_t i = tid; i < cnt; i += T) {
          const uint4 me = node[i];
          if (!(me.z >> 24)) continue;
          const uint32_t q = me.z & 0xFFFFu;
          Acc live = F[q];
          for (uint32_t z = *reinterpret_cast<const uint32_t *>(&A[q]); z != kEmpty;) {
            const uint4 o = node[z];
            if ((o.z >> 24) ? o.x > me.x : o.x <= me.x) live -= (Acc)o.y;
            z = o.w;
          }
          lds_max(&best[(me.z >> 16) & 0xFFu], live);
        }
      };
      collect(s_node, (uint32_t)lds_nodes);
      const uint32_t cnt = misc[2];
      if (cnt <= (uint32_t)lds_nodes) {
        sweep(s_node, cnt);
      } else {  // more events than the LDS holds: once more, into the block's global list
        __syncthreads();
        if (tid == 0) misc[2] = 0;
        for (int q = tid; q < n; q += T) {
          uint32_t *head = reinterpret_cast<uint32_t *>(&A[q]);
          if (*head != kEasy) *head = kEmpty;
        }
        __syncthreads();
        uint4 *node = node_all + (int64_t)blockIdx.x * node_cap;
        collect(node, (uint32_t)node_cap);
        sweep(node, misc[2]);
      }
      __syncthreads();
    }
    bool over = false;
    for (int d = tid; d < D; d += T) {
      const int64_t pk = kNarrow ? (int64_t)best[d] << sh : (int64_t)best[d];
      if (peak) peak[c * D + d] = pk;
      over |= pk > G.cap[d];
    }
    if (over) misc[3] = 1;
    __syncthreads();
    if (tid == 0) violation[c] = misc[3] ? SS_VIOLATION_MEMORY : 0;
  }
}

template <bool kNarrow>
const void *peaks_fn(bool csr, bool given, bool shift, bool ports) {
#define SS_PEAKS(c, g, s, p) reinterpret_cast<const void *>(&lds_peaks<c, g, s, p, kNarrow>)
  if (csr) return given ? SS_PEAKS(true, true, false, false) : SS_PEAKS(true, false, false, false);
  if (ports) return shift ? SS_PEAKS(false, false, true, true) : SS_PEAKS(false, false, false, true);
  if (given) return shift ? SS_PEAKS(false, true, true, false) : SS_PEAKS(false, true, false, false);
  return shift ? SS_PEAKS(false, false, true, false) : SS_PEAKS(false, false, false, false);
#undef SS_PEAKS
}

int hip_fail(hipError_t err, const char *what) {
  return ss_set_error(err == hipErrorOutOfMemory ? SS_ERR_OOM : SS_ERR_DEVICE,
                      std::string(what) + ": " + hipGetErrorString(err));
}

}  // namespace

PeaksShape ss_peaks_shape(const ss_gmg *g, bool ports, int cus, int64_t lds_block, int64_t lds_cu) {
  PeaksShape s;
  const int64_t N = g->n_ops, D = g->n_dev, n4 = (N + D + 3) / 4 * 4;
  const int64_t acc = g->view.peak_narrow ? 4 : 8;
  s.csr = !(g->n_class == 1 && g->n_link <= 2 && g->max_outdeg <= 2);
  if (N == 0 || N + D >= kMaxFlat || (ports && (s.csr || !g->view.succ2_pe))) return s;
  // about one event per ten ops falls into hard gaps when every op is placed at random
  s.lds_nodes = (int)std::max<int64_t>(64, N / 8);
  int64_t lds = n4 * (2 * acc + 4) + s.lds_nodes * 16 + (2 * D + 16) * acc + (D + 1) * 4 + 32;
  const int64_t wave_lds = s.csr ? 12 * D : 0;  // the device arrays of ops with many successors
  if (lds + wave_lds > lds_block) return s;
  // The waves per CU that the registers allow, in as many workgroups as there
  // are tables that fit it: 16 with the CSR's 108 registers, so a power of two
  // each (5,000 ops with wide successors, two tables: 3.5 ms in workgroups of
  // ten, of which a CU holds one, 2.4 in two of eight); of 24 otherwise at
  // least twenty (100,003 candidates of 2,052 ops 3.6 ms with fifteen, 3.2 with
  // twenty).  None with less than two chunks of 64 ops; the ranks' counts and
  // masks (12 bytes per wave and device) lie on A and F.
  const int64_t fit = std::max<int64_t>(1, lds_cu / lds), resident = s.csr ? 16 : 24;
  int64_t waves = 1;
  if (s.csr) {
    while (waves * fit < resident) waves *= 2;
  } else {
    waves = std::min<int64_t>(16, (20 + fit - 1) / fit);
  }
  waves = std::min(waves, (N + 2 * kWave - 1) / (2 * kWave));
  waves = std::max<int64_t>(1, std::min(waves, 2 * acc * n4 / (12 * D)));
  if (s.csr) {
    // where the table leaves room for the device arrays of one wave alone, the
    // records are faster (4,096 candidates of 11,300 ops on 128 devices at
    // random: 25.8 ms with one wave, 18.5 with records; of 10,000 ops 11.5 with
    // two waves on 64 devices, 15.8 with records on 128)
    const int64_t most = (lds_block - lds) / wave_lds;
    if (most < std::min<int64_t>(waves, 2)) return s;
    waves = std::min(waves, most);
  }
  lds += waves * wave_lds;
  s.lds = (size_t)lds;
  s.threads = (int)waves * kWave;
  // (those past the resident waves start as others run out of candidates, which
  // evens out their ranges: 32,771 candidates of 2,001 ops with wide successors
  // 6.51 ms the call, 6.58 with no more workgroups than are resident, at random
  // 7.87 and 8.00; graphs without show no difference)
  s.blocks = (int64_t)cus * std::max<int64_t>(1, std::min<int64_t>(lds_cu / lds, 32 / waves));
  s.node_cap = N + 2 * g->n_edges + 1;
  s.ok = 12 * D * waves <= 2 * acc * n4;
  return s;
}

size_t ss_peaks_slot_bytes(const ss_gmg *g, const PeaksShape &s, bool given_ranks) {
  auto align = [](size_t x) { return (x + 255) & ~size_t(255); };
  const size_t N = (size_t)g->n_ops;
  return align(N * 2) * (given_ranks ? 2 : 3) + align((size_t)s.node_cap * sizeof(uint4));
}

int ss_launch_peaks(const ss_gmg *g, const PeaksShape &s, const uint8_t *P, const uint32_t *fin, int64_t fpitch,
                    const uint32_t *arr, uint16_t *given, void *slots, int64_t n_slots, int64_t nb, uint32_t *ticket,
                    int64_t *peak, uint8_t *violation, hipStream_t stream) {
  const GmgView &G = g->view;
  auto align = [](size_t x) { return (x + 255) & ~size_t(255); };
  const int64_t N = g->n_ops, slots_n = std::min(n_slots, nb);
  auto *p = static_cast<unsigned char *>(slots);
  auto *node = reinterpret_cast<uint4 *>(p);
  p += align((size_t)s.node_cap * sizeof(uint4)) * (size_t)n_slots;
  auto *gap = reinterpret_cast<uint16_t *>(p);
  p += align((size_t)N * 2) * (size_t)n_slots;
  auto *list = reinterpret_cast<uint16_t *>(p);
  p += align((size_t)N * 2) * (size_t)n_slots;
  uint16_t *rank = given ? given : reinterpret_cast<uint16_t *>(p);
  const bool shift = G.link_shift >= 0;
  const void *fn = G.peak_narrow ? peaks_fn<true>(s.csr, given, shift, arr) : peaks_fn<false>(s.csr, given, shift, arr);
  int64_t node_cap = s.node_cap;
  int lds_nodes = s.lds_nodes;
  void *args[] = {const_cast<GmgView *>(&G), &P, &fin, &fpitch, &arr, &rank, &gap, &list, &node, &node_cap, &lds_nodes, &nb,
                  &ticket, &peak, &violation};
  hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)s.lds);
  if (err != hipSuccess) return hip_fail(err, "hipFuncSetAttribute");
  SsTimingRec *t = ss_timing_start(SS_KERNEL_MEMORY, stream);
  err = hipLaunchKernel(fn, dim3((unsigned)slots_n), dim3((unsigned)s.threads), args, s.lds, stream);
  ss_timing_stop(t, stream);
  if (err == hipSuccess) err = hipGetLastError();
  return err == hipSuccess ? SS_OK : hip_fail(err, "lds_peaks launch");
}
