// Transfer ports (SS_LINK_PORTS, Sec. 3.5.2) on 32-bit times for gfx950: the
// event-driven arbitration of port_event_schedule (simulate.hip) for graphs of
// the packed form (at most two successors per op, one device class, at most
// two link classes) whose times the loader proved to fit 32 bits, followed by
// the memory pass of peaks.hip.  One wave per candidate, candidates from a
// ticket counter.
//
// What happens at an instant depends on the pending transfers and the ports
// alone, so only two kinds of instant exist: an op finishes whose output some
// other device waits for (it posts transfers), or a transfer arrives.  Ops
// whose consumers all sit on their own device need no event: they are placed
// as soon as their inputs are known and never looked at again.  A candidate
// that moves a few ops of a partition has about 150 instants in 2,000 ops
// instead of one per op.
//
// Before the events the wave writes every op's record into its device's queue,
// 64 ops at a time: op, request, duration and for its first two inputs whether
// they are local (the producer) or remote (the edge whose arrival counts).
// Placing an op then reads one record (the next one in flight) and, where
// the input is not the op placed just before, one finish or arrival.
// Bound: the latency of those reads and of the event loop's LDS round trips;
// the waves of a CU hide each other's.  32,768 candidates of 2,052 ops that
// move up to 16 of them: 50.6 ms in port_event_schedule, 11.4 ms here; every op
// placed at random (479 of 718 ops): 5.3 and 2.6 ms the whole call.
#include <algorithm>
#include <climits>

#include "peaks.h"

namespace {

constexpr int kWave = 64;
constexpr uint32_t kNever = 0xFFFFFFFFu;   // no event; an arrival not known yet
constexpr uint32_t kNoInput = 0xFFFFFFFFu; // record: no such input
constexpr uint32_t kRemote = 0x80000000u;  // record: the input's arrival, by edge
constexpr uint32_t kMore = 0x40000000u;    // record: further inputs, from the CSR
constexpr int kPendLds = 128;              // pending transfers in LDS; more in the wave's global list
// Waves per CU, each with scratch for its queues; the registers hold 24.
// Schedule of the batch above with 8, 12, 16 and 24: 18.4, 13.8, 11.4 and
// 9.6 ms; 16,384 candidates of 322 ops 8.7, 6.2, 5.1 and 3.8 ms; 16,384 of 2,052
// ops on 128 devices 9.6, 7.3, 7.3 and 7.3 (the LDS holds twelve).
constexpr int kWavesPerCU = 16;

__device__ __forceinline__ uint32_t umax32(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint32_t umin32(uint32_t a, uint32_t b) { return a < b ? a : b; }

// Orders the wave's memory accesses (they complete in issue order).
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <int kCtrl>
__device__ __forceinline__ uint32_t row_move(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xF, 0xF, false);
}

// Smallest value of the wave, in every lane: within rows of 16 lanes by DPP
// moves, then over the four rows' values.
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  v = umin32(v, row_move<0xB1>(v));   // quad_perm {1,0,3,2}
  v = umin32(v, row_move<0x4E>(v));   // quad_perm {2,3,0,1}
  v = umin32(v, row_move<0x141>(v));  // row_half_mirror
  v = umin32(v, row_move<0x140>(v));  // row_mirror
  const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
  const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
  return umin32(umin32(a, b), umin32(c, d));
}

// A device's state, and the next op of its queue that posts transfers.
struct PortDev {
  uint32_t clk, begin, end;  // previous finish; current idle slice
  int32_t cur;               // its index
  int32_t head, qend;        // next op to place, end of the queue
  int32_t post, pend;        // next posting op in the posting list, its end
  int32_t post_at;           // that op's queue position (INT_MAX: none left)
  uint32_t post_op;          // that op
  uint32_t next_fin;         // its finish once placed, else kNever
  uint32_t send, recv;       // the ports are busy until then
  uint32_t arrive;           // arrival of the transfer entering the device, else kNever
  uint32_t dirty;            // the head's inputs may have become known
  uint32_t fill;             // counts and fill positions while the queues are written
  uint32_t pad;              // odd size: lanes of consecutive devices fall in distinct banks
};

__global__ __launch_bounds__(kWave) void port_events32(const GmgView G, const uint8_t *__restrict__ P, int64_t nb,
                                                       uint32_t *__restrict__ fin, uint32_t *__restrict__ arr_all,
                                                       uint4 *__restrict__ rec_all, uint16_t *__restrict__ posts_all,
                                                       uint4 *__restrict__ pend_all, uint32_t *__restrict__ ticket,
                                                       int64_t *__restrict__ makespan, int64_t *__restrict__ sumfin,
                                                       int64_t *__restrict__ slack, uint8_t *__restrict__ violation) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int D = G.n_dev, N = G.n_ops, R = G.n_req, K = G.n_link;
  const int E = G.pred_ptr[N];
  const int lane = threadIdx.x;
  uint4 *s_pend = reinterpret_cast<uint4 *>(lds_raw);                 // [kPendLds]
  uint64_t *mask = reinterpret_cast<uint64_t *>(s_pend + kPendLds);   // [D] a chunk's lanes on each device
  PortDev *dev = reinterpret_cast<PortDev *>(mask + D);               // [D]
  uint32_t *comp = reinterpret_cast<uint32_t *>(dev + D);             // [R]
  uint4 *rec = rec_all + (int64_t)blockIdx.x * N;
  uint16_t *posts = posts_all + (int64_t)blockIdx.x * N;
  uint4 *g_pend = pend_all + (int64_t)blockIdx.x * (E + 1);
  const uint64_t below = (1ull << lane) - 1;
  const uint32_t *m_req = G.op_meta + (int64_t)kMetaReq * G.meta_stride;
  const uint32_t *m_p01 = G.op_meta + (int64_t)kMetaP01 * G.meta_stride;
  const uint32_t *m_e0 = G.op_meta + (int64_t)kMetaE0 * G.meta_stride;
  auto link_of = [&](uint32_t a, uint32_t b) -> uint32_t {
    return (G.link_bits[a * G.link_words + (b >> 5)] >> (b & 31)) & 1u;
  };
  auto pend_at = [&](int i) -> uint4 & { return i < kPendLds ? s_pend[i] : g_pend[i]; };

  for (;;) {
    const uint32_t tk = lane == 0 ? atomicAdd(ticket, 1u) : 0u;
    const int64_t c = (uint32_t)__builtin_amdgcn_readfirstlane((int)tk);
    if (c >= nb) return;
    const uint8_t *prow = P + c * N;
    uint32_t *frow = fin + c * N;
    uint32_t *arr = arr_all + c * E;
    // a candidate naming a device outside the set is not simulated
    bool bad = false;
    for (int v = lane; v < N; v += kWave) bad = bad || prow[v] >= D;
    if (__any(bad)) {
      if (lane == 0) {
        makespan[c] = INT64_MAX;
        if (sumfin) sumfin[c] = INT64_MAX;
        violation[c] = SS_VIOLATION_INVALID;
      }
      if (slack)
        for (int r = lane; r < R; r += kWave) slack[c * R + r] = INT64_MIN;
      continue;
    }
    // ops and posting ops per device
    for (int d = lane; d < D; d += kWave) {
      dev[d].fill = 0;
      dev[d].post = 0;
      mask[d] = 0;
    }
    for (int r = lane; r < R; r += kWave) comp[r] = G.release32[r];
    wave_fence();
    auto posting = [&](int v, uint32_t d) -> bool {
      const uint32_t s2 = G.succ2[v], i0 = s2 & 0xFFFFu, i1 = s2 >> 16;
      return (i0 != 0xFFFFu && prow[i0] != d) || (i1 != 0xFFFFu && prow[i1] != d);
    };
    for (int v = lane; v < N; v += kWave) {
      const uint32_t d = prow[v];
      atomicAdd(&dev[d].fill, 1u);
      if (posting(v, d)) atomicAdd(&dev[d].post, 1);
    }
    for (int e = lane; e < E; e += kWave) arr[e] = kNever;
    wave_fence();
    {
      int q0 = 0, p0 = 0;
      for (int d0 = 0; d0 < D; d0 += kWave) {
        const int d = d0 + lane;
        const int nq = d < D ? (int)dev[d].fill : 0, np = d < D ? dev[d].post : 0;
        int sq = nq, sp = np;
        for (int o = 1; o < kWave; o <<= 1) {
          const int yq = __shfl_up(sq, o, kWave), yp = __shfl_up(sp, o, kWave);
          if (lane >= o) {
            sq += yq;
            sp += yp;
          }
        }
        if (d < D) {
          PortDev &x = dev[d];
          const int sl = G.slice_ptr[d];
          x.clk = x.send = x.recv = 0;
          x.begin = G.slice_begin32[sl];
          x.end = G.slice_end32[sl];
          x.cur = 0;
          x.head = (int)(x.fill = (uint32_t)(q0 + sq - nq));
          x.qend = q0 + sq;
          x.post = x.post_at = p0 + sp - np;  // post_at: fill position of the posting list meanwhile
          x.pend = p0 + sp;
          x.next_fin = x.arrive = kNever;
          x.dirty = 1;
        }
        q0 += __shfl(sq, kWave - 1, kWave);
        p0 += __shfl(sp, kWave - 1, kWave);
      }
    }
    wave_fence();
    // the queues' records, and the queue positions of the posting ops
    for (int v0 = 0; v0 < N; v0 += kWave) {
      const int v = min(v0 + lane, N - 1);
      const bool act = v0 + lane < N;
      const uint32_t d = prow[v];
      const bool post = act && posting(v, d);
      if (act) atomicOr(reinterpret_cast<unsigned long long *>(&mask[d]), 1ull << lane);
      const uint64_t poster = __ballot(post);
      wave_fence();
      const uint64_t peers = mask[d];
      const int at = (int)dev[d].fill + __popcll(peers & below);
      const int pat = dev[d].post_at + __popcll(peers & poster & below);
      wave_fence();
      const uint32_t rq = m_req[v], np = rq >> 16, p01 = m_p01[v], e0 = m_e0[v];
      auto code = [&](uint32_t i) -> uint32_t {
        if (i >= np) return kNoInput;
        const uint32_t u = i ? p01 >> 16 : p01 & 0xFFFFu;
        return prow[u] == d ? u : (kRemote | (e0 + i));
      };
      if (act) {
        mask[d] = 0;
        atomicAdd(&dev[d].fill, 1u);
        if (post) {
          atomicAdd(&dev[d].post_at, 1);
          posts[pat] = (uint16_t)at;
        }
        const uint32_t c1 = code(1);
        rec[at] = make_uint4((uint32_t)v | (rq & 0xFFFFu) << 16, G.dur32[v], code(0), np > 2 ? c1 | kMore : c1);
      }
      wave_fence();
    }
    __threadfence_block();
    // the next posting op of a device, read after its posting list moved on
    auto next_post = [&](PortDev &x) {
      if (x.post < x.pend) {
        x.post_at = posts[x.post];
        x.post_op = rec[x.post_at].x & 0xFFFFu;
        x.next_fin = x.post_at < x.head ? frow[x.post_op] : kNever;
      } else {
        x.post_at = INT_MAX;
        x.next_fin = kNever;
      }
    };
    for (int d = lane; d < D; d += kWave) next_post(dev[d]);
    wave_fence();

    uint32_t ms = 0;
    uint64_t sum = 0;
    int npend = 0;
    // every instant consumes at least one finish or arrival, so N + E + 1
    // instants are enough; the bound only guarantees that the wave exits
    bool stuck = false;
    for (int step = 0;; ++step) {
      if (step > N + E + 1) {
        stuck = true;
        break;
      }
      // place every queue head whose inputs are known; the next instant
      uint32_t t = kNever;
      for (int d = lane; d < D; d += kWave) {
        PortDev &x = dev[d];
        if (x.dirty) {
          x.dirty = 0;
          int h = x.head;
          const int qend = x.qend, post_at = x.post_at;
          uint32_t clk = x.clk, begin = x.begin, end = x.end, last_v = kNoInput, last_f = 0;
          uint4 r = rec[min(h, N - 1)];
          while (h < qend) {
            const uint4 rn = rec[min(h + 1, N - 1)];  // in flight while op h is placed
            const uint32_t v = r.x & 0xFFFFu, rq = r.x >> 16, w = r.y;
            bool known = true;
            auto input = [&](uint32_t k) -> uint32_t {
              if (k == kNoInput) return 0;
              if (!(k & kRemote)) return k == last_v ? last_f : frow[k];  // earlier in this queue, hence placed
              const uint32_t a = arr[k & 0xFFFFu];
              known = known && a != kNever;
              return a;
            };
            uint32_t ready = umax32(G.release32[rq], umax32(input(r.z), input(r.w == kNoInput ? kNoInput : r.w & ~kMore)));
            if (r.w != kNoInput && (r.w & kMore)) {
              const int e1 = G.pred_ptr[v + 1];
              for (int e = G.pred_ptr[v] + 2; e < e1; ++e) {
                const uint32_t u = (uint32_t)G.pred_idx[e];
                ready = umax32(ready, input(prow[u] == (uint32_t)d ? u : (kRemote | (uint32_t)e)));
              }
            }
            if (!known) break;
            const uint32_t s0 = umax32(ready, clk);
            uint32_t s = umax32(s0, begin);
            if (s + w > end) {
              int k = x.cur;
              const int sl = G.slice_ptr[d];
              do {
                ++k;
                begin = G.slice_begin32[sl + k];
                end = G.slice_end32[sl + k];
                s = umax32(s0, begin);
              } while (s + w > end);
              x.cur = k;
            }
            const uint32_t f = s + w;
            frow[v] = f;
            clk = last_f = f;
            last_v = v;
            if (h == post_at) x.next_fin = f;
            ms = umax32(ms, f);
            sum += f;
            atomicMax(&comp[rq], f);
            ++h;
            r = rn;
          }
          x.head = h;
          x.clk = clk;
          x.begin = begin;
          x.end = end;
        }
        t = umin32(t, umin32(x.next_fin, x.arrive));
      }
      t = wave_min(t);
      if (t == kNever) break;
      wave_fence();
      // arrivals at t: the ports they held are idle from t on
      for (int d = lane; d < D; d += kWave)
        if (dev[d].arrive == t) dev[d].arrive = kNever;
      // finishes at t, in producer index order: their Intents, by destination
      for (;;) {
        uint32_t key = kNever;  // op << 8 | device
        for (int d = lane; d < D; d += kWave)
          if (dev[d].next_fin == t) key = umin32(key, dev[d].post_op << 8 | (uint32_t)d);
        const uint64_t any = __ballot(key != kNever);
        if (!any) break;
        key = (any & (any - 1)) ? wave_min(key)
                                : (uint32_t)__builtin_amdgcn_readlane((int)key, __ffsll((unsigned long long)any) - 1);
        const uint32_t u = key >> 8, du = key & 0xFFu;
        if (lane == 0) {
          ++dev[du].post;
          next_post(dev[du]);
        }
        const uint32_t s2 = G.succ2[u], pe = G.succ2_pe[u];
        uint32_t e0 = (s2 & 0xFFFFu) != 0xFFFFu ? prow[s2 & 0xFFFFu] : du;
        uint32_t e1 = (s2 >> 16) != 0xFFFFu ? prow[s2 >> 16] : du;
        uint32_t pe0 = pe & 0xFFFFu, pe1 = pe >> 16;
        if (e1 < e0) {  // destinations in increasing device order
          uint32_t x = e0;
          e0 = e1;
          e1 = x;
          x = pe0;
          pe0 = pe1;
          pe1 = x;
        }
        const bool shared = e0 == e1;  // one transfer for both
        auto send = [&](uint32_t e, uint32_t edges) {  // edges: one or two, u16 each (0xFFFF: none)
          const uint32_t x = G.xfer32[u * K + (K > 1 ? link_of(du, e) : 0u)];
          if (lane == 0) {
            if (x == 0) {  // nothing moves: complete at its request
              arr[edges & 0xFFFFu] = t;
              if ((edges >> 16) != 0xFFFFu) arr[edges >> 16] = t;
              dev[e].dirty = 1;
            } else {
              pend_at(npend) = make_uint4(edges, e | du << 8, x, 0u);
            }
          }
          npend += x != 0;
        };
        if (e0 != du) send(e0, pe0 | (shared ? pe1 << 16 : 0xFFFF0000u));
        if (e1 != du && !shared) send(e1, pe1 | 0xFFFF0000u);
        wave_fence();
      }
      // arbitration at t: pending transfers in order, each started when both
      // of its ports are idle; the rest kept in order
      int kept = 0;
      for (int b0 = 0; b0 < npend; b0 += kWave) {
        const int i = b0 + lane;
        const bool valid = i < npend;
        const uint4 ent = valid ? pend_at(i) : make_uint4(0, 0, 0, 0);
        const uint32_t e = ent.y & 0xFFu, s = ent.y >> 8;
        bool started = false;
        for (;;) {
          const bool elig = valid && !started && dev[s].send <= t && dev[e].recv <= t;
          const uint64_t m = __ballot(elig);
          if (!m) break;
          if (lane == __ffsll((unsigned long long)m) - 1) {
            const uint32_t a = t + ent.z;
            dev[s].send = a;
            dev[e].recv = a;
            dev[e].arrive = a;
            dev[e].dirty = 1;
            started = true;
          }
          wave_fence();
        }
        if (started) {
          const uint32_t a = t + ent.z;
          arr[ent.x & 0xFFFFu] = a;
          if ((ent.x >> 16) != 0xFFFFu) arr[ent.x >> 16] = a;
        }
        const uint64_t km = __ballot(valid && !started);
        wave_fence();
        if (valid && !started) pend_at(kept + __popcll(km & below)) = ent;
        kept += __popcll(km);
        wave_fence();
      }
      npend = kept;
    }
    // completion-time statistics (Sec. 3.3.3); every queue has run out (a
    // queue left with ops would be a defect: its makespan reads -1)
    for (int d = lane; d < D; d += kWave) stuck = stuck || dev[d].head < dev[d].qend;
    for (int o = kWave / 2; o >= 1; o >>= 1) {
      ms = umax32(ms, (uint32_t)__shfl_xor((int)ms, o, kWave));
      sum += (uint64_t)__shfl_xor((int64_t)sum, o, kWave);
    }
    const bool failed = __any(stuck);
    if (lane == 0) {
      makespan[c] = failed ? -1 : (int64_t)ms;
      if (sumfin) sumfin[c] = (int64_t)sum;
      violation[c] = 0;
    }
    wave_fence();
    if (slack)
      for (int r = lane; r < R; r += kWave) slack[c * R + r] = G.deadline[r] - (int64_t)comp[r];
    wave_fence();
  }
}

size_t ports_lds(int64_t D, int64_t R) {
  return (size_t)kPendLds * 16 + (size_t)D * (sizeof(PortDev) + 8) + (size_t)R * 4 + 16;
}

__global__ __launch_bounds__(256) void zero_words(uint32_t *p, int n) {
  for (int i = threadIdx.x; i < n; i += 256) p[i] = 0;
}

int hip_fail(hipError_t err, const char *what) {
  return ss_set_error(err == hipErrorOutOfMemory ? SS_ERR_OOM : SS_ERR_DEVICE,
                      std::string(what) + ": " + hipGetErrorString(err));
}

}  // namespace

bool ss_ports32_ok(const ss_gmg *g) {
  if (!g->view.time32 || g->n_ops == 0 || g->n_edges == 0 || g->n_edges >= 0xFFFF || g->n_class != 1 ||
      g->n_link > 2 || g->max_outdeg > 2 || !g->view.succ2_pe || g->n_req > 4096)
    return false;
  int cus = 0, lds_block = 0, lds_cu = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, g->device) != hipSuccess ||
      hipDeviceGetAttribute(&lds_block, hipDeviceAttributeMaxSharedMemoryPerBlock, g->device) != hipSuccess ||
      hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, g->device) != hipSuccess)
    return false;
  return ss_peaks_shape(g, true, cus, lds_block, lds_cu).ok;
}

int ss_run_simulate_ports32(const ss_gmg *g, SsPlace src, int64_t *makespan, int64_t *peak, uint8_t *violation,
                            int64_t *slack, int64_t *sumfin, hipStream_t stream, SsWork &W) {
  const GmgView &G = g->view;
  const int64_t N = g->n_ops, E = g->n_edges, D = g->n_dev, R = g->n_req, B = src.B;
  int cus = 0, lds_block = 0, lds_cu = 0;
  hipError_t err = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, g->device);
  if (err == hipSuccess)
    err = hipDeviceGetAttribute(&lds_block, hipDeviceAttributeMaxSharedMemoryPerBlock, g->device);
  if (err == hipSuccess)
    err = hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, g->device);
  if (err != hipSuccess) return hip_fail(err, "hipDeviceGetAttribute");
  const PeaksShape pk = ss_peaks_shape(g, true, cus, lds_block, lds_cu);
  const size_t pk_slot = ss_peaks_slot_bytes(g, pk, false), lds = ports_lds(D, R);
  const int64_t waves = (int64_t)cus * std::max<int64_t>(1, std::min<int64_t>(kWavesPerCU, lds_cu / (int64_t)lds));
  auto align = [](size_t x) { return (x + 255) & ~size_t(255); };
  // per candidate: finish and arrival rows (and placement rows from op-major
  // input); per wave: queues, posting list and pending transfers
  const size_t sz_tk = align((size_t)(kTicketPitch + kTicketWords) * 4);
  struct Plan {
    int64_t chunk, waves, slots;
    size_t sz_fin, sz_arr, sz_rows, sz_rec, sz_post, sz_pend, sz_slots, total;
  };
  auto plan_of = [&](int64_t chunk) {
    Plan q{};
    q.chunk = chunk = std::min<int64_t>(std::max<int64_t>(1, chunk), B);
    q.waves = std::min(waves, chunk);
    q.slots = std::min(pk.blocks, chunk);
    q.sz_fin = align((size_t)(chunk * N) * 4);
    q.sz_arr = align((size_t)(chunk * E) * 4);
    q.sz_rows = src.op_major ? align((size_t)(chunk * N) + 1) : 0;
    q.sz_rec = align((size_t)(q.waves * N) * 16);
    q.sz_post = align((size_t)(q.waves * N) * 2);
    q.sz_pend = align((size_t)(q.waves * (E + 1)) * 16);
    q.sz_slots = pk_slot * (size_t)q.slots;
    q.total = q.sz_fin + q.sz_arr + q.sz_rows + q.sz_rec + q.sz_post + q.sz_pend + q.sz_slots + sz_tk;
    return q;
  };
  const int64_t per_cand = (N + E) * 4 + (src.op_major ? N : 0);
  const Plan pmin = plan_of(1), pref = plan_of((int64_t(16) << 30) / per_cand / kWave * kWave);
  if (W.query) {
    W.need_min = pmin.total;
    W.need_pref = pref.total;
    W.chunk = W.sub = pref.chunk;
    return SS_OK;
  }
  Plan pl = pref;
  SsScratch scr;
  void *scratch = nullptr;
  if (W.ptr) {  // the caller's workspace: the largest chunk that fits
    W.need_min = pmin.total;
    if (pmin.total > W.bytes)
      return ss_set_error(SS_ERR_INVALID_ARG, "workspace of " + std::to_string(W.bytes) +
                                                   " bytes is smaller than this call's minimum of " +
                                                   std::to_string(pmin.total));
    int64_t lo = 1, hi = pl.chunk;  // plan_of(lo) fits
    while (lo < hi) {
      const int64_t mid = lo + (hi - lo + 1) / 2;
      if (plan_of(mid).total <= W.bytes) lo = mid;
      else hi = mid - 1;
    }
    pl = plan_of(lo);
    scratch = W.ptr;
  } else {
    for (int64_t chunk = pl.chunk;; chunk = std::max<int64_t>(1, chunk / 2)) {
      pl = plan_of(chunk);
      err = ss_scratch_get(g->device, g->pool, pl.total, stream, &scr);
      if (err != hipErrorOutOfMemory || chunk == 1) break;
    }
    if (err != hipSuccess) return hip_fail(err, "allocating the simulation scratch");
    scratch = scr.p;
  }
  auto *p = static_cast<unsigned char *>(scratch);
  auto take = [&](size_t bytes) {
    unsigned char *q = p;
    p += bytes;
    return q;
  };
  auto *fin = reinterpret_cast<uint32_t *>(take(pl.sz_fin));
  auto *arr = reinterpret_cast<uint32_t *>(take(pl.sz_arr));
  auto *rows = take(pl.sz_rows);
  auto *rec = reinterpret_cast<uint4 *>(take(pl.sz_rec));
  auto *post = reinterpret_cast<uint16_t *>(take(pl.sz_post));
  auto *pend = reinterpret_cast<uint4 *>(take(pl.sz_pend));
  void *slots = take(pl.sz_slots);
  auto *ticket = reinterpret_cast<uint32_t *>(take(sz_tk));  // of the schedule, then of the memory pass
  int rc = SS_OK;
  err = hipFuncSetAttribute(reinterpret_cast<const void *>(&port_events32),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (err != hipSuccess) rc = hip_fail(err, "hipFuncSetAttribute");
  for (int64_t b0 = 0; b0 < B && rc == SS_OK; b0 += pl.chunk) {
    const int64_t nb = std::min(pl.chunk, B - b0);
    const uint8_t *Pc = src.p + b0 * N;
    if (src.op_major) {
      err = ss_rows_from_op_major(src.p, N, B, b0, nb, rows, stream);
      if (err != hipSuccess) {
        rc = hip_fail(err, "transpose launch");
        break;
      }
      Pc = rows;
    }
    hipLaunchKernelGGL(zero_words, dim3(1), dim3(256), 0, stream, ticket, kTicketPitch + kTicketWords);
    SsTimingRec *t = ss_timing_start(SS_KERNEL_SCHEDULE, stream);
    hipLaunchKernelGGL(port_events32, dim3((unsigned)std::min(pl.waves, nb)), dim3(kWave), lds, stream, G, Pc, nb,
                       fin, arr, rec, post, pend, ticket, makespan + b0, sumfin ? sumfin + b0 : nullptr,
                       slack ? slack + b0 * R : nullptr, violation + b0);
    ss_timing_stop(t, stream);
    err = hipGetLastError();
    if (err != hipSuccess) {
      rc = hip_fail(err, "port_events32 launch");
      break;
    }
    rc = ss_launch_peaks(g, pk, Pc, fin, N, arr, nullptr, slots, pl.slots, nb, ticket + kTicketPitch,
                         peak ? peak + b0 * D : nullptr, violation + b0, stream);
  }
  if (!W.ptr) {
    err = ss_scratch_put(g->device, &scr, stream);
    if (rc == SS_OK && err != hipSuccess) rc = hip_fail(err, "releasing the scratch");
  }
  return rc;
}
