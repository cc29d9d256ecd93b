// Whole runs of small problems in one workgroup.
//
// On a graph of a few thousand vertices a round's work takes about a
// microsecond per kernel, and the per-round kernels of the general path cost
// their launches and the chains of dependent loads behind them (a dense round
// of a 10,000-vertex graph: three kernels, 24 us; a sampled round: nine
// kernels, 55 us). Here one 1024-thread workgroup keeps the problem on its
// CU for the whole run and the rounds are separated by workgroup barriers:
//   - vertices are numbered by in-degree, highest first; thread t owns numbers
//     t, t + 1024, ... and keeps their v, dv (and Kahan term) for the whole
//     run: in registers as far as its 128 go, the rest in scratch memory
//     (registers spilled at 6, 10 and 16 vertices per thread: FP32 0, 2, 25;
//     FP32+K 0, 5, 54; FP64 0, 25, 141; weighted FP64 49, 102, 193; U32
//     distances 0, 15, 48; FP64 distances 41, 75 and 116 at 12);
//   - the message base of every vertex lies in LDS, and a thread pulls the
//     bases of its own vertices' in-neighbours into a register: LDS reads
//     run at about 25 lanes/ns per CU, FP64 LDS atomics at 7.5 (and at 0.8
//     where lanes share a target, as hubs make them), so this replaced a push
//     by LDS atomics (48,000 edges: 13 us a round);
//   - the in-neighbours stream from L2 as 16-bit numbers, four per lane and
//     load. The 64 vertices a wave pulls together have similar in-degrees and
//     are padded to the largest; a vertex of many in-edges is cut into pieces
//     that other lanes sum, added up by LDS atomics.
// A round is the one of the general kernels: the same selection (sampled and
// exact thresholds, ties to the smaller id), claim, messages, counters,
// residual and stop rule; min and max problems end bit for bit alike, sums up
// to the order of their FP64 additions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <type_traits>
#include <vector>

#include "daic_device.h"
#include "daic_problem.h"

namespace daic {

constexpr uint32_t kSmallThreads = 1024;
constexpr uint32_t kSmallPiece = 32;         // in-edges of a piece: vertices with more are cut into pieces of
                                             // as many (or twice, four times, ..., for kSmallMaxHeavy)
constexpr uint32_t kSmallMaxHeavy = 2048;    // vertices cut into pieces at most
constexpr uint32_t kSmallDegs = 768;         // distinct out-degrees (k of them take k (k - 1) / 2 edges)
constexpr uint32_t kSmallMaxN = 16384;       // message bases of 8 bytes each: 128 of the CU's 160 KiB
constexpr uint32_t kSmallMaxM = 1u << 18;    // in-edges at most: as many as were measured (see small_most_rows)
constexpr uint32_t kSmallMinEdges = 1u << 17;  // and of FP64 shortest paths (see small_most_rows),
constexpr uint32_t kSmallMinRows = 12;         // which take at most this many rows
constexpr uint32_t kSmallRounds = 4096;      // rounds per launch at most

struct SmallArgs {
  // the in-neighbours, per wave one group (four numbers per lane) after the
  // other: the groups of its first 64 vertices, of its next 64, ..., then
  // those of its slices of 64 pieces; padding: number n
  const uint2* src;
  const void* w;             // weights in the same order (EDGE_SCALE, EDGE_ADD), padding 0
  const uint32_t* wave_off;  // [16] first group of each wave
  const uint32_t* wave_sl;   // [17] first slice of pieces of each wave
  const uint32_t* len;       // [16 x 16] groups of each (wave, row of 1,024 vertices)
  const uint32_t* sl_len;    // [slices] groups of each slice of pieces
  const uint16_t* sl_num;    // [slices x 64] vertex number of each piece
  uint32_t n_heavy;          // vertices cut into pieces (they have the first numbers)
  const uint16_t* id;        // [16 x 1,024] vertex of each number (0 beyond n)
  const uint16_t* num;       // [n] number of each vertex
  const double* coef;        // [16 x 1,024] message coefficient by number (0 without out-edges)
  const uint16_t* code;      // [16 x 1,024] index of a number's out-degree among
  const uint32_t* code_deg;  // [n_code] the distinct ones,
  const double* code_coef;   // [n_code] their coefficients (not with a per-vertex alpha)
  uint32_t n_code;
  Ctl* h_ctl;                // host mirror of the control block
  double eps;
  uint64_t max_rounds;
  uint64_t k;                // exact top-k: selected vertices
  uint64_t seed;
  uint64_t n_inv;            // floor((2^64 - 1) / n)
  uint32_t sched, S, rank;
  uint32_t resume;           // continue the counters of the control block
};

// Type of an LDS accumulator and the identity of its combination.
template <int ST>
struct SmallAcc {
  using L = typename TileMM<ST>::L;
  static constexpr L ident = TileMM<ST>::ident;
};
template <> struct SmallAcc<ST_F64> { using L = double; static constexpr L ident = 0.0; };
template <> struct SmallAcc<ST_F32> { using L = double; static constexpr L ident = 0.0; };
template <> struct SmallAcc<ST_F32K> { using L = double; static constexpr L ident = 0.0; };

// Combines message x into acc (sum, minimum or maximum).
template <int ST>
__device__ __forceinline__ void small_add(typename SmallAcc<ST>::L& acc, typename SmallAcc<ST>::L x) {
  if constexpr (Tr<ST>::sum) acc += x;
  else acc = TileMM<ST>::better(x, acc) ? x : acc;
}

// One wave's walk over its groups, two at a time. The first two of the next
// slice are on their way while a slice is combined, and the next two of the
// slice while two are.
template <int ST, int G>
struct SmallWalk {
  using S = typename Tr<ST>::S;
  using L = typename SmallAcc<ST>::L;
  static constexpr bool kWeighted = G == DAIC_G_EDGE_SCALE || G == DAIC_G_EDGE_ADD;
  struct alignas(16) W4 {
    S x[4];
  };
  struct Two {
    uint2 e[2];
    W4 w[kWeighted ? 2 : 1];
  };
  const uint2* src;  // this lane's part of the coming slice's groups
  const W4* w;
  Two head;          // its first two

  __device__ __forceinline__ void load(Two& x, uint32_t g) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      x.e[i] = src[(g + i) * 64];
      if constexpr (kWeighted) x.w[i] = w[(g + i) * 64];
    }
  }
  // starts at group g of the arrays (which are padded by two groups)
  __device__ __forceinline__ void start(const SmallArgs& t, uint32_t g) {
    const uint32_t lane = threadIdx.x & 63;
    src = t.src + (uint64_t)g * 64 + lane;
    w = static_cast<const W4*>(t.w) + (uint64_t)g * 64 + lane;
    load(head, 0);
  }
  static __device__ __forceinline__ void group(const S* base, const uint2 e, const W4& y, L& acc) {
    const S m[4] = {base[e.x & 0xFFFFu], base[e.x >> 16], base[e.y & 0xFFFFu], base[e.y >> 16]};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (Tr<ST>::sum) {
        double x = (double)m[i];
        if constexpr (G == DAIC_G_EDGE_SCALE) x *= (double)y.x[i];  // 0 of a silent sender: weights are finite
        small_add<ST>(acc, x);
      } else {
        small_add<ST>(acc, tile_mm_msg<ST, G>(m[i], y.x + i, 0));
      }
    }
  }
  // the combined messages of a slice of this many (at least one) groups
  __device__ __forceinline__ L slice(const S* base, uint32_t groups) {
    Two cur = head;
    const SmallWalk here = *this;
    src += groups * 64;
    w += groups * 64;
    load(head, 0);
    L acc = SmallAcc<ST>::ident;
    uint32_t g = 0;
    for (; g + 2 < groups; g += 2) {
      Two next;
      here.load(next, g + 2);
      group(base, cur.e[0], cur.w[0], acc);
      group(base, cur.e[1], cur.w[kWeighted ? 1 : 0], acc);
      cur = next;
    }
    group(base, cur.e[0], cur.w[0], acc);
    if (g + 1 < groups) group(base, cur.e[1], cur.w[kWeighted ? 1 : 0], acc);
    return acc;
  }
};

// prio_key as a value of its own at each use (the keys of all of a thread's
// vertices kept from one use to the next would take as many registers as
// their state).
template <int ST>
__device__ __forceinline__ typename Tr<ST>::Key small_key(typename Tr<ST>::S v, typename Tr<ST>::S dv) {
  asm volatile("" : "+v"(dv));
  return prio_key<ST>(v, dv);
}

// A vertex's combined messages are taken into its dv.
template <int ST>
__device__ __forceinline__ void small_receive(typename SmallAcc<ST>::L acc, typename Tr<ST>::S v,
                                              typename Tr<ST>::S& dv) {
  using S = typename Tr<ST>::S;
  if constexpr (Tr<ST>::sum) {
    if (acc != 0.0) dv = (S)((double)dv + acc);
  } else if constexpr (ST == ST_F64MIN) {
    // compared as doubles: messages are not negative, but a starting distance
    // may be, and its bits are above every message's
    const double x = TileMM<ST>::dec(acc);
    if (x < v && x < dv) dv = x;
  } else {
    if (TileMM<ST>::better(acc, TileMM<ST>::enc(v)) && TileMM<ST>::better(acc, TileMM<ST>::enc(dv)))
      dv = (S)TileMM<ST>::dec(acc);
  }
}

// NPT: vertices per thread. One workgroup.
template <int ST, int G, int NPT>
__global__ __launch_bounds__(kSmallThreads) void k_small_run(KArgs a, SmallArgs t) {
  using S = typename Tr<ST>::S;
  using Key = typename Tr<ST>::Key;
  using L = typename SmallAcc<ST>::L;
  constexpr bool kSum = Tr<ST>::sum;
  constexpr L kIdent = SmallAcc<ST>::ident;
  __shared__ S base[NPT * kSmallThreads + 8];  // message bases; the sampled rule's keys before the claim
  __shared__ L heavy[kSmallMaxHeavy];          // sums of the heavy vertices
  __shared__ KthScratch sel;
  __shared__ double red_r[16];
  __shared__ uint32_t red_n[16];
  __shared__ double code_coef[kSmallDegs];
  __shared__ uint32_t code_deg[kSmallDegs];
  const uint32_t n = (uint32_t)a.n, tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  S silent;
  if constexpr (kSum) silent = (S)0;
  else silent = (S)TileMM<ST>::dec(kIdent);
  Ctl* ctl = a.ctl;

  S v[NPT], dv[NPT];
  float c[Tr<ST>::kahan ? NPT : 1];
  uint32_t code[NPT / 2];  // two 16-bit indices each
  for (uint32_t i = tid; i < t.n_code; i += kSmallThreads) {
    code_deg[i] = t.code_deg[i];
    code_coef[i] = t.code_coef[i];
  }
  unroll_each<NPT>([&](auto k) {
    v[k] = silent;
    dv[k] = silent;
    if constexpr (Tr<ST>::kahan) c[k] = 0.f;
    if constexpr (k % 2 == 0) code[k / 2] = 0;
    if (k * kSmallThreads + tid < n) {  // beyond n: no vertex, never pending
      const uint32_t j = t.id[k * kSmallThreads + tid];
      v[k] = static_cast<const S*>(a.v)[j];
      dv[k] = static_cast<const S*>(a.dv)[j];
      if constexpr (Tr<ST>::kahan) c[k] = a.c[j];
      code[k / 2] |= (uint32_t)t.code[k * kSmallThreads + tid] << (k % 2 * 16);
    }
  });
  for (uint32_t i = tid; i < t.n_heavy; i += kSmallThreads) heavy[i] = kIdent;
  uint64_t rounds = t.resume ? ctl->rounds : 0;
  const uint64_t act0 = t.resume ? ctl->activations : 0, pushed0 = t.resume ? ctl->pushed : 0;
  const uint64_t launch_end = rounds + kSmallRounds;
  uint32_t act = 0;  // this thread's updates and messages
  uint64_t pushed = 0;
  double res = 0.0;
  uint32_t pending = 0;
  bool done = false, stop = false;

  for (;;) {
    // the thread's index and the degree indices anew in each round: addresses
    // formed from them are not kept across rounds (they would take the
    // registers of the state)
    uint32_t tx = tid;
    asm volatile("" : "+v"(tx));
#pragma unroll
    for (int k = 0; k < NPT / 2; ++k) asm volatile("" : "+v"(code[k]));
    uint16_t at[4] = {0, 0, 0, 0};  // the sampled vertices' numbers, on their way during the reductions
    if (t.sched == DAIC_SCHED_TOPK_SAMPLED) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint64_t i = (uint64_t)tx + (uint64_t)u * kSmallThreads;
        at[u] = t.num[mod_by_inverse(splitmix64_at(t.seed, rounds * (uint64_t)t.S + i), n, t.n_inv)];
      }
    }
    // A1: the residual of the state, and the stop rule
    double rp = 0.0;
    uint32_t np = 0;
    unroll_each<NPT>([&](auto k) {
      if constexpr (kSum) {
        const double x = fabs((double)dv[k]);
        rp += x;
        np += x > 0.0 ? 1u : 0u;
      } else {
        np += small_key<ST>(v[k], dv[k]) != 0 ? 1u : 0u;
      }
    });
    if constexpr (kSum) rp = wave_sum(rp);
    np = wave_sum(np);
    if (lane == 0) {
      red_r[wave] = rp;
      red_n[wave] = np;
    }
    __syncthreads();  // also: every base of the last round was read
    res = 0.0;
    pending = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      if constexpr (kSum) res += red_r[w];
      pending += red_n[w];
    }
    done = kSum ? (res <= t.eps || pending == 0) : pending == 0;
    stop = !done && rounds >= t.max_rounds;
    if (done || stop || rounds >= launch_end) break;

    // A2: the round takes the pending vertices with key >= lo other than veto,
    // and those of `ties`, as far as `allow` has them (a bit per vertex of
    // this thread)
    Key lo = 1, veto = 0;
    uint32_t ties = 0, allow = ~0u;
    if (t.sched == DAIC_SCHED_TOPK_SAMPLED) {
      Key* keys = reinterpret_cast<Key*>(base);
      unroll_each<NPT>([&](auto k) { keys[k * kSmallThreads + tx] = small_key<ST>(v[k], dv[k]); });
      __syncthreads();
      Key ks[4];
      unroll_each<4>([&](auto u) { ks[u] = keys[at[u]]; });
      const Key tau = block_kth_sampled<Key>(sel, t.rank, t.S, pending, n, ks);
      if (tau != 0) lo = tau;  // no positive sample: every pending vertex
    } else if (t.sched == DAIC_SCHED_TOPK_EXACT) {
      if (pending > t.k) {
        uint32_t equal, rem;
        lo = block_kth<Key, NPT>(
            sel, (uint32_t)t.k, [&](auto u) { return small_key<ST>(v[u], dv[u]); },
            [&](auto u) { return small_key<ST>(v[u], dv[u]) != 0; }, &equal, &rem);
        if (equal != rem) {
          // the first rem keys equal to the threshold by id: a bit per id,
          // and for each word the bits before it
          veto = lo;
          uint32_t* bits = reinterpret_cast<uint32_t*>(base);  // [512], then the words' prefixes [512]
          uint32_t* wsum = sel.hist[0];
          if (tid < 512) bits[tid] = 0;
          __syncthreads();
          unroll_each<NPT>([&](auto k) {
            if (small_key<ST>(v[k], dv[k]) == veto) {  // positive: a vertex
              const uint32_t j = (t.id + k * kSmallThreads)[tx];
              atomicOr(&bits[j >> 5], 1u << (j & 31));
            }
          });
          __syncthreads();
          const uint32_t x = tid < 512 ? (uint32_t)__popc(bits[tid]) : 0u;
          const uint32_t incl = wave_incl_scan(x);
          if (lane == 63) wsum[wave] = incl;
          __syncthreads();
          uint32_t before = incl - x;
          for (uint32_t w = 0; w < wave; ++w) before += wsum[w];
          if (tid < 512) bits[512 + tid] = before;
          __syncthreads();
          unroll_each<NPT>([&](auto k) {
            if (small_key<ST>(v[k], dv[k]) == veto) {
              const uint32_t j = (t.id + k * kSmallThreads)[tx];
              const uint32_t r = bits[512 + (j >> 5)] + (uint32_t)__popc(bits[j >> 5] & ((1u << (j & 31)) - 1u));
              if (r < rem) ties |= 1u << k;
            }
          });
        }
      }
    } else if (t.sched == DAIC_SCHED_ROUND_ROBIN) {
      const uint32_t rr_lo = (uint32_t)(rounds % ((a.n + a.rr_chunk - 1) / a.rr_chunk) * a.rr_chunk);
      const uint32_t rr_len = (uint32_t)min((uint64_t)n, a.rr_chunk);
      allow = 0;
      unroll_each<NPT>([&](auto k) {
        if ((t.id + k * kSmallThreads)[tx] - rr_lo < rr_len) allow |= 1u << k;
      });
    }
    if (t.sched != DAIC_SCHED_ALL) __syncthreads();  // every key and tie bit was read

    // A3 + A4: claim, fold, message base
    if (kSum && !Tr<ST>::kahan && t.sched == DAIC_SCHED_ALL && a.alpha_pv == nullptr) {
      // as below with every vertex taken: one without a delta adds and sends 0
      unroll_each<NPT>([&](auto k) {
        const uint32_t ci = code[k / 2] >> (k % 2 * 16) & 0xFFFFu;
        const S delta = dv[k];
        v[k] += delta;
        dv[k] = (S)0;
        base[k * kSmallThreads + tx] = (S)(code_coef[ci] * (double)delta);
        pushed += delta != (S)0 ? code_deg[ci] : 0u;
        act += delta != (S)0 ? 1u : 0u;
        if constexpr (k % 2 == 1) asm volatile("" ::: "memory");  // the next operands stay behind (registers)
      });
    } else {
      unroll_each<NPT>([&](auto k) {
        const uint32_t ci = code[k / 2] >> (k % 2 * 16) & 0xFFFFu;
        const uint32_t dg = code_deg[ci];
        double cf = 0.0;
        if constexpr (kSum) {
          cf = code_coef[ci];
          if (a.alpha_pv != nullptr) cf = (t.coef + k * kSmallThreads)[tx];
        }
        const Key key = small_key<ST>(v[k], dv[k]);  // 0 beyond n
        const bool take = ((key >= lo && key != veto) || (ties >> k & 1u)) && (allow >> k & 1u);
        S mu = silent;
        if constexpr (kSum) {
          const S delta = dv[k];
          if constexpr (Tr<ST>::kahan) {  // as claim_fold
#pragma clang fp contract(off)
            const float y = delta - c[k];
            const float x = v[k] + y;
            const float cn = (x - v[k]) - y;
            c[k] = take ? cn : c[k];
            v[k] = take ? x : v[k];
          } else {
            v[k] = take ? v[k] + delta : v[k];
          }
          dv[k] = take ? (S)0 : delta;
          mu = take ? (S)(cf * (double)delta) : (S)0;
        } else {  // pending: dv improves v
          v[k] = take ? dv[k] : v[k];
          mu = take ? dv[k] : silent;
          dv[k] = take ? silent : dv[k];
        }
        pushed += take ? dg : 0u;
        act += take ? 1u : 0u;
        base[k * kSmallThreads + tx] = mu;
        if constexpr (k % 2 == 1) asm volatile("" ::: "memory");
      });
    }
    if (tid == 0) base[n] = silent;  // padding entries read it (number n has no vertex)
    __syncthreads();

    // A5: this thread's vertices, then its pieces of the heavy ones
    SmallWalk<ST, G> walk;
    walk.start(t, t.wave_off[wave]);
    unroll_each<NPT>([&](auto k) {
      const uint32_t groups = t.len[wave * 16 + k];
      if (groups) small_receive<ST>(walk.slice(base, groups), v[k], dv[k]);
    });
    if (t.n_heavy) {
      const uint32_t s1 = t.wave_sl[wave + 1];
      for (uint32_t s = t.wave_sl[wave]; s < s1; ++s) {
        const uint32_t r = t.sl_num[s * 64 + lane];
        const L acc = walk.slice(base, t.sl_len[s]);
        if constexpr (kSum) {
          if (acc != kIdent) atomicAdd(&heavy[r], acc);
        } else {
          if (acc != kIdent) TileMM<ST>::combine(&heavy[r], acc);
        }
      }
      __syncthreads();
      unroll_each<(NPT < kSmallMaxHeavy / kSmallThreads ? NPT : kSmallMaxHeavy / kSmallThreads)>([&](auto k) {
        if (k * kSmallThreads + tx < t.n_heavy) {
          small_receive<ST>(heavy[k * kSmallThreads + tx], v[k], dv[k]);
          heavy[k * kSmallThreads + tx] = kIdent;  // for the next round (its pieces come after barriers)
        }
      });
    }
    rounds += 1;
  }

  // the state, and the run's counters
  unroll_each<NPT>([&](auto k) {
    const uint32_t r = k * kSmallThreads + tid;
    if (r < n) {
      const uint32_t j = t.id[r];
      static_cast<S*>(a.v)[j] = v[k];
      static_cast<S*>(a.dv)[j] = dv[k];
      if constexpr (Tr<ST>::kahan) a.c[j] = c[k];
    }
  });
  const uint64_t act_all = block_sum_waves<16>((uint64_t)act), pushed_all = block_sum_waves<16>(pushed);
  if (tid == 0) {
    auto put = [&](Ctl* o) {
      o->r = kSum ? res : (double)pending;
      o->pending = pending;
      o->rounds = rounds;
      o->activations = act0 + act_all;
      o->pushed = pushed0 + pushed_all;
      o->done = done ? 1u : 0u;
      o->stop = stop ? 1u : 0u;
    };
    put(ctl);
    put(t.h_ctl);
    __threadfence_system();
  }
}

// Message coefficients by number.
template <typename S>
__global__ void k_small_coef(const uint32_t* row, const uint16_t* id, uint32_t n, bool per_degree, double alpha,
                             const S* alpha_pv, double* coef) {
  for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < n; r += gridDim.x * blockDim.x) {
    const uint32_t j = id[r], d = row[j + 1] - row[j];
    coef[r] = d == 0 ? 0.0 : per_degree ? alpha / (double)d : alpha_pv ? (double)alpha_pv[j] : alpha;
  }
}

// Weights in the order of the groups (eid: the out-edge of each entry,
// 0xFFFFFFFF for padding).
template <typename S>
__global__ void k_small_weights(const S* w, const uint32_t* eid, uint64_t count, S* out) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (uint64_t)gridDim.x * blockDim.x)
    out[i] = eid[i] == 0xFFFFFFFFu ? (S)0 : w[eid[i]];
}

// *found = 1 when a weight (the bits of a float or a double) is infinite or NaN.
template <typename S>
__global__ void k_small_nonfinite(const S* w, uint64_t m, uint64_t* found) {
  constexpr S kExp = sizeof(S) == 8 ? (S)0x7FF0000000000000ull : (S)0x7F800000u;
  bool any = false;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (uint64_t)gridDim.x * blockDim.x)
    any |= (w[i] & kExp) == kExp;
  if (any) *found = 1;
}

namespace {

// The layout of k_small_run, computed on the host (a millisecond at most for
// the sizes it takes).
struct SmallLayout {
  std::vector<uint16_t> src, id, num, sl_num;
  std::vector<uint32_t> eid, len, sl_len, wave_off, wave_sl, code_deg;
  std::vector<uint16_t> code;  // by number
  uint32_t n_heavy = 0;
};

void small_layout(uint32_t n, uint32_t m, const uint32_t* row, const uint32_t* col, bool weighted, SmallLayout& L) {
  std::vector<uint32_t> indeg(n, 0);
  for (uint32_t e = 0; e < m; ++e) ++indeg[col[e]];
  uint32_t top = 0;
  for (uint32_t d : indeg) top = std::max(top, d);
  // numbers by in-degree, highest first, ties by id
  std::vector<uint32_t> at(top + 2, 0);
  for (uint32_t d : indeg) ++at[top - d + 1];
  for (uint32_t d = 0; d <= top; ++d) at[d + 1] += at[d];
  L.id.resize(n);
  L.num.resize(n);
  for (uint32_t j = 0; j < n; ++j) {
    const uint32_t r = at[top - indeg[j]]++;
    L.id[r] = (uint16_t)j;
    L.num[j] = (uint16_t)r;
  }
  auto deg_of = [&](uint32_t r) { return indeg[L.id[r]]; };
  uint32_t piece = kSmallPiece;
  while (n > kSmallMaxHeavy && deg_of(kSmallMaxHeavy) > piece) piece *= 2;
  while (L.n_heavy < std::min(n, kSmallMaxHeavy) && deg_of(L.n_heavy) > piece) ++L.n_heavy;
  // groups of the vertices not cut, by (row of 1,024, wave)
  const uint32_t rows = (n + kSmallThreads - 1) / kSmallThreads;
  L.len.assign(16 * 16, 0);  // by (wave, row)
  uint32_t load[16] = {};
  for (uint32_t w = 0; w < 16; ++w)
    for (uint32_t k = 0; k < rows; ++k) {
      const uint32_t r0 = std::max(k * kSmallThreads + w * 64, L.n_heavy);  // in-degrees descend
      if (r0 < std::min(n, k * kSmallThreads + (w + 1) * 64)) L.len[w * 16 + k] = (deg_of(r0) + 3) / 4;
      load[w] += L.len[w * 16 + k];
    }
  // pieces, longest first, 64 to a slice, each slice to the wave with the least work
  struct Piece {
    uint32_t len, r, first;  // in-edges, vertex number, its first in-edge
  };
  std::vector<Piece> pieces;
  for (uint32_t r = 0; r < L.n_heavy; ++r)
    for (uint32_t i = 0; i < deg_of(r); i += piece) pieces.push_back({std::min(piece, deg_of(r) - i), r, i});
  std::stable_sort(pieces.begin(), pieces.end(), [](const Piece& a, const Piece& b) { return a.len > b.len; });
  std::vector<std::vector<uint32_t>> mine(16);
  for (uint32_t i = 0; i < pieces.size(); i += 64) {
    const uint32_t w = (uint32_t)(std::min_element(load, load + 16) - load);
    mine[w].push_back(i);
    load[w] += (pieces[i].len + 3) / 4;
  }
  // the waves' groups one after the other
  std::vector<uint32_t> first((size_t)rows * 16);      // first group of each (row, wave)
  std::vector<size_t> piece_at(pieces.size());         // entry of each piece's first in-edge
  std::vector<std::vector<uint32_t>> order(L.n_heavy); // pieces of each heavy vertex by their first in-edge
  L.wave_off.resize(16);
  L.wave_sl.assign(17, 0);
  uint32_t off = 0;
  for (uint32_t w = 0; w < 16; ++w) {
    L.wave_off[w] = off;
    for (uint32_t k = 0; k < rows; ++k) {
      first[k * 16 + w] = off;
      off += L.len[w * 16 + k];
    }
    for (uint32_t i0 : mine[w]) {
      const uint32_t groups = (pieces[i0].len + 3) / 4;
      L.sl_len.push_back(groups);
      for (uint32_t l = 0; l < 64; ++l) {
        const bool in = i0 + l < pieces.size();
        L.sl_num.push_back((uint16_t)(in ? pieces[i0 + l].r : 0));
        if (in) piece_at[i0 + l] = ((size_t)off * 64 + l) * 4;
      }
      off += groups;
    }
    L.wave_sl[w + 1] = (uint32_t)L.sl_len.size();
  }
  for (uint32_t i = 0; i < pieces.size(); ++i) {
    auto& o = order[pieces[i].r];
    if (o.size() <= pieces[i].first / piece) o.resize(pieces[i].first / piece + 1);
    o[pieces[i].first / piece] = i;
  }
  // the distinct out-degrees
  L.code.resize(n);
  std::vector<uint32_t> code_of;  // by degree
  for (uint32_t r = 0; r < n; ++r) {
    const uint32_t d = row[L.id[r] + 1] - row[L.id[r]];
    if (d >= code_of.size()) code_of.resize(d + 1, 0xFFFFFFFFu);
    if (code_of[d] == 0xFFFFFFFFu) {
      code_of[d] = (uint32_t)L.code_deg.size();
      L.code_deg.push_back(d);
    }
    L.code[r] = (uint16_t)code_of[d];
  }
  const size_t entries = (size_t)(off + 2) * 256;  // a walk reads up to two groups ahead
  L.src.assign(entries, (uint16_t)n);
  if (weighted) L.eid.assign(entries, 0xFFFFFFFFu);
  std::vector<uint32_t> seen(n, 0);
  for (uint32_t j = 0; j < n; ++j)
    for (uint32_t e = row[j]; e < row[j + 1]; ++e) {
      const uint32_t r = L.num[col[e]], i = seen[r]++;
      size_t pos;  // in-edge i of a lane: entry i % 4 of its group i / 4
      if (r < L.n_heavy) pos = piece_at[order[r][i / piece]] + (size_t)(i % piece / 4) * 256 + i % 4;
      else pos = ((size_t)(first[r / kSmallThreads * 16 + r % kSmallThreads / 64] + i / 4) * 64 + r % 64) * 4 + i % 4;
      L.src[pos] = L.num[j];
      if (weighted) L.eid[pos] = e;
    }
}

daic_status small_setup(daic_problem* p, hipStream_t s) {
  const GraphDev& d = p->g->dev;
  const uint32_t n = (uint32_t)d.n, m = (uint32_t)d.m;
  const size_t S = p->st == ST_F64 || p->st == ST_F64MIN ? 8 : 4;
  const bool weighted = p->gk == DAIC_G_EDGE_SCALE || p->gk == DAIC_G_EDGE_ADD;
  if (p->gk == DAIC_G_EDGE_SCALE && m) {
    // A weight that is no number must reach its target only when its sender
    // sends. The round kernels' pushes skip silent senders; here each in-edge
    // adds base x weight, and a select per in-edge to keep a silent 0 apart
    // took 0.2 to 1 us of a round's 5 to 33, so such graphs keep those kernels.
    uint64_t found = 0;  // (part_n: partials of the residual, free between rounds)
    DAIC_HIP(hipMemsetAsync(p->a.part_n, 0, 8, s));
    const dim3 grid((uint32_t)std::min<uint64_t>(256, m / 256 + 1));
    if (S == 8)
      hipLaunchKernelGGL(k_small_nonfinite<uint64_t>, grid, dim3(256), 0, s, static_cast<const uint64_t*>(p->a.w),
                         (uint64_t)m, p->a.part_n);
    else
      hipLaunchKernelGGL(k_small_nonfinite<uint32_t>, grid, dim3(256), 0, s, static_cast<const uint32_t*>(p->a.w),
                         (uint64_t)m, p->a.part_n);
    DAIC_HIP(hipMemcpyAsync(&found, p->a.part_n, 8, hipMemcpyDeviceToHost, s));
    DAIC_HIP(hipStreamSynchronize(s));
    if (found) {
      p->small_off = true;
      return DAIC_OK;
    }
  }
  std::vector<uint32_t> row(n + 1), col(m);
  DAIC_HIP(hipMemcpyAsync(row.data(), d.row, (n + 1) * 4ull, hipMemcpyDeviceToHost, s));
  if (m) DAIC_HIP(hipMemcpyAsync(col.data(), d.col, m * 4ull, hipMemcpyDeviceToHost, s));
  DAIC_HIP(hipStreamSynchronize(s));
  SmallLayout L;
  small_layout(n, m, row.data(), col.data(), weighted, L);
  // one allocation: the arrays at 256-byte offsets
  size_t bytes = 0;
  auto take = [&](size_t b) {
    const size_t at = bytes;
    bytes += (b + 255) / 256 * 256;
    return at;
  };
  const size_t np = kSmallMaxN;  // the per-number arrays cover every row of 1,024 numbers a kernel may have
  const size_t o_src = take(L.src.size() * 2), o_len = take(L.len.size() * 4), o_id = take(np * 2),
               o_num = take(n * 2ull), o_sll = take(L.sl_len.size() * 4), o_sln = take(L.sl_num.size() * 2),
               o_code = take(np * 2), o_cdeg = take(kSmallDegs * 4), o_ccoef = take(kSmallDegs * 8), o_wave = take(33 * 4), o_coef = take(np * 8),
               o_eid = take(L.eid.size() * 4), o_w = take(L.eid.size() * S);
  char* buf = nullptr;
  DAIC_HIP(hipMalloc((void**)&buf, bytes));
  p->allocs.push_back(buf);
  auto put = [&](size_t at, const void* src, size_t b) {
    return b ? hipMemcpyAsync(buf + at, src, b, hipMemcpyHostToDevice, s) : hipSuccess;
  };
  DAIC_HIP(put(o_src, L.src.data(), L.src.size() * 2));
  DAIC_HIP(put(o_len, L.len.data(), L.len.size() * 4));
  L.id.resize(np, 0);
  DAIC_HIP(put(o_id, L.id.data(), np * 2));
  DAIC_HIP(put(o_num, L.num.data(), n * 2ull));
  DAIC_HIP(put(o_sll, L.sl_len.data(), L.sl_len.size() * 4));
  DAIC_HIP(put(o_sln, L.sl_num.data(), L.sl_num.size() * 2));
  std::vector<double> code_coef;
  for (uint32_t deg : L.code_deg) code_coef.push_back(deg == 0 ? 0.0 : p->gk == DAIC_G_DEG_SCALE ? p->alpha / (double)deg : p->alpha);
  L.code.resize(np, 0);
  DAIC_HIP(put(o_code, L.code.data(), np * 2));
  DAIC_HIP(put(o_cdeg, L.code_deg.data(), L.code_deg.size() * 4));
  DAIC_HIP(put(o_ccoef, code_coef.data(), code_coef.size() * 8));
  L.wave_off.insert(L.wave_off.end(), L.wave_sl.begin(), L.wave_sl.end());
  DAIC_HIP(put(o_wave, L.wave_off.data(), 33 * 4));
  DAIC_HIP(put(o_eid, L.eid.data(), L.eid.size() * 4));
  const dim3 grid_n((uint32_t)(np / 256)), grid_w((uint32_t)std::min<size_t>(1024, L.eid.size() / 256 + 1));
  const uint32_t* drow = static_cast<const uint32_t*>(d.row);
  const uint16_t* did = reinterpret_cast<const uint16_t*>(buf + o_id);
  const uint32_t* deid = reinterpret_cast<const uint32_t*>(buf + o_eid);
  double* coef = reinterpret_cast<double*>(buf + o_coef);
  const bool per_degree = p->gk == DAIC_G_DEG_SCALE;
  if (S == 8) {
    hipLaunchKernelGGL(k_small_coef<double>, grid_n, dim3(256), 0, s, drow, did, (uint32_t)np, per_degree, p->alpha,
                       static_cast<const double*>(p->a.alpha_pv), coef);
    if (weighted)
      hipLaunchKernelGGL(k_small_weights<uint64_t>, grid_w, dim3(256), 0, s, static_cast<const uint64_t*>(p->a.w), deid,
                         (uint64_t)L.eid.size(), reinterpret_cast<uint64_t*>(buf + o_w));
  } else {
    hipLaunchKernelGGL(k_small_coef<float>, grid_n, dim3(256), 0, s, drow, did, (uint32_t)np, per_degree, p->alpha,
                       static_cast<const float*>(p->a.alpha_pv), coef);
    if (weighted)
      hipLaunchKernelGGL(k_small_weights<uint32_t>, grid_w, dim3(256), 0, s, static_cast<const uint32_t*>(p->a.w), deid,
                         (uint64_t)L.eid.size(), reinterpret_cast<uint32_t*>(buf + o_w));
  }
  DAIC_HIP(hipGetLastError());
  DAIC_HIP(hipStreamSynchronize(s));
  SmallArgs* t = new SmallArgs();
  t->src = reinterpret_cast<const uint2*>(buf + o_src);
  t->w = weighted ? buf + o_w : nullptr;
  t->wave_off = reinterpret_cast<const uint32_t*>(buf + o_wave);
  t->len = reinterpret_cast<const uint32_t*>(buf + o_len);
  t->wave_sl = t->wave_off + 16;
  t->sl_len = reinterpret_cast<const uint32_t*>(buf + o_sll);
  t->sl_num = reinterpret_cast<const uint16_t*>(buf + o_sln);
  t->n_heavy = L.n_heavy;
  t->code = reinterpret_cast<const uint16_t*>(buf + o_code);
  t->code_deg = reinterpret_cast<const uint32_t*>(buf + o_cdeg);
  t->code_coef = reinterpret_cast<const double*>(buf + o_ccoef);
  t->n_code = (uint32_t)L.code_deg.size();
  t->id = did;
  t->num = reinterpret_cast<const uint16_t*>(buf + o_num);
  t->coef = coef;
  t->h_ctl = p->h_ctl;
  t->n_inv = ~0ull / n;
  p->small = t;
  return DAIC_OK;
}

// The kernel of the smallest even number of rows (vertices per thread) that
// holds the vertices: two rows too many cost 0.4 to 3 us of a round (5,000
// vertices in 6 and 8 rows: FP64 PageRank 6.8 and 7.1 us, FP64 SSSP 14.3 and
// 16.3; 13,000 in 14 and 16: 16.6 and 22.2, 42 and 46).
template <int ST, int G, int NPT = 2>
void small_launch(daic_problem* p, const SmallArgs& t, hipStream_t s) {
  if constexpr (NPT < (int)(ST == ST_F64MIN ? kSmallMinRows : kSmallMaxN / kSmallThreads)) {
    if (p->g->dev.n > (uint64_t)NPT * kSmallThreads) return small_launch<ST, G, NPT + 2>(p, t, s);
  }
  hipLaunchKernelGGL((k_small_run<ST, G, NPT>), dim3(1), dim3(kSmallThreads), 0, s, p->a, t);
}

template <int ST>
void small_launch_sum(daic_problem* p, const SmallArgs& t, hipStream_t s) {
  if (p->gk == DAIC_G_DEG_SCALE) small_launch<ST, DAIC_G_DEG_SCALE>(p, t, s);
  else if (p->gk == DAIC_G_EDGE_SCALE) small_launch<ST, DAIC_G_EDGE_SCALE>(p, t, s);
  else small_launch<ST, DAIC_G_SRC_SCALE>(p, t, s);
}

}  // namespace

// The most rows (1,024 vertices each) that run in one workgroup, by kind of
// problem and rule: where one CU stops being faster than the chip's round
// kernels. It loses to them as its time grows with the in-edges, and with the
// rows, whose state leaves the registers for scratch memory (from 8 or 10 rows
// of 8-byte values on). us per round, this form / the round kernels, at the
// last size of a row of the table and beyond it, on a power-law graph of 11.7
// in-edges per vertex and an RMAT graph of 16:
//                                     ALL               ROUND_ROBIN       sampled           exact
//   PageRank FP32+K    n = 16,384   19 / 21, 25 / 23  21 / 28, 24 / 29  26 / 35, 31 / 36  33 / 44, 37 / 46
//   PageRank FP64      n = 14,336   18 / 22, 24 / 25  20 / 27, 24 / 31  26 / 36, 34 / 41  31 / 59, 39 / 65
//                      n = 16,384   24 / 21, 30 / 24  27 / 29, 31 / 31  34 / 38, 42 / 40  41 / 61, 48 / 65
//   Adsorption FP32    n = 14,336   21 / 23, 26 / 26  22 / 28, 27 / 32  29 / 35, 34 / 39  34 / 43, 38 / 47
//                      n = 16,384   26 / 22, 31 / 24  28 / 30, 32 / 31  33 / 37, 38 / 38  40 / 44, 44 / 46
//   Adsorption FP32+K  n = 12,288   21 / 21, 26 / 25  22 / 27, 26 / 31  29 / 34, 33 / 38  33 / 42, 36 / 46
//                      n = 14,336   25 / 23, 30 / 26  27 / 27, 31 / 32  32 / 34, 37 / 39  37 / 42, 41 / 47
//   Adsorption FP64    n =  8,192   19 / 24, 22 / 25  19 / 28, 23 / 33  26 / 36, 30 / 40  27 / 60, 30 / 64
//                      n = 10,240   25 / 24, 29 / 26  25 / 28, 29 / 33  31 / 36, 36 / 41  34 / 59, 38 / 63
//                      n = 12,288   30 / 24, 34 / 27  31 / 29, 36 / 33  37 / 37, 42 / 42  41 / 60, 45 / 64
//                      n = 14,336   35 / 25, 41 / 27  37 / 29, 42 / 33  42 / 38, 48 / 42  48 / 60, 53 / 65
//   SSSP u32           n = 16,384   24 / 34, 29 / 35  25 / 31, 28 / 29  29 / 40, 35 / 41  36 / 51, 38 / 51
//   SSSP FP64          n = 10,240   26 / 34, 34 / 34  25 / 30, 31 / 27  33 / 41, 39 / 43  41 / 63, 46 / 59
//                      n = 12,288   36 / 33, 45 / 37  35 / 31, 43 / 28  43 / 40, 51 / 44  54 / 64, 61 / 60
//                      n = 14,336   46 / 32, 52 / 31  46 / 31, 49 / 28  54 / 40, 58 / 45  73 / 65, 72 / 60
// (2^18 edges on 1,025 vertices: PageRank FP32+K 21 / 119, Adsorption FP64 28 / 120,
// SSSP FP64 30 / 80.) FP64 shortest paths by round-robin, and all pending beyond
// eight rows, also need few edges: a round sends along a fraction of them, which
// the round kernels push and this form walks whole (8,192 vertices, ROUND_ROBIN:
// 131,072 edges 23 / 27, 262,144 36 / 28).
static uint32_t small_most_rows(const daic_problem* p, daic_sched sched) {
  enum { U32_I32, SUM_F32, SUM_F64, WSUM_F32, WSUM_F32K, WSUM_F64, MIN_F64 };
  static constexpr uint32_t rows[7][4] = {
      // ALL, ROUND_ROBIN, sampled, exact
      {16, 16, 16, 16},  // U32_I32
      {16, 16, 16, 16},  // SUM_F32
      {14, 16, 16, 16},  // SUM_F64
      {14, 16, 16, 16},  // WSUM_F32
      {12, 16, 16, 16},  // WSUM_F32K
      {8, 10, 12, 16},   // WSUM_F64
      {10, 10, 10, kSmallMinRows},  // MIN_F64
  };
  const bool weighted = p->gk == DAIC_G_EDGE_SCALE;
  const int kind = p->st == ST_F64MIN ? MIN_F64
                   : p->st == ST_U32 || p->st == ST_I32 ? U32_I32
                   : p->st == ST_F64 ? (weighted ? WSUM_F64 : SUM_F64)
                   : !weighted ? SUM_F32 : p->st == ST_F32 ? WSUM_F32 : WSUM_F32K;
  switch (sched) {
    case DAIC_SCHED_ALL: return rows[kind][0];
    case DAIC_SCHED_ROUND_ROBIN: return rows[kind][1];
    case DAIC_SCHED_TOPK_SAMPLED: return rows[kind][2];
    case DAIC_SCHED_TOPK_EXACT: return rows[kind][3];
    default: return 0;
  }
}

bool small_applies(const daic_problem* p, const daic_run_opts* o) {
  const GraphDev& d = p->g->dev;
  if (d.m > kSmallMaxM || !d.row32 || p->small_off) return false;
  if (d.n > (uint64_t)small_most_rows(p, o->sched) * kSmallThreads) return false;
  const bool whole = o->sched == DAIC_SCHED_ROUND_ROBIN || (o->sched == DAIC_SCHED_ALL && d.n > 8 * kSmallThreads);
  if (p->st == ST_F64MIN && whole && d.m > kSmallMinEdges) return false;
  // a setting that asks for one form of the per-round kernels gets it
  for (const char* e : {"DAIC_NO_SMALL", "DAIC_NO_GRAPH", "DAIC_NO_FUSE", "DAIC_NO_PULL", "DAIC_NO_TILE",
                        "DAIC_PULL_DIV", "DAIC_PULL_EDGE_DIV", "DAIC_TILE_EDGES", "DAIC_TILE_BITS",
                        "DAIC_TILE_ID_ORDER"})
    if (std::getenv(e)) return false;
  return true;
}

daic_status small_prepare(daic_problem* p, hipStream_t s) { return p->small ? DAIC_OK : small_setup(p, s); }

daic_status small_run(daic_problem* p, const daic_run_opts* o, hipStream_t s) {
  const uint32_t n = (uint32_t)p->g->dev.n;
  SmallArgs t = *p->small;
  t.eps = o->eps;
  t.max_rounds = o->max_rounds ? o->max_rounds : ~0ull;
  t.k = std::max<uint64_t>(1, (uint64_t)std::ceil(o->priority_fraction * (double)n));
  t.seed = o->seed;
  t.sched = (uint32_t)o->sched;
  t.S = o->n_samples ? o->n_samples : kMaxSamples;
  t.rank = (uint32_t)std::max(1.0, std::ceil(o->priority_fraction * (double)t.S));
  for (;;) {
    switch (p->st) {
      case ST_F64: small_launch_sum<ST_F64>(p, t, s); break;
      case ST_F32: small_launch_sum<ST_F32>(p, t, s); break;
      case ST_F32K: small_launch_sum<ST_F32K>(p, t, s); break;
      case ST_U32: small_launch<ST_U32, DAIC_G_EDGE_ADD>(p, t, s); break;
      case ST_F64MIN: small_launch<ST_F64MIN, DAIC_G_EDGE_ADD>(p, t, s); break;
      default: small_launch<ST_I32, DAIC_G_COPY>(p, t, s); break;
    }
    DAIC_HIP(hipGetLastError());
    DAIC_HIP(hipEventRecord(p->ev1, s));
    DAIC_HIP(hipEventSynchronize(p->ev1));
    if (p->h_ctl->done || p->h_ctl->stop) return DAIC_OK;
    t.resume = 1;
  }
}

void small_release(daic_problem* p) {
  delete p->small;
  p->small = nullptr;
}

}  // namespace daic
