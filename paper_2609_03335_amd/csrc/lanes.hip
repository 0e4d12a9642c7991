// The lane-per-plan scoring kernel: every lane of a wave scores a plan of its
// own, walking all of the plan's units level by level in resource order.
// Same results as the general kernel of score_kernel.h.
//
// Why: the kernels that give a lane to each (plan, device) walk a level in as
// many trips as its busiest device has units, over all plans of the wave --
// 73 trips for 8 plans of 256 activations on 8 devices, 44% of the lane-trips
// working.  A lane per plan has one unit per trip in every lane, table
// indices of the order sweep and of the releases are wave-uniform, and the
// plans' LDS arrays are [entry][lane], free of bank conflicts whatever the
// entry.  (The window's tables are not: each lane gathers them by its own
// unit, model or device, and those reads conflict: SQ_LDS_BANK_CONFLICT counts
// 183 M over the 93 M LDS instructions of the workload below.)
// The price is LDS: 64 plans' state per wave, so few waves per CU fit, and
// each wave hides its latency by reading a unit's tables and its device's
// state one unit ahead.  Batches too small for that take the other kernels.
//
// Per group of 64 plans:
//   1. the resource order (Eq. 10) is built level by level, the last one
//      first: slot = priority when the heads' priorities are distinct values
//      of the level's index range, else by (priority, index), which the whole
//      wave ranks for the plans that need it; a unit is marked
//      when no later one uses its model on its device, which the walk, first
//      level first, could not know.  The order goes to a scratch area in HBM
//      ([slot][lane], read back as whole rows): in LDS it and the unit counts
//      that would replace the marks took 40% of a wave's region;
//   2. per level, a host-made list of operations over the plan's live times
//      (slots) computes releases (Eq. 2): a time's slot is given to another
//      once its last reader is past, so a plan holds about one level's times;
//   3. the walk: residency, reclamation, memory and timeline of one unit per
//      trip (Eq. 5, 7, 11) on the device state in LDS.
// Window tables that only the walk needs per lane are in LDS.
//
// Bound by LDS capacity: 1,048,576 plans of 256 activations on 8 devices keep
// 84 live times and 24 words of device state each, so five waves share a CU and
// each waits for its own LDS reads (about 1,130 cycles per unit against some
// 130 vector instructions).  2,645 us there against 3,490 us with a lane per
// (plan, device): 343 GB/s of plan rows and records, 49,000 against 79,000
// vector lane-instructions per plan; with the scratch rows the HBM traffic is
// four times the rows and records (3.6 against 0.91 GB), which the walk hides.
// With the order in LDS (three waves per CU) it took 4,482 us.
#include <type_traits>

#include "kernels.h"
#include "mutation.h"

namespace wfp {
namespace {

template <typename T>
using Uniform = const __attribute__((address_space(4))) T*;  // read with scalar loads

template <typename T>
__device__ __forceinline__ Uniform<T> uniform_at(const unsigned char* base, int off) {
  return (Uniform<T>)(uintptr_t)(base + off);
}

__device__ __forceinline__ void wsync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }

// saturating (one instruction either way): where the host has not proven
// that no time reaches 2^32, a saturated time ends in the latest finish
__device__ __forceinline__ uint32_t tadd(uint32_t a, uint32_t b) {
  return __builtin_elementwise_add_sat(a, b);
}

template <typename T>
__device__ __forceinline__ T load_any(const void* p) {  // any alignment
  T v;
  __builtin_memcpy(&v, p, sizeof(T));
  return v;
}

// A candidate as the incumbent's rows plus its changed sites, lane-major in
// LDS: per site (activation | priority << 16), and (device & 255 | flag bits
// << 8) in 16 bits.
struct LaneSites {
  uint32_t* p;
  uint16_t* q;
  int n;
  const int8_t* idev;
  const uint16_t* iprio;
  const uint8_t* iflags;
  __device__ __forceinline__ uint32_t& w(int k) const { return p[k << 6]; }
  __device__ __forceinline__ uint16_t& x(int k) const { return q[k << 6]; }
  __device__ __forceinline__ int find(int i) const {
    for (int k = 0; k < n; ++k)
      if ((int)(w(k) & 0xffffu) == i) return k;
    return -1;
  }
  __device__ __forceinline__ int site(int i) {
    int k = find(i);
    if (k < 0) {
      k = n++;
      w(k) = (uint32_t)i | ((uint32_t)iprio[i] << 16);
      x(k) = (uint16_t)((uint32_t)(uint8_t)idev[i] |
                        ((((uint32_t)iflags[i >> 2] >> ((i & 3) << 1)) & 3u) << 8));
    }
    return k;
  }
  __device__ __forceinline__ int dev(int i) const {
    const int k = find(i);
    return k >= 0 ? (int)(int8_t)(x(k) & 0xffu) : (int)idev[i];
  }
  __device__ __forceinline__ int prio(int i) const {
    const int k = find(i);
    return k >= 0 ? (int)(w(k) >> 16) : (int)iprio[i];
  }
  __device__ __forceinline__ uint32_t flags(int i) const {
    const int k = find(i);
    return k >= 0 ? ((uint32_t)x(k) >> 8) & 3u
                  : ((uint32_t)iflags[i >> 2] >> ((i & 3) << 1)) & 3u;
  }
  __device__ __forceinline__ void set_dev(int i, int d) {
    const int k = site(i);
    x(k) = (uint16_t)((x(k) & ~0xffu) | ((uint32_t)d & 0xffu));
  }
  __device__ __forceinline__ void swap_prio(int i, int j) {
    const int ki = site(i), kj = site(j);
    const uint32_t pi = w(ki) >> 16, pj = w(kj) >> 16;
    w(ki) = (uint32_t)i | (pj << 16);
    w(kj) = (uint32_t)j | (pi << 16);
  }
  __device__ __forceinline__ void toggle_flag(int i, int bit) {
    const int k = site(i);
    x(k) = (uint16_t)(x(k) ^ (0x100u << bit));
  }
  __device__ __forceinline__ void set_prefetch(int i, bool on) {
    const int k = site(i);
    x(k) = (uint16_t)(on ? x(k) | 0x200u : x(k) & ~0x200u);
  }
};

// Rows of eight consecutive activations: devices, priorities, flag bits.
struct Chunk {
  uint64_t dv;
  uint64_t p0, p1;
  uint32_t fl;
  uint32_t a[8];  // activation words (uniform)
  uint32_t lw[8];  // first index of the level | width << 16 (uniform)
  bool plain;     // none of them may be fused (uniform)
  uint32_t cb[8];  // fuse bits of the chain successors (bit 0)
};

// QB, F: reclamation queue of QB bits holding F-bit model ids (F = 4: at most
// 16 models; F = 5: at most 32 models, 12 entries).  SEARCH: candidates
// around an incumbent.  PHI: ranking keys (Eq. 12).  RCAP: replica caps.
template <int QB, int F, bool SEARCH, bool PHI, bool RCAP>
__global__ __launch_bounds__(64 * kLanesWaves) void score_lanes(
    ScoreParams sp, LanesParams lp, const int8_t* __restrict__ dev_all,
    const uint16_t* __restrict__ prio_all, const uint8_t* __restrict__ flags_all, int64_t P,
    wf_plan_score* __restrict__ scores, SearchArgs sa) {
  using QT = std::conditional_t<QB == 32, uint32_t, uint64_t>;
  constexpr QT kOnes = F == 4 ? (QT)0x1111111111111111ull : (QT)0x084210842108421ull;
  constexpr QT kHigh = kOnes << (F - 1);
  constexpr uint32_t kId = (1u << F) - 1u;
  // state words of a device: queue, busy-until, free memory and queue lengths
  constexpr int kQw = QB / 32, kFree = kQw, kPack = kQw + 1, kRec = kQw + 2;
  constexpr int kRm = kQw + 2 + (PHI ? 1 : 0);
  constexpr int SW = kQw + 2 + (PHI ? 1 : 0) + (RCAP ? 1 : 0);
  // order entry of a level being sorted (16 bits): 1 + (index in the level |
  // device << ub | prefetch | fused successor), 0 for none; of the whole
  // order: activation | device | model | fused successor | the model's last
  // use on the device | prefetch | occupied
  constexpr uint32_t kPf16 = 1u << 14, kChain16 = 1u << 15;
  constexpr uint32_t kChain = 1u << 28, kLast = 1u << 29, kPf = 1u << 30, kValid = 1u << 31;
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = sp.N, W = sp.W, M = sp.M, D = sp.D, NB = sp.NB;
  {
    const uint4* src = reinterpret_cast<const uint4*>(lp.tab);
    uint4* dst = reinterpret_cast<uint4*>(lds);
    for (int i = tid; i < (lp.t.lds_bytes >> 4); i += blockDim.x) dst[i] = src[i];
  }
  int* s_next = reinterpret_cast<int*>(lds + lp.t.lds_bytes);
  if (tid == 0) *s_next = lp.waves;
  __syncthreads();
  const unsigned char* tg = lp.tab;
  const uint4* t_rec = reinterpret_cast<const uint4*>(lds + lp.t.rec);
  const uint4* t_wm = reinterpret_cast<const uint4*>(lds + lp.t.wm);
  const uint32_t* t_ld = reinterpret_cast<const uint32_t*>(lds + lp.t.ld);
  const int2* t_um = reinterpret_cast<const int2*>(tg + lp.t.um);
  const uint32_t* t_op = reinterpret_cast<const uint32_t*>(tg + lp.t.op);
  const Uniform<uint32_t> u_act = uniform_at<uint32_t>(tg, lp.t.act);
  const Uniform<uint32_t> u_alv = uniform_at<uint32_t>(tg, lp.t.alv);
  const uint32_t* t_alv = reinterpret_cast<const uint32_t*>(tg + lp.t.alv);
  const Uniform<int32_t> u_grp = uniform_at<int32_t>(tg, lp.t.grp);
  const Uniform<int32_t> u_ooff = uniform_at<int32_t>(tg, lp.t.ooff);
  const Uniform<int32_t> u_loff = uniform_at<int32_t>(tg, lp.t.loff);
  const Uniform<int32_t> u_run = uniform_at<int32_t>(tg, lp.t.run);
  const Uniform<int32_t> u_cap = uniform_at<int32_t>(tg, lp.t.cap);
  const Uniform<uint32_t> u_res0 = uniform_at<uint32_t>(tg, lp.t.res0);
  const Uniform<uint32_t> u_free0 = uniform_at<uint32_t>(tg, lp.t.free0);
  const Uniform<uint32_t> u_arr = uniform_at<uint32_t>(tg, lp.t.arr);
  const Uniform<int32_t> u_wmib = uniform_at<int32_t>(tg, lp.t.wmib);
  const Uniform<int32_t> u_rcap = uniform_at<int32_t>(tg, lp.t.rcap);

  unsigned char* wl = lds + lp.t.lds_bytes + 16 + lp.wave_bytes * wid;
  uint32_t* s_slot = reinterpret_cast<uint32_t*>(wl) + lane;
  uint32_t* s_st = reinterpret_cast<uint32_t*>(wl + lp.st) + lane;
  uint16_t* s_ord = reinterpret_cast<uint16_t*>(wl + lp.ord) + lane;
  uint32_t* s_site = reinterpret_cast<uint32_t*>(wl + lp.site) + lane;

  const int ub = lp.ub;
  const uint32_t umask = (1u << ub) - 1u, dmask = (1u << (14 - ub)) - 1u;
  const int kk = (95 * W + 99) / 100;
  const int64_t n_groups = (P + 63) >> 6;
  uint32_t* g_ord = reinterpret_cast<uint32_t*>(lp.scratch) +
                    ((int64_t)blockIdx.x * lp.waves + wid) * ((int64_t)(N + 4) * 64) + lane;

  // the workgroup's groups are blockIdx.x + k gridDim.x; a wave takes the
  // next one when it is free (waves that share a SIMD are slower)
  int take = wid;
  for (;;) {
    const int64_t grp = (int64_t)blockIdx.x + (int64_t)take * gridDim.x;
    if (grp >= n_groups) break;
    const int64_t pl = grp * 64 + lane;
    const int64_t pr_ = pl < P ? pl : P - 1;  // lanes past the end repeat the last plan
    const int8_t* rdev = SEARCH ? dev_all : dev_all + pr_ * N;
    const uint16_t* rprio = SEARCH ? prio_all : prio_all + pr_ * N;
    const uint8_t* rfl = SEARCH ? flags_all : flags_all + pr_ * NB;
    LaneSites sites{s_site, reinterpret_cast<uint16_t*>(wl + lp.site2) + lane, 0, dev_all, prio_all, flags_all};
    int n_sites = 0;  // the most any lane has
    if constexpr (SEARCH) {
      mutate_rows((uint64_t)(sa.first + pr_), sa, N, sa.elig,
                  reinterpret_cast<const uint32_t*>(tg + lp.t.alv), sites);
      const int mine = sites.n;
      for (int b = 16; b >= 0; --b)
        if (__ballot(mine > n_sites + (1 << b) - 1) != 0ull) n_sites += 1 << b;
    }
    // activations o .. o + 7 of the lane's plan (o + 8 <= N)
    auto chunk = [&](int o) -> Chunk {
      Chunk c;
      c.dv = load_any<uint64_t>(rdev + o);
      c.p0 = load_any<uint64_t>(rprio + o);
      c.p1 = load_any<uint64_t>(rprio + o + 4);
      const int fo = (o >> 2) < NB - 4 ? (o >> 2) : NB - 4;
      c.fl = load_any<uint32_t>(rfl + fo) >> (2 * o - 8 * fo);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        c.a[j] = u_act[o + j];
        c.lw[j] = u_alv[o + j];
      }
      uint32_t any = 0u, all = ~0u;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        any |= c.a[j];
        all &= c.a[j];
      }
      c.plain = !(any & 64u) && (all >> 16) == 0xffffu;
#pragma unroll
      for (int j = 0; j < 8; ++j) c.cb[j] = 0u;
      if (!SEARCH && !c.plain) {
#pragma unroll
        for (int j = 0; j < 8; ++j)  // (shifted where it is used: no wait here)
          if ((c.a[j] >> 16) != 0xffffu) c.cb[j] = rfl[c.a[j] >> 18];
      }
      if constexpr (SEARCH) {
        for (int k = 0; k < n_sites; ++k) {
          const uint32_t w0 = sites.w(k);
          const uint32_t at = (w0 & 0xffffu) - (uint32_t)o;
          if (k < sites.n && at < 8u) {
            const uint32_t w1 = sites.x(k);
            c.dv = (c.dv & ~(0xffull << (8 * at))) | ((uint64_t)(w1 & 0xffu) << (8 * at));
            const uint32_t sh = (at & 3u) * 16u;
            const uint64_t keep = ~(0xffffull << sh), put = (uint64_t)(w0 >> 16) << sh;
            if (at < 4u)
              c.p0 = (c.p0 & keep) | put;
            else
              c.p1 = (c.p1 & keep) | put;
            c.fl = (c.fl & ~(3u << (2 * at))) | (((w1 >> 8) & 3u) << (2 * at));
          }
        }
      }
      return c;
    };
    auto fuse_of = [&](int v) -> bool {
      if constexpr (SEARCH) {
        return (sites.flags(v) & 1u) != 0u;
      } else {
        return (((uint32_t)rfl[v >> 2] >> ((v & 3) << 1)) & 1u) != 0u;
      }
    };

    // ---- the resource order (Eq. 10), last levels first: as many
    // consecutive levels as fit the live times' storage are sorted in LDS at
    // a time and written out one row per slot, every unit marked when no
    // later one uses its model on its device (a device out of range makes
    // the plan ineligible; it is walked on the last device) ----
    uint32_t inel = 0u, dmax = 0u;
    for (int d = 0; d < D; ++d) s_st[(d * SW) << 6] = 0u;  // models used later, per device
    auto first_of = [&](int lv) {
      const int c8 = u_loff[lv] & ~7;
      return chunk(c8 < N - 8 ? c8 : N - 8);
    };
    // (of plan b of the wave, read by every lane: activation u's priority,
    // flag bits and device)
    struct Gene {
      uint32_t pr, fb, d;
    };
    const int64_t last = P - 1 - grp * 64;  // the group's last plan
    auto gene_of = [&](int b, int u) -> Gene {
      if constexpr (SEARCH) {
        LaneSites sb = sites;
        sb.p += b - lane;
        sb.q += b - lane;
        sb.n = __builtin_amdgcn_readlane(sites.n, b);
        const int k = sb.find(u);
        if (k >= 0)
          return {sb.w(k) >> 16, ((uint32_t)sb.x(k) >> 8) & 3u, (uint32_t)sb.x(k) & 0xffu};
        return {prio_all[u], ((uint32_t)flags_all[u >> 2] >> ((u & 3) << 1)) & 3u,
                (uint32_t)(uint8_t)dev_all[u]};
      } else {
        const int64_t p = grp * 64 + b;
        return {prio_all[p * N + u],
                ((uint32_t)flags_all[p * NB + (u >> 2)] >> ((u & 3) << 1)) & 3u,
                (uint32_t)(uint8_t)dev_all[p * N + u]};
      }
    };
    int at_grp = lp.n_grp - 1, lb = sp.n_levels, la = u_grp[at_grp];
    Chunk first = first_of(la);
    while (lb > 0) {
      const int lo = u_loff[la], hi = u_loff[lb], w = hi - lo;
      // the rows, and the two after them, start empty; every head is put at
      // its priority (a last row takes those outside their level's range),
      // and when as many rows are occupied, over all lanes, as there are
      // heads, none was hit twice
      const int n16 = (w + 2) * 8;
      const uint32_t out = (uint32_t)lp.rows + 2u;
      uint4* o16 = reinterpret_cast<uint4*>(wl + lp.ord);
      for (int i = lane; i < n16; i += 64) o16[i] = make_uint4(0u, 0u, 0u, 0u);
      wsync();
      int fused = 0;  // of the lane's plan: activations that are no heads
      auto place = [&](const Chunk& c, int j, uint32_t base, auto plain) {
        const uint32_t d = (uint32_t)(c.dv >> (8 * j)) & 0xffu;
        const uint32_t pr = (uint32_t)((j < 4 ? c.p0 : c.p1) >> (16 * (j & 3))) & 0xffffu;
        const uint32_t fb = c.fl >> (2 * j);
        uint32_t e = (base + (uint32_t)j) + (umin(d, (uint32_t)D - 1u) << ub) + ((fb & 2u) << 13);
        uint32_t at = pr - (c.lw[j] & 0xffffu);
        at = at < (c.lw[j] >> 16) ? pr - (uint32_t)lo : out;
        if constexpr (decltype(plain)::value) {
          dmax = umax(dmax, d);
        } else {
          const uint32_t a = c.a[j];
          if ((a >> 16) != 0xffffu) {
            uint32_t cb = c.cb[j];
            if constexpr (SEARCH) cb = sites.flags((int)(a >> 16)) << ((a >> 15) & 6u);
            e += ((cb >> ((a >> 15) & 6u)) & 1u) << 15;
          }
          if (a & 64u) {
            const bool head = !(fb & 1u);
            fused += head ? 0 : 1;
            at = head ? at : out;
            dmax = head ? umax(dmax, d) : dmax;
          } else {
            dmax = umax(dmax, d);
          }
        }
        s_ord[at << 6] = (uint16_t)e;
      };
      {
        Chunk c = first;
        for (int c8 = lo & ~7; c8 < hi; c8 += 8) {
          const int o = c8 < N - 8 ? c8 : N - 8;
          const int on = c8 + 8 < hi ? (c8 + 8 < N - 8 ? c8 + 8 : N - 8) : o;
          const Chunk cn = chunk(on);
          const int ua = lo > c8 ? lo : c8;
          const uint32_t base = (uint32_t)(o - lo) + 1u;  // entries are stored plus 1
          if (c.plain && ua == o && o + 8 <= hi) {
#pragma unroll
            for (int j = 0; j < 8; ++j) place(c, j, base, std::true_type{});
          } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
              if (o + j >= ua && o + j < hi) place(c, j, base, std::false_type{});
          }
          c = cn;
        }
      }
      wsync();
      bool ranked;
      {
        uint32_t mine = (uint32_t)fused;
        for (int i = lane; i < n16; i += 64) {
          const uint4 v = o16[i];
          mine += (uint32_t)((v.x & 0xffffu) != 0u) + (uint32_t)((v.x >> 16) != 0u) +
                  (uint32_t)((v.y & 0xffffu) != 0u) + (uint32_t)((v.y >> 16) != 0u) +
                  (uint32_t)((v.z & 0xffffu) != 0u) + (uint32_t)((v.z >> 16) != 0u) +
                  (uint32_t)((v.w & 0xffffu) != 0u) + (uint32_t)((v.w >> 16) != 0u);
        }
        int sum = 0;  // occupied rows and fused activations
        for (int b = 0; (8 * ((n16 + 63) >> 6) + w) >> b; ++b)
          sum += __popcll(__ballot((mine >> b) & 1u)) << b;
        ranked = sum != 64 * w;
      }
      if (ranked) {
        // the plans whose priorities are no such permutation, one after the
        // other by the whole wave: a lane takes an activation of a run of
        // levels (up to 64 activations, or one wider level in pieces of 64)
        // and counts the keys below its own: (level, priority, index), a
        // fused activation behind its level's heads.  (One such plan in a wave
        // is common where a few percent of the plans are such; ranked by its
        // own lane alone, it takes w^2 steps per level that every lane waits
        // for.  131,072 plans of 400 activations in four levels with 2% such
        // plans: 15,300 us that way, 1,124 us this way, 914 us with none; all
        // such: 4,810 us, the kernel with a lane per (plan, device) 18,500.)
        int own = fused;
        for (int i = 0; i < w; ++i) own += s_ord[i << 6] != 0 ? 1 : 0;
        for (uint64_t bad = __ballot(own != w && lane <= last); bad; bad &= bad - 1ull) {
          const int b = __builtin_ctzll(bad);
          uint16_t* ob = s_ord + (b - lane);
          for (int lv = la, le; lv < lb; lv = le) {
            le = u_run[lv];
            const int l0 = u_loff[lv], rw = u_loff[le] - l0, sh = rw <= 64 ? 6 : 11;
            auto key_of = [&](int i, uint32_t& e) -> uint32_t {  // e: the row's entry
              if (i >= rw) return ~0u;
              const int u = l0 + i;
              const uint4 r = t_rec[u];
              const Gene g = gene_of(b, u);
              const bool chain = r.w != 0xffffu && (gene_of(b, (int)r.w).fb & 1u);
              const bool member = (r.x & 64u) && (g.fb & 1u);
              e = member ? 0u
                         : (uint32_t)(u - lo) + 1u + (umin(g.d, (uint32_t)D - 1u) << ub) +
                               ((g.fb & 2u) << 13) + (chain ? kChain16 : 0u);
              const uint32_t lv0 = (t_alv[u] & 0xffffu) - (uint32_t)l0;
              return (lv0 << 23) | ((member ? 0x10000u : g.pr) << sh) | (uint32_t)i;
            };
            for (int c0 = 0; c0 < rw; c0 += 64) {
              uint32_t e = 0u, e2 = 0u, rank = 0u;
              const uint32_t key = key_of(c0 + lane, e);
              for (int c2 = 0; c2 < rw; c2 += 64) {
                const uint32_t k2 = c2 == c0 ? key : key_of(c2 + lane, e2);
                const int n = rw - c2 < 64 ? rw - c2 : 64;
                for (int j0 = 0; j0 < n; j0 += 16)
#pragma unroll
                  for (int j = 0; j < 16; ++j)
                    rank += (uint32_t)__builtin_amdgcn_readlane((int)k2, j0 + j) < key ? 1u : 0u;
              }
              if (c0 + lane < rw) ob[(l0 - lo + (int)rank) << 6] = (uint16_t)e;
            }
          }
        }
        wsync();
      }
      // the next levels, their first rows read ahead
      const int lb2 = la;
      const int la2 = lb2 > 0 ? u_grp[--at_grp] : 0;
      first = first_of(la2);
      {
        // the unit after next is read, and the next one's model and its
        // device's mask, while this one is marked
        struct Row {
          uint32_t e, u, d, m, seen;
          bool valid;
        };
        auto fetch = [&](uint32_t e, Row& R) {
          R.valid = e != 0u;
          R.e = e ? e - 1u : 0u;
          R.u = (uint32_t)lo + (R.e & umask);
          R.d = (R.e >> ub) & dmask;
          R.m = t_rec[R.u].x & 63u;
        };
        auto mark = [&](int i, uint32_t en, Row& R, Row& Q) {
          fetch(en, Q);
          Q.seen = s_st[(Q.d * SW) << 6];
          const uint32_t bit = R.valid ? 1u << (R.m & 31u) : 0u;
          const uint32_t row = (R.seen & bit) ? 0u : kLast;
          const uint32_t x = R.u | (R.d << 16) | (R.m << 22) | row | ((R.e & kPf16) << 16) |
                             ((R.e & kChain16) << 13) | kValid;
          g_ord[(lo + i) << 6] = R.valid ? x : 0u;
          R.seen |= bit;
          s_st[(R.d * SW) << 6] = R.seen;
          if (Q.d == R.d) Q.seen = R.seen;
        };
        Row A, B;
        fetch(s_ord[(w - 1) << 6], A);
        A.seen = s_st[(A.d * SW) << 6];
        uint32_t e = w > 1 ? s_ord[(w - 2) << 6] : 0u;
        for (int i = w - 1; i >= 0; i -= 2) {
          uint32_t e2 = i > 1 ? s_ord[(i - 2) << 6] : 0u;
          mark(i, e, A, B);
          e = i > 2 ? s_ord[(i - 3) << 6] : 0u;
          if (i > 0) mark(i - 1, e2, B, A);
        }
      }
      wsync();
      la = la2;
      lb = lb2;
    }
    if (dmax >= (uint32_t)D) inel = 1u;
    // ---- device state: resident models, those with no remaining use first ----
    int32_t pe = (int32_t)0x80000000;
    for (int d = 0; d < D; ++d) {
      QT q = 0, qa = 0;
      uint32_t nd = 0u, na = 0u;
      int32_t fm = u_cap[d];
      const uint32_t res = u_res0[d], seen = s_st[(d * SW) << 6];
      for (uint32_t r = res; r; r &= r - 1u) {
        const uint32_t m = (uint32_t)__builtin_ctz(r);
        fm -= u_wmib[m];
        const bool used = ((seen >> m) & 1u) != 0u;
        q |= used ? (QT)0 : (QT)m << nd;
        qa |= used ? (QT)m << na : (QT)0;
        nd += used ? 0u : F;
        na += used ? F : 0u;
      }
      if (na) q |= qa << nd;
      pe = -fm > pe ? -fm : pe;
      uint32_t* st = s_st + ((d * SW) << 6);
      st[0] = (uint32_t)q;
      if constexpr (QB == 64) st[64] = (uint32_t)((uint64_t)q >> 32);
      st[kFree << 6] = u_free0[d];
      st[kPack << 6] = ((uint32_t)fm << 10) | (((nd + na) / F) << 5) | (nd / F);
      if constexpr (PHI) st[kRec << 6] = 0u;
      if constexpr (RCAP) st[kRm << 6] = res | (res << 16);
    }
    for (int i = 0; i < lp.n_zero; ++i) s_slot[i << 6] = 0u;

    uint32_t mk = 0u, p95 = 0u, nld = 0u, nev = 0u, over = 0u;
    uint32_t ph_cf = 0u, ph_pn = 0u;
    unsigned long long ph_adm = 0ull, ph_h = 0ull;
    wsync();

    // ---- operations over the live times before level lv (after the last
    // level: what completions still need) ----
    auto ops_at = [&](int base, int oe) -> uint32_t { return base + lane < oe ? t_op[base + lane] : 0u; };
    uint32_t ops = ops_at(u_ooff[0], u_ooff[1]);  // the first ones, read ahead
    auto boundary = [&](int lv) {
      const int ob = u_ooff[lv], oe = u_ooff[lv + 1];
      uint32_t acc = 0u;
      unsigned char* sb = wl + 4 * lane;
      for (int base = ob; base < oe; base += 64) {
        const uint32_t w = base == ob ? ops : ops_at(base, oe);
        const int n = oe - base < 64 ? oe - base : 64;  // a multiple of 8
        for (int i = 0; i < n; i += 8) {
          uint32_t o[8], v[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            o[k] = (uint32_t)__builtin_amdgcn_readlane((int)w, i + k);
            v[k] = *reinterpret_cast<const uint32_t*>(sb + (o[k] & 0x3ff00u));
          }
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            // (without the store bit the target is the slot nobody reads)
            acc = umax(acc, v[k]);
            *reinterpret_cast<uint32_t*>(sb + ((o[k] >> 10) & 0x3ff00u)) = acc;
            acc &= ~(uint32_t)((int32_t)o[k] >> 31);
          }
        }
      }
    };

    for (int lv = 0; lv < sp.n_levels; ++lv) {
      const int lo = u_loff[lv], hi = u_loff[lv + 1], w = hi - lo;
      const uint32_t e0 = g_ord[lo << 6];
      uint32_t e1 = g_ord[(lo + 1) << 6], e2 = g_ord[(lo + 2) << 6];
      boundary(lv);
      ops = ops_at(u_ooff[lv + 1], u_ooff[lv + 2]);
      // ---- the walk ----
      struct Unit {
        uint32_t e, d, u;
        uint4 a;     // activation word, arrival, release slot | finish slot << 16, chain successor
        int2 um;     // run time, memory
        uint4 wm;    // model weights, model id in every queue field
        uint32_t ld, r;
      };
      auto fetch_a = [&](uint32_t e, Unit& X) {
        X.e = e;
        X.u = e & 0xffffu;
        X.d = (e >> 16) & 63u;
        X.a = t_rec[X.u];
        X.um = t_um[__umul24(X.d, (uint32_t)N) + X.u];
      };
      auto fetch_b = [&](Unit& X) {
        const uint32_t m = (X.e >> 22) & 31u;
        X.wm = t_wm[m];
        X.ld = t_ld[__umul24(X.d, (uint32_t)M) + m];
        X.r = umax(s_slot[(X.a.z & 0xffffu) << 6], X.a.y);
      };
      struct State {
        QT q;
        uint32_t freet, pack, rec, rm;
      };
      auto read_state = [&](uint32_t d, State& S) {
        const uint32_t* st = s_st + ((d * SW) << 6);
        S.q = st[0];
        if constexpr (QB == 64) S.q |= (QT)((uint64_t)st[64] << 32);
        S.freet = st[kFree << 6];
        S.pack = st[kPack << 6];
        if constexpr (PHI) S.rec = st[kRec << 6];
        if constexpr (RCAP) S.rm = st[kRm << 6];
      };
      // (rows past the level's are the next one's: masked where they are used,
      // so that every load is issued whatever the level and waits for none)
      auto get = [&](int i) -> uint32_t { return g_ord[(lo + i) << 6]; };
      // one unit: X with its device's state S; Y and T are the next one's
      auto step = [&](int s, Unit& X, State& S, Unit& Y, State& T) {
        fetch_a(s + 1 < w ? e1 : 0u, Y);
        e1 = e2;
        e2 = get(s + 3);
        const bool valid = (X.e & kValid) != 0u;
        const uint32_t m = (X.e >> 22) & 31u;
        // run time and memory of the unit (Eq. 4: a fused chain's largest)
        int32_t mx = X.um.y;
        const bool chain = valid && (X.e & kChain) != 0u;
        if (valid) inel |= (uint32_t)X.um.x >> 31;
        if (chain) {
          for (uint32_t v = X.a.w;;) {
            const int2 lm = t_um[X.d * N + v];
            inel |= (uint32_t)lm.x >> 31;
            mx = lm.y > mx ? lm.y : mx;
            const uint32_t c = t_rec[v].w;
            if (c == 0xffffu || !fuse_of((int)c)) break;
            v = c;
          }
        }
        // residency: m among the queue's entries; a hit takes it out (it
        // re-enters below as the most recent)
        QT Q = S.q;
        int32_t fm = (int32_t)S.pack >> 10;
        uint32_t nq = ((S.pack >> 5) & 31u) * F, nd = (S.pack & 31u) * F;
        QT mq = (QT)X.wm.y;
        if constexpr (QB == 64) mq |= (QT)((uint64_t)X.wm.z << 32);
        const QT x = Q ^ mq;
        QT z = (x - kOnes) & ~x & kHigh;  // lowest flag: first matching field
        const QT in = nq >= (uint32_t)QB ? ~(QT)0 : (((QT)1 << nq) - (QT)1);
        z &= in;
        const bool hit = z != (QT)0;
        {
          uint32_t at;  // position of the field's top bit
          if constexpr (QB == 64)
            at = (uint32_t)__builtin_ctzll(z | (1ull << 63));
          else
            at = (uint32_t)__builtin_ctz(z | (1u << 31));
          const uint32_t pos = at - (F - 1);
          const QT low = ((QT)1 << (pos & (QB - 1))) - (QT)1;
          const QT rem = (Q & low) | ((Q >> F) & ~low);
          Q = hit ? rem : Q;
          nq -= hit ? (uint32_t)F : 0u;
        }
        int32_t ex = mx + (hit ? 0 : (int32_t)X.wm.x) - fm;
        uint32_t gone = 0u, pops = 0u;
        // reclaim (Sec. 3.5) from the queue's front; four victims without a
        // branch, any further ones in a loop
        {
          uint32_t v[4];
          int32_t wv[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            v[k] = (uint32_t)(Q >> (k * F)) & kId;
            wv[k] = (int32_t)t_wm[v[k]].x;
          }
          // victims needed: the prefixes of the weights the excess is above
          // (independent compares: weights are not negative)
          const int32_t p2 = wv[0] + wv[1], p3 = p2 + wv[2];
          uint32_t need = ex > 0 ? (uint32_t)F : 0u;
          need += ex > wv[0] ? (uint32_t)F : 0u;
          need += ex > p2 ? (uint32_t)F : 0u;
          need += ex > p3 ? (uint32_t)F : 0u;
          pops = umin(need, nq);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const bool c = pops > (uint32_t)(k * F);
            ex -= c ? wv[k] : 0;
            if constexpr (PHI || RCAP) gone |= c ? 1u << v[k] : 0u;
          }
          Q >>= pops;
          nq -= pops;
          while (valid && pops >= 4u * F && ex > 0 && nq >= (uint32_t)F) {
            const uint32_t x = (uint32_t)Q & kId;
            Q >>= F;
            nq -= F;
            pops += F;
            ex -= (int32_t)t_wm[x].x;
            if constexpr (PHI || RCAP) gone |= 1u << x;
          }
          nd = nd > pops ? nd - pops : 0u;
        }
        fetch_b(Y);
        read_state(Y.d, T);
        // m re-enters after the entries with no remaining use when this was
        // its last unit on the device, else at the end
        {
          const uint32_t pos = (X.e & kLast) ? nd : nq;
          const QT low = ((QT)1 << pos) - (QT)1;
          Q = (Q & low) | ((QT)m << pos) | ((Q & ~low) << F);
          nd += (X.e & kLast) ? (uint32_t)F : 0u;
          nq += F;
        }
        // timeline (Eq. 7): a load waits for the device and starts at the
        // release, or at the workflow arrival when prefetched
        const bool pf = (X.e & kPf) != 0u;
        const uint32_t a0 = pf ? X.a.y : X.r;
        const uint32_t ls = umax(a0, S.freet);
        const uint32_t le = tadd(ls, X.ld);
        const uint32_t start = umax(X.r, hit ? S.freet : le);
        if (valid) {
          pe = ex > pe ? ex : pe;
          nld += hit ? 0u : 1u;
          nev += pops;
          const uint32_t fr0 = S.freet;
          uint32_t f = tadd(start, (uint32_t)X.um.x);
          atomicMax(&s_slot[(X.a.z >> 16) << 6], f);
          p95 = umax(p95, f - X.a.y);
          if (chain) {  // members back to back on the head's device
            for (uint32_t v = X.a.w;;) {
              const uint4 av = t_rec[v];
              f = tadd(f, (uint32_t)t_um[X.d * N + v].x);
              atomicMax(&s_slot[(av.z >> 16) << 6], f);
              p95 = umax(p95, f - av.y);
              if (av.w == 0xffffu || !fuse_of((int)av.w)) break;
              v = av.w;
            }
          }
          mk = umax(mk, f);
          S.q = Q;
          S.freet = f;
          S.pack = ((uint32_t)(mx - ex) << 10) | ((nq / F) << 5) | (nd / F);
          if constexpr (RCAP) S.rm = ((S.rm & ~gone) | (1u << m)) | (0x10000u << m);
          if constexpr (PHI) {
            S.rec |= gone;
            const bool ready = ((X.a.x >> 7) & 1u) != 0u;
            if (!hit) {
              if ((S.rec >> m) & 1u) ph_h += (uint64_t)X.ld;  // reload of a reclaimed copy
              if (!ready && pf && le <= X.r) ++ph_pn;         // a timely prefetch
              if (ready) ph_h += (uint64_t)(start - umax(X.r, fr0));
            }
            if (ready && ex <= 0) {
              ph_adm += 1ull << (16u * ((X.a.x >> 8) & 3u));
              ph_cf = umax(ph_cf, f);
            }
          }
          uint32_t* st = s_st + ((X.d * SW) << 6);
          st[0] = (uint32_t)S.q;
          if constexpr (QB == 64) st[64] = (uint32_t)((uint64_t)S.q >> 32);
          st[kFree << 6] = S.freet;
          st[kPack << 6] = S.pack;
          if constexpr (PHI) st[kRec << 6] = S.rec;
          if constexpr (RCAP) st[kRm << 6] = S.rm;
        }
        // the next unit's device state: this unit's when the device is the same
        if (Y.d == X.d) T = S;
      };
      // (two units per trip, so that nothing is copied; one past the level's
      // last is empty)
      {
        Unit X, Y;
        State S, T;
        fetch_a(e0, X);
        fetch_b(X);
        read_state(X.d, S);
        for (int s = 0; s < w; s += 2) {
          step(s, X, S, Y, T);
          step(s + 1, Y, T, X, S);
        }
      }
      // ---- replica caps: models held as the level started or loaded in it,
      // counted over the devices in bit planes ----
      if constexpr (RCAP) {
        uint32_t b[7] = {};
        for (int d = 0; d < D; ++d) {
          uint32_t* st = s_st + ((d * SW + kRm) << 6);
          const uint32_t r = *st;
          uint32_t c = r >> 16;
#pragma unroll
          for (int k = 0; k < 7; ++k) {
            const uint32_t t = b[k] & c;
            b[k] ^= c;
            c = t;
          }
          *st = (r & 0xffffu) | (r << 16);
        }
        for (int m = 0; m < M; ++m) {
          int n = 0;
#pragma unroll
          for (int k = 0; k < 7; ++k) n += (int)((b[k] >> m) & 1u) << k;
          over |= (uint32_t)(n > u_rcap[m]);
        }
      }
      wsync();
    }

    uint32_t status = (pe > 0 ? (uint32_t)WF_ST_CAPACITY : 0u) |
                      (over ? (uint32_t)WF_ST_REPLICA : 0u);
    if (lp.checked && mk == 0xffffffffu) status |= kRescore;
    if constexpr (PHI) {
      wf_plan_key k;
      k.c_ready_us = 0;
      k.h_life_us = 0;
      for (int c = 0; c < WF_MAX_CLASSES; ++c) k.admitted[c] = 0;
      k.timely_prefetch = 0;
      k.pad = 0;
      k.status = inel ? (uint32_t)WF_ST_INELIGIBLE : status;
      if (!inel) {
        if (ph_adm) k.c_ready_us = sp.origin + (int64_t)ph_cf;
        k.h_life_us = (int64_t)ph_h;
        for (int c = 0; c < WF_MAX_CLASSES; ++c)
          k.admitted[c] = (uint16_t)((ph_adm >> (16 * c)) & 0xffffull);
        k.timely_prefetch = (uint16_t)(ph_pn > 65535u ? 65535u : ph_pn);
      }
      if (pl < P) reinterpret_cast<wf_plan_key*>(scores)[pl] = k;
    } else {
      if (kk < W) {
        // nearest-rank p95 is the (W - kk + 1)-th largest completion latency
        boundary(sp.n_levels);
        uint32_t t0 = 0u, t1 = 0u, t2 = 0u, t3 = 0u;
        for (int a = 0; a < W; ++a) {
          uint32_t v = s_slot[(2 + a) << 6] - u_arr[a], hi_;
          hi_ = umax(t0, v); v = umin(t0, v); t0 = hi_;
          hi_ = umax(t1, v); v = umin(t1, v); t1 = hi_;
          hi_ = umax(t2, v); v = umin(t2, v); t2 = hi_;
          t3 = umax(t3, v);
        }
        const int k = W - kk;
        p95 = k == 1 ? t1 : (k == 2 ? t2 : t3);
      }
      wf_plan_score sc;
      if (inel) {
        sc.makespan_us = 0;
        sc.p95_us = 0;
        sc.objective = 0.0f;
        sc.status = WF_ST_INELIGIBLE;
        sc.min_headroom_mib = 0;
        sc.n_loads = 0;
        sc.n_evicts = 0;
      } else {
        const int64_t span = sp.origin + (int64_t)mk - sp.min_arrival;
        const float x = sp.w_mk * (float)span;
        const float y = sp.w_p95 * (float)(int64_t)p95;
        sc.makespan_us = span;
        sc.p95_us = (int64_t)p95;
        sc.objective = x + y;
        sc.status = status;
        sc.min_headroom_mib = -pe;
        nev /= F;
        sc.n_loads = (uint16_t)(nld > 65535u ? 65535u : nld);
        sc.n_evicts = (uint16_t)(nev > 65535u ? 65535u : nev);
      }
      if (pl < P) scores[pl] = sc;
    }
    wsync();
    if (lane == 0) take = atomicAdd(s_next, 1);
    take = __builtin_amdgcn_readfirstlane(take);
  }
}

template <int QB, int F, bool SEARCH, bool PHI, bool RCAP>
hipError_t launch_variant(const ScoreParams& sp, const LanesParams& lp, const int8_t* dev,
                          const uint16_t* prio, const uint8_t* flags, int64_t n_plans,
                          wf_plan_score* scores, const SearchArgs& sa, hipStream_t stream) {
  auto k = score_lanes<QB, F, SEARCH, PHI, RCAP>;
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                            hipFuncAttributeMaxDynamicSharedMemorySize, lp.lds_bytes);
  hipLaunchKernelGGL(k, dim3(lp.grid), dim3(64 * lp.waves), lp.lds_bytes, stream, sp, lp, dev, prio,
                     flags, n_plans, scores, sa);
  return hipGetLastError();
}

template <bool SEARCH, bool PHI>
hipError_t launch_q(const ScoreParams& sp, const LanesParams& lp, const int8_t* dev,
                    const uint16_t* prio, const uint8_t* flags, int64_t n, wf_plan_score* o,
                    const SearchArgs& sa, hipStream_t stream) {
  if (lp.field == 5)
    return launch_variant<64, 5, SEARCH, PHI, false>(sp, lp, dev, prio, flags, n, o, sa, stream);
  if (lp.rcap) {
    if (lp.qbits == 32)
      return launch_variant<32, 4, SEARCH, PHI, true>(sp, lp, dev, prio, flags, n, o, sa, stream);
    return launch_variant<64, 4, SEARCH, PHI, true>(sp, lp, dev, prio, flags, n, o, sa, stream);
  }
  if (lp.qbits == 32)
    return launch_variant<32, 4, SEARCH, PHI, false>(sp, lp, dev, prio, flags, n, o, sa, stream);
  return launch_variant<64, 4, SEARCH, PHI, false>(sp, lp, dev, prio, flags, n, o, sa, stream);
}

}  // namespace

hipError_t launch_score_lanes(const ScoreParams& sp, const LanesParams& lp, const int8_t* dev,
                              const uint16_t* prio, const uint8_t* flags, int64_t n_plans,
                              void* out, const SearchArgs* search, bool keys, hipStream_t stream) {
  const SearchArgs sa = search ? *search : SearchArgs{};
  wf_plan_score* o = static_cast<wf_plan_score*>(out);
  if (search)
    return keys ? launch_q<true, true>(sp, lp, dev, prio, flags, n_plans, o, sa, stream)
                : launch_q<true, false>(sp, lp, dev, prio, flags, n_plans, o, sa, stream);
  return keys ? launch_q<false, true>(sp, lp, dev, prio, flags, n_plans, o, sa, stream)
              : launch_q<false, false>(sp, lp, dev, prio, flags, n_plans, o, sa, stream);
}

}  // namespace wfp
