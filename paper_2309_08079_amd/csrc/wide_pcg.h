// PCG of the 28-state path (nx = 28, nu = 14) on gangs of workgroups.
//
// A problem of N knots is cut into parts of KW consecutive knots, one workgroup per part
// and one wave per knot; the parts of a problem form a gang that meets at gang barriers,
// as in the 14-state kernel.  The four 16-lane DPP rows of a wave are the quarters of the
// knot's block row: lane i < 14 of quarter (h, c) owns row 14 h + i of the first or second
// half of the rows and the 14 columns of half c of each block, in registers for the whole
// solve: 3 x 14 doubles of S and 3 x 14 floats of Phi^-1.  The vectors r and p are kept by
// columns: that lane holds entry 14 c + i of the knot's own, the previous and the next knot,
// so a product is 42 fused broadcast-FMAs from registers, and one swap between the two
// quarters of a row half adds their partial sums.
//
// The loop is Algorithm 1 as printed, with its two inner products each met at a gang
// barrier.  The rows of the vector just formed (S p at the first barrier, Phi^-1 r at the
// second) go through LDS to the waves of the neighbouring knots, and across a part boundary
// as 16-byte tagged words (the 14-state kernel's protocol) with the partial sums.  After the
// barrier every wave updates r or p of its three knots with the same fused operations, so
// the copies stay bit-identical to the owner's and no other exchange is needed.  Partial
// sums are added in a fixed order, so every part takes the same decisions.
//
// What bounds it: rounds of resident workgroups (the rows of S and Phi^-1 fill the registers
// at three waves per SIMD), and in each iteration the latency of its two barriers, ~ 0.65 us
// each of the 2.2 us of a lone problem of 64 knots (0.87 us with no gang).  Measured on
// MI355X, 32 problems of 64 to 256 knots (three rounds of ~ 113 iterations): 835 us.  With
// the vectors' entries read from LDS as broadcasts, 42 + 42 per lane and iteration, and three
// more workgroup barriers per iteration: 1276 (2.2 us with no gang); with sums and rows
// awaited by one wave, two dependent round trips per poll: 990.
//
// Inputs are the workspace blocks the formation and preconditioner launches write (S, Phi^-1,
// the right-hand side); the output is lambda (or mu in adjoint mode) in FP64 in lamw and
// the stats; the primal step / gradients follow in wide_epilogue.  Stopping rule, status
// codes and precision are those of the 14-state kernel: FP64 S, vectors and reductions,
// FP32 Phi^-1 applied with FP32 accumulation.
#pragma once
#include "pcg_kernel.h"
#include "wide_kernels.h"

namespace mpc {
namespace wide {

constexpr int kGangKnots = 4;  // knots (waves) per workgroup

// Tagged words of one part (read by its gang): [parity][value] partial sums and
// [parity][channel][side][row] boundary rows, each a 16-byte pair (payload halves tagged).
struct WTag {
  uint64_t red[2][2][2];
  uint64_t rows[2][2][2][32][2];
};

struct GangArgs {
  void *tws;              // WTag[ntasks]
  Gang *gang;             // [problems]
  int *queue;             // [0] head, [1] workgroups finished, [2] launch generation,
                          // [4 + x] head of XCD x's list
  const ProbDesc *probs;  // per problem: k0, N, t0 (first task), nparts, id
  const Task *tasks;      // longest problem first, the parts of a problem adjacent
  const int32_t *xoff;    // [9] or nullptr: the tasks of XCD x are [xoff[x], xoff[x+1]),
                          // popped by the workgroups running on XCD x only, so that every
                          // gang runs on one XCD and its barriers use that XCD's L2
  int32_t ntasks;
  int32_t l2x;            // 1 with xoff: barrier words through the XCD's L2
  int64_t spin_limit;     // wall-clock ticks before a wait gives up
};

template <int NX, int KW>
__global__ void __launch_bounds__(KW * 64) __attribute__((amdgpu_waves_per_eu(3, 3)))
    wide_pcg_gang(const WArgs a, const GangArgs g) {
  static_assert(NX == pair::kN && KW > 2, "two halves of 14 rows; a wave for each channel beside the first");
  constexpr int H = NX / 2;
  constexpr int MM = NX * NX;
  constexpr int NT = KW * 64;
  // rows of the part's knots (slot s + 1 = knot s) and of its two neighbours: S p (at the
  // start the right-hand side, then r), Phi^-1 r (at the start lambda)
  __shared__ double us[KW + 2][32], ts[KW + 2][32];
  __shared__ double red_w[2][2][KW];                  // the knots' sums [parity of the barrier][value][wave]
  __shared__ double tot[2];
  __shared__ int sh_task, sh_abort[2];                // [parity of the barrier]

  // Lane indices are re-derived through an opaque copy of threadIdx.x at the top of every
  // PCG iteration, so that the compiler recomputes LDS and workspace addresses instead of
  // keeping them live across the loop, where the registers hold S and Phi^-1.
  int tid = threadIdx.x, wave, lane, c, r, e;
  bool rowv, rows, ents;
  auto refresh = [&]() {
    asm volatile("" : "+v"(tid));
    wave = uni(tid >> 6);
    lane = tid & 63;
    c = (lane >> 4) & 1;
    rowv = (lane & 15) < H;
    const int li = min(lane & 15, H - 1);
    r = (lane >> 5) * H + li;   // this lane's row of the blocks
    e = c * H + li;             // this lane's entry of the vectors
    rows = rowv && c == 0;      // lanes that pass a product's rows on
    ents = rowv && lane < 32;   // lanes that pass a vector's entries on
  };
  refresh();
  WTag *tws = reinterpret_cast<WTag *>(g.tws);
  const __amdgpu_buffer_rsrc_t wsr = ws_rsrc(g.tws);
  auto ws_off = [&](const void *p) { return (uint32_t)((const char *)p - (const char *)g.tws); };
  // launch generation (advanced by the last workgroup of every launch), part of every tag
  const uint64_t gen = (uint64_t)(uint32_t)uni(__hip_atomic_load(&g.queue[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  const bool l2x = g.l2x != 0;
  auto put_pair = [&](uint32_t off, uint32_t tag, double v) {
    if (l2x)
      store_pair_l2(wsr, off, tag, v);
    else
      store_pair(wsr, off, tag, v);
  };
  auto get_pair = [&](uint32_t off) -> u32x4 {
    u32x4 w;
    if (l2x)
      w = load_pair_l2(wsr, off);
    else
      w = load_pair(wsr, off);
    return w;
  };

  for (;;) {
    __syncthreads();
    if (tid == 0) {
      if (g.xoff) {
        unsigned x;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
        x &= 7u;
        const int t = g.xoff[x] + atomicAdd(&g.queue[4 + x], 1);
        sh_task = t < g.xoff[x + 1] ? t : g.ntasks;  // this XCD's list is empty
      } else {
        sh_task = atomicAdd(&g.queue[0], 1);
      }
    }
    __syncthreads();
    const int task = uni(sh_task);
    if (task >= g.ntasks) break;
    const Task tk = g.tasks[task];
    const ProbDesc pd = g.probs[tk.prob];
    const int part = tk.part, G = pd.nparts, N = pd.N;
    const bool multi = G > 1;
    const int b = part * KW + wave;
    const bool act = b < N;
    const bool mine = act && rowv;  // this lane holds part of an existing knot
    const int64_t kb = pd.k0 + (act ? b : 0);
    const int my_t = pd.t0 + part;
    Gang *gang = g.gang + tk.prob;
    int nsync = 0;
    bool aborted = false;
    if (tid < 2) sh_abort[tid] = 0;
    for (int t = tid; t < (KW + 2) * 32; t += NT) {
      (&us[0][0])[t] = 0.0;
      (&ts[0][0])[t] = 0.0;
    }

    // rows of S and Phi^-1: this lane's half of the columns of blocks (b,b-1), (b,b), (b,b+1)
    double S[3][H];
    float P[3][H];
    {
      const double *sb = a.S + kb * 3 * MM + c * H * NX + r;  // blocks by columns
      const float *pb = a.P + kb * 3 * MM + c * H * NX + r;
#pragma unroll
      for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int j = 0; j < H; ++j) {
          const double sv = sb[s * MM + j * NX];
          const float pv = pb[s * MM + j * NX];
          S[s][j] = mine ? sv : 0.0;
          P[s][j] = mine ? pv : 0.0f;
        }
    }
    const bool adj = a.adjoint != 0;
    const bool warm = !adj && a.warm;
    double lam = (warm && mine) ? (double)a.lam[kb * NX + e] : 0.0;

    // ---- products with the vectors' entries of knots b-1, b, b+1: this lane's row r
    auto s_prod = [&](const double (&x)[3]) {
      double acc = 0.0, lo, hi;
#pragma unroll
      for (int s = 0; s < 3; ++s) row_fma14_f64(acc, x[s], S[s]);
      pair::dup(acc, lo, hi);
      return lo + hi;
    };
    auto p_prod = [&](const double (&x)[3]) {
      float acc = 0.0f;
#pragma unroll
      for (int s = 0; s < 3; ++s) row_fma14_f32(acc, (float)x[s], P[s]);
      const uint32_t u = __builtin_bit_cast(uint32_t, acc);
      const auto v = __builtin_amdgcn_permlane16_swap(u, u, false, false);
      return __builtin_bit_cast(float, (uint32_t)v[0]) + __builtin_bit_cast(float, (uint32_t)v[1]);
    };
    // the three knots' entries of rows that are in LDS
    auto entries = [&](const double (&v)[KW + 2][32], double (&x)[3]) {
#pragma unroll
      for (int s = 0; s < 3; ++s) x[s] = v[wave + s][e];
    };
    // this wave's knot's share of an inner product, the row halves' sums added in order (the
    // entries and the product's rows meet in the lanes with r == e)
    auto put_red = [&](int v, double x) {
      const uint64_t u = __builtin_bit_cast(uint64_t, group_sum_to_last(act && rowv && r == e ? x : 0.0));
      const uint32_t lo0 = __builtin_amdgcn_readlane((uint32_t)u, 15), hi0 = __builtin_amdgcn_readlane((uint32_t)(u >> 32), 15);
      const uint32_t lo1 = __builtin_amdgcn_readlane((uint32_t)u, 63), hi1 = __builtin_amdgcn_readlane((uint32_t)(u >> 32), 63);
      if (lane == 0)
        red_w[nsync & 1][v][wave] =
            __builtin_bit_cast(double, ((uint64_t)hi0 << 32) | lo0) + __builtin_bit_cast(double, ((uint64_t)hi1 << 32) | lo1);
    };
    // row i of the knot (lanes `on`) to the part and, of its first and last knot, to the gang
    // (channel ch; first knot: side 0, last knot: side 1)
    auto put_row = [&](int ch, double (&v)[KW + 2][32], bool on, int i, double x) {
      if (on) v[wave + 1][i] = x;
      if (multi && on) {
        const uint32_t tag = loop_tag(gen, nsync);
        if (wave == 0) put_pair(ws_off(tws[my_t].rows[nsync & 1][ch][0][i]), tag, x);
        if (wave == KW - 1) put_pair(ws_off(tws[my_t].rows[nsync & 1][ch][1][i]), tag, x);
      }
    };
    // (a wait's clock starts at its 64th poll: most end before)
    auto poll_spin = [&](int &polls, long long &t_start) -> bool {
      __builtin_amdgcn_s_sleep(1);
      if ((++polls & 63) == 0) {
        if (__hip_atomic_load(&gang->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return true;
        const long long now = wall_clock64();
        if (t_start == 0) t_start = now;
        if (now - t_start > g.spin_limit) {
          __hip_atomic_store(&gang->abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          return true;
        }
      }
      return false;
    };
    // Barrier of the problem: the totals of nv inner products, and nc channels of rows, whose
    // neighbours' rows land in v0s (and v1s).  A problem of one part needs one workgroup
    // barrier, after which every wave adds the knots' sums itself.  In a gang wave 0 adds and
    // publishes them and waits for the other parts' sums, 64 parts at a time, and wave 1 + ch
    // for channel ch of the neighbours' rows (lane: side, row): one word per lane and value,
    // all in flight at once, so that a poll is one round trip.  (Publishing every knot's sum
    // instead, without the first workgroup barrier, measured 5% faster for 4 parts and 3 to 7%
    // slower for 64 parts and for a full device.)
    double total[2] = {0.0, 0.0};
    auto sync = [&](int nv, int nc, double (&v0s)[KW + 2][32], double (&v1s)[KW + 2][32]) {
      const int par = nsync & 1;
      lds_barrier();
      if (!multi || aborted) {
        for (int v = 0; v < nv; ++v) {
          double t = 0.0;
#pragma unroll
          for (int w = 0; w < KW; ++w) t += red_w[par][v][w];
          total[v] = uni(t);
        }
        ++nsync;
        return;
      }
      const uint32_t tag = loop_tag(gen, nsync);
      // the whole workgroup waits for these waves: they issue ahead of co-resident ones
      if (wave <= nc) __builtin_amdgcn_s_setprio(2);
      if (wave == 0 && lane < nv) {  // this part's sums, its waves in order
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < KW; ++w) t += red_w[par][lane][w];
        put_pair(ws_off(tws[my_t].red[par][lane]), tag, t);
      }
      // device scope: the last part's words land ~1 us after the first part arrives; through
      // one XCD's L2 a round takes ~0.4 us and polling at once is fastest
      if (!l2x) __builtin_amdgcn_s_sleep(24);
      long long t_start = 0;
      int polls = 0;
      bool ab = false;
      if (wave == 0 && nv > 0) {
        double v[2] = {0.0, 0.0};
        for (int g0 = 0; g0 < G && !ab; g0 += 64) {
          const bool want = g0 + lane < G;
          const uint32_t o = ws_off(tws[pd.t0 + (want ? g0 + lane : 0)].red[par][0]);
          u32x4 w0, w1;
          while (true) {
            w0 = get_pair(o);
            w1 = w0;
            if (nv > 1) w1 = get_pair(o + 16);
            if (__ballot(!want || (pair_has(w0, tag) && pair_has(w1, tag))) == ~0ull) break;
            if ((ab = poll_spin(polls, t_start))) break;
          }
          if (want) {
            v[0] += pair_value(w0);
            v[1] += pair_value(w1);
          }
        }
        const double s0 = wave_sum(v[0]), s1 = nv > 1 ? wave_sum(v[1]) : 0.0;
        if (lane == 0) {
          tot[0] = s0;
          tot[1] = s1;
        }
      } else if (wave > 0 && wave <= nc) {
        const int side = lane >= NX, row = min(lane - side * NX, NX - 1);
        const int nb = side ? part + 1 : part - 1;
        const bool want = lane < 2 * NX && nb >= 0 && nb < G;
        const uint32_t o = ws_off(tws[want ? pd.t0 + nb : my_t].rows[par][wave - 1][side ^ 1][row]);
        u32x4 q;
        while (true) {
          q = get_pair(o);
          if (__ballot(!want || pair_has(q, tag)) == ~0ull) break;
          if ((ab = poll_spin(polls, t_start))) break;
        }
        if (want && !ab) (wave == 1 ? v0s : v1s)[side ? KW + 1 : 0][row] = pair_value(q);
      }
      if (ab) sh_abort[par] = 1;
      __builtin_amdgcn_s_setprio(0);
      lds_barrier();
      ++nsync;
      aborted = aborted || uni(sh_abort[par]) != 0;
      total[0] = uni(tot[0]);
      total[1] = uni(tot[1]);
    };

    // ---- setup: right-hand side (and warm-start) of the three knots
    double rs[3], ps[3], ms[3];
    __syncthreads();  // us and ts are zero
    put_row(0, us, ents, e, mine ? a.rhs[kb * NX + e] : 0.0);
    if (warm) put_row(1, ts, ents, e, lam);
    sync(0, warm ? 2 : 1, us, ts);
    entries(us, rs);
    if (warm) {
      // r = gamma - S lambda_0; eta_ref = gamma^T Phi^-1 gamma needs Phi^-1 gamma as well
      entries(ts, ms);
      const double ref = rs[1] * (double)p_prod(rs);
      __syncthreads();  // us and ts have been read
      put_row(0, us, rows, r, (mine ? a.rhs[kb * NX + r] : 0.0) - s_prod(ms));
      sync(0, 1, us, us);
      entries(us, rs);
      put_red(1, ref);
    }
    float rt = p_prod(rs);
    put_red(0, rs[1] * (double)rt);
    put_row(0, ts, rows, r, (double)rt);
    sync(warm ? 2 : 1, 1, ts, ts);
    double eta = total[0], eta_new = eta;
    const double eta_ref = warm ? total[1] : eta;
    entries(ts, ps);
    const double tau = a.stop_abs ? (double)a.eps : (double)a.eps * (double)a.eps * eta_ref;
    // two barriers per iteration: the cap keeps barrier indices within the tags' 24 bits
    const int max_iter = min(a.max_iter > 0 ? a.max_iter : N * NX, 1 << 22);
    int status = MPCPCG_NOT_CONVERGED, it = 0;
    if (!(eta == eta) || !(eta_ref == eta_ref) || __builtin_isinf(eta) || __builtin_isinf(eta_ref)) {
      status = MPCPCG_BREAKDOWN;
    } else if (eta <= tau) {
      status = MPCPCG_OK;
    } else {
      __syncthreads();  // the setup's sums and rows have been read
      for (it = 1; it <= max_iter && !aborted; ++it) {
        refresh();
        // Upsilon = S p, upsilon = p^T Upsilon
        const double ups_row = s_prod(ps);
        put_row(0, us, rows, r, ups_row);
        put_red(0, ps[1] * ups_row);
        sync(1, 1, us, us);
        entries(us, ms);
        const double ups = total[0];
        if (!(ups > 0.0) || __builtin_isinf(ups)) {
          status = MPCPCG_BREAKDOWN;
          break;
        }
        const double alpha = eta / ups;
        lam = __builtin_fma(alpha, ps[1], lam);
#pragma unroll
        for (int s = 0; s < 3; ++s) rs[s] = __builtin_fma(-alpha, ms[s], rs[s]);
        // r~ = Phi^-1 r, eta' = r^T r~
        rt = p_prod(rs);
        put_row(0, ts, rows, r, (double)rt);
        put_red(0, rs[1] * (double)rt);
        sync(1, 1, ts, ts);
        entries(ts, ms);
        eta_new = total[0];
        if (!(eta_new == eta_new) || __builtin_isinf(eta_new)) {
          status = MPCPCG_BREAKDOWN;
          break;
        }
        if (eta_new < tau) {
          status = MPCPCG_OK;
          break;
        }
        const double beta = eta_new / eta;
#pragma unroll
        for (int s = 0; s < 3; ++s) ps[s] = __builtin_fma(beta, ps[s], ms[s]);
        eta = eta_new;
      }
      if (it > max_iter) it = max_iter;
    }
    if (aborted) status = MPCPCG_TIMEOUT;
    if (mine && lane < 32) a.lamw[kb * NX + e] = lam;
    if (tid == 0 && part == 0)
      put_stats(a.stats + pd.id, it, status,
                eta_ref > 0.0 ? (float)__builtin_sqrt(eta_new > 0.0 ? eta_new / eta_ref : 0.0) : 0.0f);

    // ---- gang teardown: the last part out zeroes the gang's tagged words
    if (multi) {
      __syncthreads();
      if (tid == 0) {
        // a relaxed count after the barrier, which waited for every wave's stores (part 0's
        // stats, the abort flag): no L2 write-back at every task's end
        __builtin_amdgcn_s_waitcnt(0);
        const int d = __hip_atomic_fetch_add(&gang->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh_task = d == G - 1;
      }
      __syncthreads();
      if (uni(sh_task)) {
        constexpr int kWords = sizeof(WTag) / sizeof(uint64_t);
        for (int i = tid; i < G * kWords; i += NT) {
          uint64_t *w = reinterpret_cast<uint64_t *>(&tws[pd.t0 + i / kWords]) + i % kWords;
          __hip_atomic_store(w, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (tid == 0) {
          const int ab = __hip_atomic_load(&gang->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (ab) __hip_atomic_store(reinterpret_cast<int *>(a.stats + pd.id) + 1, (int)MPCPCG_TIMEOUT,
                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&gang->abort, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&gang->done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
  }

  // ---- launch teardown: the last workgroup out resets the queue
  __syncthreads();
  if (tid == 0) {
    __builtin_amdgcn_s_waitcnt(0);
    const int d = __hip_atomic_fetch_add(&g.queue[1], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (d == (int)gridDim.x - 1) {
      // a list whose XCD ran no workgroup of this launch (a placement the host did not
      // expect) leaves its problems unsolved: they report TIMEOUT instead of stale stats
      if (g.xoff) {
        for (int x = 0; x < 8; ++x) {
          const int popped = __hip_atomic_load(&g.queue[4 + x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          for (int t = g.xoff[x] + max(popped, 0); t < g.xoff[x + 1]; ++t) {
            const Task tk = g.tasks[t];
            if (tk.part == 0) put_stats(a.stats + g.probs[tk.prob].id, 0, MPCPCG_TIMEOUT, 0.0f);
          }
        }
      }
      __hip_atomic_store(&g.queue[0], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      for (int x = 0; x < 8; ++x) __hip_atomic_store(&g.queue[4 + x], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(&g.queue[2], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&g.queue[1], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

}  // namespace wide
}  // namespace mpc
