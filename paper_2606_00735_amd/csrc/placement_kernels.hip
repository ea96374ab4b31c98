// ViBE's placement control path on the GPU (Section 4.2; Algorithms 1 and 2):
// the per-GPU latency model f_g, the latency-aware greedy placement, the
// incremental swap solver and the cosine-distance drift detector, one block
// per MoE layer. The inputs (per-layer expert loads) are produced on the GPU
// by the expert histogram, so the control path needs no host round trip.
//
// All decisions are taken in fp64 with every operation rounded on its own
// (contraction off) and every sum in a fixed order, so results do not depend
// on scheduling.
#include "common.hpp"
#include "launch.hpp"

#pragma clang fp contract(off)

namespace moe {

constexpr int kPlaceThreads = 256;
constexpr int kPlaceMaxG = 64;    // GPUs (one wave holds them)

// the bitonic sort's length: the power of two that holds E entries
__host__ __device__ inline int place_pow2(int E) {
  int P = 1;
  while (P < E) P <<= 1;
  return P;
}

// f(n) of one GPU's model: knots (kn[k], kt[k]), k < nk, kn strictly
// increasing and positive. f = 0 for n <= 0, kt[0] up to kn[0], linear
// between knots, the last segment's slope beyond the last knot (with one
// knot: kt[0] n / kn[0]). The segment is found by bisection: a chain of at
// most six dependent reads where a scan from the first knot takes nk.
__device__ double latency_at(const double* kn, const double* kt, int nk, double n) {
  if (n <= 0.0) return 0.0;
  if (n <= kn[0]) return kt[0];
  if (nk == 1) return kt[0] * (n / kn[0]);
  int lo = 1, hi = nk;  // the first knot k >= 1 with n <= kn[k], nk if there is none
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (n <= kn[mid]) hi = mid; else lo = mid + 1;
  }
  if (lo < nk) return kt[lo - 1] + (kt[lo] - kt[lo - 1]) * ((n - kn[lo - 1]) / (kn[lo] - kn[lo - 1]));
  const double lo_n = kn[nk - 2], hi_n = kn[nk - 1], lo_t = kt[nk - 2], hi_t = kt[nk - 1];
  return hi_t + (hi_t - lo_t) * ((n - hi_n) / (hi_n - lo_n));
}

// The G models, in LDS if STAGED: every block evaluates them many times, each
// time a chain of dependent reads. All of a block's LDS that depends on the
// sizes is one dynamic array (8-byte aligned), cut in order by Lds, so that a
// launch of many layers keeps several blocks on a CU (see staged).
extern __shared__ double s_dyn[];
struct Lds {
  char* p;
  __device__ __forceinline__ Lds() : p(reinterpret_cast<char*>(s_dyn)) {}
  template <class T>
  __device__ __forceinline__ T* take(int n) {
    T* r = reinterpret_cast<T*>(p);
    p += (size_t)n * sizeof(T);
    return r;
  }
};
struct Models {
  const double *n, *t;
};
template <bool STAGED>
__device__ __forceinline__ Models load_models(Lds& lds, const double* knots_n, const double* knots_t, int G, int nk) {
  if constexpr (!STAGED) return {knots_n, knots_t};
  double* n = lds.take<double>(G * nk);
  double* t = lds.take<double>(G * nk);
  for (int i = threadIdx.x; i < G * nk; i += blockDim.x) {
    n[i] = knots_n[i];
    t[i] = knots_t[i];
  }
  return {n, t};
}

// Sum of w[e] over the experts with a[e] == g, in ascending e (both in LDS; all
// lanes read the same words). Unrolled, so that only the adds are a chain.
__device__ __forceinline__ double owned_sum(const double* w, const int* a, int E, int g) {
  double n = 0.0;
#pragma unroll 8
  for (int e = 0; e < E; ++e) {
    const double s = n + w[e];
    n = a[e] == g ? s : n;
  }
  return n;
}

__device__ __forceinline__ double shfl_f64(double v, int src) {
  const int2 p = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__shfl(p.x, src, kWave), __shfl(p.y, src, kWave)));
}

// (value, index) arg-max over lanes [0, 2^LOG): larger value, then lower index;
// every one of those lanes gets the result (the others get that of their own
// group). A strict order, so the shape of the reduction does not matter. The
// exchanges within 16 lanes are DPP moves (a few cycles; a shuffle through LDS
// takes about a hundred): lanes l ^ 1 and l ^ 2 of a quad, then the mirrored
// lane of 8 and of 16, which holds the other half's result.
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ void take_better(double& v, int& i, double ov, int oi) {
  const bool other = ov > v || (ov == v && oi < i);
  v = other ? ov : v;
  i = other ? oi : i;
}
template <int CTRL>
__device__ __forceinline__ void argmax_dpp(double& v, int& i) {
  const int2 p = __builtin_bit_cast(int2, v);
  take_better(v, i, __builtin_bit_cast(double, make_int2(dpp_i32<CTRL>(p.x), dpp_i32<CTRL>(p.y))), dpp_i32<CTRL>(i));
}
template <int LOG>
__device__ __forceinline__ void group_argmax(double& v, int& i) {
  if constexpr (LOG >= 1) argmax_dpp<0xB1>(v, i);   // quad_perm 1, 0, 3, 2
  if constexpr (LOG >= 2) argmax_dpp<0x4E>(v, i);   // quad_perm 2, 3, 0, 1
  if constexpr (LOG >= 3) argmax_dpp<0x141>(v, i);  // row_half_mirror
  if constexpr (LOG >= 4) argmax_dpp<0x140>(v, i);  // row_mirror
#pragma unroll
  for (int off = 16; off < (1 << LOG); off <<= 1) {
    const int src = (threadIdx.x & 63) ^ off;
    take_better(v, i, shfl_f64(v, src), __shfl(i, src, kWave));
  }
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const int2 p = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(p.x, lane), __builtin_amdgcn_readlane(p.y, lane)));
}

// The greedy of one wave over experts in the sorted order (key: load, id:
// expert): lane g holds tau_g, its load n and its expert count; G <= 2^LOG.
// 64 experts at a time sit in the wave's registers and are broadcast from
// there, so a step is the arg-max and the winner's update.
template <int LOG>
__device__ __forceinline__ double greedy_assign(const double* key, const int* id, int E, int G, int cap, double tau,
                                                int* s_assign) {
  const int g = threadIdx.x;
  double n = 0.0;
  int cnt = 0;
  for (int r0 = 0; r0 < E; r0 += kWave) {
    const int mine = min(r0 + g, E - 1);
    const double my_key = key[mine];
    const int my_id = id[mine];
    int my_gpu = 0;
    const int m = min(kWave, E - r0);
    for (int r = 0; r < m; ++r) {
      double gap = (g < G && (cap == 0 || cnt < cap)) ? tau - n : -__builtin_inf();
      int best = g < G ? g : 0x7fffffff;
      group_argmax<LOG>(gap, best);
      best = __builtin_amdgcn_readfirstlane(best);
      const double w = readlane_f64(my_key, r);
      if (g == best) {
        n += w;
        ++cnt;
      }
      if (g == r) my_gpu = best;
    }
    if (g < m && my_id < E) s_assign[my_id] = my_gpu;  // (unordered loads could bring a padding id here)
  }
  return n;
}

// ---------------------------------------------------------------------------
// Algorithm 1, Phase 2: speed-proportional targets and descending-load greedy.
// ---------------------------------------------------------------------------
template <bool STAGED>
__global__ __launch_bounds__(kPlaceThreads) void place_greedy_kernel(const double* __restrict__ W, int E,
                                                                     const double* __restrict__ knots_n,
                                                                     const double* __restrict__ knots_t, int G,
                                                                     int nk, int cap, int32_t* __restrict__ assign,
                                                                     double* __restrict__ loads,
                                                                     double* __restrict__ targets) {
  __shared__ double s_speed[kPlaceMaxG];
  __shared__ double s_N, s_S;
  const int l = blockIdx.x, tid = threadIdx.x;
  const double* w = W + (size_t)l * E;
  const int P = place_pow2(E);
  Lds lds;
  const Models m = load_models<STAGED>(lds, knots_n, knots_t, G, nk);
  double* s_key = lds.take<double>(P);  // sort keys: load, descending
  int* s_id = lds.take<int>(P);         // expert ids, ascending among equal loads
  int* s_assign = lds.take<int>(E);

  for (int i = tid; i < P; i += kPlaceThreads) {
    if (i < E) {
      s_key[i] = w[i];
      s_id[i] = i;
      s_assign[i] = 0;
    } else {
      s_key[i] = -__builtin_inf();
      s_id[i] = 0x7fffffff;
    }
  }
  __syncthreads();
  if (tid == 0) {  // N = sum_e w_e in ascending e (the keys are not sorted yet)
    double N = 0.0;
#pragma unroll 16
    for (int e = 0; e < E; ++e) N += s_key[e];
    s_N = N;
  }
  __syncthreads();
  const double N = s_N;
  if (tid < G) {
    s_speed[tid] = N > 0.0 ? 1.0 / latency_at(m.n + tid * nk, m.t + tid * nk, nk, N / E) : 1.0;
  }
  __syncthreads();
  if (tid == 0) {
    double S = 0.0;
    for (int g = 0; g < G; ++g) S += s_speed[g];
    s_S = S;
  }
  // bitonic sort of (key desc, id asc) over P entries
  for (int k = 2; k <= P; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      __syncthreads();
      for (int i = tid; i < P; i += kPlaceThreads) {
        const int p = i ^ j;
        if (p > i) {
          const bool up = (i & k) == 0;  // this run sorts "before" first
          const double ka = s_key[i], kb = s_key[p];
          const int ia = s_id[i], ib = s_id[p];
          const bool b_first = kb > ka || (kb == ka && ib < ia);  // b belongs before a
          if (b_first == up) {
            s_key[i] = kb;
            s_key[p] = ka;
            s_id[i] = ib;
            s_id[p] = ia;
          }
        }
      }
    }
  __syncthreads();
  if (tid < kWave) {
    const int g = tid;
    const double tau = g < G ? N * s_speed[g] / s_S : 0.0;
    double n;
    if (G <= 8)
      n = greedy_assign<3>(s_key, s_id, E, G, cap, tau, s_assign);
    else if (G <= 16)
      n = greedy_assign<4>(s_key, s_id, E, G, cap, tau, s_assign);
    else
      n = greedy_assign<6>(s_key, s_id, E, G, cap, tau, s_assign);
    if (g < G) {
      if (loads) loads[(size_t)l * G + g] = n;
      if (targets) targets[(size_t)l * G + g] = tau;
    }
  }
  __syncthreads();
  for (int e = tid; e < E; e += kPlaceThreads) assign[(size_t)l * E + e] = s_assign[e];
}

// ---------------------------------------------------------------------------
// Algorithm 2: swaps between the slowest and the fastest GPU.
// ---------------------------------------------------------------------------
template <bool STAGED>
__global__ __launch_bounds__(kPlaceThreads) void place_incremental_kernel(
    const double* __restrict__ W, int E, const double* __restrict__ knots_n, const double* __restrict__ knots_t,
    int G, int nk, double eps, int max_swaps, int32_t* __restrict__ assign, int32_t* __restrict__ n_swaps) {
  __shared__ double s_n[kPlaceMaxG], s_lat[kPlaceMaxG];
  __shared__ int s_hi, s_lo, s_nhi, s_nlo, s_stop;
  __shared__ double s_red_v[kPlaceThreads / kWave];
  __shared__ int s_red_i[kPlaceThreads / kWave];
  const int l = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double* w = W + (size_t)l * E;
  int32_t* a = assign + (size_t)l * E;
  Lds lds;
  const Models m = load_models<STAGED>(lds, knots_n, knots_t, G, nk);
  double* s_w = lds.take<double>(E);
  int* s_a = lds.take<int>(E);
  int* s_hi_list = lds.take<int>(E);
  int* s_lo_list = lds.take<int>(E);
  for (int e = tid; e < E; e += kPlaceThreads) {
    s_w[e] = w[e];
    const int g = a[e];
    s_a[e] = (g >= 0 && g < G) ? g : 0;  // placements out of range are read as GPU 0
  }
  __syncthreads();
  if (tid < G) s_n[tid] = owned_sum(s_w, s_a, E, tid);  // n_g in ascending expert id
  __syncthreads();
  auto lat_of = [&](int g, double n) {
    return latency_at(m.n + g * nk, m.t + g * nk, nk, n);
  };
  int swaps = 0;
  for (;;) {
    if (tid < G) s_lat[tid] = lat_of(tid, s_n[tid]);
    __syncthreads();
    if (tid == 0) {
      double tot = 0.0;
      for (int g = 0; g < G; ++g) tot += s_lat[g];
      const double fbar = tot / G;
      int hi = 0, lo = 0;
      for (int g = 1; g < G; ++g) {
        if (s_lat[g] > s_lat[hi]) hi = g;
        if (s_lat[g] < s_lat[lo]) lo = g;
      }
      s_hi = hi;
      s_lo = lo;
      s_stop = (swaps >= max_swaps || s_lat[hi] <= (1.0 + eps) * fbar || hi == lo) ? 1 : 0;
    }
    __syncthreads();
    if (s_stop) break;
    const int hi = s_hi, lo = s_lo;
    // experts of hi and lo in ascending id (wave 0 compacts with ballots)
    if (wave == 0) {
      int nh = 0, nl = 0;
      for (int base = 0; base < E; base += kWave) {
        const int e = base + lane;
        const bool in_h = e < E && s_a[e] == hi, in_l = e < E && s_a[e] == lo;
        const uint64_t bh = __ballot(in_h), bl = __ballot(in_l);
        const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
        if (in_h) s_hi_list[nh + __popcll(bh & below)] = e;
        if (in_l) s_lo_list[nl + __popcll(bl & below)] = e;
        nh += __popcll(bh);
        nl += __popcll(bl);
      }
      if (lane == 0) {
        s_nhi = nh;
        s_nlo = nl;
      }
    }
    __syncthreads();
    const int nh = s_nhi, nl = s_nlo;
    const double lat_hi = s_lat[hi], n_hi = s_n[hi], n_lo = s_n[lo];
    // best swap: largest gain, then lowest (position in hi list, position in lo list)
    double best = 0.0;
    int best_p = 0x7fffffff;
    const int pairs = nh * nl;
    for (int p = tid; p < pairs; p += kPlaceThreads) {
      const int ei = s_hi_list[p / nl], ej = s_lo_list[p % nl];
      const double nhi = n_hi - s_w[ei] + s_w[ej];
      const double nlo = n_lo - s_w[ej] + s_w[ei];
      const double lh = lat_of(hi, nhi), ll = lat_of(lo, nlo);
      const double gain = lat_hi - (lh > ll ? lh : ll);
      if (gain > best) {  // p increases within a thread: the first maximum is kept
        best = gain;
        best_p = p;
      }
    }
    // block arg-max over (gain, -p)
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      const double ov = shfl_f64(best, lane ^ off);
      const int op = __shfl(best_p, lane ^ off, kWave);
      if (ov > best || (ov == best && op < best_p)) {
        best = ov;
        best_p = op;
      }
    }
    if (lane == 0) {
      s_red_v[wave] = best;
      s_red_i[wave] = best_p;
    }
    __syncthreads();
    if (tid == 0) {
      double bv = 0.0;
      int bp = 0x7fffffff;
      for (int q = 0; q < kPlaceThreads / kWave; ++q)
        if (s_red_v[q] > bv || (s_red_v[q] == bv && s_red_i[q] < bp)) {
          bv = s_red_v[q];
          bp = s_red_i[q];
        }
      if (bp == 0x7fffffff) {
        s_stop = 1;  // no swap lowers the pair's latency
      } else {
        const int ei = s_hi_list[bp / nl], ej = s_lo_list[bp % nl];
        const double nhi = n_hi - s_w[ei] + s_w[ej];
        const double nlo = n_lo - s_w[ej] + s_w[ei];
        s_a[ei] = lo;
        s_a[ej] = hi;
        s_n[hi] = nhi;
        s_n[lo] = nlo;
      }
    }
    __syncthreads();
    if (s_stop) break;
    ++swaps;
  }
  for (int e = tid; e < E; e += kPlaceThreads) a[e] = s_a[e];
  if (tid == 0 && n_swaps) n_swaps[l] = swaps;
}

// ---------------------------------------------------------------------------
// Predicted cost of a placement (Section 4.2.3): per layer and GPU, the load
// n_g = sum_{e in S_g} w_e (ascending e), f_g(n_g), and the grouped reading
// sum_{e in S_g} f_g(w_e). The layer latency is the maximum over GPUs.
// ---------------------------------------------------------------------------
template <bool STAGED>
__global__ __launch_bounds__(kPlaceThreads) void placement_cost_kernel(const double* __restrict__ W,
                                                                       const int32_t* __restrict__ assign, int E,
                                                                       const double* __restrict__ knots_n,
                                                                       const double* __restrict__ knots_t, int G,
                                                                       int nk, double* __restrict__ loads,
                                                                       double* __restrict__ lat,
                                                                       double* __restrict__ lat_grouped) {
  const int l = blockIdx.x, tid = threadIdx.x;
  Lds lds;
  const Models m = load_models<STAGED>(lds, knots_n, knots_t, G, nk);
  double* s_w = lds.take<double>(E);
  double* s_f = lds.take<double>(E);
  int* s_a = lds.take<int>(E);
  for (int e = tid; e < E; e += kPlaceThreads) {
    s_w[e] = W[(size_t)l * E + e];
    s_a[e] = assign[(size_t)l * E + e];
  }
  __syncthreads();
  // every expert's own latency side by side, then two sums per GPU
  for (int e = tid; e < E; e += kPlaceThreads) {
    const int g = s_a[e];
    if (g >= 0 && g < G) s_f[e] = latency_at(m.n + g * nk, m.t + g * nk, nk, s_w[e]);
  }
  __syncthreads();
  const int g = tid & (kPlaceMaxG - 1), which = tid / kPlaceMaxG;  // one wave per sum
  if (g >= G) return;
  if (which == 0) {
    const double n = owned_sum(s_w, s_a, E, g);
    if (loads) loads[(size_t)l * G + g] = n;
    lat[(size_t)l * G + g] = latency_at(m.n + g * nk, m.t + g * nk, nk, n);
  } else if (which == 1 && lat_grouped) {
    lat_grouped[(size_t)l * G + g] = owned_sum(s_f, s_a, E, g);
  }
}

// ---------------------------------------------------------------------------
// Drift detector (Section 4.2.4): window sums and cosine distance per layer.
// ---------------------------------------------------------------------------
__global__ void window_push_kernel(const int32_t* __restrict__ counts, int32_t* __restrict__ ring_slot,
                                   double* __restrict__ sums, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t c = counts[i];
  sums[i] = sums[i] + (double)c - (double)ring_slot[i];
  ring_slot[i] = c;
}

__device__ __forceinline__ double cosine_distance(double dot, double na, double nb) {
  if (na == 0.0 || nb == 0.0) return (na == nb) ? 0.0 : 1.0;
  return 1.0 - dot / (__builtin_sqrt(na) * __builtin_sqrt(nb));
}

// One block, so that the trigger (the OR of d > delta over all layers, written
// by thread 0) needs no atomics and no memset. Each of its 16 waves takes
// kDriftLayers layers at a time: the lanes read 64 experts of each, coalesced,
// and put the products u v, u u and v v into LDS; one lane per (layer, sum) then
// adds them in ascending expert id. A lane of its own per layer read its
// vectors alone, two dependent loads an expert.
constexpr int kDriftThreads = 1024;
constexpr int kDriftLayers = 4;
__global__ __launch_bounds__(kDriftThreads) void drift_distance_kernel(const double* __restrict__ w_cur,
                                                                       const double* __restrict__ w_ref, int L, int E,
                                                                       double delta, double* __restrict__ d,
                                                                       int32_t* __restrict__ trigger) {
  constexpr int NW = kDriftThreads / kWave, NS = 3 * kDriftLayers, LD = kWave + 1;  // rows off a bank
  __shared__ double s_p[NW][NS * LD];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double* p = s_p[wave];
  bool over = false;
  for (int l0 = 0; l0 < L; l0 += NW * kDriftLayers) {
    const int lw = l0 + wave * kDriftLayers;  // this wave's first layer
    double sum = 0.0;                         // lane q < NS: sum q % 3 of layer lw + q / 3
    for (int e0 = 0; e0 < E; e0 += kWave) {
      const int e = e0 + lane;
      double u[kDriftLayers], v[kDriftLayers];
#pragma unroll
      for (int q = 0; q < kDriftLayers; ++q) {
        const bool in = lw + q < L && e < E;
        u[q] = in ? w_cur[(size_t)(lw + q) * E + e] : 0.0;
        v[q] = in ? w_ref[(size_t)(lw + q) * E + e] : 0.0;
      }
      __syncthreads();  // the sums below are done with the products before
#pragma unroll
      for (int q = 0; q < kDriftLayers; ++q) {
        p[(3 * q) * LD + lane] = u[q] * v[q];
        p[(3 * q + 1) * LD + lane] = u[q] * u[q];
        p[(3 * q + 2) * LD + lane] = v[q] * v[q];
      }
      __syncthreads();
      const int m = min(kWave, E - e0);
      if (lane < NS) {
#pragma unroll 16
        for (int i = 0; i < m; ++i) sum += p[lane * LD + i];
      }
    }
    const double dot = shfl_f64(sum, (3 * lane) & 63), na = shfl_f64(sum, (3 * lane + 1) & 63),
                 nb = shfl_f64(sum, (3 * lane + 2) & 63);
    if (lane < kDriftLayers && lw + lane < L) {
      const double dist = cosine_distance(dot, na, nb);
      d[lw + lane] = dist;
      over = over || dist > delta;
    }
  }
  const int any = __syncthreads_or(over ? 1 : 0);
  if (threadIdx.x == 0 && trigger) *trigger = any ? 1 : 0;
}

// The same sums with a thread per layer, for layers of so few experts that the
// waves above would be mostly empty (see launch_drift_distance).
__global__ __launch_bounds__(256) void drift_distance_few_kernel(const double* __restrict__ w_cur,
                                                                 const double* __restrict__ w_ref, int L, int E,
                                                                 double delta, double* __restrict__ d,
                                                                 int32_t* __restrict__ trigger) {
  bool over = false;
  for (int l = threadIdx.x; l < L; l += 256) {
    const double* u = w_cur + (size_t)l * E;
    const double* v = w_ref + (size_t)l * E;
    double dot = 0.0, na = 0.0, nb = 0.0;
    for (int e = 0; e < E; ++e) {
      dot += u[e] * v[e];
      na += u[e] * u[e];
      nb += v[e] * v[e];
    }
    const double dist = cosine_distance(dot, na, nb);
    d[l] = dist;
    over = over || dist > delta;
  }
  const int any = __syncthreads_or(over ? 1 : 0);
  if (threadIdx.x == 0 && trigger) *trigger = any ? 1 : 0;
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Models go to LDS where they are small (16 KB: three blocks a CU or more with
// the largest layers) or where a CU gets one block anyway; else blocks read
// them from the caches. Room for the largest models in every block left one
// block a CU; us, so / by sizes: 1000 layers of 64 experts, 8 GPUs of 4 knots,
// greedy 84 / 24, incremental 63 / 31; 600 layers of 1024 experts, 64 GPUs of
// 64 knots (not staged), greedy 1524 / 550, incremental 407 / 162, cost 90 / 42;
// 58 layers of 256, 8 of 14: greedy 72.9 / 73.6, incremental 74.6 / 74.3. Below
// one block a CU staging is what pays: 64 layers of 1024, 64 of 64, incremental
// 277 from the caches, 138 from LDS.
static bool staged(int L, int G, int nk) { return G * nk <= 1024 || L <= device_cu_count(); }
static size_t model_bytes(bool st, int G, int nk) { return st ? (size_t)2 * G * nk * sizeof(double) : 0; }

hipError_t launch_place_greedy(const double* W, int L, int E, const double* kn, const double* kt, int G, int nk,
                               int cap, int32_t* assign, double* loads, double* targets, hipStream_t s) {
  if (L == 0) return hipSuccess;
  const bool st = staged(L, G, nk);
  const size_t lds = model_bytes(st, G, nk) + (size_t)place_pow2(E) * 12 + (size_t)E * 4;
  const auto kernel = st ? place_greedy_kernel<true> : place_greedy_kernel<false>;
  kernel<<<L, kPlaceThreads, lds, s>>>(W, E, kn, kt, G, nk, cap, assign, loads, targets);
  return hipGetLastError();
}

hipError_t launch_place_incremental(const double* W, int L, int E, const double* kn, const double* kt, int G,
                                    int nk, double eps, int max_swaps, int32_t* assign, int32_t* n_swaps,
                                    hipStream_t s) {
  if (L == 0) return hipSuccess;
  const bool st = staged(L, G, nk);
  const auto kernel = st ? place_incremental_kernel<true> : place_incremental_kernel<false>;
  kernel<<<L, kPlaceThreads, model_bytes(st, G, nk) + (size_t)E * 20, s>>>(W, E, kn, kt, G, nk, eps, max_swaps,
                                                                           assign, n_swaps);
  return hipGetLastError();
}

hipError_t launch_placement_cost(const double* W, const int32_t* assign, int L, int E, const double* kn,
                                 const double* kt, int G, int nk, double* loads, double* lat, double* lat_grouped,
                                 hipStream_t s) {
  if (L == 0) return hipSuccess;
  const bool st = staged(L, G, nk);
  const auto kernel = st ? placement_cost_kernel<true> : placement_cost_kernel<false>;
  kernel<<<L, kPlaceThreads, model_bytes(st, G, nk) + (size_t)E * 20, s>>>(W, assign, E, kn, kt, G, nk, loads, lat,
                                                                           lat_grouped);
  return hipGetLastError();
}

hipError_t launch_window_push(const int32_t* counts, int32_t* ring, double* sums, int L, int E, int slot,
                              hipStream_t s) {
  const size_t n = (size_t)L * E;
  if (n == 0) return hipSuccess;
  window_push_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(counts, ring + (size_t)slot * n, sums, n);
  return hipGetLastError();
}

hipError_t launch_drift_distance(const double* w_cur, const double* w_ref, int L, int E, double delta, double* d,
                                 int32_t* trigger, hipStream_t s) {
  // A round of drift_distance_kernel (64 layers x 64 experts, or what there is)
  // takes about 13 times an expert of drift_distance_few_kernel's 256 layers:
  // 4000 layers of 16 experts 149 / 60 us, 1000 of 64 56 / 57, 300 of 128
  // 32 / 43, 58 of 256 13.6 / 32.
  const long long rounds = (long long)((L + 63) / 64) * ((E + kWave - 1) / kWave);
  if (13 * rounds > (long long)((L + 255) / 256) * E && E < kWave)
    drift_distance_few_kernel<<<1, 256, 0, s>>>(w_cur, w_ref, L, E, delta, d, trigger);
  else
    drift_distance_kernel<<<1, kDriftThreads, 0, s>>>(w_cur, w_ref, L, E, delta, d, trigger);
  return hipGetLastError();
}

}  // namespace moe
