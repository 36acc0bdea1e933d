// hcao_recombination.hip -- gfx950 kernels of the exact forward recombination
// probability (set-up work, not part of the step).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hcao_tables.h"

namespace hcao {
namespace {

constexpr double kBoltz = 1.380649e-23;

// energy of level i of mode m: harmonic bends, tabulated stretches
__device__ __forceinline__ double mode_energy(const SpeciesTab &S, const double *lev, uint32_t m, uint32_t i) {
  if (m < S.n_bend) return ((double)i + 0.5) * S.kt[m];
  return lev[S.lev_off[m] + i];
}

// ---------------------------------------------------------------------------
// Eq. recomb-correct: forward probability summed over every combination of
// vibrational levels (set-up work, not part of the step)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double level_above_ground(const SpeciesTab &S, const double *lev, uint32_t m, uint32_t j) {
  return mode_energy(S, lev, m, j) - mode_energy(S, lev, m, 0);
}

// C(n + k - 1, k - 1): ways k bends share n quanta (exact while it fits a
// double; the products before each division are multiples of the divisor)
__device__ __forceinline__ double shares(uint32_t n, uint32_t k) {
  double g = 1.0;
  for (uint32_t i = 1; i < k; ++i) g = g * (double)(n + i) / (double)i;
  return g;
}

// One step of the walk: the energy of a prefix, its weight, and the last
// stretch's level with its place in the run of identical stretches (place,
// and how many of the run so far have that level)
struct RecNode {
  double s, w;
  uint32_t j, place, equal;
};

__device__ __forceinline__ double unit_energy(const SpeciesTab &S, const double *lev, const RecUnits &U, uint32_t u,
                                              uint32_t j) {
  return level_above_ground(S, lev, U.mode[u], j);
}

// the prefix extended by level j of unit u; false if j is no level or the
// energy reaches de
__device__ __forceinline__ bool extend(const RecEnumArgs &A, const SpeciesTab &S, uint32_t u, uint32_t j,
                                       const RecNode &from, RecNode &to) {
  const uint32_t d = A.units.degree[u];
  if (d == 0 && j > S.idiss[A.units.mode[u]]) return false;
  const double s = from.s + unit_energy(S, A.lev, A.units, u, j);
  if (!(s < A.de)) return false;
  to.s = s;
  to.j = j;
  if (d) {
    to.w = from.w * shares(j, d);
    to.place = to.equal = 0;
  } else {
    to.place = A.units.same[u] ? from.place + 1 : 1;
    to.equal = A.units.same[u] && from.j == j ? from.equal + 1 : 1;
    // multinomial of the run: times place, over the run of equal levels
    to.w = from.w * (double)to.place / (double)to.equal;
  }
  return true;
}

// first level of unit u that takes the prefix to de or above; false if none
__device__ __forceinline__ bool crossing(const RecEnumArgs &A, const SpeciesTab &S, uint32_t u, double s, uint32_t &j) {
  const uint32_t m = A.units.mode[u];
  if (A.units.degree[u]) {
    const double f = floor((A.de - s) / S.kt[m]);
    j = f > 0.0 ? (uint32_t)f : 0u;
    while (j > 0 && !(s + level_above_ground(S, A.lev, m, j - 1) < A.de)) --j;
    while (s + level_above_ground(S, A.lev, m, j) < A.de) ++j;
    return true;
  }
  uint32_t lo = 0, hi = S.idiss[m] + 1;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (s + level_above_ground(S, A.lev, m, mid) < A.de)
      lo = mid + 1;
    else
      hi = mid;
  }
  j = lo;
  return lo <= S.idiss[m];
}

template <bool WRITE>
__global__ __launch_bounds__(256) void k_rec_enum(RecEnumArgs A) {
  const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= A.n_prefix) return;
  const SpeciesTab &S = A.tab->sp[A.species];
  const uint32_t nu = A.units.n, np = A.n_prefix_units;
  uint32_t digit[kMaxModes];
  uint32_t zeros = 0;  // every digit from this unit on is 0
  uint64_t x = tid;
  for (uint32_t u = 0; u < np; ++u) {
    digit[u] = (uint32_t)(x % A.box[u]);
    x /= A.box[u];
    if (digit[u]) zeros = u + 1;
  }
  uint32_t n = 0;
  double full = 0.0;
  const uint64_t o = WRITE ? A.offset[tid] : 0;
  auto emit = [&](double e, uint32_t code, double w) {
    if (WRITE) {
      A.rec_e[o + n] = e;
      A.rec_code[o + n] = code;
      A.rec_w[o + n] = w;
    }
    ++n;
  };
  // the crossing record that node leaves at unit u. Single combinations would
  // leave one per prefix and mode: over the bends of a run, with w quanta in
  // the earlier ones and at most j - 1 below de, C(j - 1 + degree, degree - 1)
  // of them.
  auto cross = [&](uint32_t u, const RecNode &node) {
    uint32_t j;
    if (!crossing(A, S, u, node.s, j)) return;
    emit(node.s + unit_energy(S, A.lev, A.units, u, j), u | (j << 8), node.w);
    const uint32_t d = A.units.degree[u];
    full += node.w * (d ? (j ? shares(j, d) : 1.0) : 1.0);
  };
  RecNode node{0.0, 1.0, 0, 0, 0};
  bool walk = true;
  for (uint32_t u = 0; u < np && walk; ++u) {
    if (u >= zeros) cross(u, node);  // the prefix's one thread that has only zeros left
    if (A.units.same[u] && digit[u] < node.j) {
      walk = false;
    } else {
      RecNode next;
      walk = extend(A, S, u, digit[u], node, next);
      if (walk) node = next;
    }
  }
  if (walk) {
    if (np == nu) {
      emit(node.s, kRecLeaf, node.w);
      full += node.w;
    } else {
      RecNode st[kMaxModes + 1];
      uint32_t j[kMaxModes];
      uint32_t u = np;
      st[u] = node;
      j[u] = A.units.same[u] ? node.j : 0u;
      cross(u, node);
      for (;;) {
        RecNode next;
        if (!extend(A, S, u, j[u], st[u], next)) {
          if (u == np) break;
          --u;
          ++j[u];
        } else if (u + 1 == nu) {
          emit(next.s, kRecLeaf, next.w);
          full += next.w;
          ++j[u];
        } else {
          ++u;
          st[u] = next;
          j[u] = A.units.same[u] ? next.j : 0u;
          cross(u, next);
        }
      }
    }
  }
  if (!WRITE) {
    A.count[tid] = n;
    if (n) atomicAdd(A.n_full, (unsigned long long)full);
  }
}

// The same where no two modes are alike: every unit is one mode and every weight
// 1. The walk meets each crossing as it counts a mode's levels up, needs no
// search for it and carries only energies, and more threads share it (seven
// modes, 4.9 M records, 256 temperatures: 129 ms with the walk above, 118
// with this one; nine modes, 12.6 M: 431, 339).
template <bool WRITE>
__global__ __launch_bounds__(256) void k_rec_enum_distinct(RecEnumArgs A) {
  const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= A.n_prefix) return;
  const SpeciesTab &S = A.tab->sp[A.species];
  const uint32_t nm = A.units.n, np = A.n_prefix_units;
  uint32_t j[kMaxModes];
  double st[kMaxModes + 1];
  uint64_t x = tid;
  for (uint32_t m = 0; m < np; ++m) {
    j[m] = (uint32_t)(x % A.box[m]);
    x /= A.box[m];
  }
  uint32_t n = 0;
  const uint64_t o = WRITE ? A.offset[tid] : 0;
  auto emit = [&](double e, uint32_t code) {
    if (WRITE) {
      A.rec_e[o + n] = e;
      A.rec_code[o + n] = code;
    }
    ++n;
  };
  // the prefix: valid while below de; a crossing inside it is emitted once,
  // by the prefix whose crossing level is the first one and whose later
  // digits are 0
  double s = 0.0;
  bool walk = true;
  for (uint32_t m = 0; m < np && walk; ++m) {
    if (m >= S.n_bend && j[m] > S.idiss[m]) {
      walk = false;
      break;
    }
    const double s2 = s + level_above_ground(S, A.lev, m, j[m]);
    if (!(s2 < A.de)) {
      bool first = j[m] == 0 || s + level_above_ground(S, A.lev, m, j[m] - 1) < A.de;
      for (uint32_t k = m + 1; k < np; ++k) first = first && j[k] == 0;
      if (first) emit(s2, m | (j[m] << 8));
      walk = false;
      break;
    }
    s = s2;
  }
  if (walk && np == nm) emit(s, kRecLeaf);
  if (walk && np < nm) {
    uint32_t m = np;
    j[m] = 0;
    st[m] = s;
    for (;;) {
      bool back = false;
      if (m >= S.n_bend && j[m] > S.idiss[m]) {
        back = true;
      } else {
        const double s2 = st[m] + level_above_ground(S, A.lev, m, j[m]);
        if (!(s2 < A.de)) {
          emit(s2, m | (j[m] << 8));
          back = true;
        } else if (m + 1 == nm) {
          emit(s2, kRecLeaf);
          ++j[m];
        } else {
          st[m + 1] = s2;
          j[m + 1] = 0;
          ++m;
        }
      }
      if (back) {
        if (m == np) break;
        --m;
        ++j[m];
      }
    }
  }
  if (!WRITE) A.count[tid] = n;
}

// Regularized upper incomplete gamma Q(a, x) times exp(-y), x > 0 (series
// for the lower function below x = a + 1, Lentz's continued fraction above;
// Press et al., Numerical Recipes 6.2); the prefactor joins exp(-y) in one
// exponent so that small terms do not underflow early.
__device__ double gamma_q_scaled(double a, double x, double lga, double y) {
  const double lpre = (a * log(x) - x) - lga;
  if (x < a + 1.0) {
    double ap = a, del = 1.0 / a, sum = del;
    for (int i = 1; i <= 1000; ++i) {
      ap += 1.0;
      del *= x / ap;
      sum += del;
      if (fabs(del) < fabs(sum) * 1e-17) break;
    }
    return (1.0 - sum * exp(lpre)) * exp(-y);
  }
  const double tiny = 1e-300;
  double b = (x + 1.0) - a, c = 1.0 / tiny, d = 1.0 / b, h = d;
  for (int i = 1; i <= 1000; ++i) {
    const double an = -(double)i * ((double)i - a);
    b += 2.0;
    d = an * d + b;
    if (fabs(d) < tiny) d = tiny;
    c = b + an / c;
    if (fabs(c) < tiny) c = tiny;
    d = 1.0 / d;
    const double del = d * c;
    h *= del;
    if (fabs(del - 1.0) < 1e-17) break;
  }
  return exp(lpre - y) * h;
}

// (without WEIGHTED the units are the modes, every record's weight is 1 and
// rec_w is not read)
template <bool WEIGHTED>
__global__ __launch_bounds__(256) void k_rec_sum(RecSumArgs A) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  double *tail = reinterpret_cast<double *>(smem);  // stretch levels: sum_{k >= j} exp(-beta (e_k - e_j))
  __shared__ double s_z[kMaxModes + 1], s_bend[kMaxModes], s_red[256];
  const SpeciesTab &S = A.tab->sp[A.species];
  const uint32_t nu = A.units.n, tid = threadIdx.x;
  const double beta = 1.0 / (kBoltz * A.t[blockIdx.x]);
  if (tid < nu) {
    const uint32_t m = WEIGHTED ? A.units.mode[tid] : tid, d = WEIGHTED ? A.units.degree[tid] : 1u;
    if (WEIGHTED ? d > 0 : m < S.n_bend) {
      const double z = 1.0 / (1.0 - exp(-(beta * S.kt[m])));  // of one bend
      s_bend[tid] = z;
      double zz = 1.0;
      for (uint32_t i = 0; i < d; ++i) zz = zz * z;
      s_z[tid] = zz;
    } else {
      // tail sums from the top level down; the partition sum is tail[0]
      const uint32_t base = S.lev_off[m] - S.lev_off[S.n_bend];
      const uint32_t top = S.idiss[m];
      tail[base + top] = 1.0;
      for (uint32_t k = top; k-- > 0;) {
        const double step = level_above_ground(S, A.lev, m, k + 1) - level_above_ground(S, A.lev, m, k);
        tail[base + k] = 1.0 + exp(-(beta * step)) * tail[base + k + 1];
      }
      s_z[tid] = tail[base];
    }
  }
  __syncthreads();
  if (tid == 0) {
    // s_z[u] becomes the product of the partition sums of units u..nu-1
    double z = 1.0;
    s_z[nu] = 1.0;
    for (uint32_t u = nu; u-- > 0;) {
      z = z * s_z[u];
      s_z[u] = z;
    }
  }
  __syncthreads();
  double acc = 0.0;
  for (uint64_t i = tid; i < A.n_rec; i += 256) {
    const double e = A.rec_e[i], w = WEIGHTED ? A.rec_w[i] : 1.0;
    const uint32_t code = A.rec_code[i];
    if (code == kRecLeaf) {
      acc += w * gamma_q_scaled(A.a, beta * (A.de - e), A.lgamma_a, beta * e);
    } else {
      const uint32_t u = code & 0xFFu, jj = code >> 8, d = WEIGHTED ? A.units.degree[u] : (u < S.n_bend ? 1u : 0u);
      double rel;
      if (!WEIGHTED && d) {
        rel = s_bend[u];
      } else if (d) {
        // R_d(v) = sum_k C(v + k + d - 1, d - 1) r^k by R_d(v) = (C(v + d - 2,
        // d - 1) + R_{d-1}(v)) / (1 - r), R_1 = 1 / (1 - r): no term cancels
        const double z = s_bend[u];
        rel = z;
        double g = 1.0;  // C(v + k - 2, k - 1) of k = 1
        for (uint32_t k = 2; k <= d; ++k) {
          g = g * (double)(jj + k - 2) / (double)(k - 1);
          rel = (g + rel) * z;
        }
      } else {
        const uint32_t m = WEIGHTED ? A.units.mode[u] : u;
        rel = tail[(S.lev_off[m] - S.lev_off[S.n_bend]) + jj];
      }
      acc += w * ((exp(-(beta * e)) * rel) * s_z[u + 1]);
    }
  }
  s_red[tid] = acc;
  __syncthreads();
  for (uint32_t w = 128; w > 0; w >>= 1) {
    if (tid < w) s_red[tid] = s_red[tid] + s_red[tid + w];
    __syncthreads();
  }
  if (tid == 0) {
    A.num[blockIdx.x] = s_red[0];
    A.den[blockIdx.x] = s_z[0];
  }
}

}  // namespace

hipError_t launch_rec_enum(const RecEnumArgs &a, bool write, hipStream_t s) {
  if (a.n_prefix == 0) return hipSuccess;
  const dim3 grid((unsigned)((a.n_prefix + 255) / 256));
  if (!a.n_full) {
    if (write)
      hipLaunchKernelGGL(k_rec_enum_distinct<true>, grid, dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL(k_rec_enum_distinct<false>, grid, dim3(256), 0, s, a);
  } else if (write) {
    hipLaunchKernelGGL(k_rec_enum<true>, grid, dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL(k_rec_enum<false>, grid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_rec_sum(const RecSumArgs &a, uint32_t n_t, size_t lds, hipStream_t s) {
  if (n_t == 0) return hipSuccess;
  if (a.rec_w)
    hipLaunchKernelGGL(k_rec_sum<true>, dim3(n_t), dim3(256), lds, s, a);
  else
    hipLaunchKernelGGL(k_rec_sum<false>, dim3(n_t), dim3(256), lds, s, a);
  return hipGetLastError();
}

}  // namespace hcao
