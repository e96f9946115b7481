// Auxiliary ion Monte Carlo (Sec. II.C) on gfx950: swarms of one ion species
// in prescribed uniform fields E0 and a Maxwellian background gas, giving the
// stationary drift u from which the mobility u/E0 and, by Eq (2.6), the
// momentum-exchange frequency follow.  The field is uniform and the domain
// periodic, so positions never enter and every ion is independent: one
// thread owns one ion for a whole launch of many steps, its velocity and
// running sums stay in registers, and HBM is touched only at the ends of the
// launch.  The null-collision rate table sits in LDS.
#include "hd_device.h"

namespace hd {
namespace {

// 2 u - 1 of the uniform u = u01_f64(hi, lo).  u is a multiple of 2^-53 below
// 1, so 2 u - 1 and the intermediate lo' 2^-52 - 1 are multiples of 2^-52 no
// larger than 1 in magnitude: every operation is exact.
__device__ __forceinline__ double sym_f64(uint32_t hi, uint32_t lo) {
  return fma((double)hi, 0x1p-31, fma((double)(lo >> 11), 0x1p-52, -1.0));
}

// Two standard normal deviates by Marsaglia's polar method from FP64
// uniforms; (0, 0) after kSphereTries points outside the unit disk.
template <bool V>
__device__ __forceinline__ void normal_pair(StreamT<V>& st, double& g0, double& g1) {
  for (int t = 0; t < kSphereTries; ++t) {
    const double a = 2.0 * Uni<double>::get(st) - 1.0;
    const double b = 2.0 * Uni<double>::get(st) - 1.0;
    const double q = a * a + b * b;
    if (q < 1.0 && q > 0.0) {
      const double f = sqrt((-2.0 * fit_log(q)) / q);
      g0 = a * f;
      g1 = b * f;
      return;
    }
  }
  g0 = 0.0;
  g1 = 0.0;
}

// A Maxwellian velocity of thermal speed vth: three deviates of two polar
// pairs (the fourth is drawn and dropped), rounded to P.
template <class P, bool V>
__device__ __forceinline__ void maxwellian(StreamT<V>& st, double vth, P& x, P& y, P& z) {
  double g0, g1, g2, g3;
  normal_pair(st, g0, g1);
  normal_pair(st, g2, g3);
  x = (P)(vth * g0);
  y = (P)(vth * g1);
  z = (P)(vth * g2);
}

// Workgroups per CU that the step kernel is built for: its registers are
// held to that and the rate table (16 KB in FP32, 32 KB in FP64) allows it.
template <class P>
constexpr int kSwarmBlocks = sizeof(P) == 4 ? 8 : 4;
constexpr int64_t kSwarmCus = 256;  // compute units of an MI355X

template <class P>
__global__ __launch_bounds__(kSwarmThreads) void k_swarm_init(SwarmDev<P> w) {
  const int64_t gid = (int64_t)blockIdx.x * kSwarmThreads + threadIdx.x;
  if (gid >= (int64_t)w.n_fields * w.n_ions) return;
  const int f = (int)(gid / w.n_ions);
  const uint32_t i = (uint32_t)(gid - (int64_t)f * w.n_ions);
  Stream st(w.seed, kTagSwarmLoad + 16u * (uint32_t)f, i, 0u);
  P x, y, z;
  maxwellian<P>(st, w.vth_i0, x, y, z);
  w.vx[gid] = x;
  w.vy[gid] = y;
  w.vz[gid] = z;
  w.avz[gid] = 0.0;
  w.av2[gid] = 0.0;
}

// What a lane is doing with its ion.  The first three need a Philox block
// each time round; the others wait for the stage that serves them.
enum SwarmState : uint32_t {
  kFree,    // at the start of a step
  kPair,    // candidate: drawing the gas atom's two polar pairs
  kSphere,  // real collision: drawing the scattering direction
  kReady,   // gas atom drawn
  kTurn,    // direction drawn
  kDone,    // every step taken (or no ion yet)
  kIdle     // no ion left
};

// n_steps steps of every ion, starting at step index step0.  Each step:
// v_z += e E0 dt / M; the stream (kTagSwarm + 16 f, ion, step) gives u0;
// for u0 < P_max a gas atom's velocity is drawn, and the collision is real
// when u0 < P_max nu(eps)/nu_max at the pair's relative energy
// eps = M_r g^2/(2e) (table interpolated linearly, last interval beyond
// its end); a real collision keeps the centre-of-mass velocity and turns
// the relative velocity g to a random direction: v' = (m1 v + m2 v_t) +
// m2 |g| n.  With ACC, the step's v_z and |v|^2 join the ion's sums.
//
// Bound by VALU issue: the state is in registers.  One ion-step in seven is a
// candidate, so with the lanes in step nearly every step of a wave ran the
// gas atom, the logarithms and the scattering for about nine of its 64
// lanes.  Here each lane keeps its own step: every time round, the lanes
// that need a Philox block draw one together, whatever they need it for (the
// null-collision test, the next try of a polar pair or of a direction), and
// the long arithmetic waits until kServe / 8 of the wave's lanes want it.  A
// wave owns per_wave consecutive ions and hands the next one to each lane
// that has finished, so that lanes with many collisions do not hold the
// others up at the end.  The random numbers and the operations of an ion are
// those of one step after another.
// 16 x 2^20 ions, 256 steps: 60.4 ms (7.1e10 ion-steps/s) with the lanes in
// step, 31.5 ms (1.36e11) so; kServe 1, 2, 3, 5: 49, 39, 32.6, 32.8 ms.
constexpr uint32_t kServe = 4;  // eighths of the wave's lanes
template <class P, bool ACC>
__global__ __launch_bounds__(kSwarmThreads, kSwarmBlocks<P>) void k_swarm_step(
    SwarmDev<P> w, uint32_t step0, uint32_t n_steps, uint32_t per_wave, uint32_t blocks_per_field) {
  extern __shared__ __align__(16) unsigned char smem[];
  P* tab = reinterpret_cast<P*>(smem);
  __shared__ uint32_t cnt[2];
  constexpr bool kF32 = sizeof(P) == 4;
  const int tid = threadIdx.x;
  for (int k = tid; k < w.ne; k += kSwarmThreads) tab[k] = w.tab[k];
  if (tid < 2) cnt[tid] = 0u;
  __syncthreads();
  const uint32_t f = blockIdx.x / blocks_per_field;
  // the wave's ions [next, last) of swarm f (uniform)
  const uint64_t first =
      ((uint64_t)(blockIdx.x - f * blocks_per_field) * (kSwarmThreads / 64) +
       (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6)) * (uint64_t)per_wave;
  uint64_t next = first;
  const uint64_t last = min((uint64_t)w.n_ions, first + per_wave);
  const int64_t base = (int64_t)f * w.n_ions;
  const P acc = w.a[f];
  const P Pmax = w.Pmax, KEr = w.KEr, inv_dE = w.inv_dE, m1 = w.m1, m2 = w.m2;
  const P top = (P)(w.ne - 1);
  const uint32_t tag = kTagSwarm + 16u * f;
  const uint32_t k0 = (uint32_t)w.seed, k1 = (uint32_t)(w.seed >> 32);
  const uint64_t lt = lanemask_lt();
  uint32_t n_coll = 0, n_over = 0;
  uint32_t st = kDone, ion = 0, s = 0, blk = 0, tries = 0;
  bool mine = false;               // the lane holds an ion
  P vx = 0, vy = 0, vz = 0, u0 = 0;
  double az = 0.0, a2 = 0.0;
  uint32_t h1 = 0, h2 = 0, h3 = 0;  // words of the last block not yet used (FP64: h2, h3)
  double pa0 = 0.0, pb0 = 0.0, pa1 = 0.0, pb1 = 0.0;  // accepted points of the two pairs
  bool second = false;             // the first pair is drawn
  P tx = 0, ty = 0, tz = 0, g2 = 0, da = 0, db = 0;   // gas atom, g^2, point of the direction
  auto end_step = [&]() {
    if constexpr (ACC) {
      const double x = (double)vx, y = (double)vy, z = (double)vz;
      az = az + z;
      a2 = a2 + ((x * x + y * y) + z * z);
    }
    s += 1u;
    blk = 0u;
    st = s == n_steps ? kDone : kFree;
  };
  // One point of the square for the direction; true once it is settled
  // ((0, 0), the direction (0, 0, 1), after kSphereTries misses).
  auto point = [&](P a, P b) {
    const P q = a * a + b * b;
    tries += 1u;
    const bool in = q < (P)1;
    if (in || tries == (uint32_t)kSphereTries) {
      da = in ? a : (P)0;
      db = in ? b : (P)0;
      st = kTurn;
      return true;
    }
    return false;
  };
  for (;;) {
    // ---- stage 1: one Philox block for every lane that needs one
    if (st <= kSphere) {
      uint32_t w0, w1, w2, w3;
      philox4x32_10_v(ion, step0 + s, blk, tag, k0, k1, w0, w1, w2, w3);
      blk += 1u;
      if (st == kFree) {
        vz = vz + acc;
        if constexpr (kF32)
          u0 = (P)u01_f32(w0);
        else
          u0 = (P)u01_f64(w0, w1);
        if (u0 < Pmax) {
          st = kPair;
          tries = 0u;
          second = false;
        } else {
          end_step();
        }
      } else if (st == kPair) {
        const double a = kF32 ? sym_f64(h1, h2) : sym_f64(h2, h3);
        const double b = kF32 ? sym_f64(h3, w0) : sym_f64(w0, w1);
        const double q = a * a + b * b;
        const bool in = q < 1.0 && q > 0.0;
        tries += 1u;
        if (in || tries == (uint32_t)kSphereTries) {  // (0, 0): both deviates 0
          const double sa = in ? a : 0.0, sb = in ? b : 0.0;
          pa0 = second ? pa0 : sa;
          pb0 = second ? pb0 : sb;
          pa1 = sa;
          pb1 = sb;
          st = second ? kReady : kPair;
          second = true;
          tries = 0u;
        }
      } else {
        if constexpr (kF32) {
          if (!point((P)2 * (P)u01_f32(h3) - (P)1, (P)2 * (P)u01_f32(w0) - (P)1))
            point((P)2 * (P)u01_f32(w1) - (P)1, (P)2 * (P)u01_f32(w2) - (P)1);
        } else {
          point((P)sym_f64(h2, h3), (P)sym_f64(w0, w1));
        }
      }
      h1 = w1;
      h2 = w2;
      h3 = w3;
    }
    // ---- stage 2: the lanes that wait, once there are enough of them
    const uint64_t busy = __ballot(st <= kSphere);
    const uint32_t idle = (uint32_t)__popcll(__ballot(st == kIdle));
    const uint32_t waiting = 64u - (uint32_t)__popcll(busy) - idle;
    if (busy != 0 && waiting * 8u < (64u - idle) * kServe) continue;
    if (st == kReady) {
      auto radius = [](double a, double b) {
        const double q = a * a + b * b;
        return q > 0.0 ? sqrt((-2.0 * fit_log(q)) / q) : 0.0;
      };
      const double f0 = radius(pa0, pb0), f1 = radius(pa1, pb1);
      tx = (P)(w.vth_n * (pa0 * f0));
      ty = (P)(w.vth_n * (pb0 * f0));
      tz = (P)(w.vth_n * (pa1 * f1));
      const P gx = vx - tx, gy = vy - ty, gz = vz - tz;
      g2 = (gx * gx + gy * gy) + gz * gz;
      const P sc = (KEr * g2) * inv_dE;
      int j;
      P t;
      if (!(sc < top)) {  // beyond the table (or not a number)
        j = w.ne - 2;
        t = (P)1;
        n_over += 1u;
      } else {
        j = (int)sc;
        t = sc - (P)j;
      }
      const P pc = tab[j] + t * (tab[j + 1] - tab[j]);
      if (u0 < pc) {
        st = kSphere;
        tries = 0u;
        // FP32: the last block still holds the words of the first point
        if constexpr (kF32) point((P)2 * (P)u01_f32(h1) - (P)1, (P)2 * (P)u01_f32(h2) - (P)1);
      } else {
        end_step();
      }
    }
    if (st == kTurn) {
      const P q = da * da + db * db;
      const P r2 = (P)2 * sqrt((P)1 - q);
      const P nx = da * r2, ny = db * r2, nz = (P)1 - (P)2 * q;
      const P r = m2 * sqrt(g2);
      vx = (m1 * vx + m2 * tx) + r * nx;
      vy = (m1 * vy + m2 * ty) + r * ny;
      vz = (m1 * vz + m2 * tz) + r * nz;
      n_coll += 1u;
      end_step();
    }
    const uint64_t done = __ballot(st == kDone);
    if (done) {
      if (st == kDone) {
        if (mine) {
          const int64_t k = base + ion;
          w.vx[k] = vx;
          w.vy[k] = vy;
          w.vz[k] = vz;
          if constexpr (ACC) {
            w.avz[k] = az;
            w.av2[k] = a2;
          }
        }
        const uint64_t i = next + (uint32_t)__popcll(done & lt);
        mine = i < last;
        st = kIdle;
        if (mine) {
          ion = (uint32_t)i;
          const int64_t k = base + ion;
          vx = w.vx[k];
          vy = w.vy[k];
          vz = w.vz[k];
          if constexpr (ACC) {
            az = w.avz[k];
            a2 = w.av2[k];
          }
          s = 0u;
          blk = 0u;
          st = kFree;
        }
      }
      next += (uint64_t)__popcll(done);
      if (__ballot(st != kIdle) == 0) break;
    }
  }
  if (n_coll) atomicAdd(&cnt[0], n_coll);
  if (n_over) atomicAdd(&cnt[1], n_over);
  __syncthreads();
  if (tid == 0 && cnt[0])
    atomicAdd(reinterpret_cast<unsigned long long*>(&w.coll[f]), (unsigned long long)cnt[0]);
  if (tid == 1 && cnt[1])
    atomicAdd(reinterpret_cast<unsigned long long*>(&w.over[f]), (unsigned long long)cnt[1]);
}

// The same for a few steps of swarms of few ions, one ion per lane and the
// lanes in step: bound by the launch and the chain of one step, which the
// stages of k_swarm_step lengthen, while there is nothing for its lanes to be
// apart for (launch_swarm_step).
template <class P, bool ACC>
__global__ __launch_bounds__(kSwarmThreads) void k_swarm_few(SwarmDev<P> w, uint32_t step0,
                                                             uint32_t n_steps,
                                                             uint32_t blocks_per_field) {
  extern __shared__ __align__(16) unsigned char smem[];
  P* tab = reinterpret_cast<P*>(smem);
  __shared__ uint32_t cnt[2];
  const int tid = threadIdx.x;
  for (int k = tid; k < w.ne; k += kSwarmThreads) tab[k] = w.tab[k];
  if (tid < 2) cnt[tid] = 0u;
  __syncthreads();
  const uint32_t f = blockIdx.x / blocks_per_field;
  const uint32_t i = (blockIdx.x - f * blocks_per_field) * kSwarmThreads + (uint32_t)tid;
  uint32_t n_coll = 0, n_over = 0;
  if ((int64_t)i < w.n_ions) {
    const int64_t k = (int64_t)f * w.n_ions + i;
    P vx = w.vx[k], vy = w.vy[k], vz = w.vz[k];
    double az = ACC ? w.avz[k] : 0.0, a2 = ACC ? w.av2[k] : 0.0;
    const P acc = w.a[f];
    const P Pmax = w.Pmax, KEr = w.KEr, inv_dE = w.inv_dE, m1 = w.m1, m2 = w.m2;
    const P top = (P)(w.ne - 1);
    const uint32_t tag = kTagSwarm + 16u * f;
    for (uint32_t s = 0; s < n_steps; ++s) {
      StreamT<true> st(w.seed, tag, i, step0 + s);  // one ion per lane
      vz = vz + acc;
      const P u0 = Uni<P>::get(st);
      if (u0 < Pmax) {
        P tx, ty, tz;
        maxwellian<P>(st, w.vth_n, tx, ty, tz);
        const P gx = vx - tx, gy = vy - ty, gz = vz - tz;
        const P g2 = (gx * gx + gy * gy) + gz * gz;
        const P sc = (KEr * g2) * inv_dE;
        int j;
        P t;
        if (!(sc < top)) {  // beyond the table (or not a number)
          j = w.ne - 2;
          t = (P)1;
          n_over += 1u;
        } else {
          j = (int)sc;
          t = sc - (P)j;
        }
        const P pc = tab[j] + t * (tab[j + 1] - tab[j]);
        if (u0 < pc) {
          P nx, ny, nz;
          sphere<P>(st, nx, ny, nz);
          const P r = m2 * sqrt(g2);
          vx = (m1 * vx + m2 * tx) + r * nx;
          vy = (m1 * vy + m2 * ty) + r * ny;
          vz = (m1 * vz + m2 * tz) + r * nz;
          n_coll += 1u;
        }
      }
      if constexpr (ACC) {
        const double x = (double)vx, y = (double)vy, z = (double)vz;
        az = az + z;
        a2 = a2 + ((x * x + y * y) + z * z);
      }
    }
    w.vx[k] = vx;
    w.vy[k] = vy;
    w.vz[k] = vz;
    if constexpr (ACC) {
      w.avz[k] = az;
      w.av2[k] = a2;
    }
  }
  if (n_coll) atomicAdd(&cnt[0], n_coll);
  if (n_over) atomicAdd(&cnt[1], n_over);
  __syncthreads();
  if (tid == 0 && cnt[0])
    atomicAdd(reinterpret_cast<unsigned long long*>(&w.coll[f]), (unsigned long long)cnt[0]);
  if (tid == 1 && cnt[1])
    atomicAdd(reinterpret_cast<unsigned long long*>(&w.over[f]), (unsigned long long)cnt[1]);
}

// Clears the per-swarm counters and sums (a fill kernel rather than a
// memset, so that the launch may be captured into a graph).
template <class P>
__global__ void k_swarm_clear(SwarmDev<P> w) {
  const int f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= w.n_fields) return;
  w.coll[f] = 0;
  w.over[f] = 0;
  w.sums[2 * f] = 0.0;
  w.sums[2 * f + 1] = 0.0;
}

// Sums over the ions of one swarm (block f) in a fixed order: strided
// per-thread sums, then a pairwise tree in LDS.
constexpr int kRedThreads = 1024;
template <class P>
__global__ __launch_bounds__(kRedThreads) void k_swarm_reduce(SwarmDev<P> w) {
  __shared__ double r1[kRedThreads], r2[kRedThreads];
  const int f = blockIdx.x, tid = threadIdx.x;
  const double* az = w.avz + (int64_t)f * w.n_ions;
  const double* a2 = w.av2 + (int64_t)f * w.n_ions;
  double s1 = 0.0, s2 = 0.0;
  // one workgroup reads a whole swarm: bound by the round trips of its loads,
  // so a thread issues those of kRedBatch terms before it adds them in order
  constexpr int kRedBatch = 16;
  int64_t i = tid;
  for (; i + (int64_t)(kRedBatch - 1) * kRedThreads < w.n_ions; i += (int64_t)kRedBatch * kRedThreads) {
    double x1[kRedBatch], x2[kRedBatch];
#pragma unroll
    for (int u = 0; u < kRedBatch; ++u) {
      x1[u] = az[i + u * kRedThreads];
      x2[u] = a2[i + u * kRedThreads];
    }
#pragma unroll
    for (int u = 0; u < kRedBatch; ++u) {
      s1 = s1 + x1[u];
      s2 = s2 + x2[u];
    }
  }
  for (; i < w.n_ions; i += kRedThreads) {
    s1 = s1 + az[i];
    s2 = s2 + a2[i];
  }
  r1[tid] = s1;
  r2[tid] = s2;
  __syncthreads();
  for (int h = kRedThreads / 2; h > 0; h >>= 1) {
    if (tid < h) {
      r1[tid] = r1[tid] + r1[tid + h];
      r2[tid] = r2[tid] + r2[tid + h];
    }
    __syncthreads();
  }
  if (tid == 0) {
    w.sums[2 * f] = r1[0];
    w.sums[2 * f + 1] = r2[0];
  }
}

}  // namespace

template <class P>
hipError_t launch_swarm_init(const SwarmDev<P>& w, hipStream_t s) {
  const int64_t total = (int64_t)w.n_fields * w.n_ions;
  const unsigned grid = (unsigned)((total + kSwarmThreads - 1) / kSwarmThreads);
  hipLaunchKernelGGL(k_swarm_init<P>, dim3(grid), dim3(kSwarmThreads), 0, s, w);
  return hipGetLastError();
}

// Ions per wave: one per lane while the swarms leave the device's wave slots
// unfilled, else as many as make the launch fit them at once, each field's
// workgroups alike (a launch that outgrows the device slightly would wait
// for a nearly empty second round).
template <class P>
hipError_t launch_swarm_step(const SwarmDev<P>& w, uint32_t step0, int n_steps, int accumulate,
                             hipStream_t s) {
  constexpr int64_t waves = kSwarmThreads / 64, slots = kSwarmCus * kSwarmBlocks<P>;
  const size_t lds = (size_t)w.ne * sizeof(P);
  // A few steps with the lanes in step, unless a field's workgroups are so
  // many that they wait for each other at its counters.  Where the lines lie,
  // in us in step and apart: 7 x 2,048 ions 4 steps 25.9, 30.4, 8 steps 35.8,
  // 38.0, 12 steps 46.4, 42.4; 300 x 2,048 (1.2 ions per lane of the device) 4
  // steps 63.2, 64.3, 6 steps 84.8, 79.1; 1,100 x 1,024 (2.1) 2 steps 58.8, 62.8,
  // 4 steps 94.8, 91.6; 16 x 65,536 (256 workgroups each) one step 63.0, 47.0.
  constexpr int64_t lanes = slots * kSwarmThreads, kFewBlocks = 64;
  const int64_t blocks = (w.n_ions + kSwarmThreads - 1) / kSwarmThreads;
  const int64_t ions = (int64_t)w.n_fields * w.n_ions;
  if (blocks <= kFewBlocks && n_steps <= 8 && (ions <= lanes || n_steps * ions <= 5 * lanes)) {
    const auto k = accumulate ? k_swarm_few<P, true> : k_swarm_few<P, false>;
    hipLaunchKernelGGL(k, dim3((unsigned)(blocks * w.n_fields)), dim3(kSwarmThreads), lds, s, w,
                       step0, (uint32_t)n_steps, (uint32_t)blocks);
    return hipGetLastError();
  }
  const int64_t fit = slots / w.n_fields > 1 ? slots / w.n_fields : 1;  // workgroups per field
  const int64_t per = (w.n_ions + fit * kSwarmThreads - 1) / (fit * kSwarmThreads) * 64;
  const int64_t bpf = (w.n_ions + per * waves - 1) / (per * waves);
  const unsigned grid = (unsigned)(bpf * w.n_fields);
  const auto k = accumulate ? k_swarm_step<P, true> : k_swarm_step<P, false>;
  hipLaunchKernelGGL(k, dim3(grid), dim3(kSwarmThreads), lds, s, w, step0, (uint32_t)n_steps,
                     (uint32_t)per, (uint32_t)bpf);
  return hipGetLastError();
}

// Steps of one launch: the lanes of a wave end a launch apart (they have had
// different numbers of collisions), which costs a one-ion-per-lane launch of
// 256 steps 6 % against 1,024; many ions hide it, and their launches stay
// near 30 ms.
int swarm_launch_steps(int64_t ions) { return ions > ((int64_t)1 << 22) ? 256 : 1024; }

template <class P>
hipError_t launch_swarm_clear(const SwarmDev<P>& w, hipStream_t s) {
  hipLaunchKernelGGL(k_swarm_clear<P>, dim3((w.n_fields + 255) / 256), dim3(256), 0, s, w);
  return hipGetLastError();
}

template <class P>
hipError_t launch_swarm_reduce(const SwarmDev<P>& w, hipStream_t s) {
  hipLaunchKernelGGL(k_swarm_reduce<P>, dim3(w.n_fields), dim3(kRedThreads), 0, s, w);
  return hipGetLastError();
}

template hipError_t launch_swarm_init<float>(const SwarmDev<float>&, hipStream_t);
template hipError_t launch_swarm_init<double>(const SwarmDev<double>&, hipStream_t);
template hipError_t launch_swarm_step<float>(const SwarmDev<float>&, uint32_t, int, int,
                                             hipStream_t);
template hipError_t launch_swarm_step<double>(const SwarmDev<double>&, uint32_t, int, int,
                                              hipStream_t);
template hipError_t launch_swarm_reduce<float>(const SwarmDev<float>&, hipStream_t);
template hipError_t launch_swarm_clear<float>(const SwarmDev<float>&, hipStream_t);
template hipError_t launch_swarm_clear<double>(const SwarmDev<double>&, hipStream_t);
template hipError_t launch_swarm_reduce<double>(const SwarmDev<double>&, hipStream_t);

}  // namespace hd
